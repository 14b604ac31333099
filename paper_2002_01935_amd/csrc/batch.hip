// Many independent small networks in one graph launch.
//
// Workloads such as the QAOA energy (Sec. 4.5: one light-cone network per
// edge) or a batch of sampled bitstrings (Sec. 4.7.3) are many small networks
// whose contractions are mostly tiny.  Launched one kernel per pairwise
// contraction they are bound by launch latency.  Here the groups of small
// contractions at the bottom of all networks (tiny.h) run in one launch, a
// workgroup per group.  The contractions that remain in each network are
// sorted into levels: one per chain of dependences, where two of a network's
// ops depend on each other if one writes arena memory that the other touches
// (its arena was laid out for its own order).  A level's medium-sized
// contractions, of all networks, run in one launch whose workgroups look up
// their contraction in a table; its large ones are launched with the ordinary
// kernels, on parallel branches.  The whole sequence is captured once per
// workspace into a HIP graph and replayed by tn_batch_contract.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cstring>
#include <map>
#include <mutex>
#include <string>
#include <vector>

#include "exec.h"
#include "kernels.h"
#include "plan.h"

namespace tn {

#define GMEM __attribute__((address_space(1)))
#define CMEM __attribute__((address_space(4)))
#define TN_WAVE_SYNC() __builtin_amdgcn_wave_barrier()
// A value the same in every lane of the wavefront, made known to the compiler as such.
#define TN_UNIFORM(x) __builtin_amdgcn_readfirstlane(x)

#include "rowops.h"
#include "tiny_kernel.h"

constexpr int kLevelBits = 24;      // bit-list capacity of a medium contraction
constexpr int kLevelWorkBits = 22;  // log2 (outputs x summed values) of the largest one
// GEMM-class ones are asked for by TN_FLAG_GEMM_ALL_SIZES (none is smaller than
// 2^25 without it): larger ones run on the matrix cores, as the flag says
constexpr int kLevelGemmBits = 16;
constexpr int kLevelThreads = 256;
constexpr int kLongSum = 6;         // log2 summed values from which the planner splits a sum over lanes
constexpr int kLevelStep = 3;       // log2 summed values of a thread's step
constexpr int kLevelTree = 5;       // levels of a thread's addition tree above a step
// log2 summed values of the longest contraction: 2^8 per thread of a
// workgroup.  Above, the sum would be one compute unit's serial chain, and the
// split-K kernels spread it over the chip: a batch of one 2^17 sum 47 us per
// call by one workgroup, 35 by them; of 2^16, 40 and 35 (eight of them 40 and
// 151), of eight 2^22 2494 and 429.
constexpr int kLevelSumBits = kLevelStep + kLevelTree + 8;
// parallel branches of a level's large contractions in the captured graph
// (one per hardware queue a process gets by default)
constexpr int kBranches = 4;

// A position list as at most kLevelRuns runs (entries as in BitRuns).
constexpr int kLevelRuns = 8;
struct LevelList {
  int32_t n;
  uint32_t r[kLevelRuns];
};

// One medium contraction: for each of 2^n_out outputs,
//   C[o] = sum over 2^n_k summed values of opA(A[o, k]) * opB(B[o, k])
// (opX = complex conjugate when conj_x), or C[o] = A[o] without B.  The lists
// place o in A / B / C (oa, ob, oc), the threads of one output over its lowest
// summed bits (ta, tb) and the summed values above those, kLevelStep bits at first
// (step_a, step_b: their offsets) and the rest (ha, hb).
struct LevelOp {
  Ref a, b, c;
  uint32_t net;
  int32_t n_out, n_k, mode;
  int32_t has_b, conj_a, conj_b, pad;
  uint32_t step_a[kLevelStep], step_b[kLevelStep];
  LevelList oa, ob, oc, ta, tb, ha, hb;
  int32_t pad2;
};
static_assert(sizeof(LevelOp) % 8 == 0, "LevelOp layout");

// A workgroup's contraction and its block of that contraction's outputs.
struct LevelBlock {
  uint32_t op, block;
};

// Threads of one output (LevelOp::mode): one thread, one wavefront (lanes over
// the lowest six summed bits) or the whole workgroup (the lowest eight).
enum { kPerThread = 0, kPerWave = 1, kPerGroup = 2 };

// Offset of v through a list (uniform: scalar loads, a uniform branch per run).
__device__ __forceinline__ uint32_t place(uint32_t v, const LevelList& l) {
  uint32_t off = 0;
#pragma unroll
  for (int i = 0; i < kLevelRuns; i++) {
    if (i >= l.n) break;
    const uint32_t w = l.r[i];
    off |= ((v >> (w & 0xFF)) & (~0u >> (32 - (w >> 16)))) << ((w >> 8) & 0xFF);
  }
  return off;
}

// One thread's 2^walk products, 2^LO per step (uniform offsets, their loads in
// flight together).  SERIAL: added one after another, as the row kernel does.
// Else as a balanced tree: sum[l] waits for its neighbour of 2^l steps.  With
// the lanes and wavefronts a value then passes n_k additions, no more than in
// the split-K kernels: 2^16 values per output in complex64 have an error of
// 1.6e-7 (split-K kernels 2.4e-7, one running sum per thread 6.7e-7), at the
// same time per call.
template <typename T, int LO, bool SERIAL>
__device__ __forceinline__ typename C2<T>::t thread_sum(GMEM const typename C2<T>::t* A, GMEM const typename C2<T>::t* B,
                                                        CMEM const LevelOp* op, int walk, T ca, T cb) {
  using V = typename C2<T>::t;
  constexpr int N = 1 << LO;
  const LevelList ha = cload(&op->ha), hb = cload(&op->hb);
  uint32_t da[N], db[N];
  da[0] = db[0] = 0;
#pragma unroll
  for (int l = 0; l < LO; l++)
#pragma unroll
    for (int i = 0; i < (1 << l); i++) {
      da[(1 << l) + i] = da[i] + op->step_a[l];
      db[(1 << l) + i] = db[i] + op->step_b[l];
    }
  V acc, sum[kLevelTree];
  acc.x = 0;
  acc.y = 0;
  const uint32_t steps = 1u << (walk - LO);
  for (uint32_t s = 0; s < steps; s++) {
    const uint32_t xa = place(s, ha), xb = place(s, hb);
    V a[N], b[N];
#pragma unroll
    for (int i = 0; i < N; i++) {
      a[i] = ld(A + xa + da[i]);
      b[i] = ld(B + xb + db[i]);
    }
#pragma unroll
    for (int i = 0; i < N; i++) {
      a[i].y *= ca;
      b[i].y *= cb;
      if constexpr (SERIAL) acc = cfma(acc, a[i], b[i]);
      else a[i] = cmul(a[i], b[i]);
    }
    if constexpr (!SERIAL) {
#pragma unroll
      for (int n = N / 2; n >= 1; n /= 2)
#pragma unroll
        for (int i = 0; i < n; i++) a[i] = cadd(a[i], a[i + n]);
      acc = a[0];
#pragma unroll
      for (int l = 0; l < kLevelTree; l++) {
        if (((s >> l) & 1u) == 0) {
          sum[l] = acc;
          break;
        }
        acc = cadd(sum[l], acc);
      }
    }
  }
  return acc;
}

// A level's medium contractions of all networks.  Latency bound (a few
// microseconds of dependent loads); a launch per contraction would pay that
// and the launch each time.  81 QAOA terms: 12 levels, 62 launches per call in
// place of 624, 4.56 -> 1.59 ms against one workgroup per network running up
// to 2^16 multiply-adds per contraction (410 us per launch) between launches.
template <typename T>
__global__ __launch_bounds__(kLevelThreads) void level_kernel(CMEM const Ctx* ctxs, CMEM const LevelOp* ops,
                                                              CMEM const LevelBlock* blocks) {
  using V = typename C2<T>::t;
  const LevelBlock e = cload(blocks + blockIdx.x);
  CMEM const LevelOp* op = ops + e.op;
  const Ctx ctx = cload(ctxs + op->net);
  const int n_out = op->n_out, n_k = op->n_k, mode = op->mode, has_b = op->has_b;
  const uint32_t tid = threadIdx.x;
  const Ref ra = cload(&op->a), rb = cload(&op->b), rc = cload(&op->c);
  GMEM const V* A = reinterpret_cast<GMEM const V*>(resolve(ctx, ra, 0, 0, sizeof(V)));
  GMEM const V* B = has_b ? reinterpret_cast<GMEM const V*>(resolve(ctx, rb, 0, 0, sizeof(V))) : A;
  GMEM V* C = reinterpret_cast<GMEM V*>(resolve(ctx, rc, 0, 0, sizeof(V)));
  const int ts = mode == kPerThread ? 0 : (mode == kPerWave ? 6 : 8);   // log2 threads per output
  const uint32_t o = (e.block * kLevelThreads + tid) >> ts, q = tid & ((1u << ts) - 1u);
  const bool active = (o >> n_out) == 0;
  const uint32_t oo = active ? o : 0u;
  V acc;
  acc.x = 0;
  acc.y = 0;
  if (!has_b) {
    acc = ld(A + place(oo, cload(&op->oa)));
  } else {
    const T ca = op->conj_a ? T(-1) : T(1), cb = op->conj_b ? T(-1) : T(1);
    GMEM const V* Ao = A + place(oo, cload(&op->oa)) + place(q, cload(&op->ta));
    GMEM const V* Bo = B + place(oo, cload(&op->ob)) + place(q, cload(&op->tb));
    const int walk = n_k - ts;
    if (n_k < kLongSum) {
      switch (walk) {
        case 0: acc = thread_sum<T, 0, true>(Ao, Bo, op, walk, ca, cb); break;
        case 1: acc = thread_sum<T, 1, true>(Ao, Bo, op, walk, ca, cb); break;
        case 2: acc = thread_sum<T, 2, true>(Ao, Bo, op, walk, ca, cb); break;
        default: acc = thread_sum<T, 3, true>(Ao, Bo, op, walk, ca, cb);
      }
    } else {
      switch (walk) {
        case 0: acc = thread_sum<T, 0, false>(Ao, Bo, op, walk, ca, cb); break;
        case 1: acc = thread_sum<T, 1, false>(Ao, Bo, op, walk, ca, cb); break;
        case 2: acc = thread_sum<T, 2, false>(Ao, Bo, op, walk, ca, cb); break;
        default: acc = thread_sum<T, 3, false>(Ao, Bo, op, walk, ca, cb);
      }
    }
  }
  if (mode != kPerThread) {                      // fixed order: butterfly, then the four wavefronts
    acc.x = wave_sum(acc.x);
    acc.y = wave_sum(acc.y);
    if (mode == kPerGroup) {
      __shared__ V part[kLevelThreads / 64];
      if ((tid & 63) == 0) part[tid >> 6] = acc;
      __syncthreads();
      acc = cadd(cadd(part[0], part[1]), cadd(part[2], part[3]));
    }
  }
  if (active && q == 0) st(C + place(o, cload(&op->oc)), acc);
}

// The small-contraction launches that begin each network's program, all in one
// launch: workgroup b runs group entry[b].group of the blob at entry[b].blob
// bytes from the workspace base, for network entry[b].net.
struct BatchGroup {
  uint32_t net, group;
  uint64_t blob;
};
template <typename T>
__global__ __launch_bounds__(512) void tiny_batch_kernel(uint64_t base, CMEM const Ctx* ctxs, CMEM const BatchGroup* entries) {
  extern __shared__ __attribute__((aligned(16))) char smem[];
  const BatchGroup e = cload(entries + blockIdx.x);
  const Ctx ctx = cload(ctxs + e.net);
  tiny_group<T>(ctx, base + e.blob, (int)e.group, 0, 0, smem);
}

// Runs of n entries of a position list; false when there are too many.
static bool level_runs(const int8_t* pos, int n, LevelList& l) {
  BitRuns R;
  make_runs(pos, n, R);
  l.n = R.n;
  if (R.n > kLevelRuns) return false;
  for (int i = 0; i < R.n; i++) l.r[i] = R.r[i];
  return true;
}

// Whether op is a medium contraction, and its descriptor if so.
static bool as_level(const Op& op, int prec, LevelOp& t) {
  std::memset(&t, 0, sizeof t);
  int8_t oa[kLevelBits], ob[kLevelBits], oc[kLevelBits], ka[kLevelBits], kb[kLevelBits];
  for (int j = 0; j < kLevelBits; j++) oa[j] = ob[j] = oc[j] = ka[j] = kb[j] = -1;
  auto fits = [&](int n_out, int n_k) {
    t.n_out = n_out;
    t.n_k = n_k;
    return n_out <= kLevelBits && n_k <= kLevelSumBits && n_out + n_k <= kLevelWorkBits;
  };
  if (op.kind == OpKind::Row) {
    const RowOp& r = op.row;
    if (r.accumulate || !fits(r.n_rows + r.n_in, r.n_k)) return false;
    for (int j = 0; j < r.n_rows; j++) { oa[j] = r.row_a[j]; ob[j] = r.row_b[j]; oc[j] = r.row_c[j]; }
    for (int j = 0; j < r.n_in; j++) { ob[r.n_rows + j] = r.in_b[j]; oc[r.n_rows + j] = r.in_c[j]; }
    for (int j = 0; j < r.n_k; j++) { ka[j] = r.k_a[j]; kb[j] = r.k_b[j]; }
    t.a = r.a; t.b = r.b; t.c = r.c;
    t.has_b = 1;
    t.conj_a = r.conj_a; t.conj_b = r.conj_b;
  } else if (op.kind == OpKind::Gemm) {
    const GemmOp& g = op.gemm;
    if (g.accumulate || g.ab_split || g.k_split_bits + g.k_fold_bits > 0 || !fits(g.n_h + g.n_m + g.n_n, g.n_k)) return false;
    if (t.n_out + t.n_k > kLevelGemmBits) return false;
    int j = 0;
    for (int i = 0; i < g.n_h; i++, j++) { oa[j] = g.a_h[i]; ob[j] = g.b_h[i]; oc[j] = g.c_h[i]; }
    for (int i = 0; i < g.n_m; i++, j++) { oa[j] = g.a_m[i]; oc[j] = g.c_m[i]; }
    for (int i = 0; i < g.n_n; i++, j++) { ob[j] = g.b_n[i]; oc[j] = g.c_n[i]; }
    for (int i = 0; i < g.n_k; i++) { ka[i] = g.a_k[i]; kb[i] = g.b_k[i]; }
    t.a = g.a; t.b = g.b; t.c = g.c;
    t.has_b = 1;
    t.conj_a = g.conj_a; t.conj_b = g.conj_b;
  } else if (op.kind == OpKind::Permute) {
    const PermuteOp& pm = op.perm;
    const int c128 = prec == TN_C128;
    if (pm.accumulate || !fits(pm.n_bits, 0) || pm.src_c128 != c128 || pm.dst_c128 != c128 || pm.per_slice_serial) return false;
    for (int j = 0; j < pm.n_bits; j++) { oa[j] = pm.src_pos[j]; oc[j] = pm.dst_pos[j]; }
    t.a = pm.src; t.c = pm.dst;
  } else {
    return false;
  }
  // Short sums by one thread (a step takes about 1 us of load latency), long
  // ones shared by a wavefront; with 2^14 outputs a wavefront per output pays
  // from 2^8 values on, with 2^16 the threads fill the chip.
  const bool per_thread = t.n_k < kLongSum || t.n_out >= 16 || (t.n_out >= 14 && t.n_k < 8);
  t.mode = per_thread ? kPerThread : (t.n_k >= 12 && t.n_out <= 8 ? kPerGroup : kPerWave);
  const int ts = t.mode == kPerThread ? 0 : (t.mode == kPerWave ? 6 : 8), lo = std::min(kLevelStep, t.n_k - ts);
  if (t.n_k - ts > kLevelStep + kLevelTree) return false;
  for (int i = 0; i < lo; i++) {
    t.step_a[i] = 1u << ka[ts + i];
    t.step_b[i] = 1u << kb[ts + i];
  }
  return level_runs(oa, t.n_out, t.oa) && level_runs(ob, t.n_out, t.ob) && level_runs(oc, t.n_out, t.oc) &&
         level_runs(ka, ts, t.ta) && level_runs(kb, ts, t.tb) && level_runs(ka + ts + lo, t.n_k - ts - lo, t.ha) &&
         level_runs(kb + ts + lo, t.n_k - ts - lo, t.hb);
}

// Arena bytes an op reads and writes (elements of eb bytes; operands there are
// compact); false when that is not known.
struct ArenaUse {
  std::vector<std::pair<int64_t, int64_t>> reads, writes;   // [begin, end)
  bool known = true;
};

// Levels of a network's ops: the level of the last op that wrote, and of those
// that read since, for every stretch of the arena.  An op goes one level above
// all earlier ones that write what it touches or read what it writes.
class ArenaLevels {
 public:
  int place(const ArenaUse& use) {
    int level = floor_;
    if (!use.known) {
      level = floor_ = top_ + 1;                            // after all before it, before all behind it
      top_ = floor_++;
      return level;
    }
    for (auto& r : use.reads) each(r, [&](Part& p) { level = std::max(level, p.written + 1); });
    for (auto& w : use.writes) each(w, [&](Part& p) { level = std::max(level, std::max(p.written, p.read) + 1); });
    for (auto& r : use.reads) each(r, [&](Part& p) { p.read = std::max(p.read, level); });
    for (auto& w : use.writes) each(w, [&](Part& p) { p.written = level; p.read = -1; });
    top_ = std::max(top_, level);
    return level;
  }

 private:
  struct Part { int64_t end; int written, read; };
  std::map<int64_t, Part> parts_;                           // by begin, disjoint
  int floor_ = 0, top_ = -1;
  void split(int64_t at) {
    auto it = parts_.upper_bound(at);
    if (it == parts_.begin()) return;
    --it;
    if (it->first == at || it->second.end <= at) return;
    const Part rest = it->second;
    it->second.end = at;
    parts_[at] = rest;
  }
  template <typename F>
  void each(const std::pair<int64_t, int64_t>& range, F&& f) {
    split(range.first);
    split(range.second);
    auto it = parts_.lower_bound(range.first);
    for (int64_t at = range.first; at < range.second; ++it) {
      if (it == parts_.end() || it->first > at) {
        const int64_t end = it == parts_.end() ? range.second : std::min(range.second, it->first);
        it = parts_.insert(it, {at, Part{end, -1, -1}});
      }
      f(it->second);
      at = it->second.end;
    }
  }
};

static ArenaUse arena_use(const Op& op, int eb) {
  ArenaUse u;
  auto add = [&](std::vector<std::pair<int64_t, int64_t>>& v, const Ref& r, int bits, int bytes) {
    if (r.kind == 1) v.push_back({r.off, r.off + (int64_t(bytes) << bits)});
  };
  auto count = [](const int8_t* p, int n) { int c = 0; for (int i = 0; i < n; i++) c += p[i] >= 0; return c; };
  switch (op.kind) {
    case OpKind::Row: {
      const RowOp& r = op.row;
      const int out = r.n_rows + r.n_in;
      add(u.reads, r.a, count(r.row_a, r.n_rows) + r.n_k, eb);
      add(u.reads, r.b, count(r.row_b, r.n_rows) + count(r.in_b, r.n_in) + r.n_k, eb);
      add(u.writes, r.c, out, eb);
      if (r.k_split_bits > 0) add(u.writes, r.part, out + r.k_split_bits, eb);
      break;
    }
    case OpKind::RowReduce:
      add(u.reads, op.row.part, op.row.n_rows + op.row.n_in + op.row.k_split_bits, eb);
      add(u.writes, op.row.c, op.row.n_rows + op.row.n_in, eb);
      break;
    case OpKind::Gemm: {
      const GemmOp& g = op.gemm;
      if (g.ab_split) { u.known = false; break; }
      add(u.reads, g.a, g.n_h + g.n_m + g.n_k, eb);
      add(u.reads, g.b, g.n_h + g.n_n + g.n_k, eb);
      add(u.writes, g.c, g.n_h + g.n_m + g.n_n, eb);
      if (g.k_split_bits > 0) add(u.writes, g.part, g.n_h + g.n_m + g.n_n + g.k_split_bits, eb);
      break;
    }
    case OpKind::Permute:
      add(u.reads, op.perm.src, op.perm.n_bits, op.perm.src_c128 ? 16 : 8);
      add(u.writes, op.perm.dst, op.perm.n_bits, op.perm.dst_c128 ? 16 : 8);
      break;
    case OpKind::Tiny:
      for (auto& x : op.tiny->reads) {
        TinyLoad l;
        std::memcpy(&l, op.tiny->blob.data() + x.first, sizeof l);
        u.reads.push_back({256 * (int64_t)l.src, 256 * (int64_t)l.src + (int64_t(eb) << l.n_bits)});
      }
      for (auto& x : op.tiny->writes) {
        TinyOp t;
        std::memcpy(&t, op.tiny->blob.data() + x.first, sizeof t);
        if (t.dst_kind == 1) u.writes.push_back({256 * (int64_t)t.dst, 256 * (int64_t)t.dst + (int64_t(eb) << t.n_out)});
      }
      break;
    default: u.known = false;
  }
  return u;
}

}  // namespace tn

using namespace tn;

struct tn_batch_s {
  std::mutex mu;
  int prec = TN_C64_4M;
  int n_nets = 0, n_levels = 0;
  std::vector<int32_t> n_leaves;             // per network
  std::vector<uint64_t> region_off;          // per network: its plan workspace inside the batch workspace
  std::vector<Ctx> ctx_rel;                  // per network, ws relative to the batch workspace base
  std::vector<LevelOp> ops;                  // medium contractions
  std::vector<LevelBlock> blocks;            // ordered by level
  std::vector<uint32_t> level_block;         // per level: its first block; then the total
  // [level][network] -> large ops, in the network's order
  std::vector<std::vector<std::vector<Op>>> big;
  // leading small-contraction groups of all networks: blobs, workgroup table
  std::vector<char> blobs;
  std::vector<BatchGroup> groups;
  int64_t n_grouped = 0;                     // contractions in them
  uint32_t group_threads = 64, group_lds = 0;
  uint64_t blob_off = 0, group_off = 0;
  uint64_t ctx_off = 0, ops_off = 0, blocks_off = 0, ptr_off = 0, ws_bytes = 0;
  int ptr_stride = 0;                        // pointer-table slots per network
  int64_t n_launches = 0;
  // prepared workspaces: graph per workspace address, at most kMaxGraphs
  std::map<uint64_t, tn_plan_s::GraphEntry> graphs;
  uint64_t clock = 0;
};

static void batch_drop(tn_plan_s::GraphEntry& e) {
  if (e.done) {
    (void)hipEventSynchronize((hipEvent_t)e.done);
    (void)hipEventDestroy((hipEvent_t)e.done);
  }
  if (e.exec) (void)hipGraphExecDestroy((hipGraphExec_t)e.exec);
  e = tn_plan_s::GraphEntry{};
}

#define BATCH_TRY(expr)                                                                   \
  do {                                                                                    \
    hipError_t _e = (expr);                                                               \
    if (_e != hipSuccess)                                                                 \
      return set_error(TN_E_DEVICE, std::string(#expr) + ": " + hipGetErrorString(_e));   \
  } while (0)

extern "C" int tn_batch(int32_t n_plans, const tn_plan_t* plans, tn_batch_t* batch) {
  if (!batch) return set_error(TN_E_INVALID, "batch is null");
  *batch = nullptr;
  if (n_plans < 1 || !plans) return set_error(TN_E_INVALID, "no plans");
  for (int j = 0; j < n_plans; j++)
    if (!plans[j]) return set_error(TN_E_INVALID, "plan " + std::to_string(j) + " is null");
  const int prec = plans[0]->prec;
  for (int j = 0; j < n_plans; j++) {
    if (plans[j]->prec != prec) return set_error(TN_E_INVALID, "plans of a batch share one precision");
    if (plans[j]->d_sliced != 1 || plans[j]->n_batch != 1)
      return set_error(TN_E_UNSUPPORTED, "batched plans must be unsliced (plan " + std::to_string(j) + ")");
  }
  tn_batch_s* b = new tn_batch_s();
  b->prec = prec;
  b->n_nets = n_plans;
  // per network: the mode-0 program's leading groups, then levels
  const int N = n_plans;
  const int eb = prec == TN_C128 ? 16 : 8;
  std::vector<std::vector<uint32_t>> medium;               // [level] -> indices into b->ops
  for (int j = 0; j < N; j++) {
    tn_plan_s* p = plans[j];
    std::lock_guard<std::mutex> lk(p->mu);
    const std::vector<Op> prog = forward_program(p, 0);
    bool leading = true;
    ArenaLevels levels;
    auto at_level = [&](int l) {
      if ((int)medium.size() <= l) {
        medium.resize((size_t)l + 1);
        b->big.resize((size_t)l + 1, std::vector<std::vector<Op>>(N));
      }
    };
    for (size_t i = 0; i < prog.size(); i++) {
      const Op& op = prog[i];
      if (op.kind == OpKind::Counter || op.kind == OpKind::Fill) continue;
      // groups that read no arena value depend on nothing; the next stage of a
      // set that was cut reads theirs and is launched as a large op
      if (op.kind == OpKind::Tiny && leading && op.tiny->reads.empty()) {
        for (uint32_t g = 0; g < op.tiny->n_groups; g++) b->groups.push_back({(uint32_t)j, g, b->blobs.size()});
        b->blobs.insert(b->blobs.end(), op.tiny->blob.begin(), op.tiny->blob.end());
        b->blobs.resize((b->blobs.size() + 63) / 64 * 64, 0);
        b->group_threads = std::max(b->group_threads, op.tiny->threads);
        b->group_lds = std::max(b->group_lds, op.tiny->lds_bytes);
        b->n_grouped += (int64_t)op.tiny->nodes.size();
        continue;
      }
      leading = false;
      ArenaUse use = arena_use(op, eb);
      const bool reduced = i + 1 < prog.size() && prog[i + 1].kind == OpKind::RowReduce;
      if (reduced) {                                        // a split row op and its reduce pass: one unit
        const ArenaUse r = arena_use(prog[i + 1], eb);
        use.reads.insert(use.reads.end(), r.reads.begin(), r.reads.end());
        use.writes.insert(use.writes.end(), r.writes.begin(), r.writes.end());
      }
      const int level = levels.place(use);
      at_level(level);
      LevelOp t;
      if (as_level(op, prec, t)) {
        t.net = (uint32_t)j;
        medium[(size_t)level].push_back((uint32_t)b->ops.size());
        b->ops.push_back(t);
      } else {
        b->big[(size_t)level][(size_t)j].push_back(op);
        if (reduced) b->big[(size_t)level][(size_t)j].push_back(prog[i + 1]);
      }
      if (reduced) i++;
    }
    b->n_leaves.push_back(p->n_leaves);
    b->ptr_stride = std::max(b->ptr_stride, p->n_leaves + 2);
  }
  b->n_levels = (int)medium.size();
  for (auto& lvl : medium) {
    b->level_block.push_back((uint32_t)b->blocks.size());
    // longest sums first: they end last
    std::stable_sort(lvl.begin(), lvl.end(), [&](uint32_t x, uint32_t y) { return b->ops[x].n_k > b->ops[y].n_k; });
    for (uint32_t o : lvl) {
      const LevelOp& t = b->ops[o];
      const int per = t.mode == kPerThread ? 8 : (t.mode == kPerWave ? 2 : 0);   // log2 outputs per workgroup
      const uint32_t n = t.n_out > per ? 1u << (t.n_out - per) : 1u;
      for (uint32_t k = 0; k < n; k++) b->blocks.push_back({o, k});
    }
  }
  b->level_block.push_back((uint32_t)b->blocks.size());
  // workspace: contexts | medium contractions | their blocks | pointer tables | per-network plan workspaces
  auto up = [](uint64_t x) { return (x + 255) / 256 * 256; };
  b->ctx_off = 0;
  b->ops_off = up(b->ctx_off + sizeof(Ctx) * (uint64_t)N);
  b->blocks_off = up(b->ops_off + sizeof(LevelOp) * (uint64_t)b->ops.size());
  b->ptr_off = up(b->blocks_off + sizeof(LevelBlock) * (uint64_t)b->blocks.size());
  b->blob_off = up(b->ptr_off + 8 * (uint64_t)b->ptr_stride * N);
  b->group_off = up(b->blob_off + b->blobs.size());
  for (BatchGroup& g : b->groups) g.blob += b->blob_off;
  uint64_t off = up(b->group_off + sizeof(BatchGroup) * (uint64_t)b->groups.size());
  for (int j = 0; j < N; j++) {
    tn_plan_s* p = plans[j];
    b->region_off.push_back(off);
    Ctx c = make_ctx(p, reinterpret_cast<void*>(off), p->arena_bytes);   // relative to the batch base
    c.ptrtab_off = (int64_t)(b->ptr_off + 8 * (uint64_t)b->ptr_stride * j) - (int64_t)off;
    b->ctx_rel.push_back(c);
    off = up(off + p->workspace_bytes);
  }
  b->ws_bytes = off;
  int64_t launches = b->groups.empty() ? 0 : 1;
  for (int l = 0; l < b->n_levels; l++) {
    launches += b->level_block[(size_t)l] < b->level_block[(size_t)l + 1];
    for (int j = 0; j < N; j++) launches += (int64_t)b->big[(size_t)l][(size_t)j].size();
  }
  b->n_launches = launches;
  *batch = b;
  return TN_OK;
}

extern "C" int tn_batch_info(tn_batch_t b, uint64_t* workspace_bytes, int32_t* n_levels, int64_t* n_tiny,
                             int64_t* n_launches) {
  if (!b) return set_error(TN_E_INVALID, "batch is null");
  std::lock_guard<std::mutex> lk(b->mu);
  if (workspace_bytes) *workspace_bytes = b->ws_bytes;
  if (n_levels) *n_levels = b->n_levels;
  if (n_tiny) *n_tiny = b->n_grouped + (int64_t)b->ops.size();
  if (n_launches) *n_launches = b->n_launches;
  return TN_OK;
}

// Context of network j over the batch workspace at `base`.
static Ctx batch_ctx(const tn_batch_s* b, int j, uint64_t base) {
  Ctx c = b->ctx_rel[(size_t)j];
  c.ws += base;
  return c;
}

extern "C" int tn_batch_prepare(tn_batch_t b, void* workspace, uint64_t workspace_bytes, void* stream) {
  if (!b) return set_error(TN_E_INVALID, "batch is null");
  std::lock_guard<std::mutex> lk(b->mu);
  if (!workspace || workspace_bytes < b->ws_bytes)
    return set_error(TN_E_WORKSPACE, "workspace of " + std::to_string(b->ws_bytes) + " bytes required");
  hipStream_t s = static_cast<hipStream_t>(stream);
  const uint64_t base = reinterpret_cast<uint64_t>(workspace);
  char* w = static_cast<char*>(workspace);
  std::vector<Ctx> ctxs;
  for (int j = 0; j < b->n_nets; j++) ctxs.push_back(batch_ctx(b, j, base));
  BATCH_TRY(hipMemcpyAsync(w + b->ctx_off, ctxs.data(), sizeof(Ctx) * ctxs.size(), hipMemcpyHostToDevice, s));
  if (!b->ops.empty()) {
    BATCH_TRY(hipMemcpyAsync(w + b->ops_off, b->ops.data(), sizeof(LevelOp) * b->ops.size(), hipMemcpyHostToDevice, s));
    BATCH_TRY(hipMemcpyAsync(w + b->blocks_off, b->blocks.data(), sizeof(LevelBlock) * b->blocks.size(), hipMemcpyHostToDevice, s));
  }
  if (!b->groups.empty()) {
    BATCH_TRY(hipMemcpyAsync(w + b->blob_off, b->blobs.data(), b->blobs.size(), hipMemcpyHostToDevice, s));
    BATCH_TRY(hipMemcpyAsync(w + b->group_off, b->groups.data(), sizeof(BatchGroup) * b->groups.size(), hipMemcpyHostToDevice, s));
  }
  // each network's batch counter and slice-id list: 0 (one slice, id 0)
  for (int j = 0; j < b->n_nets; j++) {
    const Ctx c = ctxs[(size_t)j];
    BATCH_TRY(launch_fill(c.ws + c.counter_off, 8, s));
    BATCH_TRY(launch_fill(c.ws + c.sid_off, 8, s));
  }
  auto it = b->graphs.find(base);
  if (it != b->graphs.end()) {
    batch_drop(it->second);
    b->graphs.erase(it);
  }
  if (b->graphs.size() >= tn_plan_s::kMaxGraphs) {
    auto lru = b->graphs.begin();
    for (auto j = b->graphs.begin(); j != b->graphs.end(); ++j)
      if (j->second.last_use < lru->second.last_use) lru = j;
    batch_drop(lru->second);
    b->graphs.erase(lru);
  }
  // capture: the groups, then level by level the medium contractions' launch
  // beside the large ops on parallel branches (a level's ops are independent;
  // the graph may run the branches concurrently), joined before the next level
  hipStream_t cs[kBranches] = {};
  hipEvent_t fork[kBranches] = {}, join[kBranches] = {};
  hipError_t e = hipSuccess;
  for (int i = 0; i < kBranches && e == hipSuccess; i++) {
    e = hipStreamCreateWithFlags(&cs[i], hipStreamNonBlocking);
    if (e == hipSuccess) e = hipEventCreateWithFlags(&fork[i], hipEventDisableTiming);
    if (e == hipSuccess) e = hipEventCreateWithFlags(&join[i], hipEventDisableTiming);
  }
  if (e == hipSuccess) e = hipStreamBeginCapture(cs[0], hipStreamCaptureModeThreadLocal);
  const int N = b->n_nets;
  if (e == hipSuccess && !b->groups.empty()) {
    CMEM const Ctx* dctx = reinterpret_cast<CMEM const Ctx*>(base + b->ctx_off);
    CMEM const BatchGroup* dgrp = reinterpret_cast<CMEM const BatchGroup*>(base + b->group_off);
    const dim3 grid((unsigned)b->groups.size()), block(b->group_threads);
    if (b->prec == TN_C128) hipLaunchKernelGGL(tiny_batch_kernel<double>, grid, block, b->group_lds, cs[0], base, dctx, dgrp);
    else hipLaunchKernelGGL(tiny_batch_kernel<float>, grid, block, b->group_lds, cs[0], base, dctx, dgrp);
    e = hipGetLastError();
  }
  for (int l = 0; l < b->n_levels && e == hipSuccess; l++) {
    CMEM const Ctx* dctx = reinterpret_cast<CMEM const Ctx*>(base + b->ctx_off);
    CMEM const LevelOp* dops = reinterpret_cast<CMEM const LevelOp*>(base + b->ops_off);
    const uint32_t first = b->level_block[(size_t)l], n = b->level_block[(size_t)l + 1] - first;
    CMEM const LevelBlock* dblk = reinterpret_cast<CMEM const LevelBlock*>(base + b->blocks_off) + first;
    bool large = false;
    for (int j = 0; j < N; j++) large = large || !b->big[(size_t)l][(size_t)j].empty();
    // the large ones on the other branches, beside the medium ones' launch
    for (int i = 1; i < kBranches && e == hipSuccess && large; i++) {
      e = hipEventRecord(fork[i], cs[0]);
      if (e == hipSuccess) e = hipStreamWaitEvent(cs[i], fork[i], 0);
    }
    if (n > 0 && e == hipSuccess) {
      if (b->prec == TN_C128) hipLaunchKernelGGL(level_kernel<double>, dim3(n), dim3(kLevelThreads), 0, cs[0], dctx, dops, dblk);
      else hipLaunchKernelGGL(level_kernel<float>, dim3(n), dim3(kLevelThreads), 0, cs[0], dctx, dops, dblk);
      e = hipGetLastError();
    }
    int at = 0;
    for (int j = 0; j < N && e == hipSuccess; j++) {
      if (b->big[(size_t)l][(size_t)j].empty()) continue;
      hipStream_t branch = cs[n > 0 ? 1 + at % (kBranches - 1) : at % kBranches];
      at++;
      for (const Op& op : b->big[(size_t)l][(size_t)j]) {
        e = launch_op(b->prec, ctxs[(size_t)j], op, branch);
        if (e != hipSuccess) break;
      }
    }
    for (int i = 1; i < kBranches && e == hipSuccess && large; i++) {
      e = hipEventRecord(join[i], cs[i]);
      if (e == hipSuccess) e = hipStreamWaitEvent(cs[0], join[i], 0);
    }
  }
  hipGraph_t graph = nullptr;
  hipError_t e2 = cs[0] ? hipStreamEndCapture(cs[0], &graph) : hipErrorInvalidValue;
  for (int i = 0; i < kBranches; i++) {
    if (cs[i]) (void)hipStreamDestroy(cs[i]);
    if (fork[i]) (void)hipEventDestroy(fork[i]);
    if (join[i]) (void)hipEventDestroy(join[i]);
  }
  if (e != hipSuccess || e2 != hipSuccess) {
    if (graph) (void)hipGraphDestroy(graph);
    return set_error(TN_E_DEVICE, std::string("batch capture: ") + hipGetErrorString(e != hipSuccess ? e : e2));
  }
  hipGraphExec_t exec = nullptr;
  e = hipGraphInstantiate(&exec, graph, nullptr, nullptr, 0);
  (void)hipGraphDestroy(graph);
  if (e != hipSuccess) return set_error(TN_E_DEVICE, std::string("hipGraphInstantiate: ") + hipGetErrorString(e));
  hipEvent_t done = nullptr;
  e = hipEventCreateWithFlags(&done, hipEventDisableTiming);
  if (e != hipSuccess) {
    (void)hipGraphExecDestroy(exec);
    return set_error(TN_E_DEVICE, std::string("hipEventCreateWithFlags: ") + hipGetErrorString(e));
  }
  tn_plan_s::GraphEntry ent;
  ent.exec = exec;
  ent.done = done;
  ent.last_use = ++b->clock;
  b->graphs[base] = ent;
  return TN_OK;
}

extern "C" int tn_batch_contract(tn_batch_t b, const void* const* leaves, void* const* outs, void* workspace,
                                 uint64_t workspace_bytes, void* stream) {
  if (!b) return set_error(TN_E_INVALID, "batch is null");
  std::lock_guard<std::mutex> lk(b->mu);
  if (!leaves || !outs) return set_error(TN_E_INVALID, "leaves or outs is null");
  if (!workspace || workspace_bytes < b->ws_bytes)
    return set_error(TN_E_WORKSPACE, "workspace of " + std::to_string(b->ws_bytes) + " bytes required");
  const uint64_t base = reinterpret_cast<uint64_t>(workspace);
  auto it = b->graphs.find(base);
  if (it == b->graphs.end()) return set_error(TN_E_WORKSPACE, "workspace not prepared (tn_batch_prepare)");
  std::vector<uint64_t> tab((size_t)b->ptr_stride * b->n_nets, 0);
  size_t li = 0;
  for (int j = 0; j < b->n_nets; j++) {
    uint64_t* t = &tab[(size_t)b->ptr_stride * j];
    for (int v = 0; v < b->n_leaves[(size_t)j]; v++, li++) {
      if (!leaves[li]) return set_error(TN_E_INVALID, "leaf pointer " + std::to_string(li) + " is null");
      t[v] = reinterpret_cast<uint64_t>(leaves[li]);
    }
    if (!outs[j]) return set_error(TN_E_INVALID, "output " + std::to_string(j) + " is null");
    t[b->n_leaves[(size_t)j]] = reinterpret_cast<uint64_t>(outs[j]);
  }
  hipStream_t s = static_cast<hipStream_t>(stream);
  BATCH_TRY(hipMemcpyAsync(static_cast<char*>(workspace) + b->ptr_off, tab.data(), tab.size() * 8,
                           hipMemcpyHostToDevice, s));
  it->second.last_use = ++b->clock;
  BATCH_TRY(hipGraphLaunch((hipGraphExec_t)it->second.exec, s));
  BATCH_TRY(hipEventRecord((hipEvent_t)it->second.done, s));
  return TN_OK;
}

extern "C" void tn_batch_destroy(tn_batch_t b) {
  if (!b) return;
  {
    std::lock_guard<std::mutex> lk(b->mu);
    for (auto& kv : b->graphs) batch_drop(kv.second);
    b->graphs.clear();
  }
  delete b;
}
