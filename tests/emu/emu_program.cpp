// Runs the planner's forward and reverse programs op by op on the host, as a
// simulation of what their launches read and write (not of the kernels'
// arithmetic, which is done in double): every arena byte starts as NaN, a
// launch's operands are all read before any of its results is written, and
// the partial sums of split contractions overwrite their whole buffer.  An op
// that is launched before the op whose value it reads, or a buffer whose
// memory is given away too early, shows up as NaN or a wrong value.
//
//   emu_program net.txt leaves.bin out.bin
//
// net.txt: as in the test (network, tree, sliced indices, slice ids, leaves to
// differentiate, options); leaves.bin: the leaves and the output cotangent,
// complex128; out.bin: the sum of the root values, then the gradients.
#include <cmath>
#include <complex>
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <functional>
#include <limits>
#include <string>
#include <vector>

#include "plan.h"

using namespace tn;
typedef std::complex<double> Z;

static int g_eb;                          // bytes of a stored value
static std::vector<char> g_arena;         // of one slice
static std::vector<std::vector<Z>> g_slot;
static int64_t g_sid;

// One operand: an arena range (rounded to the storage type) or a slot of values.
struct Mem {
  char* arena = nullptr;
  std::vector<Z>* slot = nullptr;
  uint64_t off = 0;
  int eb = 0;
  Z get(uint64_t i) const {
    if (slot) return slot->at(off + i);
    check(i);
    if (eb == 8) return Z(reinterpret_cast<float*>(arena)[2 * i], reinterpret_cast<float*>(arena)[2 * i + 1]);
    return Z(reinterpret_cast<double*>(arena)[2 * i], reinterpret_cast<double*>(arena)[2 * i + 1]);
  }
  void set(uint64_t i, Z v) const {
    if (slot) { slot->at(off + i) = v; return; }
    check(i);
    if (eb == 8) {
      reinterpret_cast<float*>(arena)[2 * i] = (float)v.real();
      reinterpret_cast<float*>(arena)[2 * i + 1] = (float)v.imag();
    } else {
      reinterpret_cast<double*>(arena)[2 * i] = v.real();
      reinterpret_cast<double*>(arena)[2 * i + 1] = v.imag();
    }
  }
  void check(uint64_t i) const {
    if (arena + (i + 1) * eb > g_arena.data() + g_arena.size()) {
      fprintf(stderr, "arena access out of range\n");
      exit(5);
    }
  }
};

static Mem at(const Ref& r, int eb = 0) {
  Mem m;
  m.eb = eb ? eb : g_eb;
  if (r.kind == 1) {
    m.arena = g_arena.data() + r.off;
    return m;
  }
  m.slot = &g_slot.at((size_t)r.slot);
  for (int i = 0; i < r.n_slice; i++) m.off |= uint64_t((g_sid >> r.slice_bit[i]) & 1) << r.slice_pos[i];
  return m;
}

static Mem arena_at(uint64_t off) {
  Ref r{};
  r.kind = 1;
  r.off = (int64_t)off;
  return at(r);
}

static uint64_t place(uint64_t v, const int8_t* pos, int n) {
  uint64_t o = 0;
  for (int i = 0; i < n; i++)
    if (pos[i] >= 0) o |= ((v >> i) & 1) << pos[i];
  return o;
}

static Z cj(Z v, int c) { return c ? std::conj(v) : v; }

typedef std::vector<std::function<void()>> Writes;

static void row(const RowOp& r, Writes& w) {
  const int ks = r.k_split_bits > 0 ? r.k_split_bits : 0;
  for (uint64_t o = 0; o < (uint64_t(1) << r.n_rows); o++)
    for (uint64_t j = 0; j < (uint64_t(1) << r.n_in); j++) {
      const uint64_t a0 = place(o, r.row_a, r.n_rows);
      const uint64_t b0 = place(o, r.row_b, r.n_rows) + place(j, r.in_b, r.n_in);
      const uint64_t c = place(o, r.row_c, r.n_rows) + place(j, r.in_c, r.n_in);
      Z s = 0;
      for (uint64_t k = 0; k < (uint64_t(1) << r.n_k); k++)
        s += cj(at(r.a).get(a0 + place(k, r.k_a, r.n_k)), r.conj_a) * cj(at(r.b).get(b0 + place(k, r.k_b, r.n_k)), r.conj_b);
      if (r.accumulate) s += at(r.c).get(c);
      const uint64_t p = ((o << r.n_in) + j) << ks;
      if (ks) {
        const Mem m = at(r.part);
        w.push_back([=] { for (uint64_t i = 0; i < (uint64_t(1) << ks); i++) m.set(p + i, i ? Z(0) : s); });
      } else {
        const Mem m = at(r.c);
        w.push_back([=] { m.set(c, s); });
      }
    }
}

static void reduce(const RowOp& r, Writes& w) {
  for (uint64_t o = 0; o < (uint64_t(1) << r.n_rows); o++)
    for (uint64_t j = 0; j < (uint64_t(1) << r.n_in); j++) {
      Z s = 0;
      for (uint64_t i = 0; i < (uint64_t(1) << r.k_split_bits); i++)
        s += at(r.part).get((((o << r.n_in) + j) << r.k_split_bits) + i);
      const Mem m = at(r.c);
      const uint64_t c = place(o, r.row_c, r.n_rows) + place(j, r.in_c, r.n_in);
      w.push_back([=] { m.set(c, s); });
    }
}

static void gemm(const GemmOp& g, Writes& w) {
  if (g.k_split_bits > 0) {
    const Mem p = at(g.part);
    const uint64_t n = uint64_t(1) << (g.n_h + g.n_m + g.n_n + g.k_split_bits);
    w.push_back([=] { for (uint64_t i = 0; i < n; i++) p.set(i, Z(NAN, NAN)); });
  }
  for (uint64_t h = 0; h < (uint64_t(1) << g.n_h); h++)
    for (uint64_t m = 0; m < (uint64_t(1) << g.n_m); m++)
      for (uint64_t n = 0; n < (uint64_t(1) << g.n_n); n++) {
        const uint64_t a0 = place(h, g.a_h, g.n_h) + place(m, g.a_m, g.n_m);
        const uint64_t b0 = place(h, g.b_h, g.n_h) + place(n, g.b_n, g.n_n);
        const uint64_t c = place(h, g.c_h, g.n_h) + place(m, g.c_m, g.n_m) + place(n, g.c_n, g.n_n);
        Z s = 0;
        for (uint64_t k = 0; k < (uint64_t(1) << g.n_k); k++)
          s += cj(at(g.a).get(a0 + place(k, g.a_k, g.n_k)), g.conj_a) * cj(at(g.b).get(b0 + place(k, g.b_k, g.n_k)), g.conj_b);
        if (g.accumulate) s += at(g.c).get(c);
        const Mem m2 = at(g.c);
        w.push_back([=] { m2.set(c, s); });
      }
}

static void permute(const PermuteOp& p, Writes& w) {
  for (uint64_t i = 0; i < (uint64_t(1) << p.n_bits); i++) {
    Z v = at(p.src, p.src_c128 ? 16 : 8).get(place(i, p.src_pos, p.n_bits));
    const Mem d = at(p.dst, p.dst_c128 ? 16 : 8);
    const uint64_t o = place(i, p.dst_pos, p.n_bits);
    const bool acc = p.accumulate != 0;
    w.push_back([=] { d.set(o, acc ? d.get(o) + v : v); });
  }
}

template <typename S>
static S read(const std::vector<char>& blob, size_t off) {
  S s;
  std::memcpy(&s, blob.data() + off, sizeof s);
  return s;
}

static uint64_t nibbles(uint64_t v, uint64_t list, int n) {
  uint64_t o = 0;
  for (int i = 0; i < n; i++) {
    const int p = (list >> (4 * i)) & 15;
    if (p != kTinyAbsent) o |= ((v >> i) & 1) << p;
  }
  return o;
}

static void tiny(const TinyLaunch& L, Writes& w) {
  for (uint32_t g = 0; g < L.n_groups; g++) {
    const TinyDir d = read<TinyDir>(L.blob, g * sizeof(TinyDir));
    std::vector<Z> lds((L.lds_bytes - 16 * d.tab_units) / g_eb, Z(NAN, NAN));
    for (uint32_t i = 0; i < d.n_loads; i++) {
      const TinyLoad ld = read<TinyLoad>(L.blob, d.ld_off + i * sizeof(TinyLoad));
      for (uint64_t e = 0; e < (uint64_t(1) << ld.n_bits); e++) {
        Z v;
        if (ld.kind == 2) {
          const TinyExt x = read<TinyExt>(L.blob, d.ext_off + ld.src * sizeof(TinyExt));
          v = at(x.ref).get(place(e, x.pos, ld.n_bits));
        } else if (ld.kind == 1) {
          v = arena_at(256 * uint64_t(ld.src)).get(e);
        } else {
          v = g_slot.at(ld.src).at(e);
        }
        lds.at(ld.lds + e) = v;
      }
    }
    for (uint32_t l = 0; l < d.n_levels; l++) {
      const TinyLevel lev = read<TinyLevel>(L.blob, d.tab_off + l * sizeof(TinyLevel));
      std::vector<std::pair<size_t, Z>> stores;            // of the level, after all its reads
      uint32_t begin = 0;
      for (int c = 0; c < kTinyClasses; c++) {
        const uint32_t count = (lev.end[c] - begin) >> (kTinyMaxThreadBits - c - 2);
        begin = lev.end[c];
        for (uint32_t j = 0; j < count; j++) {
          const TinyOp t = read<TinyOp>(L.blob, d.tab_off + d.ops_off + (lev.first[c] + j) * sizeof(TinyOp));
          for (uint64_t o = 0; o < (uint64_t(1) << t.n_out); o++) {
            Z s = 0;
            for (uint64_t k = 0; k < (uint64_t(1) << t.n_k); k++)
              s += cj(lds.at(t.a + nibbles(o, t.oa, t.n_out) + nibbles(k, t.ka, t.n_k)), t.conj & 1) *
                   cj(lds.at(t.b + nibbles(o, t.ob, t.n_out) + nibbles(k, t.kb, t.n_k)), t.conj & 2);
            if (t.lds_c) stores.push_back({t.c + o, s});
            if (t.dst_kind) {
              const Mem m = arena_at(256 * uint64_t(t.dst));
              w.push_back([=] { m.set(o, s); });
            }
          }
        }
      }
      for (auto& x : stores) lds.at(x.first) = x.second;
    }
  }
}

static void scatter(const TinyLaunch& L, Writes& w) {
  for (uint32_t g = 0; g < L.n_groups; g++) {
    const ScatterEntry e = read<ScatterEntry>(L.blob, g * sizeof(ScatterEntry));
    uint64_t off = 0;
    for (int j = 0; j < e.n_slice; j++) off |= uint64_t((g_sid >> e.slice_bit[j]) & 1) << e.slice_pos[j];
    for (uint64_t i = 0; i < (uint64_t(1) << e.n_bits); i++) {
      uint64_t to = off;
      for (int j = 0; j < e.n_bits; j++) to |= ((i >> j) & 1) << e.pos[j];
      const Z v = arena_at(256 * uint64_t(e.src)).get(i);
      std::vector<Z>* s = &g_slot.at(e.slot);
      w.push_back([=] { s->at(to) += v; });
    }
  }
}

static int run(const std::vector<Op>& prog, uint64_t bytes) {
  g_arena.assign((size_t)bytes, 0);
  const double nan = std::numeric_limits<double>::quiet_NaN();
  const float nanf = std::numeric_limits<float>::quiet_NaN();
  for (size_t i = 0; i + g_eb / 2 <= g_arena.size(); i += g_eb / 2) {
    if (g_eb == 8) std::memcpy(g_arena.data() + i, &nanf, 4);
    else std::memcpy(g_arena.data() + i, &nan, 8);
  }
  for (const Op& op : prog) {
    Writes w;
    switch (op.kind) {
      case OpKind::Row: row(op.row, w); break;
      case OpKind::RowReduce: reduce(op.row, w); break;
      case OpKind::Gemm: gemm(op.gemm, w); break;
      case OpKind::Permute: permute(op.perm, w); break;
      case OpKind::Tiny: tiny(*op.tiny, w); break;
      case OpKind::Scatter: scatter(*op.tiny, w); break;
      default: return 4;
    }
    for (auto& f : w) f();
  }
  return 0;
}

template <typename T>
static std::vector<T> list(FILE* f) {
  long n = 0, x;
  if (fscanf(f, "%ld", &n) != 1) exit(1);
  std::vector<T> v;
  for (long i = 0; i < n; i++) {
    if (fscanf(f, "%ld", &x) != 1) exit(1);
    v.push_back((T)x);
  }
  return v;
}

int main(int argc, char** argv) {
  if (argc != 4) return 1;
  FILE* f = fopen(argv[1], "r");
  if (!f) return 1;
  tn_plan_s p;
  p.rank = list<int32_t>(f);
  p.leaf_idx = list<int64_t>(f);
  p.idx_dim = list<int64_t>(f);
  p.out_idx = list<int64_t>(f);
  p.left = list<int32_t>(f);
  p.right = list<int32_t>(f);
  p.sliced = list<int64_t>(f);
  const std::vector<int64_t> ids = list<int64_t>(f);
  const std::vector<int32_t> wrt = list<int32_t>(f);
  const std::vector<int32_t> opt = list<int32_t>(f);       // precision, flags, group_small[, slices in flight: list the row ops only]
  fclose(f);
  const int nl = p.n_leaves = (int)p.rank.size();
  p.n_idx = (int)p.idx_dim.size();
  p.n_out = (int)p.out_idx.size();
  p.n_sliced = (int)p.sliced.size();
  p.prec = opt[0];
  p.opt.prec = opt[0];
  p.opt.flags = opt[1];
  p.group_small = opt[2] != 0;
  if (opt.size() > 3) p.opt.max_inflight_slices = opt[3];
  g_eb = p.elem_bytes = p.prec == TN_C128 ? 16 : 8;
  std::string err;
  if (build_plan(&p, err) || (!wrt.empty() && build_backward(&p, wrt, err))) {
    fprintf(stderr, "plan: %s\n", err.c_str());
    return 2;
  }
  if (opt.size() > 3) {                                    // row ops: reverse, rows, in-thread, summed, chunk bits
    for (int rev = 0; rev < 2; rev++)
      for (const Op& op : rev ? p.bwd : p.fwd)
        if (op.kind == OpKind::Row)
          printf("%d %d %d %d %d\n", rev, op.row.n_rows, op.row.n_in, op.row.n_k, op.row.k_split_bits);
    return 0;
  }
  g_slot.resize((size_t)p.n_slots);
  FILE* in = fopen(argv[2], "rb");
  if (!in) return 1;
  size_t at_idx = 0;
  auto fill = [&](std::vector<Z>& v, size_t n) {
    v.resize(n);
    if (fread(v.data(), 16, n, in) != n) exit(1);
  };
  std::vector<size_t> size(nl, 1);
  for (int v = 0; v < nl; v++) {
    for (int i = 0; i < p.rank[v]; i++) size[v] *= (size_t)p.idx_dim[p.leaf_idx[at_idx++]];
    fill(g_slot[v], size[v]);
  }
  size_t outs = 1;
  for (int64_t e : p.out_idx) outs *= (size_t)p.idx_dim[e];
  fill(g_slot[p.slot_gout], outs);
  fclose(in);
  for (size_t i = 0; i < wrt.size(); i++) g_slot[p.slot_grad0 + i].assign(size[wrt[i]], Z(0));
  std::vector<Z> total(outs, Z(0));
  for (int64_t sid : ids) {
    g_sid = sid;
    if (run(p.fwd, p.arena_bytes)) return 4;
    for (size_t i = 0; i < outs; i++) total[i] += arena_at((uint64_t)p.root_off).get(i);
    if (!wrt.empty() && run(p.bwd, p.bwd_arena_bytes)) return 4;
  }
  FILE* fo = fopen(argv[3], "wb");
  fwrite(total.data(), 16, outs, fo);
  for (size_t i = 0; i < wrt.size(); i++) fwrite(g_slot[p.slot_grad0 + i].data(), 16, size[wrt[i]], fo);
  fclose(fo);
  return 0;
}
