// Collects the small contractions of a program into launches of the
// small-contraction kernel (tiny.h).  Included by plan.cpp inside namespace tn,
// after Prog.
#pragma once

// Largest contraction a group takes: log2 of outputs x summed values, and of
// the values of an operand or output.  A workgroup of 512 threads does 2^12
// multiply-adds in eight steps, well under the ~5 us a launch of its own
// costs; above that, the launch spreads the work over many compute units.
constexpr int kTinyWorkBits = 12;
constexpr int kTinyTensorBits = 10;
constexpr int kTinyGroupOps = 170;         // contractions of one group (tables of that many fit below)
constexpr int kTinyGroupTable = 16384;     // bytes of their table and the levels'
constexpr int kTinyGroupLds = 61440;       // bytes of LDS, tables included

namespace tiny_detail {

// Operand or output of a small contraction: buffer id or leaf slot.
struct Operand {
  bool leaf = false;
  int id = -1;
  Ref ref;
  int n = 0;
  int8_t pos[kTinyTensorBits] = {};  // positions of its bits, ascending
  int lds = 0;                       // LDS element offset
};

struct Item {
  int op = -1;                       // index in the program
  Operand a, b;
  int c = -1, c_lds = 0, n_out = 0, n_k = 0;
  uint64_t oa = 0, ob = 0, ka = 0, kb = 0;
  int conj = 0;
  bool split = false;                // a contraction of the split-K kernel
  int group = -1, stage = 0, level = 0;
};

inline int rank_of(const Operand& o, int p) {
  for (int i = 0; i < o.n; i++)
    if (o.pos[i] == p) return i;
  return kTinyAbsent;
}

// Fills `it` from a contraction op; false when the op is not a small one.
// Without `splits`, contractions of the split-K kernel are left to it.
inline bool describe(const Op& op, bool splits, Item& it) {
  if (op.kind != OpKind::Row) return false;
  const RowOp& r = op.row;
  if (r.accumulate || (r.k_split_bits >= 0 && !splits)) return false;
  const int n_out = r.n_rows + r.n_in, n_k = r.n_k;
  if (n_out + n_k > kTinyWorkBits || n_out > kTinyTensorBits) return false;
  if (r.c.kind != 1 || r.a.kind == 2 || r.b.kind == 2) return false;
  int8_t ca[kMaxBits], cb[kMaxBits], ka[kMaxBits], kb[kMaxBits];   // by position in C / summed bit
  for (int i = 0; i < r.n_rows; i++) { ca[r.row_c[i]] = r.row_a[i]; cb[r.row_c[i]] = r.row_b[i]; }
  for (int i = 0; i < r.n_in; i++) { ca[r.in_c[i]] = -1; cb[r.in_c[i]] = r.in_b[i]; }
  for (int i = 0; i < n_k; i++) { ka[i] = r.k_a[i]; kb[i] = r.k_b[i]; }
  it.split = r.k_split_bits >= 0;
  it.conj = (r.conj_a ? 1 : 0) | (r.conj_b ? 2 : 0);
  auto operand = [&](const Ref& ref, const int8_t* c, const int8_t* k, Operand& o, uint64_t& on, uint64_t& kn) {
    o.leaf = ref.kind == 0;
    o.id = o.leaf ? ref.slot : (int)ref.off;
    o.ref = ref;
    int n = n_k;
    for (int i = 0; i < n_out; i++) n += c[i] >= 0;
    if (n > kTinyTensorBits) return false;
    for (int i = 0; i < n_out; i++) if (c[i] >= 0) o.pos[o.n++] = c[i];
    for (int i = 0; i < n_k; i++) o.pos[o.n++] = k[i];
    std::sort(o.pos, o.pos + o.n);
    for (int i = 0; i < n_out; i++) on |= uint64_t(c[i] < 0 ? kTinyAbsent : rank_of(o, c[i])) << (4 * i);
    for (int i = 0; i < n_k; i++) kn |= uint64_t(rank_of(o, k[i])) << (4 * i);
    return true;
  };
  it.n_out = n_out;
  it.n_k = n_k;
  it.c = (int)r.c.off;
  return operand(r.a, ca, ka, it.a, it.oa, it.ka) && operand(r.b, cb, kb, it.b, it.ob, it.kb);
}

// Threads per output (log2).  A sum that the row kernel would run in index
// order stays one thread's (at most 32 values unless rows are many): grouping
// does not change its rounding.  The longer sums of the split-K kernel (at most
// 2^10 values, operands being that small) are shared by threads of one
// wavefront, 2^2 to 2^4 values each.
inline int split_bits(const Item& it) {
  if (!it.split) return 0;
  return std::max(0, std::min(std::min(it.n_k - 2, 6), kTinyMaxThreadBits - it.n_out));
}
inline int thread_bits(const Item& it) {
  return std::min(kTinyMaxThreadBits, std::max(kTinyMinThreadBits, it.n_out + split_bits(it)));
}

}  // namespace tiny_detail

// Buffers an op reads and writes (buffer ids).  A split row op counts as
// writing C too, so that C never shares memory with its operands: a batch runs
// the op and its reduce pass as one contraction.
template <typename F>
static void op_refs(Op& op, F&& f) {
  switch (op.kind) {
    case OpKind::Row: f(op.row.a, false); f(op.row.b, false); if (op.row.k_split_bits > 0) f(op.row.part, true); f(op.row.c, true); break;
    case OpKind::RowReduce: f(op.row.part, false); f(op.row.c, true); break;
    case OpKind::Gemm: f(op.gemm.a, false); f(op.gemm.b, false); if (op.gemm.k_split_bits > 0) f(op.gemm.part, true); f(op.gemm.c, true); break;
    case OpKind::Accum: f(op.accum.src, false); break;
    case OpKind::Permute: f(op.perm.src, false); f(op.perm.dst, true); break;
    case OpKind::Split: f(op.split.src, false); f(op.split.dst, true); break;
    default: break;
  }
}

// `prog` with its small contractions grouped.  `root_buf`: buffer of
// the root value (read after the program).  Only the op order and the buffer
// lifetimes change; every value is computed from the same operands.
static Prog group_small(const tn_plan_s* p, Prog& prog, int root_buf) {
  using namespace tiny_detail;
  // complex64 forward values keep the rounding of the split-K kernel's
  // butterfly, so that sums over slices do not depend on the grouping
  const bool splits = p->prec == TN_C128 || root_buf < 0;
  const int nops = (int)prog.ops.size(), nbuf = (int)prog.bufs.size();
  std::vector<Item> item(nops);
  std::vector<char> small(nops, 0), dropped(nops, 0);
  for (int i = 0; i < nops; i++) {
    item[i].op = i;
    small[i] = describe(prog.ops[i], splits, item[i]);
  }
  std::vector<int> producer(nbuf, -1);                   // op that completes each buffer
  std::vector<std::vector<int>> readers(nbuf);
  for (int i = 0; i < nops; i++) {
    if (prog.ops[i].kind == OpKind::RowReduce && i > 0 && small[i - 1]) { dropped[i] = 1; continue; }
    op_refs(prog.ops[i], [&](Ref& r, bool w) {
      if (r.kind != 1) return;
      if (w) producer[(size_t)r.off] = i;
      else readers[(size_t)r.off].push_back(i);
    });
    if (small[i]) producer[(size_t)item[i].c] = i;
  }
  std::vector<int> rep(nops);
  std::vector<std::vector<int>> members;                   // per group, program order
  std::vector<uint32_t> lds_elems;
  // values by key: buffers, then leaves; `seen` marks those of the group at hand
  auto key_of = [&](const tiny_detail::Operand& o) { return o.leaf ? nbuf + o.id : o.id; };
  struct Val { int size = 0, first = 0, last = 0, lds = 0; };
  std::vector<Val> vals((size_t)nbuf + p->n_leaves);
  std::vector<int> seen((size_t)nbuf + p->n_leaves, -1);
  int mark = 0;
  auto find = [&](int x) { while (rep[x] != x) x = rep[x] = rep[rep[x]]; return x; };
  auto inputs = [&](int i, auto&& f) {
    if (small[i]) {
      for (const tiny_detail::Operand* o : {&item[i].a, &item[i].b}) if (!o->leaf) f(producer[o->id]);
    } else if (!dropped[i]) {
      op_refs(prog.ops[i], [&](Ref& r, bool w) { if (r.kind == 1 && !w) f(producer[(size_t)r.off]); });
    }
  };
  std::vector<int> stage(nops, 0);
  // Groups: small contractions connected through values they pass on, with no
  // other op in between (`stage` counts the alternations, so no path leaves a
  // group and returns to it).  A group that exceeds the limits is cut: a
  // contraction with too many others below it (forward) or the readers of one
  // with too many above it (reverse) start groups of the next stage.  A pass
  // cuts every group at all places, so that a few passes do for any length.
  std::vector<char> cut(nops, 0);
  for (;;) {
    for (int i = 0; i < nops; i++) rep[i] = i;
    for (int i = 0; i < nops; i++) {
      int s = 0;
      inputs(i, [&](int q) { if (q >= 0) s = std::max(s, stage[q] + (small[i] && (!small[q] || cut[i]) ? 1 : 0)); });
      // the partial sums of a split op are read by the op behind it
      if (prog.ops[i].kind == OpKind::RowReduce && !dropped[i]) s = std::max(s, stage[i - 1]);
      stage[i] = s;
      if (small[i]) {
        int lev = 0;
        inputs(i, [&](int q) {
          if (q >= 0 && small[q] && stage[q] == s) { rep[find(q)] = find(i); lev = std::max(lev, item[q].level + 1); }
        });
        item[i].level = lev;
      }
    }
    members.clear();
    std::vector<int> ids(nops, -1);
    for (int i = 0; i < nops; i++)
      if (small[i]) {
        int& id = ids[(size_t)find(i)];
        if (id < 0) {
          id = (int)members.size();
          members.emplace_back();
        }
        item[i].group = id;
        members[(size_t)item[i].group].push_back(i);
      }
    lds_elems.assign(members.size(), 0);
    bool fits = true;
    std::vector<int> below(nops, 0), above(nops, 0);
    for (size_t g = 0; g < members.size(); g++) {
      // LDS offsets from lifetimes in levels (first fit): loads live from the
      // start, outputs from their level, until their last reading level
      std::vector<int> keys;
      int levels = 0, ext = 0;
      mark++;
      for (int i : members[g]) {
        levels = std::max(levels, item[i].level + 1);
        for (const tiny_detail::Operand* o : {&item[i].a, &item[i].b}) {
          const int k = key_of(*o);
          if (seen[k] != mark) {
            seen[k] = mark;
            keys.push_back(k);
            vals[k] = Val{1 << o->n, -1, 0, 0};
            ext++;
          }
          vals[k].last = std::max(vals[k].last, item[i].level);
        }
        seen[item[i].c] = mark;
        keys.push_back(item[i].c);
        vals[item[i].c] = Val{1 << item[i].n_out, item[i].level, item[i].level, 0};
      }
      std::vector<std::vector<int>> born((size_t)levels + 1), dies((size_t)levels + 1);
      for (int k : keys) { born[(size_t)(vals[k].first + 1)].push_back(k); dies[(size_t)(vals[k].last + 1)].push_back(k); }
      std::vector<std::pair<int, int>> used;               // (offset, size), ascending
      int peak = 0;
      for (int t = 0; t <= levels; t++) {
        for (int k : born[(size_t)t]) {
          const int sz = (vals[k].size + 3) / 4 * 4;
          int cur = 0;
          size_t at = 0;
          for (; at < used.size() && used[at].first - cur < sz; at++) cur = used[at].first + used[at].second;
          used.insert(used.begin() + at, {cur, sz});
          vals[k].lds = cur;
          peak = std::max(peak, cur + sz);
        }
        for (int k : dies[(size_t)t])
          used.erase(std::lower_bound(used.begin(), used.end(), std::make_pair(vals[k].lds, 0)));
      }
      for (int i : members[g]) {
        item[i].a.lds = vals[key_of(item[i].a)].lds;
        item[i].b.lds = vals[key_of(item[i].b)].lds;
        item[i].c_lds = vals[item[i].c].lds;
      }
      lds_elems[g] = (uint32_t)peak;
      const int table = (levels * (int)sizeof(TinyLevel) + 15) / 16 * 16 + (int)(members[g].size() * sizeof(TinyOp));
      const int loads = ext * (int)(sizeof(TinyLoad) + sizeof(TinyExt));
      if (members[g].size() <= (size_t)kTinyGroupOps && table <= kTinyGroupTable &&
          table + loads + 64 <= kTinyBlobLarge && table + 64 + peak * p->elem_bytes <= kTinyGroupLds)
        continue;
      fits = false;
      // cut into parts of at most `limit` contractions (half, where LDS or the
      // tables are the limit): counting from the inputs, then from the readers
      const int size = (int)members[g].size(), limit = size > kTinyGroupOps ? kTinyGroupOps : std::max(1, size / 2);
      bool done = false;
      for (int i : members[g]) {
        below[i] = 1;
        inputs(i, [&](int q) { if (q >= 0 && small[q] && item[q].group == (int)g) below[i] = std::min(below[i] + below[q], size + 1); });
        if (below[i] > limit && !cut[i]) {
          cut[i] = 1;
          below[i] = 1;
          done = true;
        }
      }
      if (!done)
        for (auto r = members[g].rbegin(); r != members[g].rend(); ++r) {
          const int i = *r;
          above[i] = 1;
          for (int q : readers[item[i].c])
            if (small[q] && item[q].group == (int)g && !cut[q]) above[i] = std::min(above[i] + above[q], size + 1);
          if (above[i] <= limit) continue;
          for (int q : readers[item[i].c])
            if (small[q] && item[q].group == (int)g && !cut[q]) { cut[q] = 1; done = true; }
          above[i] = 1;
        }
      if (!done) {
        std::vector<int> open;
        for (int i : members[g])
          if (!cut[i]) open.push_back(i);
        for (size_t i = open.size() / 2; i < open.size(); i++) { cut[open[i]] = 1; done = true; }
      }
      if (!done) {                                       // cannot be cut: its last contraction is launched by itself
        const int i = members[g].back();
        small[i] = 0;
        if (i + 1 < nops && dropped[i + 1]) {            // with its reduce pass
          dropped[i + 1] = 0;
          producer[(size_t)item[i].c] = i + 1;
        }
      }
    }
    if (fits) break;
  }
  const int G = (int)members.size();
  auto at_end = [&](int i) {                             // copy of a leaf's cotangent into its gradient
    const Op& o = prog.ops[i];
    return o.kind == OpKind::Permute && o.perm.accumulate && o.perm.per_slice_serial && o.perm.n_bits <= kTinyTensorBits;
  };
  // Order of the other ops: the program's, except that an op which reads a
  // group's result comes after all ops that the group waits for.  A group of a
  // reverse program can hold a forward value that an early op reads and, up
  // its connected set, a cotangent that needs a later op.  Groups and ops form
  // no cycle (see `stage`), so a walk that visits inputs first finds the order.
  std::vector<int> others;
  {
    std::vector<char> seen_unit((size_t)nops + G, 0);      // ops, then groups
    std::vector<std::pair<int, bool>> todo;                // unit, inputs done
    for (int i0 = 0; i0 < nops; i0++) {
      if (small[i0] || dropped[i0] || at_end(i0)) continue;
      todo.push_back({i0, false});
      while (!todo.empty()) {
        const auto [u, ready] = todo.back();
        todo.pop_back();
        if (ready) {
          if (u < nops) others.push_back(u);
          continue;
        }
        if (seen_unit[(size_t)u]) continue;
        seen_unit[(size_t)u] = 1;
        todo.push_back({u, true});
        const size_t from = todo.size();
        auto need = [&](int q) {
          if (q < 0) return;
          const int v = small[q] ? nops + item[q].group : q;
          if (v != u && !seen_unit[(size_t)v]) todo.push_back({v, false});
        };
        if (u < nops) inputs(u, need);
        else for (int i : members[(size_t)(u - nops)]) inputs(i, need);
        std::stable_sort(todo.begin() + (int64_t)from, todo.end(), [](auto& x, auto& y) { return x.first > y.first; });
      }
    }
  }
  // Launch positions in the sequence of the other ops (a group at position q
  // runs before the q-th of them): as soon as the external operands are
  // there, or at the end when nothing but gradient copies reads the results.
  std::vector<int> pos(nops, -1);
  int seq = 0;
  for (int i : others) pos[i] = seq++;
  std::vector<int> gpos(G, 0), order(G);
  std::vector<char> has_reader(G, 0);
  for (int g = 0; g < G; g++) {
    order[g] = g;
    for (int i : members[g])
      for (int q : readers[item[i].c]) has_reader[g] |= !(at_end(q)) && !(small[q] && item[q].group == g);
    for (int i : members[g]) has_reader[g] |= item[i].c == root_buf;
  }
  std::stable_sort(order.begin(), order.end(), [&](int x, int y) { return stage[members[x][0]] < stage[members[y][0]]; });
  for (int g : order) {
    int q = 0;
    for (int i : members[g])
      inputs(i, [&](int x) {
        if (x < 0) return;
        if (!small[x]) q = std::max(q, pos[x] + 1);
        else if (item[x].group != g) q = std::max(q, gpos[item[x].group]);
      });
    gpos[g] = has_reader[g] ? q : seq;
  }
  // a group placed at the end that another group reads would have a reader, so
  // groups at one position in stage order respect their dependencies
  std::map<std::pair<int, int>, std::vector<int>> launches;   // (position, stage; one stage at the end)
  for (int g : order) launches[{gpos[g], stage[members[g][0]]}].push_back(g);
  {
    // at the end only values that nobody else reads are computed: one stage
    std::map<std::pair<int, int>, std::vector<int>> merged;
    for (auto& l : launches)
      for (int g : l.second) merged[{l.first.first, has_reader[g] ? l.first.second : 1 << 30}].push_back(g);
    launches.swap(merged);
  }
  Prog out;
  out.bufs = prog.bufs;
  for (Buf& b : out.bufs) b.first = b.last = b.off = -1;
  auto emit = [&](const std::vector<int>& groups) {
    size_t count = 0;
    for (int g : groups) count += members[(size_t)g].size();
    if (count < 2) {                                     // nothing to share: the op as it was
      for (int g : groups)
        for (int i : members[(size_t)g]) {
          out.ops.push_back(prog.ops[i]);
          if (i + 1 < nops && dropped[i + 1]) out.ops.push_back(prog.ops[i + 1]);
        }
      return;
    }
    size_t at = 0;
    while (at < groups.size()) {
      auto L = std::make_shared<TinyLaunch>();
      // as many groups as the largest blob holds
      auto bytes_of = [&](int g) {
        int levels = 0;
        for (int i : members[(size_t)g]) levels = std::max(levels, item[i].level + 1);
        return (int)sizeof(TinyDir) + (levels * (int)sizeof(TinyLevel) + 15) / 16 * 16 +
               (int)(members[(size_t)g].size() * (sizeof(TinyOp) + 2 * (sizeof(TinyLoad) + sizeof(TinyExt)))) + 48;
      };
      size_t end = at;
      int total = 64;
      while (end < groups.size() && (end == at || total + bytes_of(groups[end]) <= kTinyBlobLarge)) total += bytes_of(groups[end++]);
      L->n_groups = (uint32_t)(end - at);
      std::vector<char>& blob = L->blob;
      auto align = [&] { blob.resize((blob.size() + 15) / 16 * 16, 0); };
      auto put = [&](const void* d, size_t n) { blob.insert(blob.end(), (const char*)d, (const char*)d + n); };
      blob.resize(sizeof(TinyDir) * L->n_groups, 0);
      Op op;
      op.kind = OpKind::Tiny;
      uint32_t max_threads = 64, max_lds = 0;
      for (size_t gi = at; gi < end; gi++) {
        const int g = groups[gi];
        std::vector<int> ops = members[(size_t)g];
        std::stable_sort(ops.begin(), ops.end(), [&](int x, int y) {
          if (item[x].level != item[y].level) return item[x].level < item[y].level;
          return thread_bits(item[x]) > thread_bits(item[y]);
        });
        TinyDir d{};
        align();
        d.tab_off = (uint32_t)blob.size();
        d.n_levels = (uint32_t)item[ops.back()].level + 1;
        std::vector<TinyLevel> lev(d.n_levels);
        std::memset(lev.data(), 0, lev.size() * sizeof(TinyLevel));
        size_t j = 0;
        for (uint32_t l = 0; l < d.n_levels; l++) {
          uint32_t units = 0;
          for (int c = 0; c < kTinyClasses; c++) {
            lev[l].first[c] = (uint16_t)j;
            for (; j < ops.size() && item[ops[j]].level == (int)l && thread_bits(item[ops[j]]) == kTinyMaxThreadBits - c; j++)
              units += 1u << (kTinyMaxThreadBits - c - 2);
            lev[l].end[c] = (uint16_t)units;
          }
          while (max_threads < 4 * units && max_threads < 512) max_threads *= 2;
        }
        put(lev.data(), lev.size() * sizeof(TinyLevel));
        align();
        d.ops_off = (uint32_t)blob.size() - d.tab_off;
        std::vector<const tiny_detail::Operand*> ext;
        mark++;
        for (int i : ops) {
          const Item& it = item[i];
          const uint32_t here = (uint32_t)blob.size();
          TinyOp t;
          std::memset(&t, 0, sizeof t);
          auto off = [&](const tiny_detail::Operand& o) {
            const int k = key_of(o);
            if ((o.leaf || !small[producer[o.id]] || item[producer[o.id]].group != g) && seen[k] != mark) {
              seen[k] = mark;
              ext.push_back(&o);
            }
            return (uint16_t)o.lds;
          };
          t.a = off(it.a);
          t.b = off(it.b);
          t.c = (uint16_t)it.c_lds;
          t.n_out = (uint8_t)it.n_out;
          t.n_k = (uint8_t)it.n_k;
          t.ks = (uint8_t)split_bits(it);
          t.conj = (uint8_t)it.conj;
          t.oa = it.oa; t.ob = it.ob; t.ka = it.ka; t.kb = it.kb;
          for (int q : readers[it.c]) {
            if (small[q] && item[q].group == g) t.lds_c = 1;
            else t.dst_kind = 1;
          }
          if (it.c == root_buf) { t.dst_kind = 1; L->root_op = here; }
          if (t.dst_kind) L->writes.push_back({here, it.c});
          put(&t, sizeof t);
          L->nodes.push_back(prog.ops[i].node);
          op.node = prog.ops[i].node;
          op.flops += prog.ops[i].flops;
          op.bytes += prog.ops[i].bytes;
          op.grid_rows += 1;
        }
        d.tab_units = ((uint32_t)blob.size() - d.tab_off) / 16;
        align();
        d.ld_off = (uint32_t)blob.size();
        d.n_loads = (uint32_t)ext.size();
        std::vector<TinyExt> exts;
        for (const tiny_detail::Operand* e : ext) {
          const tiny_detail::Operand& o = *e;
          TinyLoad ld;
          ld.lds = (uint16_t)o.lds;
          ld.n_bits = (uint8_t)o.n;
          bool plain = o.ref.n_slice == 0;
          for (int i = 0; i < o.n; i++) plain = plain && o.pos[i] == i;
          if (!o.leaf) {
            ld.kind = 1;
            ld.src = 0;
            L->reads.push_back({(uint32_t)blob.size(), o.id});
          } else if (plain) {
            ld.kind = 0;
            ld.src = (uint32_t)o.ref.slot;
          } else {
            ld.kind = 2;
            ld.src = (uint32_t)exts.size();
            TinyExt x;
            std::memset(&x, 0, sizeof x);
            x.ref = o.ref;
            std::memcpy(x.pos, o.pos, (size_t)o.n);
            exts.push_back(x);
          }
          put(&ld, sizeof ld);
        }
        align();
        d.ext_off = (uint32_t)blob.size();
        put(exts.data(), exts.size() * sizeof(TinyExt));
        std::memcpy(blob.data() + sizeof(TinyDir) * (gi - at), &d, sizeof d);
        max_lds = std::max(max_lds, d.tab_units * 16 + lds_elems[(size_t)g] * (uint32_t)p->elem_bytes);
      }
      align();
      L->threads = max_threads;
      L->lds_bytes = max_lds;
      op.tiny = L;
      out.ops.push_back(op);
      at = end;
    }
  };
  auto launch_at = [&](int q) {
    for (auto it = launches.lower_bound({q, 0}); it != launches.end() && it->first.first == q; ++it) emit(it->second);
  };
  for (int i : others) {
    launch_at(pos[i]);
    out.ops.push_back(prog.ops[i]);
  }
  launch_at(seq);
  // the gradient copies, in launches of up to as many entries as a blob holds
  std::vector<int> copies;
  for (int i = 0; i < nops; i++)
    if (at_end(i)) copies.push_back(i);
  constexpr size_t kMost = kTinyBlobLarge / sizeof(ScatterEntry);
  for (size_t at = 0; at < copies.size(); at += kMost) {
    auto L = std::make_shared<TinyLaunch>();
    Op op;
    op.kind = OpKind::Scatter;
    for (size_t j = at; j < std::min(copies.size(), at + kMost); j++) {
      const Op& o = prog.ops[copies[j]];
      ScatterEntry e;
      std::memset(&e, 0, sizeof e);
      e.slot = (uint32_t)o.perm.dst.slot;
      e.n_bits = (uint8_t)o.perm.n_bits;
      e.n_slice = (uint8_t)o.perm.dst.n_slice;
      std::memcpy(e.slice_bit, o.perm.dst.slice_bit, sizeof e.slice_bit);
      std::memcpy(e.slice_pos, o.perm.dst.slice_pos, sizeof e.slice_pos);
      for (int i = 0; i < o.perm.n_bits; i++) e.pos[i] = (uint8_t)o.perm.dst_pos[i];
      L->reads.push_back({(uint32_t)L->blob.size(), (int)o.perm.src.off});
      L->blob.insert(L->blob.end(), (const char*)&e, (const char*)&e + sizeof e);
      L->n_groups++;
      op.node = o.node;
    }
    op.tiny = L;
    out.ops.push_back(op);
  }
  // lifetimes in the new order
  for (int i = 0; i < (int)out.ops.size(); i++) {
    Op& op = out.ops[i];
    if (op.kind == OpKind::Tiny || op.kind == OpKind::Scatter) {
      auto touch = [&](int b) { Ref r = buf_ref(b); out.touch(r, i); };
      for (auto& x : op.tiny->reads) touch(x.second);
      for (auto& x : op.tiny->writes) touch(x.second);
    } else {
      op_refs(op, [&](Ref& r, bool) { out.touch(r, i); });
    }
  }
  return out;
}
