// Device side of the small-contraction kernel (tiny.h): one workgroup runs one
// group.  Included inside namespace tn after rowops.h.
#pragma once

// Offset of the low n bits of v through a nibble list of positions (absent
// bits land at kTinyAbsent, above every LDS operand, and are masked off).
__device__ __forceinline__ uint32_t nibbles(uint32_t v, uint64_t list, int n) {
  uint32_t off = 0;
  for (int i = 0; i < n; i++) off |= ((v >> i) & 1u) << ((uint32_t)(list >> (4 * i)) & 15u);
  return off & ((1u << kTinyAbsent) - 1u);
}

template <typename V>
__device__ __forceinline__ V lane_xor(V v, int m) {
  v.x = __shfl_xor(v.x, m, 64);
  v.y = __shfl_xor(v.y, m, 64);
  return v;
}

// Group g of the blob at `blob`, for in-flight slice z.
template <typename T>
__device__ __forceinline__ void tiny_group(const Ctx& ctx, uint64_t blob, int g, int z, int64_t sid, char* smem) {
  using V = typename C2<T>::t;
  typedef uint32_t u4 __attribute__((ext_vector_type(4)));
  const TinyDir d = cload(reinterpret_cast<CMEM const TinyDir*>(blob) + g);
  const uint32_t tid = threadIdx.x, nt = blockDim.x;
  V* data = reinterpret_cast<V*>(smem + 16 * d.tab_units);
  for (uint32_t i = tid; i < d.tab_units; i += nt)
    reinterpret_cast<u4*>(smem)[i] = reinterpret_cast<GMEM const u4*>(blob + d.tab_off)[i];
  // external operands, 16 threads each: all loads of the group in flight together
  GMEM const uint64_t* ptrs = reinterpret_cast<GMEM const uint64_t*>(ctx.ws + ctx.ptrtab_off);
  for (uint32_t i = tid >> 4; i < d.n_loads; i += nt >> 4) {
    const uint64_t w = reinterpret_cast<GMEM const uint64_t*>(blob + d.ld_off)[i];
    const uint32_t src = (uint32_t)w, lds = (uint32_t)(w >> 32) & 0xFFFFu;
    const uint32_t kind = (uint32_t)(w >> 48) & 0xFFu, n_bits = (uint32_t)(w >> 56);
    if (kind != 2) {
      const uint64_t base = kind == 0 ? ptrs[src] : ctx.ws + ctx.arena_off + uint64_t(z) * ctx.arena_stride + 256 * uint64_t(src);
      for (uint32_t e = tid & 15; e < (1u << n_bits); e += 16) data[lds + e] = ld(reinterpret_cast<GMEM const V*>(base) + e);
    } else {
      GMEM const TinyExt* x = reinterpret_cast<GMEM const TinyExt*>(blob + d.ext_off) + src;
      uint64_t off = 0;
      const int ns = x->ref.n_slice;
      for (int j = 0; j < ns; j++) off |= uint64_t((sid >> x->ref.slice_bit[j]) & 1) << x->ref.slice_pos[j];
      GMEM const V* S = reinterpret_cast<GMEM const V*>(ptrs[x->ref.slot]) + off;
      for (uint32_t e = tid & 15; e < (1u << n_bits); e += 16) {
        uint32_t o = 0;
        for (uint32_t j = 0; j < n_bits; j++) o |= ((e >> j) & 1u) << x->pos[j];
        data[lds + e] = ld(S + o);
      }
    }
  }
  __syncthreads();
  const TinyOp* ops = reinterpret_cast<const TinyOp*>(smem + d.ops_off);
  for (uint32_t l = 0; l < d.n_levels; l++) {
    const TinyLevel* L = reinterpret_cast<const TinyLevel*>(smem) + l;
    uint32_t total = 0;
    for (int c = 0; c < kTinyClasses; c++) total += (uint32_t)L->cnt[c] << (kTinyMaxThreadBits - c);
    for (uint32_t t0 = 0; t0 < total; t0 += nt) {
      // this thread's contraction and its place in it: thread counts are
      // powers of two in falling order, so every contraction starts at a
      // multiple of its own count
      uint32_t r = t0 + tid, op_i = L->first;
      bool found = false;
      for (int c = 0; c < kTinyClasses; c++) {
        const uint32_t n = L->cnt[c], s = kTinyMaxThreadBits - c;
        if (!found) {
          if (r < (n << s)) {
            op_i += r >> s;
            r &= (1u << s) - 1u;
            found = true;
          } else {
            r -= n << s;
            op_i += n;
          }
        }
      }
      const TinyOp* op = ops + (found ? op_i : L->first);
      const int n_out = op->n_out, n_k = op->n_k, ks = op->ks, conj = op->conj;
      const uint64_t ka = op->ka, kb = op->kb;
      const int kk = n_k - ks;
      const T ca = (conj & 1) ? T(-1) : T(1), cb = (conj & 2) ? T(-1) : T(1);
      const uint32_t o = r >> ks, q = r & ((1u << ks) - 1u);
      const bool active = found && (o >> n_out) == 0;
      const V* A = data + op->a + nibbles(o, op->oa, n_out) + nibbles(q, ka >> (4 * kk), ks);
      const V* B = data + op->b + nibbles(o, op->ob, n_out) + nibbles(q, kb >> (4 * kk), ks);
      V acc;
      acc.x = 0;
      acc.y = 0;
      if (active) {
        // four summed values at a time: their loads are independent
        const uint32_t a0 = kk >= 1 ? nibbles(1, ka, 1) : 0u, b0 = kk >= 1 ? nibbles(1, kb, 1) : 0u;
        const uint32_t a1 = kk >= 2 ? nibbles(1, ka >> 4, 1) : 0u, b1 = kk >= 2 ? nibbles(1, kb >> 4, 1) : 0u;
        for (uint32_t j = 0; j < (1u << kk); j += 4) {
          const uint32_t xa = kk > 2 ? nibbles(j >> 2, ka >> 8, kk - 2) : 0u, xb = kk > 2 ? nibbles(j >> 2, kb >> 8, kk - 2) : 0u;
          V a[4], b[4];
          a[0] = A[xa]; b[0] = B[xb];
          a[1] = A[xa + a0]; b[1] = B[xb + b0];
          a[2] = A[xa + a1]; b[2] = B[xb + b1];
          a[3] = A[xa + a0 + a1]; b[3] = B[xb + b0 + b1];
#pragma unroll
          for (int u = 0; u < 4; u++) {
            a[u].y *= ca;
            b[u].y *= cb;
            if (u < 1 || (u < 2 && kk >= 1) || kk >= 2) acc = cfma(acc, a[u], b[u]);
          }
        }
      }
      // the 2^ks partial sums of an output sit in neighbouring lanes: fixed order
      for (int b = 0; b < 6; b++) {
        if (!__any(ks > b)) break;
        const V v = lane_xor(acc, 1 << b);
        if (ks > b) {
          acc.x += v.x;
          acc.y += v.y;
        }
      }
      if (active && q == 0) {
        if (op->lds_c) data[op->c + o] = acc;
        if (op->dst_kind) {
          const uint64_t base = op->dst_kind == 1 ? ctx.ws + ctx.arena_off + uint64_t(z) * ctx.arena_stride + 256 * uint64_t(op->dst)
                                                  : ptrs[op->dst];
          st(reinterpret_cast<GMEM V*>(base) + o, acc);
        }
      }
    }
    __syncthreads();
  }
}
