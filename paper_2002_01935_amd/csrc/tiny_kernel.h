// Device side of the small-contraction kernel (tiny.h): one workgroup runs one
// group.  Included inside namespace tn after rowops.h.
#pragma once

// Offset of the low n <= 10 bits of v through a nibble list of positions
// (absent bits land at kTinyAbsent, above every LDS operand, and are masked
// off).  The list is shifted through two 32-bit registers.
__device__ __forceinline__ uint32_t nibbles(uint32_t v, uint64_t list, int n) {
  uint32_t off = 0, lo = (uint32_t)list, hi = (uint32_t)(list >> 32);
  for (int i = 0; i < n; i++) {
    off |= (v & 1u) << (lo & 15u);
    v >>= 1;
    lo = (lo >> 4) | (hi << 28);
    hi >>= 4;
  }
  return off & ((1u << kTinyAbsent) - 1u);
}

template <typename V>
__device__ __forceinline__ V lane_xor(V v, int m) {
  v.x = __shfl_xor(v.x, m, 64);
  v.y = __shfl_xor(v.y, m, 64);
  return v;
}

// cfma with its four roundings spelled out, as the row kernel's code has them:
// left to the compiler, products shared with the other branch below would be
// rounded before they are added.
__device__ __forceinline__ float fused(float a, float b, float c) { return __builtin_fmaf(a, b, c); }
__device__ __forceinline__ double fused(double a, double b, double c) { return __builtin_fma(a, b, c); }
template <typename V>
__device__ __forceinline__ V cfma_in_order(V acc, V a, V b) {
  acc.x = fused(-a.y, b.y, fused(a.x, b.x, acc.x));
  acc.y = fused(a.y, b.x, fused(a.x, b.y, acc.y));
  return acc;
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
  // external operands, 16 threads each, or more where they are few (three of 2^10
  // values 65 us with 16, 12 with 128): all loads of the group in flight together
  GMEM const uint64_t* ptrs = reinterpret_cast<GMEM const uint64_t*>(ctx.ws + ctx.ptrtab_off);
  uint32_t lanes = 16;
  while (2 * lanes <= nt && 2 * lanes * d.n_loads <= nt) lanes *= 2;
  const uint32_t first = tid & (lanes - 1);
  for (uint32_t i = tid / lanes; i < d.n_loads; i += nt / lanes) {
    const uint64_t w = reinterpret_cast<GMEM const uint64_t*>(blob + d.ld_off)[i];
    const uint32_t src = (uint32_t)w, lds = (uint32_t)(w >> 32) & 0xFFFFu;
    const uint32_t kind = (uint32_t)(w >> 48) & 0xFFu, n_bits = (uint32_t)(w >> 56);
    if (kind != 2) {
      const uint64_t base = kind == 0 ? ptrs[src] : ctx.ws + ctx.arena_off + uint64_t(z) * ctx.arena_stride + 256 * uint64_t(src);
      for (uint32_t e = first; e < (1u << n_bits); e += lanes) data[lds + e] = ld(reinterpret_cast<GMEM const V*>(base) + e);
    } else {
      GMEM const TinyExt* x = reinterpret_cast<GMEM const TinyExt*>(blob + d.ext_off) + src;
      uint64_t off = 0;
      const int ns = x->ref.n_slice;
      for (int j = 0; j < ns; j++) off |= uint64_t((sid >> x->ref.slice_bit[j]) & 1) << x->ref.slice_pos[j];
      GMEM const V* S = reinterpret_cast<GMEM const V*>(ptrs[x->ref.slot]) + off;
      for (uint32_t e = first; e < (1u << n_bits); e += lanes) {
        uint32_t o = 0;
        for (uint32_t j = 0; j < n_bits; j++) o |= ((e >> j) & 1u) << x->pos[j];
        data[lds + e] = ld(S + o);
      }
    }
  }
  __syncthreads();
  for (uint32_t l = 0; l < d.n_levels; l++) {
    // the level's record in three 128-bit reads: 16-bit ends, then firsts
    const u4* L = reinterpret_cast<const u4*>(smem) + 3 * l;
    const u4 w0 = L[0], w1 = L[1], w2 = L[2];
    const uint32_t w[9] = {w0[0], w0[1], w0[2], w0[3], w1[0], w1[1], w1[2], w1[3], w2[0]};
    const uint32_t total = 4 * (w[4] & 0xFFFFu);
    for (uint32_t t0 = 0; t0 < total; t0 += nt) {
      // this thread's contraction and its place in it
      const uint32_t t = t0 + tid, unit = t >> 2;
      uint32_t start = 0, op_i = w[4] >> 16, s = kTinyMaxThreadBits;
#pragma unroll
      for (int c = 0; c < kTinyClasses - 1; c++) {
        const uint32_t end = (c & 1) ? w[c >> 1] >> 16 : w[c >> 1] & 0xFFFFu;
        const int f = kTinyClasses + c + 1;                        // first[c + 1] among the 16-bit values
        const uint32_t nf = (f & 1) ? w[f >> 1] >> 16 : w[f >> 1] & 0xFFFFu;
        if (unit >= end) {
          start = end;
          op_i = nf;
          s = kTinyMaxThreadBits - 1 - c;
        }
      }
      const bool found = t < total;
      uint32_t r = t - 4 * start;
      op_i = found ? op_i + (r >> s) : 0u;
      r &= (1u << s) - 1u;
      const u4* P = reinterpret_cast<const u4*>(smem + d.ops_off) + 3 * op_i;
      const u4 p0 = P[0], p1 = P[1], p2 = P[2];
      // TinyOp: dst | a, b | c, n_out, n_k | ks, conj, dst_kind, lds_c | oa | ob | ka | kb
      const uint32_t dst = p0[0], a_lds = p0[1] & 0xFFFFu, b_lds = p0[1] >> 16, c_lds = p0[2] & 0xFFFFu;
      const int n_out = (p0[2] >> 16) & 0xFF, n_k = p0[2] >> 24;
      const int ks = p0[3] & 0xFF, conj = (p0[3] >> 8) & 0xFF;
      const uint32_t dst_kind = (p0[3] >> 16) & 0xFF, lds_c = p0[3] >> 24;
      const uint64_t oa = p1[0] | uint64_t(p1[1]) << 32, ob = p1[2] | uint64_t(p1[3]) << 32;
      const uint64_t ka = p2[0] | uint64_t(p2[1]) << 32, kb = p2[2] | uint64_t(p2[3]) << 32;
      const int kk = n_k - ks;
      const T ca = (conj & 1) ? T(-1) : T(1), cb = (conj & 2) ? T(-1) : T(1);
      const uint32_t o = r >> ks, q = r & ((1u << ks) - 1u);
      const bool active = found && (o >> n_out) == 0;
      const V* A = data + a_lds + nibbles(o, oa, n_out) + nibbles(q, ka >> (4 * kk), ks);
      const V* B = data + b_lds + nibbles(o, ob, n_out) + nibbles(q, kb >> (4 * kk), ks);
      V acc, half, quarter;
      acc.x = half.x = quarter.x = 0;
      acc.y = half.y = quarter.y = 0;
      if (active) {
        // four summed values at a time: their loads are independent
        const uint32_t a0 = kk >= 1 ? 1u << (ka & 15) : 0u, b0 = kk >= 1 ? 1u << (kb & 15) : 0u;
        const uint32_t a1 = kk >= 2 ? 1u << ((ka >> 4) & 15) : 0u, b1 = kk >= 2 ? 1u << ((kb >> 4) & 15) : 0u;
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
          }
          if (ks == 0) {
#pragma unroll
            for (int u = 0; u < 4; u++)
              if (u < 1 || (u < 2 && kk >= 1) || kk >= 2) acc = cfma_in_order(acc, a[u], b[u]);
          } else {
            // a shared sum, 2^2 to 2^4 values per thread: a balanced tree over
            // them and the lanes, as many additions per value (n_k) as in the
            // split-K kernel that runs it alone
            acc = cadd(cadd(cmul(a[0], b[0]), cmul(a[1], b[1])), cadd(cmul(a[2], b[2]), cmul(a[3], b[3])));
            const uint32_t step = j >> 2;
            if ((step & 1u) == 0) {
              half = acc;
            } else {
              acc = cadd(half, acc);
              if ((step & 2u) == 0) quarter = acc;
              else acc = cadd(quarter, acc);
            }
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
        if (lds_c) data[c_lds + o] = acc;
        if (dst_kind) {
          const uint64_t base = dst_kind == 1 ? ctx.ws + ctx.arena_off + uint64_t(z) * ctx.arena_stride + 256 * uint64_t(dst)
                                                  : ptrs[dst];
          st(reinterpret_cast<GMEM V*>(base) + o, acc);
        }
      }
    }
    __syncthreads();
  }
}
