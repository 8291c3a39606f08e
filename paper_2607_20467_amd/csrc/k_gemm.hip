// MFMA bf16 GEMM family for gfx950 with fused epilogues.
//
//   C[w, t] = sum_k W[w, k] * X[t, k]      W: bf16 [Nw, K] (weights, nn.Linear layout)
//                                           X: bf16 [T, K]  (activations, one row per token)
// Both operands are K-contiguous, so every MFMA fragment is one 16-byte load. Weights play the
// MFMA "A" role: a lane of a 16x16 accumulator tile then holds four consecutive weight rows of one
// token, which makes the fused epilogues local to a lane:
//   QKV    + bias, rotate-half RoPE (rotation pairs were interleaved into adjacent rows at load),
//          scattered to q [B,H,S,dh], k [B,Hkv,S,dh] and key-contiguous v [B,Hkv,dh,Sp];
//   RESID  r[t, w] += C (float32 residual stream);
//   SWIGLU a[t, f] = bf16(silu(gate) * up) (gate/up rows interleaved at load);
//   LMHEAD per (token, 128-id vocabulary tile): top-1, top-2, sum exp(l - top1) and the entropy
//          sum — logits stay in registers and never reach memory;
//   PARTIAL float32 split-K slice, folded into the residual stream by the next RMSNorm;
//   F32    plain float32 store (debug logits).
// Tiles: BW weight rows x BT tokens per workgroup, K staged through a multi-stage LDS ring of 64-deep
// slices (128-deep for at most 64 tokens) filled by direct-to-LDS DMA. Two kernels: gemm_pp_kernel, whose two
// waves per SIMD alternate between reading and multiplying (the large tiles), and gemm_kernel (few tokens, K
// tails, and two tiles of one round of units). The unit ->
// workgroup map is XCD-aware: tiles that share operands land on the same XCD and its L2. The
// configuration comes from a cost model with measured constants per configuration (gemm_tuned.inc).
#include <float.h>
#include <limits.h>

#include <algorithm>
#include <cmath>
#include <type_traits>

#include "dcl_internal.h"

namespace dcl {


__device__ __forceinline__ f32x4_t mfma16(const bf16x8_t& a, const bf16x8_t& b, const f32x4_t& c) {
  return __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, b, c, 0, 0, 0);
}

// ---------------------------------------------------------------- epilogues
// apply(): acc[i][j] holds C[wb + 16 i + 4 (lane/16) + r][tb + 16 JS j + lane%16], r = 0..3 (JS: the stride
// of a wave's token fragments, in fragments).

enum { kEpiPlain, kEpiQkv, kEpiResid, kEpiLm, kEpiDebug };

struct EpiResid {
  float* r;
  static constexpr int kKind = kEpiResid;
  template <int SW, int ST, int JS = 1>
  __device__ __forceinline__ void apply(f32x4_t (&acc)[SW][ST], int wb, int tb, int lane, int Nw, int T, int, int) const {
    const int wq = wb + 4 * (lane >> 4), tl = tb + (lane & 15);
#pragma unroll
    for (int j = 0; j < ST; ++j) {
      const int t = tl + 16 * JS * j;
      if (t >= T) continue;
#pragma unroll
      for (int i = 0; i < SW; ++i) {
        const int w = wq + 16 * i;
        if (w >= Nw) continue;
        float4* p = reinterpret_cast<float4*>(r + (size_t)t * Nw + w);
        float4 v = *p;
        v.x += acc[i][j][0]; v.y += acc[i][j][1]; v.z += acc[i][j][2]; v.w += acc[i][j][3];
        *p = v;
      }
    }
  }
};

// g / (1 + e^-g): the quotient by reciprocal and one correction step (exact remainder), at two thirds of the IEEE
// division's instructions. It is within an ulp of that where the denominator is below 2^126 (g > -87.3; past it the
// reciprocal and the remainder leave the normal range) and g is finite (the correction of inf is NaN). `range` adds up
// the denominators, and a correction that is not finite makes it NaN: with range < 2^126 every quotient that it has
// seen holds.
constexpr float kSiluRange = 0x1p126f;
__device__ __forceinline__ float silu(float g, float& range) {
  const float x = 1.0f + __expf(-g);
  const float r = __builtin_amdgcn_rcpf(x);
  const float q = g * r;
  const float c = fmaf(fmaf(-q, x, g), r, q);
  range = fmaf(c, 0.0f, range + x);
  return c;
}
__device__ __forceinline__ float silu_ieee(float g) { return g / (1.0f + __expf(-g)); }

// Transposes over the four 16-lane groups. Lane group p holds piece p (rows 4 p ..) of each fragment of a wave's
// column; a store needs consecutive rows of one fragment in one lane.
// N = 4: h[i] = this group's piece of fragment i -> the four pieces, in order, of fragment p.
// N = 2: -> pieces 2 (p / 2) and 2 (p / 2) + 1 of fragment p % 2.
__device__ __forceinline__ uint4 gather_pieces(uint32_t h0, uint32_t h1, uint32_t h2, uint32_t h3) {
  const auto a0 = __builtin_amdgcn_permlane32_swap(h0, h2, false, false);
  const auto a1 = __builtin_amdgcn_permlane32_swap(h1, h3, false, false);
  const auto b0 = __builtin_amdgcn_permlane16_swap(a0[0], a1[0], false, false);
  const auto b1 = __builtin_amdgcn_permlane16_swap(a0[1], a1[1], false, false);
  return make_uint4(b0[0], b0[1], b1[0], b1[1]);
}
__device__ __forceinline__ uint2 gather_pieces(uint32_t h0, uint32_t h1) {
  const auto a = __builtin_amdgcn_permlane16_swap(h0, h1, false, false);
  return make_uint2(a[0], a[1]);
}

// What the epilogue costs: a 192 x 192 unit at 24576 x 384 x 4096 takes 66 us without one and 76 us with one
// 4-byte store per fragment; four fragments' pieces gathered into 16-byte stores (64 contiguous bytes per
// token): 73 us, 37888 x 3072 x 3584 617 -> 604 us, 24576 x 512 x 4096 (192 x 256) 92 -> 87 us.
struct EpiSwiglu {
  bf16_t* a;  // [T, Nw/2]; Nw / 2 is a multiple of 16, so the stores are aligned
  static constexpr int kKind = kEpiPlain;
  template <int SW, int ST, int JS = 1>
  __device__ __forceinline__ void apply(f32x4_t (&acc)[SW][ST], int wb, int tb, int lane, int Nw, int T, int, int) const {
    const int F = Nw >> 1;
    const int p = lane >> 4, tl = tb + (lane & 15);
#pragma unroll
    for (int j = 0; j < ST; ++j) {
      const int t = tl + 16 * JS * j;
      if (tb + 16 * JS * j >= T) continue;  // wave-uniform: every lane takes part in the swaps
      bf16_t* dst = a + (size_t)t * F;
      uint32_t h[SW];  // this lane's piece of each fragment: two products
      float range = 0.f;
#pragma unroll
      for (int i = 0; i < SW; ++i) {
        const f32x4_t v = acc[i][j];
        h[i] = f2bf2(silu(v[0], range) * v[1], silu(v[2], range) * v[3]);
      }
      if (!(range < kSiluRange)) {
#pragma unroll
        for (int i = 0; i < SW; ++i) {
          const f32x4_t v = acc[i][j];
          h[i] = f2bf2(silu_ieee(v[0]) * v[1], silu_ieee(v[2]) * v[3]);
        }
      }
#pragma unroll
      for (int i = 0; i + 4 <= SW; i += 4) {
        const uint4 x = gather_pieces(h[i], h[i + 1], h[i + 2], h[i + 3]);
        const int w = wb + 16 * (i + p);
        if (t < T && w < Nw) *reinterpret_cast<uint4*>(dst + (w >> 1)) = x;
      }
      if constexpr (SW % 4 >= 2) {
        constexpr int i = SW / 4 * 4;
        const uint2 x = gather_pieces(h[i], h[i + 1]);
        const int w = wb + 16 * (i + (p & 1));
        if (t < T && w < Nw) *reinterpret_cast<uint2*>(dst + (w >> 1) + 4 * (p >> 1)) = x;
      }
      if constexpr (SW % 2) {
        const int w = wb + 16 * (SW - 1) + 4 * p;
        if (t < T && w < Nw) *reinterpret_cast<uint32_t*>(dst + (w >> 1)) = h[SW - 1];
      }
    }
  }
};

// Offsets are 32-bit element counts: gemm_qkv rejects outputs of 2^31 elements or more.
struct EpiQkv {
  QkvOut o;
  static constexpr int kKind = kEpiQkv;
  template <int SW, int ST, int JS = 1>
  __device__ __forceinline__ void apply(f32x4_t (&acc)[SW][ST], int wb, int tb, int lane, int Nw, int T, int, int) const {
    const int DH = o.dh, HALF = DH >> 1, LOG2DH = DH == 128 ? 7 : 6;  // head_dim 64 or 128
    const int qrows = o.H * DH, qkrows = qrows + o.Hkv * DH;
    const int Sk = o.Sk ? o.Sk : o.S;  // fresh key rows per (sequence, kv head); token s sits in slot koff + s
    const int p = lane >> 4, tl = tb + (lane & 15);
#pragma unroll
    for (int j = 0; j < ST; ++j) {
      const int t = tl + 16 * JS * j;
      if (tb + 16 * JS * j >= T) continue;  // wave-uniform: every lane takes part in the swaps
      const bool valid = t < T;
      const int b = min(t, T - 1) / o.S, s = min(t, T - 1) - b * o.S;
      const int pos = o.pos0 + s;
      // per token: element offsets of (head 0, position s) in q, k, and of (row 0, key s) in v^T
      const uint32_t qt = (uint32_t)(b * o.H * o.S + s) * DH;
      const uint32_t kt = (uint32_t)(b * o.Hkv * Sk + o.koff + s) * DH;
      const uint32_t vtt = (uint32_t)b * o.Hkv * DH * o.Sp + o.koff + s;
      const float2* rope_t = o.rope ? o.rope + (size_t)pos * HALF : nullptr;
      // rows w .. w + 3 of this lane with bias
      auto biased = [&](int i) {
        f32x4_t v = acc[i][j];
        if (o.bias) {
          const int w = wb + 16 * i + 4 * p;
          if (w < Nw) v += *reinterpret_cast<const f32x4_t*>(o.bias + w);
        }
        return v;
      };
      // rotated q / k pairs of fragment i: (first halves of two pairs, second halves)
      auto rotated = [&](int i, uint32_t& lo, uint32_t& hi) {
        f32x4_t v = biased(i);
        if (rope_t) {
          const int jp = ((wb + 16 * i + 4 * p) & (DH - 1)) >> 1;  // pairs (v0, v1) -> jp, (v2, v3) -> jp + 1
          const float4 cs = *reinterpret_cast<const float4*>(rope_t + jp);
          v = f32x4_t{v[0] * cs.x - v[1] * cs.y, v[1] * cs.x + v[0] * cs.y, v[2] * cs.z - v[3] * cs.w,
                      v[3] * cs.z + v[2] * cs.w};
        }
        lo = f2bf2(v[0], v[2]);
        hi = f2bf2(v[1], v[3]);
      };
      // first element of the pair of weight row w (a multiple of 2) in q or k
      auto qk_dst = [&](int w) {
        const bool isq = w < qrows;
        const int wl = isq ? w : w - qrows, head = wl >> LOG2DH, jp = (wl & (DH - 1)) >> 1;
        return (isq ? o.q + qt + (uint32_t)head * o.S * DH : o.k + kt + (uint32_t)head * Sk * DH) + jp;
      };
      auto single = [&](int i) {  // one fragment, q / k or v (the regions start at multiples of 64 rows)
        const int w = wb + 16 * i + 4 * p;
        if (wb + 16 * i < qkrows) {
          uint32_t lo, hi;
          rotated(i, lo, hi);
          if (!valid || w >= Nw) return;
          bf16_t* dst = qk_dst(w);
          *reinterpret_cast<uint32_t*>(dst) = lo;
          *reinterpret_cast<uint32_t*>(dst + HALF) = hi;
        } else if (valid && w < Nw) {
          const f32x4_t v = biased(i);
          bf16_t* base = o.vt + vtt + (uint32_t)(w - qkrows) * o.Sp;  // w - qkrows = head * DH + dimension
          base[0] = f2bf(v[0]);
          base[o.Sp] = f2bf(v[1]);
          base[2 * o.Sp] = f2bf(v[2]);
          base[3 * o.Sp] = f2bf(v[3]);
          if (s == o.S - 1) {  // the last token also clears the padding slots [koff + S, Sp) of its four rows
            for (int z = 1; o.koff + s + z < o.Sp; ++z)
              for (int rr = 0; rr < 4; ++rr) base[rr * o.Sp + z] = 0;
          }
        }
      };
      // four (two) q / k fragments at a time: 16-byte (8-byte) stores of 8 (4) consecutive pairs
#pragma unroll
      for (int i = 0; i + 4 <= SW; i += 4) {
        if (wb + 16 * (i + 3) < qkrows) {
          uint32_t lo[4], hi[4];
#pragma unroll
          for (int x = 0; x < 4; ++x) rotated(i + x, lo[x], hi[x]);
          const uint4 l4 = gather_pieces(lo[0], lo[1], lo[2], lo[3]), h4 = gather_pieces(hi[0], hi[1], hi[2], hi[3]);
          const int w = wb + 16 * (i + p);
          if (valid && w < Nw) {
            bf16_t* dst = qk_dst(w);
            *reinterpret_cast<uint4*>(dst) = l4;
            *reinterpret_cast<uint4*>(dst + HALF) = h4;
          }
        } else {
#pragma unroll
          for (int x = 0; x < 4; ++x) single(i + x);
        }
      }
      if constexpr (SW % 4 >= 2) {
        constexpr int i = SW / 4 * 4;
        if (wb + 16 * (i + 1) < qkrows) {
          uint32_t lo[2], hi[2];
          rotated(i, lo[0], hi[0]);
          rotated(i + 1, lo[1], hi[1]);
          const uint2 l2 = gather_pieces(lo[0], lo[1]), h2 = gather_pieces(hi[0], hi[1]);
          const int w = wb + 16 * (i + (p & 1)) + 8 * (p >> 1);
          if (valid && w < Nw) {
            bf16_t* dst = qk_dst(w);
            *reinterpret_cast<uint2*>(dst) = l2;
            *reinterpret_cast<uint2*>(dst + HALF) = h2;
          }
        } else {
          single(i);
          single(i + 1);
        }
      }
      if constexpr (SW % 2) single(SW - 1);
    }
  }
  // A ragged cached prefix: the koff newest cached keys and values go in front of the fresh ones, slots [0, koff)
  // of every k and v^T row of a sequence. The workgroup whose tile holds a sequence's first token copies the rows of
  // its weight rows, one row per thread with all its loads in flight together, while the first stages of the main loop
  // are under way. A layer of 3 x 60 tokens, 4096 wide, takes 185 us over 256 cached keys and 189 over 261 (196 when the
  // wave that held a sequence's first token copied element after element in the epilogue); 1 x 64 over 323: 134 (131
  // over 320; a copy launch of its own added 4.5).
  __device__ __forceinline__ void carry(int w0, int bw, int t0, int t1, int Nw, int tid, int nthr) const {
    const int DH = o.dh, LOG2DH = DH == 128 ? 7 : 6, qrows = o.H * DH, kvrows = o.Hkv * DH;
    const int w_lo = max(w0, qrows), n = min(w0 + bw, Nw) - w_lo;  // the tile's k and v rows
    const int b0 = (t0 + o.S - 1) / o.S, nb = (t1 + o.S - 1) / o.S - b0;  // sequences that start in the tile
    for (int e = tid; e < n * nb; e += nthr) {
      const int x = e / n, w = w_lo + (e - x * n) - qrows, b = b0 + x;
      const int key = o.pos0 - o.koff;
      const bf16_t* src;
      bf16_t* dst;
      int ld;  // elements between keys
      if (w < kvrows) {  // pairs of rows are dimensions jp and jp + DH / 2
        const size_t head = (size_t)b * o.Hkv + (w >> LOG2DH);
        const int wl = w & (DH - 1), d = (wl >> 1) + (wl & 1) * (DH >> 1);
        src = o.kc + (head * o.Pc + key) * DH + d;
        dst = o.k + head * o.Sk * DH + d;
        ld = DH;
      } else {
        const size_t row = (size_t)b * kvrows + (w - kvrows);
        src = o.vc + row * o.Pc + key;
        dst = o.vt + row * o.Sp;
        ld = 1;
      }
      bf16_t v[7];
#pragma unroll
      for (int z = 0; z < 7; ++z)
        v[z] = src[min(z, o.koff - 1) * ld];
      // vmcnt(0) in a form that the compiler counts: with these loads open on some path it would wait for all of the
      // main loop's DMA wherever that reuses their registers (d5120, 64 tokens: 183 -> 218 us a layer)
      __builtin_amdgcn_s_waitcnt(0x0F70);
#pragma unroll
      for (int z = 0; z < 7; ++z)
        if (z < o.koff) dst[z * ld] = v[z];
    }
  }
};

struct EpiF32 {
  float* out;
  static constexpr int kKind = kEpiDebug;
  template <int SW, int ST, int JS = 1>
  __device__ __forceinline__ void apply(f32x4_t (&acc)[SW][ST], int wb, int tb, int lane, int Nw, int T, int, int) const {
    const int wq = wb + 4 * (lane >> 4), tl = tb + (lane & 15);
#pragma unroll
    for (int j = 0; j < ST; ++j) {
      const int t = tl + 16 * JS * j;
      if (t >= T) continue;
#pragma unroll
      for (int i = 0; i < SW; ++i)
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          const int w = wq + 16 * i + r;
          if (w < Nw) out[(size_t)t * Nw + w] = acc[i][j][r];
        }
    }
  }
};

// Split-K slice: unit `split` writes its float32 partial C to P + split * stride ([T, Nw] each);
// the consumer (the next RMSNorm) adds the slices up in split order and the sum to the residual stream.
struct EpiPartial {
  float* P;
  size_t stride;
  static constexpr int kKind = kEpiResid;
  template <int SW, int ST, int JS = 1>
  __device__ __forceinline__ void apply(f32x4_t (&acc)[SW][ST], int wb, int tb, int lane, int Nw, int T, int,
                                        int split) const {
    float* base = P + (size_t)split * stride;
    const int wq = wb + 4 * (lane >> 4), tl = tb + (lane & 15);
#pragma unroll
    for (int j = 0; j < ST; ++j) {
      const int t = tl + 16 * JS * j;
      if (t >= T) continue;
#pragma unroll
      for (int i = 0; i < SW; ++i) {
        const int w = wq + 16 * i;
        if (w >= Nw) continue;
        *reinterpret_cast<float4*>(base + (size_t)t * Nw + w) =
            make_float4(acc[i][j][0], acc[i][j][1], acc[i][j][2], acc[i][j][3]);
      }
    }
  }
};

__device__ __forceinline__ bool better(float va, int ia, float vb, int ib) {
  return va > vb || (va == vb && ia < ib);
}
struct Part {
  float m1, m2, s, t;  // s = sum exp(l - m1), t = sum exp(l - m1) (l - m1), both relative to m1
  int i1, i2;
};
__device__ __forceinline__ void top2_push(Part& p, float v, int id) {
  if (better(v, id, p.m1, p.i1)) {
    p.m2 = p.m1; p.i2 = p.i1; p.m1 = v; p.i1 = id;
  } else if (better(v, id, p.m2, p.i2)) {
    p.m2 = v; p.i2 = id;
  }
}
__device__ __forceinline__ Part part_merge(const Part& a, const Part& b) {
  Part o;
  if (better(a.m1, a.i1, b.m1, b.i1)) {
    o.m1 = a.m1; o.i1 = a.i1;
    if (better(a.m2, a.i2, b.m1, b.i1)) { o.m2 = a.m2; o.i2 = a.i2; } else { o.m2 = b.m1; o.i2 = b.i1; }
  } else {
    o.m1 = b.m1; o.i1 = b.i1;
    if (better(b.m2, b.i2, a.m1, a.i1)) { o.m2 = b.m2; o.i2 = b.i2; } else { o.m2 = a.m1; o.i2 = a.i1; }
  }
  // sums are relative to each side's own top-1 value; moving t to the new reference m adds
  // s (m1 - m) (each term exp(l - m1) (l - m1) becomes exp(l - m1) (l - m))
  const float da = (a.m1 == -INFINITY) ? 0.f : a.m1 - o.m1, db = (b.m1 == -INFINITY) ? 0.f : b.m1 - o.m1;
  const float ea = (a.m1 == -INFINITY) ? 0.f : __expf(da), eb = (b.m1 == -INFINITY) ? 0.f : __expf(db);
  o.s = a.s * ea + b.s * eb;
  o.t = ea * (a.t + a.s * da) + eb * (b.t + b.s * db);
  return o;
}

// Value of lane ^ 16 and lane ^ 32 paired with the lane's own by the lane-swap instructions (no LDS round
// trip): op gets both values, in an order that is the same in both lanes, so it must be symmetric.
template <class Op>
__device__ __forceinline__ float pair_lanes(float v, bool far, Op op) {
  const int b = __builtin_bit_cast(int, v);
  if (far) {
    const auto p = __builtin_amdgcn_permlane32_swap(b, b, false, false);
    return op(__builtin_bit_cast(float, (int)p[0]), __builtin_bit_cast(float, (int)p[1]));
  }
  const auto p = __builtin_amdgcn_permlane16_swap(b, b, false, false);
  return op(__builtin_bit_cast(float, (int)p[0]), __builtin_bit_cast(float, (int)p[1]));
}

// Statistics of one token fragment j over the wave's 16 * SW ids, every lane of a token's four ends with them:
// a scan over the lane's values (in id order, so a strict > keeps the lowest id of equal values), a butterfly
// over the four lanes of the token, then the sums relative to the wave's top-1 value. VALU-bound: about 7
// operations a value for the top two with their ids and 8 for the sums (the exponential counts 4), against
// about 28 with ties, the vocabulary's end and the left-out id tested per value (the general version below):
// 126464 x 4096 at 32 / 256 rows 202 -> 183 / 266 -> 251 us, 152064 x 3584 at 1920 rows 1850 -> 1707 us. Returns
// false where a value is not finite enough for the short cuts (NaN, infinities, fewer than two values above -inf); the
// general version then gives that fragment.
template <int SW, int ST>
__device__ __forceinline__ bool lm_fragment(const f32x4_t (&acc)[SW][ST], int j, int wq, Part& p) {
  float m1 = fmaxf(acc[0][j][0], acc[0][j][1]), m2 = fminf(acc[0][j][0], acc[0][j][1]);
  int n1 = acc[0][j][1] > acc[0][j][0] ? 1 : 0, n2 = 1 - n1;
#pragma unroll
  for (int n = 2; n < 4 * SW; ++n) {
    const float v = acc[n >> 2][j][n & 3];
    const int id = 16 * (n >> 2) + (n & 3);
    const bool c1 = v > m1, c2 = v > m2;
    n2 = c1 ? n1 : (c2 ? id : n2);
    n1 = c1 ? id : n1;
    m2 = __builtin_amdgcn_fmed3f(m1, m2, v);
    m1 = fmaxf(m1, v);
  }
  int i1 = wq + n1, i2 = wq + n2;
#pragma unroll
  for (int far = 0; far < 2; ++far) {
    // both halves of the swap: (x, y) are the two lanes' values, in the same order in both lanes
    auto both = [&](int v, int& x, int& y) {
      if (far) {
        const auto q = __builtin_amdgcn_permlane32_swap(v, v, false, false);
        x = (int)q[0];
        y = (int)q[1];
      } else {
        const auto q = __builtin_amdgcn_permlane16_swap(v, v, false, false);
        x = (int)q[0];
        y = (int)q[1];
      }
    };
    int ma, mb, sa, sb, ia, ib, ja, jb;
    both(__builtin_bit_cast(int, m1), ma, mb);
    both(__builtin_bit_cast(int, m2), sa, sb);
    both(i1, ia, ib);
    both(i2, ja, jb);
    const float a1 = __builtin_bit_cast(float, ma), b1 = __builtin_bit_cast(float, mb);
    const float a2 = __builtin_bit_cast(float, sa), b2 = __builtin_bit_cast(float, sb);
    const bool first = better(a1, ia, b1, ib);
    const float lose = first ? b1 : a1, sec = first ? a2 : b2;
    const int ilose = first ? ib : ia, isec = first ? ja : jb;
    const bool keep = better(sec, isec, lose, ilose);
    m1 = first ? a1 : b1;
    i1 = first ? ia : ib;
    m2 = keep ? sec : lose;
    i2 = keep ? isec : ilose;
  }
  float s = 0.f, t = 0.f;
#pragma unroll
  for (int n = 0; n < 4 * SW; ++n) {
    const float d = acc[n >> 2][j][n & 3] - m1;
    const float e = __expf(d);
    s += e;
    t += e * d;
  }
  auto add = [](float x, float y) { return x + y; };
  s = pair_lanes(s, false, add);
  s = pair_lanes(s, true, add);
  t = pair_lanes(t, false, add);
  t = pair_lanes(t, true, add);
  p = Part{m1, m2, s, t, i1, i2};
  const float chk = s + t;
  return __builtin_amdgcn_ballot_w64(!(fabsf(chk) < INFINITY)) == 0;
}
// The same with every id tested: ids at or past Nw and the left-out id do not count.
template <int SW, int ST>
__device__ __forceinline__ void lm_fragment_general(const f32x4_t (&acc)[SW][ST], int j, int wq, int Nw, int exclude,
                                                    Part& p) {
  p = {-INFINITY, -INFINITY, 0.f, 0.f, INT_MAX, INT_MAX};
#pragma unroll
  for (int i = 0; i < SW; ++i)
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const int w = wq + 16 * i + r;
      if (w < Nw && w != exclude) top2_push(p, acc[i][j][r], w);
    }
#pragma unroll
  for (int off = 16; off <= 32; off <<= 1) {
    Part x;
    x.m1 = __shfl_xor(p.m1, off, 64); x.m2 = __shfl_xor(p.m2, off, 64);
    x.i1 = __shfl_xor(p.i1, off, 64); x.i2 = __shfl_xor(p.i2, off, 64);
    x.s = 0.f;
    x.t = 0.f;
    Part y = part_merge(p, x);  // symmetric: ids differ, so argument order does not matter
    p.m1 = y.m1; p.m2 = y.m2; p.i1 = y.i1; p.i2 = y.i2;
  }
  float s = 0.f, t = 0.f;
#pragma unroll
  for (int i = 0; i < SW; ++i)
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const int w = wq + 16 * i + r;
      if (w < Nw && w != exclude) {
        const float d = acc[i][j][r] - p.m1;
        const float e = __expf(d);
        s += e;
        t += e * d;
      }
    }
  s += __shfl_xor(s, 16, 64);
  s += __shfl_xor(s, 32, 64);
  t += __shfl_xor(t, 16, 64);
  t += __shfl_xor(t, 32, 64);
  p.s = s;
  p.t = t;
}

// LM head: one partial per (token, vocabulary tile of kLmTile ids). Within a wave: per-lane scan of
// its values, butterfly over the four lanes holding the same token, then a second pass for the sum
// of exp(l - m1_wave). A wave whose weight rows span a whole vocabulary tile (16 * SW == kLmTile)
// writes that tile's partial itself; otherwise the WW waves of a BW = kLmTile workgroup tile split
// its vocabulary rows and merge through LDS in wave order.
template <int BW, int WW>
struct EpiLm {
  LmOut o;
  static constexpr int kKind = kEpiLm;
  // [wave along W][token fragment slot within the workgroup tile]; only the split-tile layout uses it
  template <int NTOK>
  __device__ static Part (*xch_slot())[NTOK] {
    __shared__ Part xch[WW][NTOK];
    return xch;
  }
  template <int SW, int ST, int JS = 1>
  __device__ __forceinline__ void apply(f32x4_t (&acc)[SW][ST], int wb, int tb, int lane, int Nw, int T, int tile_w, int) const {
    constexpr bool kOwn = 16 * SW == kLmTile;  // this wave covers a whole vocabulary tile
    // any other layout is never planned for the LM head (plan_gemm's lm_ok); nothing to instantiate
    if constexpr (!kOwn && !(BW == kLmTile && 16 * SW * WW == BW)) return;
    const int wid = threadIdx.x >> 6;
    // the wave grids of gemm_kernel (JS = 1) and gemm_pp_kernel (token fragments JS apart)
    const int wave_w = JS == 1 ? wid % WW : wid / JS, wave_t = JS == 1 ? wid / WW : wid % JS;
    constexpr int NTOK = ST * 16 * (8 / WW);  // tokens of the workgroup tile (8 waves)
    const int R = o.count ? *o.count : T;
    const int vt = kOwn ? wb / kLmTile : tile_w;  // vocabulary tile of this wave's partial
    const int wq = wb + 4 * (lane >> 4), tl = tb + (lane & 15);
    // the wave's ids all exist and none is left out
    const bool inside = wb + 16 * SW <= Nw && (o.exclude < wb || o.exclude >= wb + 16 * SW);
#pragma unroll
    for (int j = 0; j < ST; ++j) {
      if (tb + 16 * JS * j >= T && (kOwn || WW == 1)) continue;  // no valid token in this fragment
      Part p;
      bool general = !inside;
      if (inside) general = !lm_fragment<SW, ST>(acc, j, wq, p);
      if (general) lm_fragment_general<SW, ST>(acc, j, wq, Nw, o.exclude, p);
      if constexpr (kOwn || WW == 1) {
        const int t = tl + 16 * JS * j;
        if (lane < 16 && t < R && t < T && vt < o.n_vt) {
          const size_t idx = (size_t)t * o.n_vt + vt;
          o.pm1[idx] = p.m1; o.pi1[idx] = p.i1; o.pm2[idx] = p.m2; o.pi2[idx] = p.i2; o.ps[idx] = p.s;
          o.pt[idx] = p.t;
        }
      } else {
        if (lane < 16) xch_slot<NTOK>()[wave_w][(wave_t * ST + j) * 16 + lane] = p;
      }
    }
    if constexpr (!kOwn && WW > 1) {
      Part(*xch)[NTOK] = xch_slot<NTOK>();
      __syncthreads();
      if (wave_w == 0) {
#pragma unroll
        for (int j = 0; j < ST; ++j) {
          const int t = tl + 16 * JS * j;
          if (lane < 16 && t < R && t < T) {
            Part p = xch[0][(wave_t * ST + j) * 16 + lane];
#pragma unroll
            for (int v = 1; v < WW; ++v) p = part_merge(p, xch[v][(wave_t * ST + j) * 16 + lane]);
            const size_t idx = (size_t)t * o.n_vt + tile_w;
            o.pm1[idx] = p.m1; o.pi1[idx] = p.i1; o.pm2[idx] = p.m2; o.pi2[idx] = p.i2; o.ps[idx] = p.s;
            o.pt[idx] = p.t;
          }
        }
      }
    }
  }
};

// ---------------------------------------------------------------- the kernel
// Direct-to-LDS multi-stage pipeline: each stage holds a BW x KD weight slice and a BT x KD
// activation slice (KD = 64 or 128 K elements), written by global_load_lds_dwordx4 (16 bytes per
// lane straight into LDS, no register staging). A row is KD/8 chunks of 16 bytes, XOR-swizzled
// (chunk c of row r at c ^ (r mod KD/8)) so the MFMA fragment reads are bank-conflict free.
// All STAGES buffers are in flight at once: buffer k mod STAGES is refilled with stage
// k + STAGES as soon as every wave holds stage k's fragments in registers. Fragments are double
// buffered per 32-wide K substep: the LDS reads of substep s + 1 are in flight while the MFMAs of
// substep s run, and the first substep of stage k + 1 is read across the stage boundary.
//
// The DMA instructions are issued through dma16_lds (inline assembly), so the compiler's wait-count
// pass does not treat them as pending LDS traffic and keeps its LDS waits fine-grained; their
// completion is tracked here with vmcnt waits on this wave's own
// outstanding stages, and a bare s_barrier (no vmcnt(0) fence) publishes a stage to the other
// waves. Vector-memory loads complete in issue order, and no other vector-memory load is issued
// inside the K loop, so "at most n outstanding" means "all but the newest n landed".
//
// Split-K: unit (tile, split) accumulates K-steps [split*per, ...) and hands its partial to a
// slice epilogue (EpiPartial: one float32 slice per split, no unit waits on another); the consumer
// adds the slices in split order, so results are bitwise reproducible. nsplit > 1 is only used with
// a slice epilogue.
static __device__ __attribute__((aligned(64))) uint4 g_zero_chunk[4];

// dma16_at with the LDS destination already wave-uniform (a scalar register)
__device__ __forceinline__ void dma16_lds(const void* g, uint32_t lds_addr) {
  asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, off" ::"s"(lds_addr), "v"(g) : "memory", "m0");
}

template <int N>
__device__ __forceinline__ void wait_vmcnt() {
  static_assert(N >= 0 && N < 64, "vmcnt range");
  __builtin_amdgcn_s_waitcnt((N & 15) | (7 << 4) | (15 << 8) | ((N >> 4) << 14));
}

template <int IPW, int MAXN>
__device__ __forceinline__ void wait_stages(int n) {  // all but this wave's newest n stages (IPW loads each) landed
  if constexpr (MAXN > 0) {
    if (n >= MAXN) {
      wait_vmcnt<MAXN * IPW>();
      return;
    }
    wait_stages<IPW, MAXN - 1>(n);
  } else {
    wait_vmcnt<0>();
  }
}

__device__ __forceinline__ void lds_barrier() { asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory"); }

// Waves per SIMD that the registers must allow. The K-tail kernel's 64 KB ring lets a CU hold two workgroups of two waves
// per SIMD, which takes at most 128 registers; one more halves the waves (q/k/v of 1280 tokens x 6144 x 2000: 75 us with
// 129 registers, 51 with 128). Its LM head needs 145.
template <class Epi, bool KTAIL>
constexpr int kMinWaves = KTAIL && Epi::kKind != kEpiLm ? 4 : 1;

template <int BW, int BT, int KD, int STAGES, int WW, int WT, class Epi, bool KTAIL>
__global__ void __launch_bounds__(WW * WT * 64, (kMinWaves<Epi, KTAIL>))
gemm_kernel(const bf16_t* __restrict__ W, const bf16_t* __restrict__ X, int Nw, int T, int K,
            const int32_t* __restrict__ t_count, int nsplit, Epi epi) {
  constexpr int NWAVE = WW * WT;
  constexpr int CPR = KD / 8, KS = KD / 32;  // 16-byte chunks per row, 32-wide substeps per stage
  constexpr int TW = BW / WW, TT = BT / WT, SW = TW / 16, ST = TT / 16;
  constexpr int CH = (BW + BT) * CPR;        // chunks per stage
  constexpr int IPW = CH / 64 / NWAVE;       // load instructions per wave per stage
  static_assert(TW % 16 == 0 && TT % 16 == 0 && CH % (64 * NWAVE) == 0 && (BW * CPR) % 64 == 0, "tile shape");
  static_assert((KD == 64 || KD == 128) && STAGES >= 2 && IPW * (STAGES - 1) < 64, "pipeline shape");
  extern __shared__ __attribute__((aligned(1024))) uint4 sm[];

  // Units: (split, weight tile, token tile), token tile innermost so neighbours share a weight
  // slice, split outermost so an XCD's run covers one or two K ranges and its L2 holds only that
  // part of the activations. Only token tiles holding valid rows (t_count, when given) are units.
  // XCD x (= blockIdx % 8) walks a contiguous run of units, its workgroups striding through it.
  const int Tv = t_count ? min(T, *t_count) : T;
  const int nW = (Nw + BW - 1) / BW, nTt = (Tv + BT - 1) / BT;
  const int units = nW * nsplit * nTt;
  const int per = (units + 7) / 8;
  const int xcd = blockIdx.x & 7, stride = gridDim.x >> 3;
  const int run_end = min(units, (xcd + 1) * per);
  const int tid = threadIdx.x, lane = tid & 63, wid = tid >> 6;
  const int wave_w = wid % WW, wave_t = wid / WW;
  const int frow = lane & 15, fchunk = lane >> 4;
  for (int L = xcd * per + (blockIdx.x >> 3); L < run_end; L += stride) {
    const int tile_t = L % nTt, rest = L / nTt;
    const int tile_w = rest % nW, split = rest / nW;
    const int w0 = tile_w * BW, t0 = tile_t * BT;
    const int nk_all = (K + KD - 1) / KD;
    const int kper = (nk_all + nsplit - 1) / nsplit;
    const int kb = min(nk_all, split * kper);
    const int nk = min(nk_all, kb + kper) - kb;

    // Per-lane source of this wave's load instructions at K offset 0. A row outside the operand
    // is clamped to the last valid row: its data only reaches accumulators of rows / tokens that
    // every epilogue skips, so no zero fill is needed. The source of stage kt is this pointer plus
    // (kb + kt) * KD elements; with KTAIL (K not a multiple of KD), chunks past K read the zero chunk.
    const bf16_t* gsrc[IPW];
    int kc[IPW];
#pragma unroll
    for (int i = 0; i < IPW; ++i) {
      const int q = wid * IPW + i;
      const int pos = q * 64 + lane;
      const bool isw = q * 64 < BW * CPR;
      const int p2 = isw ? pos : pos - BW * CPR;
      const int row = p2 / CPR, c = (p2 % CPR) ^ (row & (CPR - 1));
      const int grow = min((isw ? w0 : t0) + row, (isw ? Nw : Tv) - 1);
      gsrc[i] = (isw ? W : X) + (size_t)grow * K + c * 8;
      kc[i] = c * 8;
    }
    const uint32_t lds0 = lds_addr_of(sm) + (uint32_t)(__builtin_amdgcn_readfirstlane(wid) * IPW) * 1024u;
    auto issue = [&](int kt) {
      const uint32_t stage = lds0 + (uint32_t)((kt % STAGES) * CH) * 16u;
      const int k0 = (kb + kt) * KD;
#pragma unroll
      for (int i = 0; i < IPW; ++i) {
        const bf16_t* g = gsrc[i] + k0;
        if constexpr (KTAIL)
          if (k0 + kc[i] >= K) g = reinterpret_cast<const bf16_t*>(g_zero_chunk);
        dma16_lds(g, stage + (uint32_t)i * 1024u);
      }
    };
    auto frag = [&](int kt, int ks, bf16x8_t(&a)[SW], bf16x8_t(&b)[ST]) {
      const uint4* stage = sm + (kt % STAGES) * CH;
      const int c = 4 * ks + fchunk;
#pragma unroll
      for (int i = 0; i < SW; ++i) {
        const int r = wave_w * TW + 16 * i + frow;
        a[i] = __builtin_bit_cast(bf16x8_t, stage[r * CPR + (c ^ (r & (CPR - 1)))]);
      }
#pragma unroll
      for (int j = 0; j < ST; ++j) {
        const int r = wave_t * TT + 16 * j + frow;
        b[j] = __builtin_bit_cast(bf16x8_t, stage[BW * CPR + r * CPR + (c ^ (r & (CPR - 1)))]);
      }
    };
    f32x4_t acc[SW][ST];
#pragma unroll
    for (int i = 0; i < SW; ++i)
#pragma unroll
      for (int j = 0; j < ST; ++j) acc[i][j] = f32x4_t{0.f, 0.f, 0.f, 0.f};
    auto mma = [&](const bf16x8_t(&a)[SW], const bf16x8_t(&b)[ST]) {
#pragma unroll
      for (int i = 0; i < SW; ++i)
#pragma unroll
        for (int j = 0; j < ST; ++j) acc[i][j] = mfma16(a[i], b[j], acc[i][j]);
    };

    auto mma_rows = [&](const bf16x8_t(&a)[SW], const bf16x8_t(&b)[ST], int i0, int i1) {
#pragma unroll
      for (int i = 0; i < SW; ++i)
        if (i >= i0 && i < i1)
#pragma unroll
          for (int j = 0; j < ST; ++j) acc[i][j] = mfma16(a[i], b[j], acc[i][j]);
    };
#pragma unroll
    for (int st = 0; st < STAGES; ++st)
      if (st < nk) issue(st);
    if constexpr (Epi::kKind == kEpiQkv)
      if (epi.o.kc) epi.carry(w0, BW, t0, min(t0 + BT, Tv), Nw, tid, NWAVE * 64);
    wait_stages<IPW, STAGES - 1>(min(STAGES, nk) - 1);  // stage 0 landed
    lds_barrier();
    bf16x8_t fa[2][SW], fb[2][ST];
    if (nk > 0) frag(0, 0, fa[0], fb[0]);
    for (int kt = 0; kt + 1 < nk; ++kt) {
#pragma unroll
      for (int s = 0; s < KS; ++s) {
        if (s + 1 < KS) {
          frag(kt, s + 1, fa[(s + 1) & 1], fb[(s + 1) & 1]);
        } else {
          // stage kt + 1 landed (stages kt + 2 .. min(nk - 1, kt + STAGES - 1) may still fly);
          // after the barrier every wave holds stage kt in registers, so its buffer is refilled
          wait_stages<IPW, STAGES - 2>(min(STAGES - 2, nk - 2 - kt));
          lds_barrier();
          if constexpr (STAGES >= 3) {
            // the next stage's first fragments go out first, and the refill is issued between two
            // halves of this substep's MFMAs, so its address work overlaps the matrix pipe
            frag(kt + 1, 0, fa[0], fb[0]);
            mma_rows(fa[s & 1], fb[s & 1], 0, (SW + 1) / 2);
            if (kt + STAGES < nk) issue(kt + STAGES);
            mma_rows(fa[s & 1], fb[s & 1], (SW + 1) / 2, SW);
            continue;
          } else {
            // one stage in flight: the refill goes out at once, ahead of everything else
            if (kt + STAGES < nk) issue(kt + STAGES);
            frag(kt + 1, 0, fa[0], fb[0]);
          }
        }
        mma(fa[s & 1], fb[s & 1]);
      }
    }
    if (nk > 0) {
#pragma unroll
      for (int s = 0; s < KS; ++s) {
        if (s + 1 < KS) frag(nk - 1, s + 1, fa[(s + 1) & 1], fb[(s + 1) & 1]);
        mma(fa[s & 1], fb[s & 1]);
      }
    }

    epi.template apply<SW, ST>(acc, w0 + wave_w * TW, t0 + wave_t * TT, lane, Nw, Tv, tile_w, split);
    lds_barrier();  // the next unit's prologue overwrites LDS the epilogue may still read
  }
}

// ---------------------------------------------------------------- the two-phase kernel
// The large tiles. Eight waves, two per SIMD, as 2 (weight rows) x 4 (tokens); the two waves of a SIMD run
// half a phase apart, so while one issues its MFMAs the other reads its fragments and issues the DMA:
//
//   interval        2j          2j+1         2j+2
//   waves 0-3    read phase j   MFMA j     read j+1
//   waves 4-7     MFMA j-1    read phase j   MFMA j       (a bare s_barrier between intervals)
//
// What bounds it: in gemm_kernel every wave of a workgroup reads fragments at the same time and then
// multiplies at the same time, so the LDS port and the matrix pipe take turns (256 x 256 tiles at 3072 x 37888
// x 3584: MFMA busy 56 % of the cycles). Half a phase apart they overlap: 69 %, at the clock that the power
// budget leaves then. In the step 679 -> 581 us (1437 TFLOP/s); 24576 x 1280 x 4096: 208 -> 183 us.
//
// A phase is one 64-deep K stage of all the wave's rows, or (two-stage rings, NPH = 2) half of the rows, so
// that half a stage's weights can be refilled a phase earlier: the LDS ring is the limit on the bytes in
// flight (64 KB per 256 x 256 stage). Order of the 1 KiB blocks of a stage, in LDS and for the DMA:
// [weight rows of phase 0][tokens][weight rows of phase 1]; block q is copied by wave q mod 8.
//   phase 0 of stage kt reads [.. tokens] and refills the previous stage's phase-1 rows (stage kt - 1 + S);
//   phase 1 reads the phase-1 rows and refills [.. tokens] of the same buffer (stage kt + S).
// A refill is safe: the rows were last read one phase earlier by the late waves (4-7), which wait for their
// reads (lgkmcnt) before the barrier that starts the refilling interval. A stage is complete: each wave waits
// for its own loads of the rows a phase needs (vmcnt; loads complete in order, and the same number per wave
// is issued after them) before the barrier that starts the first interval reading them: the late waves in
// their read interval, the early ones after their MFMAs, both in the interval just before.
// Barriers per unit, with P = nk * NPH phases: early waves 1 + 2P; late waves 1 + 1 + 2P - 1 (they start one
// interval later and skip the last). A K range without stages (nk = 0) has one barrier for both.
//
// Units as in gemm_kernel, but each XCD's run is walked in groups of `gw` weight tiles, all token tiles of
// a group in turn (weight tile innermost), so the 32 workgroups of an XCD cover about gw x 8 tiles and share
// both operands in its L2 (L2 misses limit the fill at thousands of tokens: of the case above 36 % of the requests
// miss at gw = 1, 25 % at 4). A workgroup issues the first stages of its next unit before the epilogue.
// A partly filled token tile computes only the ceil(valid / 64) token fragments a wave needs: fragment j of
// wave t is the tokens [64 j + 16 t, +16), so the valid ones spread over all waves. With COUNTED (a step's LM head) the
// same serves tiles of one fragment column fewer, where the rows fill those better (lmhead_tile_tokens).
__device__ __forceinline__ void phase_barrier() {
  __builtin_amdgcn_sched_barrier(0);
  asm volatile("s_barrier" ::: "memory");
  __builtin_amdgcn_sched_barrier(0);
}
template <int BW, int BT, int S, class Epi, bool COUNTED = false>
__global__ void __launch_bounds__(512)
gemm_pp_kernel(const bf16_t* __restrict__ W, const bf16_t* __restrict__ X, int Nw, int T, int K,
               const int32_t* __restrict__ t_count, int nsplit, int gw, uint64_t narrow, Epi epi) {
  constexpr int WW = 2, WT = 4, NPH = S == 2 ? 2 : 1;
  constexpr int TW = BW / WW, SW = TW / 16, ST = BT / 64, SWP = SW / NPH;
  constexpr int NB = (BW + BT) / 8, IPW = NB / 8;       // 1 KiB blocks per stage, loads per wave and stage
  constexpr uint32_t STAGE = (BW + BT) * 128;           // bytes per stage
  constexpr int QX = BW / 8 / NPH, Q0 = QX + BT / 8;    // blocks [0, QX) weights, [QX, Q0) tokens, [Q0, NB) weights
  static_assert(BW % 64 == 0 && BT % 64 == 0 && SW % NPH == 0 && S >= 2 && IPW * (S - 1) < 64, "tile shape");
  extern __shared__ __attribute__((aligned(1024))) uint4 sm[];

  const int Tv = t_count ? min(T, *t_count) : T;
  // tokens of a tile: with COUNTED one fragment column fewer where `narrow` says so for this many rows
  const int bt = COUNTED && Tv > 0 && (narrow >> min(63, (Tv - 1) / 64) & 1) ? BT - 64 : BT;
  const int nW = (Nw + BW - 1) / BW, nTt = (Tv + bt - 1) / bt;
  const int units = nW * nsplit * nTt;
  const int per = (units + 7) / 8;
  const int xcd = blockIdx.x & 7, stride = gridDim.x >> 3;
  const int run_end = min(units, (xcd + 1) * per);
  const int lane = threadIdx.x & 63, wid = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int wave_w = wid / WT, wave_t = wid % WT;
  const bool late = wid >= 4;
  const int frow = lane & 15, fchunk = lane >> 4;
  const uint32_t lds0 = lds_addr_of(sm);
  const int nk_all = K / 64, kper = (nk_all + nsplit - 1) / nsplit;
  // lane i of a block copies chunk i % 8 of row i / 8 (rows of 8 chunks, XOR-swizzled as in gemm_kernel)
  const uint32_t vchunk = (uint32_t)((lane & 7) ^ (lane >> 3)) * 16u;
  // a fragment read: row frow, chunk 4 ks + fchunk
  const uint32_t fo0 = (uint32_t)frow * 128u + (uint32_t)(fchunk ^ (frow & 7)) * 16u;
  const uint32_t fo1 = (uint32_t)frow * 128u + (uint32_t)((fchunk + 4) ^ (frow & 7)) * 16u;

  int L = xcd * per + (blockIdx.x >> 3);
  if (L >= run_end) return;
  const char *wbase, *xbase;
  uint32_t voff[IPW];
  int tile_w, split, w0, t0, nk, ste;
  auto setup = [&](int u) {
    split = u / (nW * nTt);
    const int r = u - split * (nW * nTt);
    const int g = r / (gw * nTt), rr = r - g * gw * nTt, gn = min(gw, nW - g * gw);
    const int tile_t = rr / gn;
    tile_w = g * gw + rr - tile_t * gn;
    w0 = tile_w * BW;
    t0 = tile_t * bt;
    ste = min(bt / 64, (Tv - t0 + 63) / 64);
    const int kb = min(nk_all, split * kper);
    nk = min(nk_all, kb + kper) - kb;
    wbase = reinterpret_cast<const char*>(W + (size_t)w0 * K + kb * 64);
    xbase = reinterpret_cast<const char*>(X + (size_t)t0 * K + kb * 64);
#pragma unroll
    for (int i = 0; i < IPW; ++i) {
      const int q = i * 8 + wid;
      int row;  // rows outside the operand are clamped to the last valid row, as in gemm_kernel
      if (q >= QX && q < Q0) {
        row = min((q - QX) * 8 + (lane >> 3), Tv - t0 - 1);
      } else {
        constexpr int HR = SWP * 16;  // weight rows of one wave and phase; LDS order: phase, wave, row
        const int slot = (q < QX ? q : q - BT / 8) * 8 + (lane >> 3);
        const int ph = slot / (WW * HR), r2 = slot % (WW * HR);
        row = min((r2 / HR) * TW + ph * HR + r2 % HR, Nw - w0 - 1);
      }
      voff[i] = (uint32_t)row * (uint32_t)K * 2u + vchunk;
    }
  };
  auto copy = [&](int kt, int i) {
    const int q = i * 8 + wid;
    dma16_sv((q >= QX && q < Q0 ? xbase : wbase) + (size_t)kt * 128, voff[i],
             lds0 + (uint32_t)(kt % S) * STAGE + (uint32_t)q * 1024u);
  };
  auto issue0 = [&](int kt) {  // phase-0 weights and tokens
#pragma unroll
    for (int i = 0; i < IPW; ++i)
      if ((i + 1) * 8 <= Q0) copy(kt, i);
      else if (i * 8 < Q0) {
        if (wid < Q0 - i * 8) copy(kt, i);
      }
  };
  auto issue1 = [&](int kt) {  // phase-1 weights (none with NPH = 1)
#pragma unroll
    for (int i = 0; i < IPW; ++i)
      if (i * 8 >= Q0) copy(kt, i);
      else if ((i + 1) * 8 > Q0) {
        if (wid >= Q0 - i * 8) copy(kt, i);
      }
  };
  auto prologue = [&]() {
#pragma unroll
    for (int st = 0; st < S; ++st)
      if (st < nk) {
        issue0(st);
        issue1(st);
      }
  };

  setup(L);
  prologue();
  while (true) {
    f32x4_t acc[SW][ST];
#pragma unroll
    for (int i = 0; i < SW; ++i)
#pragma unroll
      for (int j = 0; j < ST; ++j) acc[i][j] = f32x4_t{0.f, 0.f, 0.f, 0.f};
    if constexpr (Epi::kKind == kEpiQkv)
      if (epi.o.kc) epi.carry(w0, BW, t0, min(t0 + bt, Tv), Nw, threadIdx.x, 512);
    wait_stages<IPW, S - 1>(min(S, nk) - 1);
    phase_barrier();
    if (late && nk > 0) phase_barrier();
    // instantiated twice: for a full token tile, and with a scalar branch around each fragment column
    auto main_loop = [&](auto full_tile) {
      constexpr bool kFull = decltype(full_tile)::value;
      bf16x8_t fa[SWP][2], fb[ST][2];
      for (int kt = 0; kt < nk; ++kt) {
        const char* stage = reinterpret_cast<const char*>(sm) + (uint32_t)(kt % S) * STAGE;
#pragma unroll
        for (int ph = 0; ph < NPH; ++ph) {
          const char* sa = stage + (ph ? Q0 : 0) * 1024 + wave_w * (SWP * 2048);
          const char* sb = stage + QX * 1024 + wave_t * 2048;
          if (ph == 0) {
#pragma unroll
            for (int j = 0; j < ST; ++j)
              if (kFull || j == 0 || j < ste) {
                fb[j][0] = *reinterpret_cast<const bf16x8_t*>(sb + j * 8192 + fo0);
                fb[j][1] = *reinterpret_cast<const bf16x8_t*>(sb + j * 8192 + fo1);
              }
          }
#pragma unroll
          for (int i = 0; i < SWP; ++i) {
            fa[i][0] = *reinterpret_cast<const bf16x8_t*>(sa + i * 2048 + fo0);
            fa[i][1] = *reinterpret_cast<const bf16x8_t*>(sa + i * 2048 + fo1);
          }
          __builtin_amdgcn_sched_barrier(0);
          if (NPH == 1 || ph == 1) {
            const int nx = NPH == 1 ? kt - 1 + S : kt + S;
            if ((NPH == 2 || kt > 0) && nx < nk) issue0(nx);
          } else if (kt > 0 && kt - 1 + S < nk) {
            issue1(kt - 1 + S);
          }
          // stages that may still fly while the next phase reads
          auto landed = [&]() {
            if (NPH == 1) wait_stages<IPW, S - 2>(min(S - 2, max(0, nk - 2 - kt)));
            else wait_stages<IPW, S - 1>(min(S - 1, max(0, nk - 1 - ph - kt)));
          };
          if (late) landed();
          asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
          phase_barrier();
          __builtin_amdgcn_s_setprio(1);
          if constexpr (kFull) {
#pragma unroll
            for (int ks = 0; ks < 2; ++ks)
#pragma unroll
              for (int i = 0; i < SWP; ++i)
#pragma unroll
                for (int j = 0; j < ST; ++j)
                  acc[ph * SWP + i][j] = mfma16(fa[i][ks], fb[j][ks], acc[ph * SWP + i][j]);
          } else {
#pragma unroll
            for (int j = 0; j < ST - 1; ++j)
              if (j == 0 || j < ste)
#pragma unroll
                for (int ks = 0; ks < 2; ++ks)
#pragma unroll
                  for (int i = 0; i < SWP; ++i)
                    acc[ph * SWP + i][j] = mfma16(fa[i][ks], fb[j][ks], acc[ph * SWP + i][j]);
          }
          __builtin_amdgcn_s_setprio(0);
          __builtin_amdgcn_sched_barrier(0);
          if (!late) landed();
          if (!(late && ph == NPH - 1 && kt == nk - 1)) phase_barrier();
        }
      }
    };
    if (ST == 1 || ste == ST) main_loop(std::true_type{});
    else main_loop(std::false_type{});
    const int ew = w0, et = t0, etile = tile_w, esplit = split;
    L += stride;
    const bool more = L < run_end;
    if (more) {  // every wave's reads of the ring completed before the last barrier
      setup(L);
      prologue();
    }
    epi.template apply<SW, ST, WT>(acc, ew + wave_w * TW, et + wave_t * 16, lane, Nw,
                                COUNTED ? min(et + bt, Tv) : Tv, etile, esplit);
    if (!more) break;
  }
}

// ---------------------------------------------------------------- planning and dispatch
struct TileCfg {
  int bw, bt, kd, stages, ww, wt, pp;  // pp = 1: gemm_pp_kernel, 0: gemm_kernel
};
static const TileCfg kCfgs[] = {
    {128, 128, 64, 2, 2, 4, 0}, {64, 64, 64, 4, 2, 2, 0},   {96, 192, 64, 3, 3, 4, 0},  {256, 256, 64, 2, 2, 4, 1},
    {256, 192, 64, 2, 2, 4, 1}, {256, 128, 64, 3, 2, 4, 1}, {256, 64, 64, 4, 2, 4, 1},  {192, 256, 64, 2, 2, 4, 1},
    {192, 192, 64, 3, 2, 4, 1}, {192, 128, 64, 4, 2, 4, 1}, {192, 64, 64, 4, 2, 4, 1},  {128, 256, 64, 3, 2, 4, 1},
    {128, 192, 64, 4, 2, 4, 1}, {128, 128, 64, 4, 2, 4, 1}, {128, 64, 64, 3, 2, 4, 1},
    // one token tile of weights streamed (stream_cfg)
    {32, 32, 128, 4, 2, 2, 0},  {32, 64, 128, 6, 1, 4, 0},  {48, 64, 128, 5, 1, 4, 0},  {96, 64, 128, 3, 2, 2, 0},
    {128, 192, 64, 3, 2, 4, 0},  // residual GEMMs with full token tiles, heads of one round (plan_gemm)
};
constexpr int kModelCfgs = 15;  // the first ones: those that the cost model chooses from
constexpr int kNumCfgs = sizeof(kCfgs) / sizeof(kCfgs[0]);
constexpr int kCUs = 256;
constexpr size_t kLdsBytes = 160 * 1024;  // LDS per CU (gfx950)

static size_t cfg_lds(const TileCfg& c) { return (size_t)c.stages * (c.bw + c.bt) * (c.kd / 8) * 16; }

// force_bw != 0 (the LM head): each wave owns a whole vocabulary tile of force_bw ids, or the tile is
// force_bw weight rows split over exactly kLmWaves of the 8 waves, the layout the top-2 epilogue's cross-wave
// merge is written for.
static bool lm_ok(const TileCfg& c, int force_bw) {
  if (!force_bw) return true;
  if (c.bw / c.ww == force_bw) return true;
  return c.bw == force_bw && c.ww == kLmWaves && c.ww * c.wt == 8 &&
         cfg_lds(c) + sizeof(Part) * kLmWaves * c.bt <= kLdsBytes;
}

// Whether a step's scored rows choose the tokens per tile under LM-head plan `p` (lmhead_tile_tokens).
static bool rows_choose(const GemmPlan& p) { return p.cfg == 3 || p.cfg == 4; }

// Configurations of the LM head alone (256 x 64, 128 x 64).
static constexpr bool lm_only(int ci) { return ci == 6 || ci == 14; }

struct TileCost {
  double a, b0, b1, m;
};
static const TileCost kCost[2 * kModelCfgs] = {
#include "gemm_tuned.inc"
};

// Estimated time (us) of a GEMM with configuration `ci` and n K splits: launch + rounds of resident workgroups,
// each round a unit's fixed part plus its stages. A stage also takes no less than the weight rows that the
// resident workgroups share out need from HBM (each distinct row once) at 5.4 TB/s, the rate the streaming
// cases reach. Split-K slices are charged the read of the next RMSNorm (5 TB/s: 25 MB of them
// lengthen a norm of 384 tokens by 4.5 us, 63 MB one of 1280 by 12.5).
static double plan_cost(int ci, bool lm, int n, int Nw, int T, int K) {
  const TileCfg& c = kCfgs[ci];
  const TileCost& k = kCost[(lm ? kModelCfgs : 0) + ci];
  const int nW = (Nw + c.bw - 1) / c.bw, nT = (T + c.bt - 1) / c.bt;
  const double units = (double)nW * nT * n;
  const int nk = ((K + 63) / 64 + n - 1) / n;
  const int per_cu = std::max(1, std::min<int>(c.pp ? 2 : 4, (int)(kLdsBytes / cfg_lds(c))));
  const double slots = (double)kCUs * per_cu, active = std::min(units, slots);
  const double rounds = std::ceil(units / slots);
  // 64-token fragments computed: gemm_pp_kernel skips those past the last token
  const double full = c.bt / 64.0, last = c.pp ? (double)((T - (nT - 1) * c.bt + 63) / 64) : full;
  const double f = rounds > 1 ? (full * (nT - 1) + last) / nT : (nT > 1 ? full : last);
  double stage = k.b0 + k.b1 * f;
  if (active > kCUs) stage *= 1.0 + (std::ceil(active / kCUs) - 1.0) * k.m;  // the CUs that hold one more set the time
  const double hbm = std::max(1.0, active / nT) * c.bw * 128.0 / 5.4e6;
  const double s4 = stage * stage * stage * stage, h4 = hbm * hbm * hbm * hbm;
  stage = std::sqrt(std::sqrt(s4 + h4));
  return 4.0 + rounds * (k.a + nk * stage) + (n > 1 ? n * (double)T * Nw * 4.0 / 5e6 : 0.0);
}

#if DCL_GEMM_PART == 1
// At most 64 tokens without a K split: the time is that of streaming the weights, and what decides it is how evenly
// the CUs share them and how much each has in flight, so the smallest tile whose units fit one round of the CUs is
// taken, with 128-deep stages (256 contiguous bytes of each weight row per load) filling the LDS. Against the
// 64 x 64 tiles with 64-deep stages that the cost model picks (weights from HBM, us):
//   64 tokens: 12288 x 4096 26.4 -> 24.3 (48 rows: 256 units, 64 rows: 192), 24576 x 4096 46.7 -> 43.0 (96 rows),
//              4608 x 3584 20.0 -> 15.4 (32 rows); other widths lose (33.5 and 30.4 for 12288 with 32 and 96 rows)
//   24 tokens, 32 x 32 tiles (their activations are half the loads): 24.4 -> 23.1, 41.3 -> 36.7, 17.7 -> 11.2
//   12289 to 16384 rows: 64 x 64 tiles have the unit per CU (16384 x 2048: 19.3, 96 rows 21.4; 16 tokens 18.6, 32 x 32
//              tiles 19.9)
// More weight rows than 96 x 256 (37888 x 3584 at 24 tokens: 192 x 64 tiles 48.5, 32 x 32 tiles 50.5), and residual
// GEMMs (four K slices already give 64 x 64 tiles a unit per CU): the cost model.
static int stream_cfg(int Nw, int T, int K) {
  if (T > 64 || K % 128 != 0) return -1;
  for (int ci : {16, 17, 1, 18})
    if (Nw <= kCfgs[ci].bw * kCUs) return ci != 1 && T <= 32 ? 15 : ci;
  return -1;
}

GemmPlan plan_gemm(int Nw, int T, int K, int force_bw, int max_split) {
  GemmPlan best{0, 1, 0};
  double best_t = 1e30;
  const bool lm = force_bw != 0;
  const int nk = (K + 63) / 64;
  const int sc = lm || max_split > 1 ? -1 : stream_cfg(Nw, T, K);
  if (sc >= 0) best.cfg = sc;
  for (int ci = 0; sc < 0 && ci < kModelCfgs; ++ci) {
    // K not a multiple of the stage depth: one tail-aware configuration (128 x 128, 64-deep stages, which also
    // suits the LM head's split layout) serves every such shape, so the others carry no tail handling. It is
    // the slower kernel everywhere else; 256 x 64 and 128 x 64 tiles pay only under the LM head (they halve the last
    // round).
    if ((K % kCfgs[ci].kd != 0) != (ci == 0)) continue;
    if (!lm && lm_only(ci)) continue;
    if (!lm_ok(kCfgs[ci], force_bw)) continue;
    for (int n = 1; n <= max_split && (n == 1 || (n - 1) * ((nk + n - 1) / n) < nk); ++n) {
      const double t = plan_cost(ci, lm, n, Nw, T, K);
      if (t < best_t * 0.999) {
        best_t = t;
        best.cfg = ci;
        best.nsplit = n;
      }
    }
  }
  // 128 x 192 tiles of a residual GEMM whose last token tile has no empty fragment: the two-phase kernel has nothing
  // to skip there, and the ring kernel's three stages are 1 - 4 % faster than its four (in the layer: 4096 x 384 x 4096
  // 23.7 -> 22.7 us, K = 12288 47.9 -> 47.3, 3584 x 384 x 18944 64.6 -> 63.3; with a partly filled last tile up to 13 %
  // slower, 3584 x 448 x 18944).
  if (best.cfg == 12 && max_split > 1 && (T - 1) % 192 >= 128) best.cfg = 19;
  auto tiles = [&](int ci) {
    const TileCfg& c = kCfgs[ci];
    return ((Nw + c.bw - 1) / c.bw) * ((T + c.bt - 1) / c.bt);
  };
  // The LM head of a small vocabulary, where one round of 128 x 192 tiles holds it and the model's choice is 256 x 128 or
  // 128 x 256 ones: these leave CUs idle or fragments empty, and a unit per CU is bound by the bytes that it has in flight.
  // 32000 x 4096 at 129 - 192 rows 67 -> 55 us, 16384 x 2048 at 384 rows 38 -> 32, 6000 x 4096 at 900 rows 74 -> 53; of 66
  // such heads one is slower (14000 x 512, 384 rows: 21.0, 22.1). Where the model takes 128 x 128, 256 x 64 or 128 x 64
  // tiles those are the faster ones (16384 x 4096, 250 rows: 44, 55 here).
  if (lm && (best.cfg == 5 || best.cfg == 11) && tiles(19) <= kCUs) best.cfg = 19;
  best.tiles = tiles(best.cfg);
  return best;
}

// Tokens per tile of a step's LM head with R scored rows. A step knows its tokens on the host, the scored rows (what
// follows the prompt, less as decoding goes on) only on the device, and the plan for its tokens can be far off for
// the rows: of 126464 ids, 256 x 192 tiles, best for 384 rows, take 289 us for 256 of them, 256 x 256 tiles 220; for 300 rows
// it is 306 and 371. So where the plan is one of these two the 256 x 256 kernel runs and takes 192 or 256 tokens per
// tile by the count, 64 rows at a time. Timed both ways (vocabularies of 32000 to 152064 ids, 129 to 4000 rows) this
// rule is 0.06 % from the better one, at most 2.7 %; it asks 5 % of the model's costs for 192, which leave a quarter
// of the tile's loads unused and so are up to 7 % slower than 256 x 192 tiles (384 of 384 rows 351 us, 343).
int lmhead_tile_tokens(int V, int R, int K) {
  return plan_cost(4, true, 1, V, R, K) < 0.95 * plan_cost(3, true, 1, V, R, K) ? 192 : 256;
}

GemmPlan plan_lmhead_step(int V, int T, int K, int* tokens) {
  GemmPlan p = plan_gemm(V, T, K, kLmTile, 1);
  if (rows_choose(p)) p.cfg = 3;
  *tokens = p.cfg == 3 ? lmhead_tile_tokens(V, T, K) : kCfgs[p.cfg].bt;
  return p;
}

void gemm_cfg_shape(int cfg, int* shape) {
  const TileCfg& c = kCfgs[cfg >= 0 && cfg < kNumCfgs ? cfg : 0];
  shape[0] = c.bw;
  shape[1] = c.bt;
  shape[2] = c.kd;
  shape[3] = c.stages;
  shape[4] = c.ww;
  shape[5] = c.wt;
}
#endif

// Per instantiation: the ring plus the epilogue's static LDS fit in a CU, and (once per device) the kernel's
// dynamic-LDS limit is raised.
static bool prepare_kernel(const void* kern, size_t lds, std::atomic<int>& fits, std::atomic<uint32_t>& lds_set) {
  if (fits.load(std::memory_order_acquire) < 0) {  // -1 = not yet known
    hipFuncAttributes at{};
    fits.store(hipFuncGetAttributes(&at, kern) == hipSuccess && at.sharedSizeBytes + lds <= kLdsBytes,
               std::memory_order_release);
  }
  if (!fits.load(std::memory_order_acquire)) return false;
  ensure_dynamic_lds(kern, lds, lds_set);
  return true;
}

template <int BW, int BT, int KD, int STAGES, int WW, int WT, class Epi, bool KTAIL = false>
static bool run_cfg(const bf16_t* W, const bf16_t* X, int Nw, int T, int K, const int32_t* t_count, int nsplit,
                    const Epi& epi, hipStream_t s) {
  const int units = ((Nw + BW - 1) / BW) * ((T + BT - 1) / BT) * nsplit;
  if (units == 0) return true;
  // One workgroup per unit; with a device-side row count the grid is capped (workgroups stride
  // over the units that turn out to be active) so inactive token tiles cost no dispatch.
  int grid = 8 * ((units + 7) / 8);
  if (t_count && grid > 8 * kCUs) grid = 8 * kCUs;
  const size_t lds = (size_t)STAGES * (BW + BT) * (KD / 8) * 16;
  auto kern = gemm_kernel<BW, BT, KD, STAGES, WW, WT, Epi, KTAIL>;
  static std::atomic<int> fits{-1};
  static std::atomic<uint32_t> lds_set{0};
  if (!prepare_kernel(reinterpret_cast<const void*>(kern), lds, fits, lds_set)) return false;
  hipLaunchKernelGGL(kern, dim3(grid), dim3(WW * WT * 64), lds, s, W, X, Nw, T, K, t_count, nsplit, epi);
  return true;
}

// Weight tiles walked together by an XCD (see gemm_pp_kernel): 4 x 8 tiles of the 32 workgroups.
constexpr int kGroupW = 4;

template <int BW, int BT, int S, class Epi>
static bool run_pp(const bf16_t* W, const bf16_t* X, int Nw, int T, int K, const int32_t* t_count, int nsplit,
                   const Epi& epi, hipStream_t s) {
  const int units = ((Nw + BW - 1) / BW) * ((T + BT - 1) / BT) * nsplit;
  if (units == 0) return true;
  constexpr size_t lds = (size_t)S * (BW + BT) * 128;
  constexpr int slots = kCUs * (2 * lds <= kLdsBytes ? 2 : 1);  // resident workgroups; they stride over the units
  const int grid = std::min(8 * ((units + 7) / 8), slots);
  auto kern = gemm_pp_kernel<BW, BT, S, Epi>;
  static std::atomic<int> fits{-1};
  static std::atomic<uint32_t> lds_set{0};
  if (!prepare_kernel(reinterpret_cast<const void*>(kern), lds, fits, lds_set)) return false;
  hipLaunchKernelGGL(kern, dim3(grid), dim3(512), lds, s, W, X, Nw, T, K, t_count, nsplit, kGroupW, 0, epi);
  return true;
}

static_assert(kNumCfgs == 20, "run_plan dispatches every configuration of kCfgs");

// Whether the epilogue has a kernel for configuration CI: the LM head runs only the layouts of lm_ok, the debug
// logits (test support) one tile, and the 128 x 192 ring serves residual GEMMs and the LM head.
template <class Epi, int CI>
constexpr bool has_cfg() {
  if (Epi::kKind == kEpiLm) return (CI >= 3 && CI <= 6) || CI == 11 || CI == 13 || CI == 14 || CI == 19;
  if (Epi::kKind == kEpiDebug) return CI == 13;
  return !lm_only(CI) && (CI != 19 || Epi::kKind == kEpiResid);
}

template <class Epi>
static void run_plan(const GemmPlan& p, const bf16_t* W, const bf16_t* X, int Nw, int T, int K, const int32_t* t_count,
                     const Epi& epi, hipStream_t s) {
  const int n = p.nsplit;
  bool ok = false;
#define DCL_RING(CI, ...) \
  case CI: if constexpr (has_cfg<Epi, CI>()) ok = run_cfg<__VA_ARGS__>(W, X, Nw, T, K, t_count, n, epi, s); break
#define DCL_PP(CI, ...) \
  case CI: if constexpr (has_cfg<Epi, CI>()) ok = run_pp<__VA_ARGS__>(W, X, Nw, T, K, t_count, n, epi, s); break
  if (K % kCfgs[p.cfg].kd == 0) {
    switch (p.cfg) {
      DCL_RING(1, 64, 64, 64, 4, 2, 2);
      DCL_RING(2, 96, 192, 64, 3, 3, 4);
      DCL_PP(3, 256, 256, 2);
      DCL_PP(4, 256, 192, 2);
      DCL_PP(5, 256, 128, 3);
      DCL_PP(6, 256, 64, 4);
      DCL_PP(7, 192, 256, 2);
      DCL_PP(8, 192, 192, 3);
      DCL_PP(9, 192, 128, 4);
      DCL_PP(10, 192, 64, 4);
      DCL_PP(11, 128, 256, 3);
      DCL_PP(12, 128, 192, 4);
      DCL_PP(13, 128, 128, 4);
      DCL_PP(14, 128, 64, 3);
      DCL_RING(15, 32, 32, 128, 4, 2, 2);
      DCL_RING(16, 32, 64, 128, 6, 1, 4);
      DCL_RING(17, 48, 64, 128, 5, 1, 4);
      DCL_RING(18, 96, 64, 128, 3, 2, 2);
      DCL_RING(19, 128, 192, 64, 3, 2, 4);
    }
  }
#undef DCL_RING
#undef DCL_PP
  // Configuration 0 (K tails); also a ring that does not fit (never planned: plans respect kLdsBytes), rather
  // than a launch the runtime would reject. The tail-aware kernel is correct for every shape and always fits.
  if (!ok) run_cfg<128, 128, 64, 2, 2, 4, Epi, true>(W, X, Nw, T, K, t_count, n, epi, s);
}

// The wrappers below are compiled as three objects (DCL_GEMM_PART 1-3, in parallel).
#if DCL_GEMM_PART == 1
void gemm_qkv(const bf16_t* W, const bf16_t* X, int Nw, int T, int K, const QkvOut& o, hipStream_t s) {
  run_plan(plan_gemm(Nw, T, K, 0, 1), W, X, Nw, T, K, nullptr, EpiQkv{o}, s);
}
#endif
#if DCL_GEMM_PART == 2
int gemm_resid(const bf16_t* W, const bf16_t* X, int Nw, int T, int K, float* r, float* P, hipStream_t s) {
  const GemmPlan p = plan_gemm(Nw, T, K, 0, P ? kMaxSplit : 1);
  if (p.nsplit > 1) {
    run_plan(p, W, X, Nw, T, K, nullptr, EpiPartial{P, (size_t)T * Nw}, s);
    return p.nsplit;
  }
  run_plan(p, W, X, Nw, T, K, nullptr, EpiResid{r}, s);
  return 0;
}
#endif
#if DCL_GEMM_PART == 3
void gemm_swiglu(const bf16_t* W, const bf16_t* X, int Nw, int T, int K, bf16_t* a, hipStream_t s) {
  run_plan(plan_gemm(Nw, T, K, 0, 1), W, X, Nw, T, K, nullptr, EpiSwiglu{a}, s);
}
void gemm_store_f32(const bf16_t* W, const bf16_t* X, int Nw, int T, int K, float* out, hipStream_t s) {
  const GemmPlan p{K % 64 ? 0 : 13, 1, 0};
  run_plan(p, W, X, Nw, T, K, nullptr, EpiF32{out}, s);
}
// A step's LM head: its tokens' plan, except where that is one of the tiles of 256 ids over 192 or 256 tokens.
static bool run_counted(const GemmPlan& p, const bf16_t* W, const bf16_t* X, int V, int T, int K, const LmOut& o,
                        hipStream_t s) {
  if (!o.count || !rows_choose(p)) return false;
  uint64_t narrow = 0;
  for (int i = 0; i < 64 && 64 * i < T; ++i)
    if (lmhead_tile_tokens(V, 64 * (i + 1), K) == 192) narrow |= (uint64_t)1 << i;
  using Epi = EpiLm<kLmTile, kLmWaves>;
  constexpr size_t lds = 2 * (256 + 256) * 128;
  auto kern = gemm_pp_kernel<256, 256, 2, Epi, true>;
  static std::atomic<int> fits{-1};
  static std::atomic<uint32_t> lds_set{0};
  if (!prepare_kernel(reinterpret_cast<const void*>(kern), lds, fits, lds_set)) return false;
  const int units = ((V + 255) / 256) * ((T + 191) / 192);  // of the narrower tiles
  hipLaunchKernelGGL(kern, dim3(std::min(8 * ((units + 7) / 8), kCUs)), dim3(512), lds, s, W, X, V, T, K, o.count, 1,
                     kGroupW, narrow, Epi{o});
  return true;
}
void gemm_lmhead(const bf16_t* W, const bf16_t* X, int V, int T, int K, const LmOut& o, hipStream_t s) {
  static_assert(kLmTile == 128 && kLmWaves == 2, "the LM-head vocabulary tile is the GEMM's weight tile");
  const GemmPlan p = plan_gemm(V, T, K, kLmTile, 1);
  if (run_counted(p, W, X, V, T, K, o, s)) return;
  run_plan(p, W, X, V, T, K, o.count, EpiLm<kLmTile, kLmWaves>{o}, s);
}
#endif

}  // namespace dcl
