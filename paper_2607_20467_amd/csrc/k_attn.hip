// Non-causal (bidirectional) flash-style attention for gfx950, MHA and GQA, head_dim 64 / 128.
//
// Masked diffusion LMs attend from every position to every position; there is no causal mask, so
// the whole S x S score matrix is real work. One workgroup handles 16*NQ queries of one (batch,
// head); each wavefront owns 16 queries and walks its share of the keys in tiles of KT (32 or 64)
// with an online softmax in float32. Keys are [cached prefix (P) || the S fresh tokens].
//
// Orientation: the score tile is computed transposed, S^T = K Q^T (MFMA A = K from LDS, B = Q held
// in registers), so each lane holds 16 scores of ONE query. Its softmax probabilities then feed the
// P*V product directly as the MFMA B operand of O^T = V^T P^T, with V^T read from a key-contiguous
// LDS tile in the matching key order; no register shuffle of P is needed.
// P is split into three bf16 parts (hi + mid + lo, three MFMAs), so the probabilities enter the
// product with at least 24 significant bits, as in a float32 evaluation. Two parts (16 bits) were
// measurably less accurate than float32: on sequences of 5-8 tokens they flipped the bf16 rounding
// of about a quarter of the final hidden states of a small model against a float64 reference.
#include <type_traits>

#include "dcl_internal.h"

namespace dcl {



__device__ __forceinline__ f32x4_t mfma16a(const bf16x8_t& a, const bf16x8_t& b, const f32x4_t& c) {
  return __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, b, c, 0, 0, 0);
}

// op(v, v of lane ^ 16) and op(v, v of lane ^ 32) in every lane, through the gfx950 lane-swap
// instructions (no LDS round trip). The swap of a register with itself leaves, per lane, the
// value of both partners in the two results; op must be commutative.
template <class Op>
__device__ __forceinline__ float xor_lanes16(float v, Op op) {
  const int b = __builtin_bit_cast(int, v);
  const auto p = __builtin_amdgcn_permlane16_swap(b, b, false, false);
  return op(__builtin_bit_cast(float, (int)p[0]), __builtin_bit_cast(float, (int)p[1]));
}
template <class Op>
__device__ __forceinline__ float xor_lanes32(float v, Op op) {
  const int b = __builtin_bit_cast(int, v);
  const auto p = __builtin_amdgcn_permlane32_swap(b, b, false, false);
  return op(__builtin_bit_cast(float, (int)p[0]), __builtin_bit_cast(float, (int)p[1]));
}

// A wave-uniform address that the compiler computed in vector registers, in scalar ones.
__device__ __forceinline__ const bf16_t* uniform_ptr(const bf16_t* p) {
  const uint64_t v = reinterpret_cast<uint64_t>(p);
  const uint32_t lo = __builtin_amdgcn_readfirstlane((uint32_t)v), hi = __builtin_amdgcn_readfirstlane((uint32_t)(v >> 32));
  return reinterpret_cast<const bf16_t*>(((uint64_t)hi << 32) | lo);
}

template <int N>
__device__ __forceinline__ void attn_wait_vmcnt() {
  __builtin_amdgcn_s_waitcnt((N & 15) | (7 << 4) | (15 << 8) | ((N >> 4) << 14));
}
// Wait until all but this wave's `newer` most recently issued stages (IPW loads each) landed.
template <int IPW, int MAXN>
__device__ __forceinline__ void attn_wait_stages(int newer) {
  if constexpr (MAXN > 0) {
    static_assert(MAXN * IPW < 64, "vmcnt range");
    if (newer >= MAXN) {
      attn_wait_vmcnt<MAXN * IPW>();
      return;
    }
    attn_wait_stages<IPW, MAXN - 1>(newer);
  } else {
    attn_wait_vmcnt<0>();
  }
}

// K and V^T tiles move HBM/L2 -> LDS with global_load_lds_dwordx4 into a STAGES-deep ring (no
// register staging, no padding). K rows (DH/8 chunks of 16 bytes) are XOR-swizzled by the key
// index, V^T rows (KT/8 chunks of 8 keys) by the dimension index. Both are read in whole 16-byte
// chunks, bank-conflict free; the V^T fragments are then assembled by a lane-row swap (below).
// Chunks past the last key repeat real data (see below).
//
// What bounds it: per 16 queries x 32 keys (head_dim 128) a wave needs 512 matrix-pipe cycles (8 MFMAs for the
// scores, 24 for the three-part P V), about as many VALU cycles, and 16 KB of fragments through the LDS port
// (128 cycles, for four SIMDs again 512). So a wave takes QF x 16 queries: with QF = 2 each K and V^T fragment
// (and the lane-row swap of V^T) serves both.
//
// Key groups: the NQ * KG waves of a workgroup are NQ query waves (16 QF queries each) times KG key
// groups. Step t of the ring holds the KG key tiles t*KG .. t*KG + KG - 1; key group g works on
// tile t*KG + g, so each wave's serial chain (scores -> softmax -> P V) covers 1/KG of the keys
// and KG times as many waves hide each other's latencies. At the end the groups' running
// (max, sum, unnormalised output) are combined through LDS in group order, which keeps the result
// independent of timing.
template <int NQ, int QF, int KG, int KT, int DH, int STAGES>
__global__ void __launch_bounds__(NQ * KG * 64, 2) attn_kernel(AttnArgs a) {
  constexpr int BQ = 16 * NQ * QF, NWAVE = NQ * KG;
  constexpr int KC = DH / 8;           // chunks per K row
  constexpr int VC = KT / 8;           // chunks per V^T row
  constexpr int KCH = KT * KC;         // K chunks per tile
  constexpr int VCH = DH * VC;         // V^T chunks per tile
  constexpr int TCH = KCH + VCH;       // chunks per tile
  constexpr int SCH = KG * TCH;        // chunks per ring step
  constexpr int KI = KCH / 64 / NWAVE, TI = TCH / 64 / NWAVE;  // K / all load instructions per wave and key tile
  constexpr int IPW = KG * TI;         // load instructions per wave per ring step
  static_assert((KT == 32 || KT == 64) && (KCH / 64) % NWAVE == 0 && (VCH / 64) % NWAVE == 0 && STAGES >= 2 &&
                    IPW * (STAGES - 2) < 64 && NWAVE <= 16,
                "stage shape");
  static_assert(KG == 1 || (size_t)(KG - 1) * NQ * QF * ((DH / 16) * 64 * 16 + 64 * 8) <= (size_t)STAGES * SCH * 16,
                "the group merge reuses the ring");
  extern __shared__ __attribute__((aligned(1024))) uint4 sm[];

  // Units (batch, head, query tile), query tile innermost: XCD x (= blockIdx % 8) takes a contiguous
  // run of units, so the query tiles of one head (and the heads sharing a KV head) read their keys
  // and values through one L2.
  const int nqt = (a.S + BQ - 1) / BQ;
  const int units = nqt * a.H * a.B, per = (units + 7) / 8;
  const int L = (blockIdx.x & 7) * per + (blockIdx.x >> 3);
  if (L >= units) return;
  // in scalar registers: the quotients come from vector arithmetic, the loads below want scalar bases
  const int bh = __builtin_amdgcn_readfirstlane(L / nqt), b = __builtin_amdgcn_readfirstlane(bh / a.H);
  const int qt = L - bh * nqt, h = bh - b * a.H, g = __builtin_amdgcn_readfirstlane(h / (a.H / a.Hkv));
  const int tid = threadIdx.x, lane = tid & 63, wid = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int qw = wid % NQ, kg = wid / NQ;
  const int lq = lane & 15, lg = lane >> 4;
  const int S = a.S, P = a.P, Sk = a.Sk ? a.Sk : a.S, nkeys = P + Sk;  // S queries; P cached + Sk fresh keys
  const int q0 = qt * BQ + qw * (16 * QF);  // first query of the wave
  const int ntiles = (nkeys + KT - 1) / KT;
  const int nsteps = (ntiles + KG - 1) / KG;

  bf16x8_t qf[QF][DH / 32];
#pragma unroll
  for (int f = 0; f < QF; ++f) {
    const int qrow = q0 + 16 * f + lq;
    const bf16_t* qp = a.q + (((size_t)b * a.H + h) * S + (qrow < S ? qrow : 0)) * DH + 8 * lg;
#pragma unroll
    for (int ks = 0; ks < DH / 32; ++ks) {
      uint4 v = qrow < S ? *reinterpret_cast<const uint4*>(qp + 32 * ks) : make_uint4(0, 0, 0, 0);
      qf[f][ks] = __builtin_bit_cast(bf16x8_t, v);
    }
  }
  const size_t kvh = (size_t)b * a.Hkv + g;
  const bf16_t* kc = a.kc ? a.kc + kvh * a.Pc * DH : nullptr;
  const bf16_t* kf = a.k + kvh * Sk * DH;
  const bf16_t* vc = a.vc ? a.vc + kvh * DH * a.Pc : nullptr;
  const bf16_t* vf = a.vt + kvh * DH * a.Sp;

  f32x4_t o[QF][DH / 16];
#pragma unroll
  for (int f = 0; f < QF; ++f)
#pragma unroll
    for (int dt = 0; dt < DH / 16; ++dt) o[f][dt] = f32x4_t{0.f, 0.f, 0.f, 0.f};
  // per query: reference point m (log2 units, scaled; within 2^8 of the running maximum, see the
  // lazy rescaling below), the same in the query's four lanes, and the sum l of exp2(score - m) over
  // this lane's keys (the four lanes' sums are added at the end)
  float m[QF], l[QF];
#pragma unroll
  for (int f = 0; f < QF; ++f) {
    m[f] = -INFINITY;
    l[f] = 0.f;
  }
  const float scale = a.scale_log2;

  // DMA assignment: load i of wave w fills the 64-chunk block i * NWAVE + w of a key tile (block sizes are
  // multiples of NWAVE, so the K / V^T role of load i is compile-time). A tile that lies whole in the cache
  // or whole in the fresh keys is a scalar base plus a per-lane offset that never changes: no vector
  // arithmetic per load. Any other tile takes each chunk from the cache (key j < P) or the fresh keys / values
  // by itself. A chunk past the last key re-reads the last key's (or last 8-key chunk's) data: those keys
  // score -inf, so their probability is exactly 0 against finite values.
  int key[TI];             // key of the chunk within the tile (V^T: first of its 8)
  uint32_t voff[TI];       // byte offset from the tile's base: fresh operands
  uint32_t coff[TI];       // the same in the cache (V^T rows of pitch Pc)
#pragma unroll
  for (int i = 0; i < TI; ++i) {
    const int pos = (i * NWAVE + wid) * 64 + lane;  // chunk within the key tile
    if (i < KI) {                                    // K chunk: slot pos -> key row, chunk column
      key[i] = pos / KC;
      voff[i] = coff[i] = (uint32_t)(key[i] * DH + ((pos % KC) ^ (key[i] & (KC - 1))) * 8) * 2u;
    } else {                                          // V^T chunk: slot -> dimension row, 8-key chunk
      const int d = (pos - KCH) / VC, c = ((pos - KCH) % VC) ^ (d & (VC - 1));
      key[i] = c * 8;
      voff[i] = ((uint32_t)d * (uint32_t)a.Sp + c * 8) * 2u;
      coff[i] = ((uint32_t)d * (uint32_t)a.Pc + c * 8) * 2u;
    }
  }
  const bool near = a.Sp < (1 << 23) && a.Pc < (1 << 23);  // the 32-bit offsets reach every V^T row
  const uint32_t lds_base = lds_addr_of(sm) + (uint32_t)wid * 1024u;
  auto issue = [&](int t) {
    const uint32_t stage = lds_base + (uint32_t)((t % STAGES) * SCH) * 16u;
#pragma unroll
    for (int gg = 0; gg < KG; ++gg) {
      const int k0 = (t * KG + gg) * KT;
      const uint32_t dst = stage + (uint32_t)gg * (TCH * 16u);
      if (near && k0 >= P && k0 + KT <= nkeys) {
        const bf16_t* kb = uniform_ptr(kf + (ptrdiff_t)(k0 - P) * DH);
        const bf16_t* vb = uniform_ptr(vf + (k0 - P));
#pragma unroll
        for (int i = 0; i < TI; ++i) dma16_sv(i < KI ? kb : vb, voff[i], dst + (uint32_t)(i * NWAVE) * 1024u);
      } else if (near && k0 + KT <= P) {
        const bf16_t* kb = uniform_ptr(kc + (ptrdiff_t)k0 * DH);
        const bf16_t* vb = uniform_ptr(vc + k0);
#pragma unroll
        for (int i = 0; i < TI; ++i) dma16_sv(i < KI ? kb : vb, coff[i], dst + (uint32_t)(i * NWAVE) * 1024u);
      } else {
#pragma unroll
        for (int i = 0; i < TI; ++i) {
          // P is a multiple of 8, so no 8-key chunk straddles the two sides
          const int j = k0 + key[i];
          const bf16_t* src;
          if (i < KI) {
            const int c = (int)(voff[i] >> 1) - key[i] * DH;  // element within the row
            src = (j < P ? kc + (ptrdiff_t)j * DH : kf + (ptrdiff_t)min(j - P, Sk - 1) * DH) + c;
          } else {
            const int d = ((i * NWAVE + wid) * 64 + lane - KCH) / VC;
            src = j < P ? vc + (ptrdiff_t)d * a.Pc + j : vf + (ptrdiff_t)d * a.Sp + min(j - P, (Sk - 1) & ~7);
          }
          dma16_at(src, dst + (uint32_t)(i * NWAVE) * 1024u);
        }
      }
    }
  };

#pragma unroll
  for (int st = 0; st < STAGES - 1; ++st)
    if (st < nsteps) issue(st);
  for (int t = 0; t < nsteps; ++t) {
    // step t landed; the steps t + 1 .. min(nsteps - 1, t + STAGES - 2) may still fly
    attn_wait_stages<IPW, STAGES - 2>(min(STAGES - 2, nsteps - 1 - t));
    asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
    if (t + STAGES - 1 < nsteps) issue(t + STAGES - 1);
    const int k0 = (t * KG + kg) * KT;
    if (k0 >= nkeys) continue;  // this group's tile is past the end (uniform per wave)
    const uint4* sK = sm + (t % STAGES) * SCH + kg * TCH;
    const uint4* sV = sK + KCH;

    // S^T = K Q^T: lane holds keys 16 kt + 4 lg + r of query lq. The tile's K fragments are read
    // first and the independent accumulation chains interleaved.
    bf16x8_t kfr[KT / 16][DH / 32];
#pragma unroll
    for (int kt = 0; kt < KT / 16; ++kt) {
      const int row = 16 * kt + lq;
#pragma unroll
      for (int ks = 0; ks < DH / 32; ++ks) {
        const int c = 4 * ks + lg;
        kfr[kt][ks] = __builtin_bit_cast(bf16x8_t, sK[row * KC + (c ^ (row & (KC - 1)))]);
      }
    }
    f32x4_t sc[QF][KT / 16];
#pragma unroll
    for (int f = 0; f < QF; ++f)
#pragma unroll
      for (int kt = 0; kt < KT / 16; ++kt) sc[f][kt] = f32x4_t{0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int f = 0; f < QF; ++f)
#pragma unroll
      for (int ks = 0; ks < DH / 32; ++ks)
#pragma unroll
        for (int kt = 0; kt < KT / 16; ++kt) sc[f][kt] = mfma16a(kfr[kt][ks], qf[f][ks], sc[f][kt]);
    // V^T fragments, read while the softmax below runs: dimension 16 dt + lq at the keys
    // 32 s2 + 4 lg + {0..3} and 32 s2 + 16 + 4 lg + {0..3} (the order in which the score MFMA left
    // the probabilities in the lanes). Each lane reads one whole 16-byte chunk (bank-conflict free
    // through the XOR swizzle, as the K reads): lane groups 0 / 1 / 2 / 3 read the keys
    // 0-7 / 16-23 / 8-15 / 24-31 of the 32-key block, and neighbouring groups (0, 1) and (2, 3)
    // exchange halves with v_permlane16_swap, which swaps the odd 16-lane rows of its first operand
    // with the even rows of its second: group 0 keeps keys 0-3 and receives 16-19, group 1 receives
    // 4-7 and keeps 20-23, and likewise for groups 2 and 3.
    bf16x8_t vfr[KT / 32][DH / 16];
#pragma unroll
    for (int s2 = 0; s2 < KT / 32; ++s2) {
      const int cx = 4 * s2 + (((lg & 1) << 1) | (lg >> 1));
#pragma unroll
      for (int dt = 0; dt < DH / 16; ++dt) {
        const int d = 16 * dt + lq;
        const uint4 x = sV[d * VC + (cx ^ (d & (VC - 1)))];
        const auto s0 = __builtin_amdgcn_permlane16_swap(x.x, x.z, false, false);
        const auto s1 = __builtin_amdgcn_permlane16_swap(x.y, x.w, false, false);
        vfr[s2][dt] = __builtin_bit_cast(bf16x8_t, make_uint4(s0[0], s1[0], s0[1], s1[1]));
      }
    }
    if (k0 + KT > nkeys) {  // only the last tile holds keys past the end
      asm volatile("");     // keep it a branch: as selects it costs every tile
#pragma unroll
      for (int kt = 0; kt < KT / 16; ++kt)
#pragma unroll
        for (int r = 0; r < 4; ++r)
          if (k0 + 16 * kt + 4 * lg + r >= nkeys)
#pragma unroll
            for (int f = 0; f < QF; ++f) sc[f][kt][r] = -INFINITY;
    }
    // Lazy rescaling: the reference point m only moves when a score exceeds it by more than
    // 2^8 (probabilities up to 256 are exact to represent and sum in float32); the division by
    // the running sum at the end makes the result independent of the reference point. When no
    // lane of the wave moves (all but the first few tiles), neither the maximum over the query's four
    // lanes nor the output rescale is needed.
    float tmax[QF];  // of this lane's keys
    bool move = false;
#pragma unroll
    for (int f = 0; f < QF; ++f) {
      tmax[f] = -INFINITY;
#pragma unroll
      for (int kt = 0; kt < KT / 16; ++kt)
#pragma unroll
        for (int r = 0; r < 4; ++r) tmax[f] = fmaxf(tmax[f], sc[f][kt][r]);
      move |= tmax[f] * scale > m[f] + 8.f;
    }
    if (__builtin_amdgcn_ballot_w64(move)) {
#pragma unroll
      for (int f = 0; f < QF; ++f) {
        // the four lane groups holding one query's keys: lanes l, l^16, l^32, l^48
        float ts = xor_lanes16(tmax[f], [](float x, float y) { return fmaxf(x, y); });
        ts = xor_lanes32(ts, [](float x, float y) { return fmaxf(x, y); }) * scale;
        const float mn = ts > m[f] + 8.f ? ts : m[f];  // moves on the first processed tile (m = -inf)
        const float alpha = __builtin_amdgcn_exp2f(m[f] - mn);  // 1 in the lanes that keep m
        l[f] *= alpha;
#pragma unroll
        for (int dt = 0; dt < DH / 16; ++dt) o[f][dt] *= alpha;
        m[f] = mn;
      }
    }
    // O^T += V^T P^T over 32-key steps; P enters as three bf16 parts (hi + mid + lo)
#pragma unroll
    for (int f = 0; f < QF; ++f) {
#pragma unroll
      for (int kt = 0; kt < KT / 16; ++kt)
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          const float pv = __builtin_amdgcn_exp2f(fmaf(sc[f][kt][r], scale, -m[f]));
          sc[f][kt][r] = pv;
          l[f] += pv;
        }
#pragma unroll
      for (int s2 = 0; s2 < KT / 32; ++s2) {
        uint32_t hi[4], mi[4], lo[4];
#pragma unroll
        for (int x = 0; x < 4; ++x) {
          const float p0 = sc[f][2 * s2 + (x >> 1)][(x & 1) * 2], p1 = sc[f][2 * s2 + (x >> 1)][(x & 1) * 2 + 1];
          hi[x] = f2bf2(p0, p1);
          const float r0 = p0 - __uint_as_float(hi[x] << 16), r1 = p1 - __uint_as_float(hi[x] & 0xFFFF0000u);
          mi[x] = f2bf2(r0, r1);
          lo[x] = f2bf2(r0 - __uint_as_float(mi[x] << 16), r1 - __uint_as_float(mi[x] & 0xFFFF0000u));
        }
        const bf16x8_t phi = __builtin_bit_cast(bf16x8_t, make_uint4(hi[0], hi[1], hi[2], hi[3]));
        const bf16x8_t pmi = __builtin_bit_cast(bf16x8_t, make_uint4(mi[0], mi[1], mi[2], mi[3]));
        const bf16x8_t plo = __builtin_bit_cast(bf16x8_t, make_uint4(lo[0], lo[1], lo[2], lo[3]));
#pragma unroll
        for (int dt = 0; dt < DH / 16; ++dt) o[f][dt] = mfma16a(vfr[s2][dt], phi, o[f][dt]);
#pragma unroll
        for (int dt = 0; dt < DH / 16; ++dt) o[f][dt] = mfma16a(vfr[s2][dt], pmi, o[f][dt]);
#pragma unroll
        for (int dt = 0; dt < DH / 16; ++dt) o[f][dt] = mfma16a(vfr[s2][dt], plo, o[f][dt]);
      }
    }
  }

  if constexpr (KG > 1) {
    // groups 1 .. KG-1 park (m, l, o) in the ring; group 0 folds them in group order
    asm volatile("s_waitcnt vmcnt(0) lgkmcnt(0)\n\ts_barrier" ::: "memory");
    f32x4_t* xo = reinterpret_cast<f32x4_t*>(sm);
    float2* xml = reinterpret_cast<float2*>(xo + (size_t)(KG - 1) * NQ * QF * (DH / 16) * 64);
    if (kg > 0) {
#pragma unroll
      for (int f = 0; f < QF; ++f) {
        const int base = ((kg - 1) * NQ + qw) * QF + f;
#pragma unroll
        for (int dt = 0; dt < DH / 16; ++dt) xo[((size_t)base * (DH / 16) + dt) * 64 + lane] = o[f][dt];
        xml[base * 64 + lane] = make_float2(m[f], l[f]);
      }
    }
    asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
    if (kg > 0) return;
#pragma unroll
    for (int f = 0; f < QF; ++f)
#pragma unroll
      for (int gg = 1; gg < KG; ++gg) {
        const int base = ((gg - 1) * NQ + qw) * QF + f;
        const float2 ml = xml[base * 64 + lane];
        if (ml.x == -INFINITY) continue;  // a group that saw no key
        const float mn = fmaxf(m[f], ml.x);
        const float ea = __builtin_amdgcn_exp2f(m[f] - mn), eb = __builtin_amdgcn_exp2f(ml.x - mn);
        l[f] = l[f] * ea + ml.y * eb;
#pragma unroll
        for (int dt = 0; dt < DH / 16; ++dt)
          o[f][dt] = o[f][dt] * ea + xo[((size_t)base * (DH / 16) + dt) * 64 + lane] * eb;
        m[f] = mn;
      }
  }

#pragma unroll
  for (int f = 0; f < QF; ++f) {
    float lt = xor_lanes16(l[f], [](float x, float y) { return x + y; });
    lt = xor_lanes32(lt, [](float x, float y) { return x + y; });
    const int qrow = q0 + 16 * f + lq;
    if (qrow >= S) continue;
    const float inv = 1.0f / lt;
    bf16_t* dst = a.o + (((size_t)b * S + qrow) * a.H + h) * DH + 4 * lg;
#pragma unroll
    for (int dt = 0; dt < DH / 16; ++dt) {
      uint2 w;
      w.x = f2bf2(o[f][dt][0] * inv, o[f][dt][1] * inv);
      w.y = f2bf2(o[f][dt][2] * inv, o[f][dt][3] * inv);
      *reinterpret_cast<uint2*>(dst + 16 * dt) = w;
    }
  }
}

template <int NQ, int QF, int KG, int KT, int DH, int STAGES>
static void run_attn(const AttnArgs& a, hipStream_t s) {
  constexpr size_t lds = (size_t)STAGES * KG * (KT * (DH / 8) + DH * (KT / 8)) * 16;
  static_assert(lds <= 160 * 1024, "ring exceeds the LDS of a CU");
  const int units = ((a.S + 16 * NQ * QF - 1) / (16 * NQ * QF)) * a.H * a.B;
  if (units == 0) return;
  dim3 grid(8 * ((units + 7) / 8));
  auto kern = attn_kernel<NQ, QF, KG, KT, DH, STAGES>;
  static std::atomic<uint32_t> lds_set{0};
  ensure_dynamic_lds(reinterpret_cast<const void*>(kern), lds, lds_set);
  hipLaunchKernelGGL(kern, grid, dim3(NQ * KG * 64), lds, s, a);
}

// Rings of two steps. The layout follows from the query waves (16 queries each) that the call has and from how its
// workgroups fill the rounds of 256 CUs, which hold two (layouts of 2 x 2 waves) or three (4 x 1 x 1) of them. head_dim
// 128, kernel in the layer, us, cached keys from HBM:
//   up to 256 query waves: a workgroup per query wave whose four waves share out the keys: otherwise few CUs have work
//     at all. 32 (1 x 16 tokens over 1900 keys, kernel alone) 39.2 -> 25.1, head_dim 64, 24 (1 x 96) 4.8 -> 3.8
//     (up to 64 keys most of those waves would have none: the next layout, 2 - 7 % faster there)
//   32-query workgroups while they are one to a CU (192 of them, 2 x 180 over 1800, 16 heads, 49.0 -> 45.0), and two where
//     workgroups of 64 queries would be two as well, with half their queries empty (420 for 280, Dream, 5 x 90 over 975,
//     39.8 -> 31.2), or where all keys are fresh and warm (1 x 448 16.6 -> 16.2, 2 x 250 13.9 -> 12.0; up to 160 keys one
//     key group is 3 % faster). Over a cache the second workgroup reads it once more: 384 for 192 (6 x 40 over 1800) 69.5
//     against 56.5 with the next layout, 320 for 160 (5 x 40 over 975) 37.3 against 30.9
//   workgroups of 64 queries, one to a CU, over a cache: four query waves and two key groups, so that the CU has eight
//     waves (5 x 60 over 331 18.4 -> 17.3; 1.6 % faster than 2 x 2 x 2 on average of 189 sizes)
//   more than 768 of them: 128-query workgroups (3616 query waves, 1 x 1800, 1.15 times as fast; 16 x 70 over 331 46.4 ->
//     34.4) unless a sequence's last one would be more than half empty and they are 3/5 as many (up to 64, 129 - 192 or
//     257 - 320 tokens: 13 x 130 over 700 96.6 against 73.3 with one key group, 32 x 60 21.8 against 17.2)
//   more than 320 keys and almost two full rounds of two to a CU: as for one (32 x 60 over 331 63.2 -> 56.0)
//   up to 320 keys one key group, since a group's share would be few tiles and the merge (3 x 203 14.7 -> 13.3), and
//     where three of its workgroups to a CU beat two (1 x 1300 78.2 -> 73.3, 4 x 384 30.2 -> 27.2); otherwise two
//     query fragments per wave and two key groups (1 x 1024 40.7 -> 38.2).
// head_dim 64: 64-key tiles halve the steps of four query waves x two key groups, which is the faster layout over more
// than 320 keys where 129 to 256 or 385 to 512 of its workgroups fill one round of the CUs, or more than 640 the last one
// (1024, 1 x 1024, 20.0 -> 18.7; 2048, 1 x 2048, 48.9 -> 43.9; 3072, 4 x 768, 32.1 -> 29.5); in between 32-query
// workgroups are (1280, 1 x 1280, 1.10 times as fast).
// Over 331 sizes (4 to 32 heads, 16 to 3072 tokens, 0 to 2003 cached keys) the rule is on average 0.6 % slower than the
// fastest of eight layouts, at most 12 % (2304 to 2560 tokens of 28 or 32 heads); over 1000 more of 12 to 64 heads, 1 to
// 48 sequences of 20 to 320 tokens, without or with 70 to 1800 cached keys, 0.5 %, at most 13 %.
void launch_attention(const AttnArgs& a, hipStream_t s) {
  const long query_waves = (long)a.B * a.H * ((a.S + 15) / 16), wg64 = (long)a.B * a.H * ((a.S + 63) / 64);
  const long wg32 = (long)a.B * a.H * ((a.S + 31) / 32), wg128 = (long)a.B * a.H * ((a.S + 127) / 128);
  const int nkeys = a.P + (a.Sk ? a.Sk : a.S);
  const bool few = query_waves <= 256 && nkeys > 64;
  if (a.dh == 128) {
    if (few) run_attn<1, 1, 4, 32, 128, 2>(a, s);
    else if (wg32 <= 256 || (wg32 <= 512 && (wg64 > 256 || (!a.P && nkeys > 160)))) run_attn<2, 1, 2, 32, 128, 2>(a, s);
    else if (a.P && wg64 <= 256 && nkeys > 160) run_attn<4, 1, 2, 32, 128, 2>(a, s);
    else if (wg64 > 768 && 5 * wg128 < 3 * wg64) run_attn<4, 2, 1, 32, 128, 2>(a, s);
    else if (nkeys > 320 && wg64 > 896 && wg64 <= 1024) run_attn<4, 1, 2, 32, 128, 2>(a, s);
    else if (nkeys <= 320 || wg64 > 512) run_attn<4, 1, 1, 32, 128, 2>(a, s);
    else run_attn<2, 2, 2, 32, 128, 2>(a, s);
  } else {
    const bool filled = wg64 <= 256 ? wg64 > 128 : wg64 <= 512 ? wg64 > 384 : wg64 > 640;
    if (few) run_attn<1, 1, 4, 32, 64, 2>(a, s);
    else if (nkeys > 320 && filled) run_attn<4, 1, 2, 64, 64, 2>(a, s);
    else run_attn<2, 1, 2, 32, 64, 2>(a, s);
  }
}

// ---------------------------------------------------------------- cache write-back
// One thread per 16-byte key chunk, then one per 8-key chunk of a value row. Token s of the step sits in slot
// koff + s of the fresh buffers (k rows of Sk keys, v^T rows of pitch Sp) and goes to position P + s, and
// koff = P mod 8, so value chunks are aligned alike on both sides: whole ones are one 16-byte copy, the first and the
// last may hold tokens in part. Bound by memory (12 MB read and written at 730 tokens x 32 heads: 11.9 us with a thread
// and a division per value element, 7.7 us now).
__global__ void __launch_bounds__(256) kv_writeback_kernel(const bf16_t* __restrict__ k, const bf16_t* __restrict__ vt,
                                                          bf16_t* __restrict__ kc, bf16_t* __restrict__ vc, int BH,
                                                          int S, int Sk, int Sp, int koff, int dh, int P, int Pc) {
  const int nc = (koff + S + 7) / 8;  // value chunks of a row that hold tokens
  const bool aligned = (reinterpret_cast<uintptr_t>(vc) & 15) == 0;  // the pitches are multiples of 8
  const size_t nk = (size_t)BH * S * (dh / 8), nv = (size_t)BH * dh * nc;
  for (size_t i = blockIdx.x * (size_t)blockDim.x + threadIdx.x; i < nk + nv; i += (size_t)gridDim.x * blockDim.x) {
    if (i < nk) {
      const size_t c = i % (dh / 8), rest = i / (dh / 8);
      const size_t s = rest % S, bh = rest / S;
      *reinterpret_cast<uint4*>(kc + (bh * Pc + P + s) * dh + 8 * c) =
          *reinterpret_cast<const uint4*>(k + (bh * Sk + koff + s) * dh + 8 * c);
    } else {
      const size_t e = i - nk;
      const int c = (int)(e % nc);
      const size_t row = e / nc;  // bh * dh + d
      const bf16_t* src = vt + row * Sp + 8 * c;
      bf16_t* dst = vc + row * Pc + (P - koff) + 8 * c;
      const int lo = c == 0 ? koff : 0, hi = min(8, koff + S - 8 * c);
      if (aligned && lo == 0 && hi == 8) {
        *reinterpret_cast<uint4*>(dst) = *reinterpret_cast<const uint4*>(src);
      } else {
        for (int x = lo; x < hi; ++x) dst[x] = src[x];
      }
    }
  }
}

void launch_kv_writeback(const bf16_t* k, const bf16_t* vt, bf16_t* kc, bf16_t* vc, int B, int Hkv, int S, int Sk,
                         int Sp, int koff, int dh, int P, int Pc, hipStream_t s) {
  const size_t n = (size_t)B * Hkv * ((size_t)S * (dh / 8) + (size_t)dh * ((koff + S + 7) / 8));
  if (n == 0) return;
  const int grid = (int)((n + 255) / 256 < 8 * 1024 ? (n + 255) / 256 : 8 * 1024);
  hipLaunchKernelGGL(kv_writeback_kernel, dim3(grid), dim3(256), 0, s, k, vt, kc, vc, B * Hkv, S, Sk, Sp, koff, dh, P,
                     Pc);
}

}  // namespace dcl
