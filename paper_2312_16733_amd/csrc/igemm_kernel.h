// WeightSlice convolution / linear as an implicit GEMM on bf16 MFMA (gfx950).
//
//   Y[m, k] = sum_{r,s,c} X[n, p*st + r - pad, q*st + s - pad, c] * W[k, r0 + r, s0 + s, c]
//   m = (n, p, q) over the requests of one subnet cfg, k < K_active, c < C_active.
//
// The weight operand is the resident max-size tensor: a block reads the leading K_active rows,
// and inside each (k, r, s) the leading C_active channels, through the tensor's own strides.
// The reduction index is flattened over the ACTIVE extent only, in units of 8 channels
// (16 bytes): unit u -> (tap rs, c8) = (u / C8, u % C8), so a narrow subnet pays for its own K,
// not for the SuperNet's.  Active channel counts are multiples of 8, so a unit never straddles a
// tap and every 16-byte load is aligned.
//
// Data path: operands go from global memory straight into LDS (buffer loads with the LDS
// destination, 16 bytes per lane; an out-of-range offset writes zeros, which feeds padding taps,
// ragged rows and the K tail).  LDS holds a ring of NS stages of one K step (64 elements) each;
// rows are 128 bytes with the 16-byte chunks XOR-swizzled by (row >> 1) & 7 so that both the
// linear DMA writes and the column-wise fragment reads are bank-conflict free.  Plain rings: loads
// for step kt + NS - 1 are issued before the MFMAs of step kt; waits are explicit (s_waitcnt vmcnt
// with the number of newer loads still allowed in flight, then s_barrier); fragment reads are
// software-pipelined one 16-wide slice ahead of the v_mfma_f32_32x32x16_bf16 that use them.  Deep
// rings (launches of few tiles, long reductions): waves of their own fetch several steps ahead with
// the taps looked up in an LDS table, the others read a step's fragments (half a step's, where a wave
// has several tiles) under the MFMAs before it, and the two meet once in one or two steps.
// The epilogue (fused SubnetNorm scale/shift, residual, activation) goes through a per-wave
// fp32 LDS tile so that residual loads and output stores are 16 bytes per lane.  Blocks are
// renumbered so that consecutive tiles (which share activation rows) run on the same XCD.
// A launch is grouped: each block finds its problem (one per subnet cfg) from its tile number.
#pragma once
#include "igemm_common.h"

namespace sna {

// Waves per SIMD the register allocation must leave room for: tiles with short reductions are
// launched with a small LDS request and then run that many blocks per CU.
constexpr int igemm_min_waves(int bm, int bn, int ns) {
  return bm * bn > 128 * 128 ? 2 : (bm * bn >= 128 * 128 ? 3 : (bm * bn >= 128 * 96 || (bm * bn == 128 * 64 && ns == 2) ? 4 : 5));
}

// Deep rings: tap table, waves that only fetch, fragments read ahead across K steps.  `small`: one 32x32 tile per computing
// wave or half of one, and eight stages, for launches of few tiles; `large`: several tiles per wave and four stages, one block per CU.
constexpr bool deep_small(int bm, int bn, int n_math, int ns, int fw) { return fw > 0 && ns >= 5 && bm * bn <= n_math * 32 * 32; }
constexpr bool deep_large(int bm, int bn, int n_math, int ns, int fw) { return fw > 0 && ns >= 4 && bm * bn > n_math * 32 * 32; }

// Accesses that are coherent across the chip without cache-wide flushes: relaxed atomics at agent
// scope.  Such a store is written through to memory and such a load is not served from the CU's own
// cache.  The chunk sums that blocks on different XCDs hand to each other go through these; fences
// instead would write back and invalidate the whole L2 of an XCD under the feet of its other blocks
// (measured: forwards at batch 16 lost 15-25 %).  8 bytes per access is the widest atomic there is.
__device__ __forceinline__ void store_f8_agent(float* ptr, const float* v) {      // 8 floats, 32-byte aligned
  unsigned long long* q = (unsigned long long*)ptr;
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    const unsigned long long w = (unsigned long long)__float_as_uint(v[2 * i]) |
                                 ((unsigned long long)__float_as_uint(v[2 * i + 1]) << 32);
    __hip_atomic_store(q + i, w, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  }
}
__device__ __forceinline__ void store_f4_agent(float* ptr, const float* v) {      // 4 floats, 16-byte aligned
  unsigned long long* q = (unsigned long long*)ptr;
#pragma unroll
  for (int i = 0; i < 2; ++i)
    __hip_atomic_store(q + i, (unsigned long long)__float_as_uint(v[2 * i]) | ((unsigned long long)__float_as_uint(v[2 * i + 1]) << 32),
                       __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ void load_f8_agent(const float* ptr, float4& lo, float4& hi) {
  const unsigned long long* q = (const unsigned long long*)ptr;
  unsigned long long w[4];
#pragma unroll
  for (int i = 0; i < 4; ++i) w[i] = __hip_atomic_load(q + i, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  lo = make_float4(__uint_as_float((unsigned)w[0]), __uint_as_float((unsigned)(w[0] >> 32)),
                   __uint_as_float((unsigned)w[1]), __uint_as_float((unsigned)(w[1] >> 32)));
  hi = make_float4(__uint_as_float((unsigned)w[2]), __uint_as_float((unsigned)(w[2] >> 32)),
                   __uint_as_float((unsigned)w[3]), __uint_as_float((unsigned)(w[3] >> 32)));
}

// Sum of the fp32 chunk sums of output row m, channels k .. k+7, in chunk order, then SubnetNorm scale /
// shift, residual and activation exactly as the fused epilogue does: the same bits as one block walking
// all chunks.  `src` points at part 0's row-major [M][K] sums.  Used by the reduction kernel and by the
// matrix kernel's own last-arriving block.
// AGENT: `src0` already points at this octet inside part 0 (the matrix kernel's tile-major layout).
template <bool AGENT>
__device__ __forceinline__ void reduce_octet(const ConvProblem& p, const float* src0, int m, int k) {
  // all loads first (at most 4 chunks), then the sums in chunk order
  const float* src = AGENT ? src0 : src0 + (long)m * p.K + k;
  float4 pa[4], pb[4];
#pragma unroll
  for (int c = 0; c < 4; ++c) {
    if (c < p.parts) {
      const float* sp = (const float*)((const char*)src + (size_t)c * p.part_stride);
      if (AGENT) {
        load_f8_agent(sp, pa[c], pb[c]);      // written by other blocks of this launch
      } else {
        pa[c] = *(const float4*)sp;
        pb[c] = *(const float4*)(sp + 4);
      }
    }
  }
  float4 sc0 = make_float4(1.f, 1.f, 1.f, 1.f), sc1 = sc0, sh0 = make_float4(0.f, 0.f, 0.f, 0.f), sh1 = sh0;
  // the per-channel vectors are only guaranteed 4-byte alignment
  auto load8 = [&](const float* v, float4& lo, float4& hi) {
    if (((size_t)v & 15) == 0) {
      lo = *(const float4*)(v + k);
      hi = *(const float4*)(v + k + 4);
    } else {
      lo = make_float4(v[k], v[k + 1], v[k + 2], v[k + 3]);
      hi = make_float4(v[k + 4], v[k + 5], v[k + 6], v[k + 7]);
    }
  };
  if (p.scale) load8(p.scale, sc0, sc1);
  if (p.shift) load8(p.shift, sh0, sh1);
  uint4 r4 = make_uint4(0, 0, 0, 0);
  if (p.res) r4 = *(const uint4*)((const bf16_t*)p.res + (long)m * p.res_stride + k);
  float val[8];
#pragma unroll
  for (int e = 0; e < 8; ++e) val[e] = 0.f;
#pragma unroll
  for (int c = 0; c < 4; ++c) {
    if (c < p.parts) {
      val[0] = val[0] + pa[c].x; val[1] = val[1] + pa[c].y; val[2] = val[2] + pa[c].z; val[3] = val[3] + pa[c].w;
      val[4] = val[4] + pb[c].x; val[5] = val[5] + pb[c].y; val[6] = val[6] + pb[c].z; val[7] = val[7] + pb[c].w;
    }
  }
  const float scv[8] = {sc0.x, sc0.y, sc0.z, sc0.w, sc1.x, sc1.y, sc1.z, sc1.w};
  const float shv[8] = {sh0.x, sh0.y, sh0.z, sh0.w, sh1.x, sh1.y, sh1.z, sh1.w};
#pragma unroll
  for (int e = 0; e < 8; ++e) val[e] = fmaf(val[e], scv[e], shv[e]);
  float rv[8];
  if (p.res) {
    const unsigned ru[4] = {r4.x, r4.y, r4.z, r4.w};
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      rv[2 * e] = __uint_as_float(ru[e] << 16);
      rv[2 * e + 1] = __uint_as_float(ru[e] & 0xffff0000u);
    }
    if (!p.res_after_act) {
#pragma unroll
      for (int e = 0; e < 8; ++e) val[e] += rv[e];
    }
  }
#pragma unroll
  for (int e = 0; e < 8; ++e) val[e] = apply_act(val[e], p.act);
  if (p.res && p.res_after_act) {
#pragma unroll
    for (int e = 0; e < 8; ++e) val[e] += rv[e];
  }
  if (p.out_fp32) {
    float* yo = (float*)p.y + (long)m * p.y_stride + k;
    *(float4*)yo = make_float4(val[0], val[1], val[2], val[3]);
    *(float4*)(yo + 4) = make_float4(val[4], val[5], val[6], val[7]);
  } else {
    uint4 o;
    o.x = pack_bf16x2(val[0], val[1]);
    o.y = pack_bf16x2(val[2], val[3]);
    o.z = pack_bf16x2(val[4], val[5]);
    o.w = pack_bf16x2(val[6], val[7]);
    *(uint4*)((bf16_t*)p.y + (long)m * p.y_stride + k) = o;
  }
}

constexpr int kGateLoads = 4;               // 16-byte loads of its tile's gates that a thread has in flight
__device__ __forceinline__ int gate_request(const ConvProblem& p, int m) {      // the request that output row m belongs to
  const int t = p.Wo == 1 ? m : (int)__umulhi((unsigned)m, p.magic_wo);
  return p.Ho == 1 ? t : (int)__umulhi((unsigned)t, p.magic_ho);
}

// FW > 0 (wave-specialised): the block has FW more waves that only fetch (address arithmetic,
// global->LDS loads, the wait for them); the others only compute, and the two meet at the one
// barrier per K step.  A fetching wave stalled on the texture path no longer holds up MFMA issue,
// which matters when a CU has a single block to overlap with itself.
// GATED: the input of a pointwise stride-1 layer is multiplied by its request's squeeze-excite gate, which saves the pass
// that wrote the scaled tensor.  Every thread that fetches scales what it fetched itself, in LDS, once its loads have
// landed and ahead of the barrier that hands the step over: each element once, and beside the MFMAs of the computing waves.
// (Scaled between LDS and the matrix pipe, 20 instructions a fragment and by every wave that reads it, the 64x128
// tile took 13.6 us instead of 12.1 on 12544 x 112 outputs over 672 channels.)  Built for tiles with fetching waves alone:
// where the same waves compute, scaling lies in the chain of their steps, and on none of 114 launch shapes were 64x64,
// 128x64 and 128x32 plain rings ahead by more than 3 % (12800 x 40 over 240: 9.1, 11.0 and 10.3 us, 64x64 deep ring 7.5;
// 3200 x 112 over 480: 10.4, 14.0 and 13.0, 32x32 deep ring 8.0).  The gates of the tile's requests lie in LDS behind the
// ring's stages.
constexpr int igemm_waves(int bm, int bn, int n_math, int ns, bool chunked, int fw) {
  return fw ? (bm * bn >= 128 * 128 || deep_large(bm, bn, n_math, ns, fw) ? 2 : 4)
            : (chunked ? (bm * bn == 128 * 64 ? 3 : (bm * bn > 128 * 128 ? 1 : 2)) : igemm_min_waves(bm, bn, ns));
}
// Tile `local` of problem p, which comes by value: uniform fields live in SGPRs across the asm blocks.
template <int BM, int BN, int WARPS_M, int WARPS_N, int NS, bool CHUNKED, int FW, bool GATED>
__device__ __forceinline__ void igemm_tile(const ConvProblem p, int local) {
#if defined(__HIP_DEVICE_COMPILE__)        // the host pass needs the symbol only, not the body
  using Cfg = IgemmCfg<BM, BN, WARPS_M, WARPS_N, NS, FW>;
  constexpr bool WS = FW > 0;
  constexpr bool LARGE = deep_large(BM, BN, WARPS_M * WARPS_N, NS, FW), DEEP = LARGE || deep_small(BM, BN, WARPS_M * WARPS_N, NS, FW);
  constexpr int G = LARGE ? 1 : 2;         // deep rings: K steps between barriers
  static_assert(!DEEP || (NS % G == 0 && NS >= 3 * G && NS / G <= 7), "whole groups of stages");
  constexpr int WTM = Cfg::WTM, WTN = Cfg::WTN, TM = Cfg::TM, TN = Cfg::TN;
  constexpr bool HALF = DEEP && WTM == 16;       // a wave computes 16 pixels x 32 channels
  static_assert(TM >= 1 && TN >= 1 && (WTM % 32 == 0 || HALF) && WTN % 32 == 0, "wave tile");
  static_assert(BM % 8 == 0 && BN % 8 == 0 && Cfg::PASS_ROWS % 16 == 0, "a thread's rows in all passes share one swizzle, (row >> 1) & 7");
  constexpr int A_IT = Cfg::A_IT, B_IT = Cfg::B_IT, L = A_IT + B_IT;   // DMA loads per thread per stage
  static_assert(NS >= 1 && (NS - 2) * L < 64, "vmcnt range");
  static_assert(NS > 1 || !WS, "a fetching wave needs a second stage to run ahead");
  static_assert(BM % Cfg::PASS_ROWS == 0 && BN % Cfg::PASS_ROWS == 0, "every wave issues the same number of loads");

  extern __shared__ __attribute__((aligned(16))) char smem[];
  const unsigned lds0 = (unsigned)(size_t)(lds_char*)smem;              // LDS byte address of the tiles

  int part = 0;                            // which K range of the problem this block reduces over
  if (p.parts > 1) {
    part = p.by_tiles_base.div(local);
    local -= part * p.tiles_base;
  }
  const int tm = p.by_tiles_n.div(local), tn = local - tm * p.tiles_n;
  const int m0 = tm * BM, n0 = tn * BN;

  constexpr int NW = WARPS_M * WARPS_N;
  const int lane = threadIdx.x & 63;
  const bool fetcher = WS && (int)(threadIdx.x >> 6) >= NW;
  const bool do_load = !WS || fetcher, do_math = !WS || !fetcher;
  const int wave = (int)(threadIdx.x >> 6) - (fetcher ? NW : 0);                  // index within its role
  const int tid = wave * 64 + lane;
  const int wm = wave / WARPS_N, wn = wave % WARPS_N;
  const int lrow = tid >> 3;                               // row inside a pass
  const int kc = (tid & 7) ^ ((lrow >> 1) & 7);            // global 16-byte unit this lane's LDS slot holds

  const int C = p.C, H = p.H, Wd = p.W, S = p.S, RS = p.R * p.S;
  const int kt0 = part * p.kt_part;        // first K step of this block's range
  const int KT_all = (p.K8 + 7) >> 3;      // K steps of 64 elements in the whole reduction
  const int KT = KT_all - kt0 < p.kt_part ? KT_all - kt0 : p.kt_part;
  // bytes of the tap table in front of the ring (whole groups: the step that fills up the last one is fetched and never read)
  const int tab_steps = DEEP && RS > 1 ? (KT + G - 1) / G * G : 0;
  const unsigned tab_b = (unsigned)tab_steps * ROW_B;
  if constexpr (DEEP) {
    // Tap table: where the 8 units of every K step lie.  One 16-byte entry per unit: byte offset from a row's first tap
    // in the activations, in the weights, the tap's number, and bit 31 set past the end of the reduction.
    for (int e = threadIdx.x; e < tab_steps * 8; e += 64 * (WARPS_M * WARPS_N + FW)) {
      const unsigned u = (unsigned)(kt0 * 8 + e);
      const unsigned t = (unsigned)p.by_c8.div((int)u), o = u - t * (unsigned)p.C8;
      const int r = ((int)t * p.inv_s) >> 16, s = (int)t - r * S;
      u32x4 v = {(unsigned)(((r * Wd + s) * C + (int)o * 8) * 2), (unsigned)((r * p.wr + s * p.ws + (int)o * 8) * 2), t & 63u,
                 (int)t < RS ? 0u : 0x80000000u};
      *(u32x4*)(smem + e * 16) = v;
    }
  }

  // rows this thread fetches: byte offset of the window's first tap and which taps are in range
  int a_base[A_IT];
  unsigned long long a_mask[A_IT];      // bit rs set: tap rs of this row's window is inside the image
  unsigned long long tap_rows = 0;      // bit r * S for every window row r (uniform)
  for (int r = 0; r < p.R; ++r) tap_rows |= 1ull << (r * S);
  const bool pointwise = RS == 1 && p.stride == 1 && p.pad == 0;   // output pixel m reads input pixel m
#pragma unroll
  for (int i = 0; i < A_IT; ++i) {
    const int row = lrow + Cfg::PASS_ROWS * i;
    const int m = m0 + row;
    a_base[i] = 0;
    a_mask[i] = 0;
    if (row < BM && m < p.M) {
      if (pointwise) {
        a_base[i] = m * C * 2;
        a_mask[i] = 1;
      } else {
        // m -> (n, pp, q) with multiply-high by the host's reciprocals (exact for m * divisor < 2^32)
        const int t = p.Wo == 1 ? m : (int)__umulhi((unsigned)m, p.magic_wo);
        const int q = m - t * p.Wo;
        const int n = p.Ho == 1 ? t : (int)__umulhi((unsigned)t, p.magic_ho);
        const int pp = t - n * p.Ho;
        const int ih0 = pp * p.stride - p.pad, iw0 = q * p.stride - p.pad;
        a_base[i] = ((n * H + ih0) * Wd + iw0) * C * 2;
        // taps inside the image: columns [s_lo, s_hi) of window rows [r_lo, r_hi), without loops
        const int s_lo = iw0 < 0 ? -iw0 : 0, s_hi = Wd - iw0 < S ? Wd - iw0 : S;
        const int r_lo = ih0 < 0 ? -ih0 : 0, r_hi = H - ih0 < p.R ? H - ih0 : p.R;
        unsigned long long mk = 0;
        if (s_hi > s_lo && r_hi > r_lo) {
          const unsigned long long colm = low_bits(s_hi) & ~low_bits(s_lo);
          mk = colm * (tap_rows & low_bits(r_hi * S) & ~low_bits(r_lo * S));      // one copy of colm per window row
        }
        a_mask[i] = mk;
      }
    }
  }
  int b_base[B_IT];
  unsigned b_ok = 0;
#pragma unroll
  for (int j = 0; j < B_IT; ++j) {
    const int row = lrow + Cfg::PASS_ROWS * j;
    const int k = n0 + row;
    if (row < BN && k < p.K) b_ok |= 1u << j;
    b_base[j] = k * p.wk * 2;
  }

  // Gates of the tile's requests, [request][C] in LDS, brought by the computing waves
  const unsigned gate_lds = GATED ? (unsigned)((KT >= NS ? NS : (HALF ? (KT + G - 1) / G * G : KT)) * Cfg::STAGE_B) : 0u;
  const int gate_n0 = GATED ? gate_request(p, m0) : 0, gate_c4 = C >> 2;
  const int gate_cnt = GATED ? (gate_request(p, m0 + BM - 1 < p.M ? m0 + BM - 1 : p.M - 1) - gate_n0 + 1) * gate_c4 : 0;
  auto bring_gates = [&] {
    if constexpr (GATED) {
      const float inv = __builtin_amdgcn_rcpf((float)gate_c4);          // e / gate_c4 for e < 2^20: within 2^-22 of it, 1 / (2 gate_c4) from an integer
      for (int e0 = tid; e0 < gate_cnt; e0 += 64 * NW * kGateLoads) {
        float4 v[kGateLoads];
#pragma unroll
        for (int i = 0; i < kGateLoads; ++i) {
          const int e = e0 + i * 64 * NW, n = (int)(((float)e + 0.5f) * inv);
          v[i] = e < gate_cnt ? *(const float4*)(p.gate + (long)(gate_n0 + n) * p.gate_stride + (e - n * gate_c4) * 4) : make_float4(0.f, 0.f, 0.f, 0.f);
        }
#pragma unroll
        for (int i = 0; i < kGateLoads; ++i) {
          const int e = e0 + i * 64 * NW;
          if (e < gate_cnt) *(float4*)(smem + gate_lds + e * 16) = v[i];
        }
      }
    }
  };
  unsigned gate_row[GATED ? A_IT : 1];           // LDS address of the gates of this thread's rows, unit kc of step 0
  if constexpr (GATED) {
#pragma unroll
    for (int i = 0; i < A_IT; ++i) {
      const int m = m0 + lrow + Cfg::PASS_ROWS * i;
      gate_row[i] = lds0 + gate_lds + (unsigned)((m < p.M ? gate_request(p, m) - gate_n0 : 0) * C + kc * 8) * 4;
    }
  }

  // reduction position of this thread's unit: tap rs and channel octet c8 (the deep rings look it up instead)
  int rs = 0, c8 = 0;
  if constexpr (!DEEP) {
    rs = p.by_c8.div(kt0 * 8 + kc);
    c8 = kt0 * 8 + kc - rs * p.C8;
  }

  const __amdgpu_buffer_rsrc_t rsrc_x = __builtin_amdgcn_make_buffer_rsrc((void*)p.x, 0, (int)p.x_bytes, 0x00020000);
  const __amdgpu_buffer_rsrc_t rsrc_w = __builtin_amdgcn_make_buffer_rsrc((void*)p.w, 0, (int)p.w_bytes, 0x00020000);
  constexpr unsigned OOB = 0x80000000u;
  // LDS destination of this wave's DMA ops inside a stage: 64 lanes x 16 bytes = 8 consecutive rows
  lds_char* const dma_a = (lds_char*)smem + tab_b + (wave * 8) * ROW_B;
  lds_char* const dma_b = dma_a + BM * ROW_B;

  // Buffer offsets of the next K step to fetch.  Within a tap they advance by one step (128 bytes)
  // per fetch; only when a lane's unit crosses into the next tap are they rebuilt from (rs, c8).
  // An out-of-range entry stays out of range under the increments (it starts at 2^31).
  unsigned dma_off[L];
  auto locate = [&]() {
    const bool u_ok = rs < RS;
    const int r = (rs * p.inv_s) >> 16, s = rs - r * S;
    const int tx = ((r * Wd + s) * C + c8 * 8) * 2, tw = (r * p.wr + s * p.ws + c8 * 8) * 2;
#pragma unroll
    for (int i = 0; i < A_IT; ++i) {
      const bool ok = u_ok && ((a_mask[i] >> (rs & 63)) & 1ull);
      dma_off[i] = ok ? (unsigned)(a_base[i] + tx) : OOB;
    }
#pragma unroll
    for (int j = 0; j < B_IT; ++j) {
      const bool ok = u_ok && ((b_ok >> j) & 1u);
      dma_off[A_IT + j] = ok ? (unsigned)(b_base[j] + tw) : OOB;
    }
  };
  if constexpr (!DEEP) locate();
  // The deep rings' fetch: with the tap looked up, a load's offset is an add and two bit tests
  auto issue_at = [&](int stage, const u32x4 e) {
#pragma unroll
    for (int i = 0; i < A_IT; ++i) {
      const unsigned out = (unsigned)(~a_mask[i] >> e[2]) << 31;
      __builtin_amdgcn_raw_ptr_buffer_load_lds(rsrc_x, dma_a + stage * Cfg::STAGE_B + Cfg::PASS_ROWS * i * ROW_B, 16,
                                               ((unsigned)a_base[i] + e[0]) | e[3] | out, 0, 0, 0);
    }
#pragma unroll
    for (int j = 0; j < B_IT; ++j) {
      const unsigned out = (~b_ok >> j) << 31;
      __builtin_amdgcn_raw_ptr_buffer_load_lds(rsrc_w, dma_b + stage * Cfg::STAGE_B + Cfg::PASS_ROWS * j * ROW_B, 16,
                                               ((unsigned)b_base[j] + e[1]) | e[3] | out, 0, 0, 0);
    }
  };
  const unsigned tab_lane = lds0 + kc * 16;      // this thread's unit in the tap table
  int stage0 = 0;                                // stage of the next step to request
  // The n steps from kt on, into the stages from kt % NS on (n divides NS).  A step past the block's
  // last is fetched too, and never read (zeros, or what the next part of a split reduction begins with), except while the
  // ring fills: a launch of fewer steps than stages has no LDS for the others.
  auto request_steps = [&](int kt, auto n_c) {
    constexpr int n = decltype(n_c)::value;
    if (RS == 1) {                               // a pointwise layer has nothing to look up
#pragma unroll
      for (int i = 0; i < n; ++i) {
        const unsigned u = (unsigned)((kt0 + kt + i) * 8 + kc);
        if (n < NS || kt + i < KT) issue_at(stage0 + i, u32x4{u * 16, u * 16, 0u, u < (unsigned)p.C8 ? 0u : 0x80000000u});
      }
    } else {
      u32x4 e[n];
      unsigned at[n];
#pragma unroll
      for (int i = 0; i < n; ++i) at[i] = tab_lane + (n == NS && kt + i >= KT ? 0 : kt + i) * ROW_B;
      lds_read_b128_now(e, at);
#pragma unroll
      for (int i = 0; i < n; ++i)
        if (n < NS || kt + i < KT) issue_at(stage0 + i, e[i]);
    }
    stage0 = stage0 + n == NS ? 0 : stage0 + n;
  };
  auto issue = [&](int stage) {
#pragma unroll
    for (int i = 0; i < A_IT; ++i)
      __builtin_amdgcn_raw_ptr_buffer_load_lds(rsrc_x, dma_a + stage * Cfg::STAGE_B + Cfg::PASS_ROWS * i * ROW_B, 16,
                                               dma_off[i], 0, 0, 0);
#pragma unroll
    for (int j = 0; j < B_IT; ++j)
      __builtin_amdgcn_raw_ptr_buffer_load_lds(rsrc_w, dma_b + stage * Cfg::STAGE_B + Cfg::PASS_ROWS * j * ROW_B, 16,
                                               dma_off[A_IT + j], 0, 0, 0);
    c8 += 8;                              // advance one K step
    if (c8 >= p.C8) {
      do { c8 -= p.C8; ++rs; } while (c8 >= p.C8);
      locate();
    } else {
#pragma unroll
      for (int i = 0; i < L; ++i) dma_off[i] += BK * 2;
    }
  };

  f32x16 acc[TM][TN];                      // written at the first step of a sum

  const int frag_row = lane & 31, frag_hi = lane >> 5, frag_sw = (frag_row >> 1) & 7;
  unsigned frag_off[BK / 16];              // swizzled byte offset of this lane's chunk in each 16-wide slice
#pragma unroll
  for (int ks = 0; ks < BK / 16; ++ks) frag_off[ks] = (unsigned)(((ks * 2 + frag_hi) ^ frag_sw) * 16);
  // GATED: this thread's part of GS steps is scaled in LDS, its own loads having landed.  Reads and writes are written out,
  // since the compiler would wait for every load of the ring ahead of an LDS access of its own (36 x 160 outputs over 960
  // channels, 15 steps: 10.6 us instead of 9.6).  A unit past C is zero and stays so.
  constexpr int GS = DEEP ? G : 1;
  auto scale_steps = [&](int st, int kt) {
    if constexpr (GATED) {
      static_assert(GS * A_IT % 2 == 0, "two units at a time");
      auto two = [](unsigned w, unsigned lo, unsigned hi) { return pack_bf16x2(__uint_as_float(w << 16) * __uint_as_float(lo), __uint_as_float(w & 0xffff0000u) * __uint_as_float(hi)); };
#pragma unroll
      for (int q = 0; q < GS * A_IT; q += 2) {
        unsigned at[6];
        bool ok[2];
        u32x4 v[6];
#pragma unroll
        for (int h = 0; h < 2; ++h) {
          const int t = (q + h) / A_IT, i = (q + h) % A_IT;
          ok[h] = kt + t < KT && (kt + t) * 8 + kc < p.C8;
          const int tt = ok[h] ? t : 0;
          at[3 * h] = lds0 + (st + tt) * Cfg::STAGE_B + (wave * 8 + Cfg::PASS_ROWS * i) * ROW_B + lane * 16;
          at[3 * h + 1] = gate_row[i] + (ok[h] ? (kt + t) * 256 : 0);
          at[3 * h + 2] = at[3 * h + 1] + 16;
        }
        lds_read_b128_now(v, at);
#pragma unroll
        for (int h = 0; h < 2; ++h) {
          const u32x4 a = v[3 * h], g0 = v[3 * h + 1], g1 = v[3 * h + 2];
          if (ok[h]) lds_write_b128(at[3 * h], u32x4{two(a[0], g0[0], g0[1]), two(a[1], g0[2], g0[3]), two(a[2], g1[0], g1[1]), two(a[3], g1[2], g1[3])});
        }
      }
      asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
    }
  };
  const unsigned a_lane = lds0 + tab_b + (wm * WTM + frag_row) * ROW_B;
  const unsigned b_lane = lds0 + tab_b + (BM + wn * WTN + frag_row) * ROW_B;

  // `fresh`: the accumulators start a new sum at this step (wave tiles of one or two 32x32 tiles clear them, the larger
  // ones have the first MFMA of each take C = 0)
  auto compute = [&](int stage, const bool fresh) {
    const unsigned ab = a_lane + stage * Cfg::STAGE_B, bb = b_lane + stage * Cfg::STAGE_B;
    if constexpr (TM * TN == 1 || (TM * TN == 2 && NS == 2)) {
      if (fresh) {
#pragma unroll
        for (int i = 0; i < TM; ++i)
#pragma unroll
          for (int j = 0; j < TN; ++j)
#pragma unroll
            for (int v = 0; v < 16; ++v) acc[i][j][v] = 0.f;
      }
      // one or two 32x32 tiles per wave: a slice's MFMAs are too short to hide an LDS read, so the reads of the whole step
      // go out together and each slice waits only for its own (64x64 tiles, a lone request: 100 x 136 outputs of a 3x3
      // over 136 channels 13.6 -> 12.6 us, 32x128 tiles 13.8 -> 12.9; the smallest ResNet-shaped subnet 419 -> 412).
      // Two tiles per wave: only with the two-stage ring, which full batches use (three blocks share a CU; 64 requests of
      // the largest ResNet-shaped subnet 3083 -> 2969 us, four waves per SIMD so that nothing spills).  The plain
      // rings of three and four stages lose by it where a CU has one block (64x128 tiles, one request of the largest
      // ResNet-shaped subnet 989 -> 1013 us, before such launches went to the deep rings).
      constexpr int NSL = BK / 16, RD = TM + TN;      // slices per step, reads per slice
      static_assert(RD * NSL <= 15, "lgkmcnt range");
      u32x4 a1[NSL][TM], b1[NSL][TN];
#pragma unroll
      for (int ks = 0; ks < NSL; ++ks) {
#pragma unroll
        for (int i = 0; i < TM; ++i) a1[ks][i] = lds_read_b128(ab + frag_off[ks], i * 32 * ROW_B);
#pragma unroll
        for (int j = 0; j < TN; ++j) b1[ks][j] = lds_read_b128(bb + frag_off[ks], j * 32 * ROW_B);
      }
      auto slice = [&](auto ks_c) {
        constexpr int ks = decltype(ks_c)::value;
        __builtin_amdgcn_s_waitcnt(0xc07f | ((RD * (NSL - 1 - ks)) << 8));      // lgkmcnt: the later slices' reads
#pragma unroll
        for (int i = 0; i < TM; ++i) asm volatile("" : "+v"(a1[ks][i]));
#pragma unroll
        for (int j = 0; j < TN; ++j) asm volatile("" : "+v"(b1[ks][j]));
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int i = 0; i < TM; ++i)
#pragma unroll
          for (int j = 0; j < TN; ++j)
            acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, a1[ks][i]),
                                                                __builtin_bit_cast(bf16x8, b1[ks][j]), acc[i][j], 0, 0, 0);
      };
      static_assert(NSL == 4, "four slices per step");
      slice(std::integral_constant<int, 0>{});
      slice(std::integral_constant<int, 1>{});
      slice(std::integral_constant<int, 2>{});
      slice(std::integral_constant<int, 3>{});
      return;
    }
    u32x4 af[2][TM], bfr[2][TN];
#pragma unroll
    for (int i = 0; i < TM; ++i) af[0][i] = lds_read_b128(ab + frag_off[0], i * 32 * ROW_B);
#pragma unroll
    for (int j = 0; j < TN; ++j) bfr[0][j] = lds_read_b128(bb + frag_off[0], j * 32 * ROW_B);
#pragma unroll
    for (int ks = 0; ks < BK / 16; ++ks) {
      const int cur = ks & 1, nxt = cur ^ 1;
      // fragments of slice ks were requested one slice ago: wait for them, then request slice ks+1
      // before the MFMAs of slice ks so that the LDS latency runs under the matrix pipe
      asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
#pragma unroll
      for (int i = 0; i < TM; ++i) asm volatile("" : "+v"(af[cur][i]));
#pragma unroll
      for (int j = 0; j < TN; ++j) asm volatile("" : "+v"(bfr[cur][j]));
      if (ks + 1 < BK / 16) {
#pragma unroll
        for (int i = 0; i < TM; ++i) af[nxt][i] = lds_read_b128(ab + frag_off[ks + 1], i * 32 * ROW_B);
#pragma unroll
        for (int j = 0; j < TN; ++j) bfr[nxt][j] = lds_read_b128(bb + frag_off[ks + 1], j * 32 * ROW_B);
      }
      __builtin_amdgcn_sched_barrier(0);    // keep the requests ahead of the MFMAs that hide their latency
      if (ks == 0 && fresh) {
        const f32x16 zero = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int i = 0; i < TM; ++i)
#pragma unroll
          for (int j = 0; j < TN; ++j)
            acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, af[cur][i]),
                                                                __builtin_bit_cast(bf16x8, bfr[cur][j]), zero, 0, 0, 0);
      } else {
#pragma unroll
        for (int i = 0; i < TM; ++i)
#pragma unroll
          for (int j = 0; j < TN; ++j)
            acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, af[cur][i]),
                                                                __builtin_bit_cast(bf16x8, bfr[cur][j]), acc[i][j], 0, 0, 0);
      }
    }
  };

  // ---- main loop: ring of NS stages ----------------------------------------------------------
  if constexpr (DEEP) {
    if (RS > 1) __syncthreads();                 // the tap table is written
    if (do_load) request_steps(0, std::integral_constant<int, NS>{});
  } else if (do_load) {
#pragma unroll
    for (int st = 0; st < NS - 1; ++st)
      if (st < KT) issue(st);
  }
  if constexpr (GATED) {
    static_assert(WS && !LARGE, "not built");
    if (do_math) bring_gates();
    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
    __builtin_amdgcn_s_barrier();
    asm volatile("" ::: "memory");
  }

  // SubnetNorm scale / shift of this lane's output columns, requested behind the first stages' loads so
  // that they arrive under the main loop
  const int col_l = lane & 31, row_l = (lane >> 5) * 4;
  // reduction finished inside this launch: the blocks store bare chunk sums, the last one to arrive at a
  // tile applies scale / shift / residual / activation after adding them up
  const bool in_kernel_reduce = p.parts > 1 && p.counters != nullptr;
  float sc[TN], sh[TN];
#pragma unroll
  for (int j = 0; j < TN; ++j) {
    const int k = n0 + wn * WTN + j * 32 + col_l;
    sc[j] = (do_math && !in_kernel_reduce && p.scale && k < p.K) ? p.scale[k] : 1.f;
    sh[j] = (do_math && !in_kernel_reduce && p.shift && k < p.K) ? p.shift[k] : 0.f;
  }

  // The small deep rings have the registers to request the residual rows here, too (one round trip less at the end)
  constexpr bool DIRECT = DEEP && !LARGE;
  // DIRECT: this lane's pixel and its PIECES runs of four channels, px_k + PIECE q ..
  constexpr int PIECES = HALF ? 2 : 4, PIECE = HALF ? 16 : 8;
  const int lane_k = (HALF ? lane >> 4 : lane >> 5) * 4;
  const int px_m = m0 + wm * WTM + (lane & (HALF ? 15 : 31)), px_k = n0 + wn * WTN + lane_k;
  uint2 res_early[DIRECT ? PIECES : 1];
  if (DIRECT && do_math && p.res && !in_kernel_reduce) {
#pragma unroll
    for (int q = 0; q < PIECES; ++q)
      res_early[q] = (px_m < p.M && px_k + PIECE * q < p.K) ? *(const uint2*)((const bf16_t*)p.res + (long)px_m * p.res_stride + px_k + PIECE * q) : make_uint2(0, 0);
  }

  // CHUNKED: the reduction is summed in chunks of p.kt_chunk steps, each accumulated from zero and
  // added to a running total in fp32, so that one block reducing over all chunks gives the same
  // bits as one block per chunk plus the reduction kernel.
  f32x16 tot[CHUNKED ? TM : 1][CHUNKED ? TN : 1];
  int to_fold = p.kt_chunk;
  if (CHUNKED) {
#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
      for (int j = 0; j < TN; ++j)
#pragma unroll
        for (int v = 0; v < 16; ++v) tot[i][j][v] = 0.f;
  }
  int stage = 0, fill = NS - 1;            // stage holding step kt; stage that step kt + NS - 1 goes to
  bool fresh = true;
  if constexpr (DEEP) {
    // Few tiles on the chip: a block has a CU (almost) to itself, and what counts is how long its chain of K steps takes.
    // The plain rings spend 0.35 us (64x64) to 0.75 us (64x128) a step on it: a load round trip per two or three steps, a
    // barrier and an LDS latency per step, the address arithmetic of a tap change in the fetching wave.  Here the taps are
    // looked up, the loads run NS - 2 G steps ahead, a step's fragments are read under the MFMAs of the step before, and
    // the fetching and the computing waves meet once in G steps, in the second: then the next group has landed, and the
    // group before is in registers, its stages free.
    if (do_load) {
      // wait until at most the n newest groups are in flight (n >= NG - 1 is the start of the ring)
      constexpr int NG = NS / G;
      auto landed = [&](int n) {
        if (n >= NG - 1) __builtin_amdgcn_s_waitcnt(vmcnt_imm((NG - 1) * G * L));
        else if (n >= NG - 2) __builtin_amdgcn_s_waitcnt(vmcnt_imm((NG - 2) * G * L));
        else if (n >= NG - 3) __builtin_amdgcn_s_waitcnt(vmcnt_imm((NG - 3) * G * L));
        else if (NG > 4 && n >= NG - 4) __builtin_amdgcn_s_waitcnt(vmcnt_imm((NG > 4 ? NG - 4 : 0) * G * L));
        else if (NG > 5 && n >= NG - 5) __builtin_amdgcn_s_waitcnt(vmcnt_imm((NG > 5 ? NG - 5 : 0) * G * L));
        else if (NG > 6 && n >= NG - 6) __builtin_amdgcn_s_waitcnt(vmcnt_imm((NG > 6 ? NG - 6 : 0) * G * L));
        else __builtin_amdgcn_s_waitcnt(vmcnt_imm(0));
      };
      int requested = KT < NS ? KT : NS;
      int scaled = 0;                            // GATED: stage of the group to scale next
      auto scale_group = [&](int kt) {
        scale_steps(scaled, kt);
        scaled = scaled + G == NS ? 0 : scaled + G;
      };
      landed((requested - G) / G);
      scale_group(0);
      __builtin_amdgcn_s_barrier();              // group 0 is in LDS
#pragma unroll 1
      for (int kt = 0; kt + G < KT; kt += G) {
        landed((requested - kt - 2 * G) / G);
        scale_group(kt + G);
        __builtin_amdgcn_s_barrier();            // the group after step kt's is in LDS, the one before it is free (LARGE and HALF: step kt's too)
        if ((LARGE || HALF || kt != 0) && requested < KT) {
          request_steps(requested, std::integral_constant<int, G>{});
          requested += G;
        }
      }
    } else if constexpr (LARGE) {
      // Several 32x32 tiles per wave, one block per CU.  Half a step's fragments (two 16-wide slices) are read under the
      // MFMAs of the half before; the waves meet in a step's second half, when the step is in registers altogether and
      // the next one has landed.  128x96 tiles, 4096 x 768 outputs over 3072 channels: 29.7 -> 27.0 us (the wave-specialised
      // 128x128 tile before), 3136 x 720 of a 3x3 over 720 channels 68 -> 61.  Bound by the CU's fetch rate (28 KB a step at
      // 97 B/ns where the rows are line-aligned, 57 where not) and its LDS reads (64 KB a step); a 128x128 tile of this kind
      // takes as long per output as 128x96.
      typedef __attribute__((address_space(3))) const u32x4 lds_frag;
      u32x4 fa[2][2][TM], fb[2][2][TN];
#pragma unroll
      for (int i = 0; i < TM; ++i)
#pragma unroll
        for (int j = 0; j < TN; ++j)
#pragma unroll
          for (int v = 0; v < 16; ++v) acc[i][j][v] = 0.f;
      auto read_half = [&](int st, auto h_c) {
        constexpr int h = decltype(h_c)::value;
#pragma unroll
        for (int s2 = 0; s2 < 2; ++s2) {
#pragma unroll
          for (int i = 0; i < TM; ++i) fa[h][s2][i] = *(lds_frag*)(a_lane + st * Cfg::STAGE_B + frag_off[2 * h + s2] + i * 32 * ROW_B);
#pragma unroll
          for (int j = 0; j < TN; ++j) fb[h][s2][j] = *(lds_frag*)(b_lane + st * Cfg::STAGE_B + frag_off[2 * h + s2] + j * 32 * ROW_B);
        }
      };
      auto mfma_half = [&](auto h_c) {
        constexpr int h = decltype(h_c)::value;
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int s2 = 0; s2 < 2; ++s2)
#pragma unroll
          for (int i = 0; i < TM; ++i)
#pragma unroll
            for (int j = 0; j < TN; ++j)
              acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, fa[h][s2][i]),
                                                                  __builtin_bit_cast(bf16x8, fb[h][s2][j]), acc[i][j], 0, 0, 0);
        __builtin_amdgcn_sched_barrier(0);
      };
      typedef std::integral_constant<int, 0> h0_t;
      typedef std::integral_constant<int, 1> h1_t;
      asm volatile("" ::: "memory");
      __builtin_amdgcn_s_barrier();
      asm volatile("" ::: "memory");
      read_half(0, h0_t{});
#pragma unroll 1
      for (int kt = 0; kt + 1 < KT; ++kt) {
        read_half(stage, h1_t{});
        mfma_half(h0_t{});
        stage = stage + 1 == NS ? 0 : stage + 1;
        asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");       // step kt is in registers
        __builtin_amdgcn_s_barrier();
        asm volatile("" ::: "memory");
        read_half(stage, h0_t{});
        mfma_half(h1_t{});
        if (CHUNKED && --to_fold == 0) {                          // chunk boundary: bank the chunk's sum
          to_fold = p.kt_chunk;
#pragma unroll
          for (int i = 0; i < TM; ++i)
#pragma unroll
            for (int j = 0; j < TN; ++j)
#pragma unroll
              for (int v = 0; v < 16; ++v) {
                tot[i][j][v] = tot[i][j][v] + acc[i][j][v];
                acc[i][j][v] = 0.f;
              }
        }
      }
      read_half(stage, h1_t{});
      mfma_half(h0_t{});
      mfma_half(h1_t{});
    } else if constexpr (HALF) {
      // A 32x32 tile by two waves on v_mfma_f32_16x16x32_bf16, whose sum over 32 elements has the bits of two 32x32x16 in a
      // row (fp32 sums in steps of 8 elements, in order).  A step's LDS reads (8 KB) and MFMAs (131 clocks) were one wave's;
      // now each of two has 6 KB and 68 clocks, and requests a whole group ahead of the MFMAs of the group before.  What is
      // left to bound a step is its fetch (8 KB at 57 B/ns of a CU where rows are not line-aligned, 0.14 us; 97 where they
      // are).  One image: 196 x 360 outputs of a 3x3 over 360 channels, 51 steps 11.35 -> 10.41 us, in two parts 9.53 -> 8.54;
      // 49 x 720 of a linear layer over 2048, 32 steps 7.55 -> 6.73, 196 x 360 over 1024, 16 steps 4.87 -> 4.47.  A request
      // of the largest ResNet-shaped subnet 452 -> 412 us, of the smallest 235 -> 220; MBV3-shaped 258 -> 254, 3 sequences
      // 477 -> 472.
      typedef __attribute__((address_space(3))) const u32x4 lds_frag;
      typedef __attribute__((address_space(3))) float lds_total;
      typedef __attribute__((ext_vector_type(4))) float f32x4;
      const int fr = lane & 15, fh = lane >> 4;
      unsigned at[2];                            // by half of a step: this lane's unit of its row
#pragma unroll
      for (int h = 0; h < 2; ++h) at[h] = lds0 + tab_b + fr * ROW_B + (unsigned)(((h * 4 + fh) ^ ((fr >> 1) & 7)) * 16);
      const unsigned a_rows = wm * 16 * ROW_B, b_rows = (BM + wn * WTN) * ROW_B;
      lds_total* const tot_l = (lds_total*)(lds0 + tab_b + NS * Cfg::STAGE_B + wave * 2048 + lane * 4);
      bool first_fold = true;
      f32x4 sum[2];                              // channels 0 .. 15 and 16 .. 31 of the wave's tile
#pragma unroll
      for (int v = 0; v < 8; ++v) sum[v >> 2][v & 3] = 0.f;
      u32x4 fa[2][G][2], fb[2][G][2][2];
      auto read_group = [&](auto b_c) {
        constexpr int b = decltype(b_c)::value;
#pragma unroll
        for (int i = 0; i < G; ++i)
#pragma unroll
          for (int h = 0; h < 2; ++h) {
            const unsigned u = at[h] + (stage + i) * Cfg::STAGE_B;
            fa[b][i][h] = *(lds_frag*)(u + a_rows);
#pragma unroll
            for (int j = 0; j < 2; ++j) fb[b][i][h][j] = *(lds_frag*)(u + b_rows + j * 16 * ROW_B);
          }
        stage = stage + G == NS ? 0 : stage + G;
      };
      auto step = [&](auto b_c, auto i_c, bool more) {      // channels as rows, pixels as columns: see the epilogue
        constexpr int b = decltype(b_c)::value, i = decltype(i_c)::value;
#pragma unroll
        for (int h = 0; h < 2; ++h)
#pragma unroll
          for (int j = 0; j < 2; ++j)
            sum[j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, fb[b][i][h][j]),
                                                             __builtin_bit_cast(bf16x8, fa[b][i][h]), sum[j], 0, 0, 0);
        if (CHUNKED && more && --to_fold == 0) {            // chunk boundary: bank the chunk's sum
          to_fold = p.kt_chunk;
#pragma unroll
          for (int v = 0; v < 8; ++v) {
            tot_l[v * 64] = first_fold ? sum[v >> 2][v & 3] : tot_l[v * 64] + sum[v >> 2][v & 3];
            sum[v >> 2][v & 3] = 0.f;
          }
          first_fold = false;
        }
      };
      auto meet = [&] {                          // barrier; no LDS read moves across it
        asm volatile("" ::: "memory");
        __builtin_amdgcn_s_barrier();
        asm volatile("" ::: "memory");
      };
      typedef std::integral_constant<int, 0> i0_t;
      typedef std::integral_constant<int, 1> i1_t;
      // the group from step kt on, in buffer b: the next one is requested ahead of its MFMAs
      auto group = [&](auto b_c, int kt) {
        __builtin_amdgcn_s_waitcnt(0xc07f);      // lgkmcnt(0): the group is in registers, its stages are free
        if (kt + G < KT) {
          meet();
          read_group(std::integral_constant<int, decltype(b_c)::value ^ 1>{});
        }
        __builtin_amdgcn_sched_barrier(0);
        step(b_c, i0_t{}, kt + 1 < KT);
        if (kt + 1 < KT) step(b_c, i1_t{}, kt + 2 < KT);
      };
      static_assert(G == 2, "unrolled above");
      meet();
      read_group(i0_t{});
#pragma unroll 1
      for (int kt = 0; kt < KT; kt += 2 * G) {
        group(i0_t{}, kt);
        if (kt + G < KT) group(i1_t{}, kt + G);
      }
#pragma unroll
      for (int v = 0; v < 8; ++v) acc[0][0][v] = sum[v >> 2][v & 3];
      if (CHUNKED && !first_fold) {
#pragma unroll
        for (int v = 0; v < 8; ++v) tot[0][0][v] = tot_l[v * 64];
      }
    } else {
      u32x4 fa[2][BK / 16], fb[2][BK / 16];
#pragma unroll
      for (int v = 0; v < 16; ++v) acc[0][0][v] = 0.f;
      // The next step's fragments are requested ahead of this step's MFMAs and arrive under them (reads between the MFMAs
      // measured 0.14 us a step: the last ones are then waited for; a branch in a step costs as much as an MFMA's issue)
      // (Plain loads, whose waits the compiler places: the fragments cross the loop's back edge in flight, where it may
      // copy registers.  These waves fetch nothing, so that no wait for a fetch comes with them.)
      typedef __attribute__((address_space(3))) const u32x4 lds_frag;
      typedef __attribute__((address_space(3))) float lds_total;
      auto read_step = [&](int st, int b) {
#pragma unroll
        for (int ks = 0; ks < BK / 16; ++ks) {
          fa[b][ks] = *(lds_frag*)(a_lane + st * Cfg::STAGE_B + frag_off[ks]);
          fb[b][ks] = *(lds_frag*)(b_lane + st * Cfg::STAGE_B + frag_off[ks]);
        }
      };
      // The running total lies in LDS behind the ring: in registers it costs the fourth wave per SIMD, without which two
      // blocks of five waves do not share a CU (462 x 576 outputs of a 3x3 over 576 channels, 270 tiles: 28.4 -> 17.6 us)
      lds_total* const tot_l = (lds_total*)(lds0 + tab_b + NS * Cfg::STAGE_B + wave * 4096 + lane * 4);
      bool first_fold = true;
      auto meet = [&] {                          // barrier; no LDS read moves across it
        asm volatile("" ::: "memory");
        __builtin_amdgcn_s_barrier();
        asm volatile("" ::: "memory");
      };
      auto mfma = [&](int b, int ks) {           // channels as rows, pixels as columns: see the epilogue
        acc[0][0] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, fb[b][ks]),
                                                            __builtin_bit_cast(bf16x8, fa[b][ks]), acc[0][0], 0, 0, 0);
      };
      auto step = [&](auto i_c, auto more_c) {   // step i of a group; more: another one follows
        constexpr int b = decltype(i_c)::value & 1;
        constexpr bool more = decltype(more_c)::value;
        stage = stage + 1 == NS ? 0 : stage + 1;
        if (more) read_step(stage, b ^ 1);
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int ks = 0; ks < BK / 16; ++ks) mfma(b, ks);
        if (CHUNKED && more && --to_fold == 0) {            // chunk boundary: bank the chunk's sum
          to_fold = p.kt_chunk;
#pragma unroll
          for (int v = 0; v < 16; ++v) {
            tot_l[v * 64] = first_fold ? acc[0][0][v] : tot_l[v * 64] + acc[0][0][v];
            acc[0][0][v] = 0.f;
          }
          first_fold = false;
        }
      };
      static_assert(G == 2, "unrolled below");
      typedef std::integral_constant<bool, true> more_t;
      typedef std::integral_constant<bool, false> last_t;
      typedef std::integral_constant<int, 0> s0_t;
      typedef std::integral_constant<int, 1> s1_t;
      meet();
      read_step(0, 0);
      int kt = 0;
#pragma unroll 1
      for (; kt + G < KT; kt += G) {
        step(s0_t{}, more_t{});
        meet();                                  // the group before this one is in registers
        step(s1_t{}, more_t{});
      }
      if (KT - kt == 1) {                        // the last group: one or two steps
        step(s0_t{}, last_t{});
      } else {
        step(s0_t{}, more_t{});
        step(s1_t{}, last_t{});
      }
      if (CHUNKED && !first_fold) {
#pragma unroll
        for (int v = 0; v < 16; ++v) tot[0][0][v] = tot_l[v * 64];
      }
    }
  } else
  for (int kt = 0; kt < KT; ++kt) {
    if constexpr (NS == 1) {
      // a single stage: the step is fetched, awaited and consumed in turn.  Nothing overlaps inside the
      // block; the small LDS footprint lets more blocks share a CU, which is what short reductions need.
      if (kt > 0) __builtin_amdgcn_s_barrier();            // every wave is done reading the stage
      if (do_load) {
        issue(0);
        __builtin_amdgcn_s_waitcnt(vmcnt_imm(0));
      }
      __builtin_amdgcn_s_barrier();                        // every wave's part of step kt is in LDS
    } else {
      // step kt's loads were issued NS-1 steps ago; up to NS-2 newer steps may stay in flight
      if (do_load) {
        if (kt + NS - 1 <= KT) __builtin_amdgcn_s_waitcnt(vmcnt_imm((NS - 2) * L));
        else __builtin_amdgcn_s_waitcnt(vmcnt_imm(0));
        scale_steps(stage, kt);
      }
      __builtin_amdgcn_s_barrier();          // every wave's part of step kt is in LDS; step kt-1 fully consumed
      if (do_load && kt + NS - 1 < KT) issue(fill);
    }
    if (do_math) compute(stage, fresh);
    fresh = false;
    stage = stage + 1 == NS ? 0 : stage + 1;
    fill = fill + 1 == NS ? 0 : fill + 1;
    if (CHUNKED && --to_fold == 0 && kt + 1 < KT) {       // chunk boundary: bank the chunk's sum
      to_fold = p.kt_chunk;
      fresh = true;
#pragma unroll
      for (int i = 0; i < TM; ++i)
#pragma unroll
        for (int j = 0; j < TN; ++j)
#pragma unroll
          for (int v = 0; v < 16; ++v) tot[i][j][v] = tot[i][j][v] + acc[i][j][v];
    }
  }
  __syncthreads();
  if (WS && fetcher) return;               // no barrier below this point

  // ---- epilogue -----------------------------------------------------------------------------
  // accumulator element v of lane l is row 8*(v/4) + 4*(l/32) + v%4, column l%32 of a 32x32 tile.
  // Per 32-row strip: SubnetNorm scale/shift on the accumulators, fp32 strip into this wave's LDS
  // region, then each lane takes (row, 8 consecutive channels): residual, activation, store.
  float* epi = (float*)smem + wave * 32 * Cfg::EPI_STRIDE;
  constexpr int OCT = WTN / 8;                 // channel octets per staged row
  constexpr int PAIRS = 32 * OCT / 64;         // (row, octet) pairs per lane
  // ACT, RES (0 none, 1 added before the activation, 2 after) and F32 are uniform over the launch's
  // problem: one dispatch below instead of per-element tests.
  // Small deep rings: the product was taken transposed, so that accumulator elements 4 q .. 4 q + 3 of a lane are channels
  // 8 q + 4 (l / 32) .. + 3 of pixel l % 32 (HALF: 16 q + 4 (l / 16) .. + 3 of pixel l % 16), and go out as 8-byte pieces with no turn through LDS, which is on the
  // critical path of a launch of few tiles (0.48 us of a lone request's 3.5 us a launch).  Only SubnetNorm's vectors do.
  auto epilogue_direct = [&](auto act_c, auto res_c, auto f32_c) __attribute__((always_inline)) {
    constexpr int ACT = decltype(act_c)::value, RES = decltype(res_c)::value;
    constexpr bool F32 = decltype(f32_c)::value;
    float* const norm = (float*)smem + wave * 64;               // this wave's 32 scales, then 32 shifts
    norm[lane] = lane < 32 ? sc[0] : sh[0];
    __builtin_amdgcn_wave_barrier();
    float4 sc4[PIECES], sh4[PIECES];
#pragma unroll
    for (int q = 0; q < PIECES; ++q) {
      sc4[q] = *(const float4*)(norm + PIECE * q + lane_k);
      sh4[q] = *(const float4*)(norm + 32 + PIECE * q + lane_k);
    }
    if (px_m >= p.M) return;
#pragma unroll
    for (int q = 0; q < PIECES; ++q) {
      const int k = px_k + PIECE * q;
      const float scq[4] = {sc4[q].x, sc4[q].y, sc4[q].z, sc4[q].w}, shq[4] = {sh4[q].x, sh4[q].y, sh4[q].z, sh4[q].w};
      const float rv[4] = {__uint_as_float(res_early[DIRECT ? q : 0].x << 16), __uint_as_float(res_early[DIRECT ? q : 0].x & 0xffff0000u),
                           __uint_as_float(res_early[DIRECT ? q : 0].y << 16), __uint_as_float(res_early[DIRECT ? q : 0].y & 0xffff0000u)};
      float val[4];
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        const int v = 4 * q + e;
        val[e] = fmaf(CHUNKED ? tot[0][0][v] + acc[0][0][v] : acc[0][0][v], scq[e], shq[e]);
        if (RES == 1) val[e] += rv[e];
        val[e] = apply_act(val[e], ACT);
        if (RES == 2) val[e] += rv[e];
      }
      if (k >= p.K) continue;
      if (F32) {
        if (in_kernel_reduce)
          store_f4_agent((float*)((char*)p.part_buf + (size_t)part * p.part_stride) + (size_t)local * (BM * BN) + (px_m - m0) * BN + (k - n0), val);
        else
          *(float4*)((float*)((char*)p.y + (size_t)part * p.part_stride) + (long)px_m * p.y_stride + k) = make_float4(val[0], val[1], val[2], val[3]);
      } else {
        *(uint2*)((bf16_t*)p.y + (long)px_m * p.y_stride + k) = make_uint2(pack_bf16x2(val[0], val[1]), pack_bf16x2(val[2], val[3]));
      }
    }
  };
  auto epilogue = [&](auto act_c, auto res_c, auto f32_c) __attribute__((always_inline)) {
    if constexpr (DIRECT) {
      epilogue_direct(act_c, res_c, f32_c);
      return;
    }
    constexpr int ACT = decltype(act_c)::value, RES = decltype(res_c)::value;
    constexpr bool F32 = decltype(f32_c)::value;
    // Residual rows.  With several 32-row strips per wave they are all requested up front, so that
    // one round trip runs under the staging of the first strip instead of one per strip; with a
    // single strip the request goes after the staging writes, when the accumulators' registers are free.
    constexpr bool RES_UP_FRONT = TM > 1;
    uint4 r4[TM][PAIRS];
    auto load_res = [&](int i) {
#pragma unroll
      for (int t = 0; t < PAIRS; ++t) {
        const int id = t * 64 + lane;
        const int row = id / OCT, oct = id - row * OCT;
        const int m = m0 + wm * WTM + i * 32 + row;
        const int k = n0 + wn * WTN + oct * 8;
        r4[i][t] = (m < p.M && k < p.K) ? *(const uint4*)((const bf16_t*)p.res + (long)m * p.res_stride + k)
                                        : make_uint4(0, 0, 0, 0);
      }
    };
    if (RES != 0 && RES_UP_FRONT) {
#pragma unroll
      for (int i = 0; i < TM; ++i) load_res(i);
    }
#pragma unroll
    for (int i = 0; i < TM; ++i) {
#pragma unroll
      for (int j = 0; j < TN; ++j)
#pragma unroll
        for (int v = 0; v < 16; ++v)
          epi[(8 * (v >> 2) + row_l + (v & 3)) * Cfg::EPI_STRIDE + j * 32 + col_l] =
              fmaf(CHUNKED ? tot[i][j][v] + acc[i][j][v] : acc[i][j][v], sc[j], sh[j]);
      if (RES != 0 && !RES_UP_FRONT) load_res(i);
      // wave-private region: the wave's own LDS writes are visible to its later reads
      __builtin_amdgcn_wave_barrier();
      __builtin_amdgcn_s_waitcnt(0xc07f);        // lgkmcnt(0)
      __builtin_amdgcn_wave_barrier();
#pragma unroll
      for (int t = 0; t < PAIRS; ++t) {
        const int id = t * 64 + lane;
        const int row = id / OCT, oct = id - row * OCT;
        const int m = m0 + wm * WTM + i * 32 + row;
        const int k = n0 + wn * WTN + oct * 8;
        const float4 v0 = *(const float4*)(epi + row * Cfg::EPI_STRIDE + oct * 8);
        const float4 v1 = *(const float4*)(epi + row * Cfg::EPI_STRIDE + oct * 8 + 4);
        float val[8] = {v0.x, v0.y, v0.z, v0.w, v1.x, v1.y, v1.z, v1.w};
        float rv[8];
        if (RES != 0) {
          const unsigned ru[4] = {r4[i][t].x, r4[i][t].y, r4[i][t].z, r4[i][t].w};
#pragma unroll
          for (int e = 0; e < 4; ++e) {
            rv[2 * e] = __uint_as_float(ru[e] << 16);
            rv[2 * e + 1] = __uint_as_float(ru[e] & 0xffff0000u);
          }
        }
        if (RES == 1) {
#pragma unroll
          for (int e = 0; e < 8; ++e) val[e] += rv[e];
        }
#pragma unroll
        for (int e = 0; e < 8; ++e) val[e] = apply_act(val[e], ACT);
        if (RES == 2) {
#pragma unroll
          for (int e = 0; e < 8; ++e) val[e] += rv[e];
        }
        if (m < p.M && k < p.K) {
          if (F32) {
            if (in_kernel_reduce) {
              // tile-major: every tile's sums fill whole cache lines of their own, so that no block ever
              // pulls a line into its L2 that another tile's blocks have yet to write
              float* yo = (float*)((char*)p.part_buf + (size_t)part * p.part_stride) + (size_t)local * (BM * BN) +
                          (m - m0) * BN + (k - n0);
              store_f8_agent(yo, val);
            } else {
              float* yo = (float*)((char*)p.y + (size_t)part * p.part_stride) + (long)m * p.y_stride + k;
              *(float4*)yo = make_float4(val[0], val[1], val[2], val[3]);
              *(float4*)(yo + 4) = make_float4(val[4], val[5], val[6], val[7]);
            }
          } else {
            uint4 o;
            o.x = pack_bf16x2(val[0], val[1]);
            o.y = pack_bf16x2(val[2], val[3]);
            o.z = pack_bf16x2(val[4], val[5]);
            o.w = pack_bf16x2(val[6], val[7]);
            *(uint4*)((bf16_t*)p.y + (long)m * p.y_stride + k) = o;
          }
        }
      }
      __builtin_amdgcn_wave_barrier();
    }
  };
  using std::integral_constant;
  typedef integral_constant<bool, true> yes_t;
  typedef integral_constant<bool, false> no_t;
#define SNA_EPI(A, R) epilogue(integral_constant<int, A>{}, integral_constant<int, R>{}, no_t{})
  const int res_mode = p.res ? (p.res_after_act ? 2 : 1) : 0;
  if (in_kernel_reduce) {
    epilogue(integral_constant<int, SNA_ACT_NONE>{}, integral_constant<int, 0>{}, yes_t{});      // bare chunk sums to part_buf
    // Count arrivals at this tile.  The chunk sums went out as write-through agent-scope stores; once
    // every thread's stores have completed, the block's one atomic publishes them.  The block that sees
    // parts - 1 earlier arrivals is the last and owns the tile from here on (nobody waits for anybody).
    // It puts the counter back to zero for the next launch that uses it.
    __builtin_amdgcn_s_waitcnt(vmcnt_imm(0));
    __syncthreads();
    int* const flag = (int*)smem;               // the ring is dead by now
    if (threadIdx.x == 0) {
      int* const cnt = p.counters + local;
      const int seen = atomicAdd(cnt, 1);
      const int last = seen == p.parts - 1;
      if (last) atomicExch(cnt, 0);
      *flag = last;
    }
    __syncthreads();
    if (*flag == 0) return;
    constexpr int OCT_T = BN / 8;
    const int nthr = 64 * NW;                   // fetching waves of a wave-specialised block have left
    for (int id = threadIdx.x; id < BM * OCT_T; id += nthr) {
      const int row = id / OCT_T, oct = id - row * OCT_T;
      const int m = m0 + row, k = n0 + oct * 8;
      if (m < p.M && k < p.K) reduce_octet<true>(p, p.part_buf + (size_t)local * (BM * BN) + row * BN + oct * 8, m, k);
    }
  } else if (p.out_fp32) {                                     // logits: no activation, no residual
    if (p.act == SNA_ACT_NONE && res_mode == 0) epilogue(integral_constant<int, SNA_ACT_NONE>{}, integral_constant<int, 0>{}, yes_t{});
  } else if (p.act == SNA_ACT_RELU) {
    if (res_mode == 0) SNA_EPI(SNA_ACT_RELU, 0); else if (res_mode == 1) SNA_EPI(SNA_ACT_RELU, 1); else SNA_EPI(SNA_ACT_RELU, 2);
  } else if (p.act == SNA_ACT_NONE) {
    if (res_mode == 0) SNA_EPI(SNA_ACT_NONE, 0); else SNA_EPI(SNA_ACT_NONE, 1);
  } else if (p.act == SNA_ACT_HSWISH) {
    if (res_mode == 0) SNA_EPI(SNA_ACT_HSWISH, 0); else if (res_mode == 1) SNA_EPI(SNA_ACT_HSWISH, 1); else SNA_EPI(SNA_ACT_HSWISH, 2);
  } else {
    if (res_mode == 0) SNA_EPI(SNA_ACT_GELU, 0); else if (res_mode == 1) SNA_EPI(SNA_ACT_GELU, 1); else SNA_EPI(SNA_ACT_GELU, 2);
  }
#undef SNA_EPI
#endif
}

template <int BM, int BN, int WARPS_M, int WARPS_N, int NS, bool CHUNKED, int FW, bool GATED = false>
__global__ __launch_bounds__(64 * (WARPS_M * WARPS_N + FW), igemm_waves(BM, BN, WARPS_M * WARPS_N, NS, CHUNKED, FW))
void igemm_kernel(const ConvGroupArgs args) {
  // The first problem's descriptor sits at a fixed offset of the arguments, so its load does not wait for the problem search.
  ConvProblem p = args.p[0];
  int local;
  if (args.n > 1) {
    const TilePlace at = place_of_block(args, blockIdx.x);
    if (at.problem > 0) p = args.p[at.problem];
    local = at.tile;
  } else {
    local = tile_of_block(p);
  }
  if (local < 0) return;
  igemm_tile<BM, BN, WARPS_M, WARPS_N, NS, CHUNKED, FW, GATED>(p, local);
}

// A lone pointwise stride-1 problem on a small deep ring.  What the first loads need comes in scalar arguments, which the
// dispatch puts into registers (they lead the list: 12 of the 14 words there is room for); a struct's first use waits
// 0.36 us for a load of it, in a launch of 3 us.  The rest of the descriptor is read under the first loads.
struct PwArgs {                        // host side of the scalars
  const void *x, *w; unsigned x_bytes, w_bytes; int M, tiles; unsigned ck, tn, tn_m; int wk;
  static bool fits(const ConvProblem& p) {
    return p.R == 1 && p.S == 1 && p.stride == 1 && p.pad == 0 && p.parts == 1 && p.tile_start == 0 && p.C8 < 65536 && p.K / 8 < 65536 && p.tiles_n < (1 << 24);
  }
  static PwArgs of(const ConvProblem& p) {
    return {p.x, p.w, p.x_bytes, p.w_bytes, p.M, p.tiles, (unsigned)p.C8 | (unsigned)(p.K / 8) << 16,
            (unsigned)p.tiles_n | (unsigned)(p.by_tiles_n.shift + 1) << 24, p.by_tiles_n.m, p.wk};
  }
};
template <int BM, int BN, int WARPS_M, int WARPS_N, int NS, bool CHUNKED, int FW, bool GATED>
__global__ __launch_bounds__(64 * (WARPS_M * WARPS_N + FW), igemm_waves(BM, BN, WARPS_M * WARPS_N, NS, CHUNKED, FW))
void igemm_pw_kernel(const void* x, const void* w, unsigned x_bytes, unsigned w_bytes, int M, int tiles, unsigned ck, unsigned tn,
                     unsigned tn_m, int wk, const ConvProblem q) {
  ConvProblem p = q;
  p.x = x; p.w = w; p.x_bytes = x_bytes; p.w_bytes = w_bytes; p.M = M; p.wk = wk;
  p.C8 = (int)(ck & 0xffffu); p.K8 = p.C8; p.C = p.C8 * 8; p.K = (int)(ck >> 16) * 8;
  p.tiles = tiles; p.tile_start = 0; p.tiles_n = (int)(tn & 0xffffffu); p.by_tiles_n.m = tn_m; p.by_tiles_n.shift = (int)(tn >> 24) - 1;
  p.R = 1; p.S = 1; p.stride = 1; p.pad = 0; p.parts = 1; p.counters = nullptr; p.kt_part = 1 << 30;
  const int local = tile_of_block(p);
  if (local < 0) return;
  igemm_tile<BM, BN, WARPS_M, WARPS_N, NS, CHUNKED, FW, GATED>(p, local);
}
typedef void (*PwKernel)(const void*, const void*, unsigned, unsigned, int, int, unsigned, unsigned, unsigned, int, const ConvProblem);

// One tile variant: the kernel with and without in-register chunk sums, and what its launch needs
struct Variant {
  int bm, bn, threads, smem, ns, stage_bytes, epi_bytes;
  void (*fn)(const ConvGroupArgs); void (*fn_chunked)(const ConvGroupArgs);
  void (*fn_gated)(const ConvGroupArgs);       // nullptr: cannot scale its input
  bool slab;             // conv3_slab_kernel: 3x3 stride-1 layers only; stage_bytes is the weight ring's
  bool deep;             // a deep ring: at most kDeepMaxSteps K steps per block, which is the LDS its tap table has (and a
                         // bound for pointwise layers as well, which have no table but whose times were not measured beyond)
  bool totals_lds;       // its chunk-folding kernel keeps the running totals in LDS
  PwKernel pw = nullptr, pw_chunked = nullptr, pw_gated = nullptr;      // for a lone pointwise problem
  int group = 1;         // stages its computing waves read at a time
};
constexpr int kDeepMaxSteps = 128;
constexpr int kDeepVariantCount = 3;
extern const Variant kDeepVariants[kDeepVariantCount];

}  // namespace sna
