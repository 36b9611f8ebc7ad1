// Depthwise WeightSlice convolution (centre k x k window of a stored 7x7, leading channels) with
// fused SubnetNorm + activation, and the squeeze-excite gate.  All of it is HBM-bound streaming:
// threads own 8 consecutive channels (16-byte loads / stores, channel-fastest across lanes).
#include "common.h"

namespace sna {

__device__ __forceinline__ void unpack8(const uint4 v, float* f) {
  const unsigned u[4] = {v.x, v.y, v.z, v.w};
#pragma unroll
  for (int e = 0; e < 4; ++e) {
    f[2 * e] = __uint_as_float(u[e] << 16);
    f[2 * e + 1] = __uint_as_float(u[e] & 0xffff0000u);
  }
}
__device__ __forceinline__ uint4 pack8(const float* f) {
  uint4 o;
  o.x = pack_bf16x2(f[0], f[1]);
  o.y = pack_bf16x2(f[2], f[3]);
  o.z = pack_bf16x2(f[4], f[5]);
  o.w = pack_bf16x2(f[6], f[7]);
  return o;
}

// ---------------------------------------------------------------------------------------------
// One thread = TW adjacent output pixels of one row x 8 channels.  For every kernel row the
// thread loads the (TW-1)*STRIDE + K input columns it needs once and reuses them across its TW
// outputs, so an input element is fetched K (not K*K) times per output row from L1/L2 and once
// from HBM.  y = act(scale[c] * sum_{r,s} x * w[r0+r][s0+s][c] + shift[c]).
//
// POOL (the layer feeds a squeeze-excite gate): blocks are laid out per request, and each block
// also leaves the per-channel sum of the outputs it stored (the rounded values, which is what the
// gate's average pool is defined on), added in a fixed order: per thread over its outputs, then over
// the block's threads of one channel group in thread order.  The gate adds the blocks' sums in order.
// ---------------------------------------------------------------------------------------------
constexpr int DW_TW = 4;

template <int K, int STRIDE, bool POOL>
__global__ __launch_bounds__(256) void depthwise_kernel(const DwGroupArgs args) {
  const int g = find_problem(args, blockIdx.x);
  const DwProblem& p = args.p[g];
  const int c8n = p.C >> 3;
  const int strips = (p.Wo + DW_TW - 1) / DW_TW;
  const long per_req = (long)p.Ho * strips * c8n;
  const int block = blockIdx.x - p.tile_start;
  long idx;
  bool valid;
  if (POOL) {
    const long in_req = (long)(block % p.bpr) * 256 + threadIdx.x;
    valid = in_req < per_req;
    idx = (long)(block / p.bpr) * per_req + in_req;
  } else {
    idx = (long)block * 256 + threadIdx.x;
    valid = idx < per_req * p.N;
    if (!valid) return;
  }
  float psum[8];
#pragma unroll
  for (int e = 0; e < 8; ++e) psum[e] = 0.f;
  if (valid) {
  const int c8 = idx % c8n;
  long t = idx / c8n;
  const int qs = t % strips; t /= strips;
  const int pp = t % p.Ho;
  const int n = t / p.Ho;
  const int q0 = qs * DW_TW;
  constexpr int COLS = (DW_TW - 1) * STRIDE + K;
  constexpr int PAD = K / 2;
  const bf16_t* x = (const bf16_t*)p.x + (long)n * p.H * p.W * p.C + c8 * 8;
  const bf16_t* w = (const bf16_t*)p.w + c8 * 8;           // already at the centre window's first tap
  // The taps of a kernel row are taken two at a time with v_dot2_f32_bf16: per channel one register
  // holds (x[col], x[col + 1]) and one (w[s], w[s + 1]), built from the channel-pair words of memory with
  // byte permutes; no bf16 -> fp32 unpacking and half the multiply-add instructions.  An odd last tap
  // is paired with a zero weight.
  typedef __bf16 bf16x2_t __attribute__((ext_vector_type(2)));
  constexpr int WP = (K + 1) / 2;                          // tap pairs per kernel row
  constexpr int CSTEP = STRIDE == 2 ? 2 : 1;                 // stride 2 only ever pairs (even, odd) columns
  float acc[DW_TW][8];
#pragma unroll
  for (int o = 0; o < DW_TW; ++o)
#pragma unroll
    for (int e = 0; e < 8; ++e) acc[o][e] = 0.f;
  const int iw0 = q0 * STRIDE - PAD;
#pragma unroll
  for (int r = 0; r < K; ++r) {
    const int ih = pp * STRIDE + r - PAD;
    if (ih < 0 || ih >= p.H) continue;
    uint4 raw[COLS + 1];
#pragma unroll
    for (int cidx = 0; cidx < COLS; ++cidx) {
      const int iw = iw0 + cidx;
      raw[cidx] = (iw >= 0 && iw < p.W) ? *(const uint4*)(x + ((long)ih * p.W + iw) * p.C) : make_uint4(0, 0, 0, 0);
    }
    raw[COLS] = make_uint4(0, 0, 0, 0);
    unsigned wp[WP][8];                    // [tap pair][channel]: (w[2t], w[2t + 1])
#pragma unroll
    for (int t = 0; t < WP; ++t) {
      const uint4 w0 = *(const uint4*)(w + (long)r * p.wr + (long)(2 * t) * p.ws);
      const uint4 w1 = 2 * t + 1 < K ? *(const uint4*)(w + (long)r * p.wr + (long)(2 * t + 1) * p.ws) : make_uint4(0, 0, 0, 0);
      const unsigned a0[4] = {w0.x, w0.y, w0.z, w0.w}, a1[4] = {w1.x, w1.y, w1.z, w1.w};
#pragma unroll
      for (int d = 0; d < 4; ++d) {
        wp[t][2 * d] = __builtin_amdgcn_perm(a1[d], a0[d], 0x05040100u);
        wp[t][2 * d + 1] = __builtin_amdgcn_perm(a1[d], a0[d], 0x07060302u);
      }
    }
#pragma unroll
    for (int c = 0; c < COLS; c += CSTEP) {
      // is this column pair the start of a tap pair of some output?  (c = o * STRIDE + 2 t)
      bool used = false;
#pragma unroll
      for (int o = 0; o < DW_TW; ++o)
#pragma unroll
        for (int t = 0; t < WP; ++t) used = used || (c == o * STRIDE + 2 * t);
      if (!used) continue;
      const unsigned x0[4] = {raw[c].x, raw[c].y, raw[c].z, raw[c].w};
      const unsigned x1[4] = {raw[c + 1].x, raw[c + 1].y, raw[c + 1].z, raw[c + 1].w};
      unsigned xp[8];                      // [channel]: (x[col c], x[col c + 1])
#pragma unroll
      for (int d = 0; d < 4; ++d) {
        xp[2 * d] = __builtin_amdgcn_perm(x1[d], x0[d], 0x05040100u);
        xp[2 * d + 1] = __builtin_amdgcn_perm(x1[d], x0[d], 0x07060302u);
      }
#pragma unroll
      for (int o = 0; o < DW_TW; ++o)
#pragma unroll
        for (int t = 0; t < WP; ++t)
          if (c == o * STRIDE + 2 * t) {
#pragma unroll
            for (int e = 0; e < 8; ++e)
              acc[o][e] = __builtin_amdgcn_fdot2_f32_bf16(__builtin_bit_cast(bf16x2_t, xp[e]),
                                                          __builtin_bit_cast(bf16x2_t, wp[t][e]), acc[o][e], false);
          }
    }
  }
  if (p.raw_out) {
    float* yr = (float*)p.y + (((long)n * p.Ho + pp) * p.Wo) * p.C + c8 * 8;
#pragma unroll
    for (int o = 0; o < DW_TW; ++o) {
      if (q0 + o >= p.Wo) break;
      *(float4*)(yr + (long)(q0 + o) * p.C) = make_float4(acc[o][0], acc[o][1], acc[o][2], acc[o][3]);
      *(float4*)(yr + (long)(q0 + o) * p.C + 4) = make_float4(acc[o][4], acc[o][5], acc[o][6], acc[o][7]);
    }
    return;
  }
  float sc[8], sh[8];
#pragma unroll
  for (int e = 0; e < 8; ++e) { sc[e] = p.scale[c8 * 8 + e]; sh[e] = p.shift[c8 * 8 + e]; }
  bf16_t* y = (bf16_t*)p.y + (((long)n * p.Ho + pp) * p.Wo) * p.C + c8 * 8;
#pragma unroll
  for (int o = 0; o < DW_TW; ++o) {
    if (q0 + o >= p.Wo) break;
    float v[8];
#pragma unroll
    for (int e = 0; e < 8; ++e) v[e] = apply_act(fmaf(acc[o][e], sc[e], sh[e]), p.act);
    const uint4 packed = pack8(v);
    *(uint4*)(y + (long)(q0 + o) * p.C) = packed;
    if (POOL) {
      unpack8(packed, v);
#pragma unroll
      for (int e = 0; e < 8; ++e) psum[e] += v[e];
    }
  }
  }
  if (POOL) {
    __shared__ float red[8][256];
#pragma unroll
    for (int e = 0; e < 8; ++e) red[e][threadIdx.x] = psum[e];
    __syncthreads();
    // thread t < c8n owns the channel group of the block's t-th element; its other elements sit c8n apart
    if ((int)threadIdx.x < c8n) {
      const int in_block = block % p.bpr;
      const int c8 = (int)(((long)in_block * 256 + threadIdx.x) % c8n);
      float s8[8];
#pragma unroll
      for (int e = 0; e < 8; ++e) s8[e] = 0.f;
      for (int t = threadIdx.x; t < 256; t += c8n)
#pragma unroll
        for (int e = 0; e < 8; ++e) s8[e] += red[e][t];
      float* out = p.pool_part + ((long)block * p.C) + c8 * 8;     // block = n * bpr + in_block
      *(float4*)out = make_float4(s8[0], s8[1], s8[2], s8[3]);
      *(float4*)(out + 4) = make_float4(s8[4], s8[5], s8[6], s8[7]);
    }
  }
}

hipError_t launch_depthwise(const DwGroupArgs& a, hipStream_t s) {
  // one launch per (kernel size, stride, with / without pool) present among the problems
  for (int pool = 0; pool < 2; ++pool)
    for (int k = 3; k <= 7; k += 2)
      for (int st = 1; st <= 2; ++st) {
        DwGroupArgs b;
        b.n = 0;
        int start = 0;
        for (int i = 0; i < a.n; ++i) {
          if (a.p[i].k != k || a.p[i].stride != st || (a.p[i].pool_part != nullptr) != (pool == 1)) continue;
          DwProblem p = a.p[i];
          const long strips = (p.Wo + DW_TW - 1) / DW_TW;
          const long per_req = (long)p.Ho * strips * (p.C / 8);
          if (pool) {
            // every block must meet every channel group, or some sums would never be written
            if (p.C / 8 > 256 || p.bpr != (int)((per_req + 255) / 256)) return hipErrorInvalidValue;
            p.tiles = p.N * p.bpr;
          } else {
            p.tiles = (int)((per_req * p.N + 255) / 256);
          }
          p.tile_start = start;
          start += p.tiles;
          b.p[b.n++] = p;
        }
        if (!b.n) continue;
#define SNA_DW(KK, SS)                                                                                              \
  if (k == KK && st == SS) {                                                                                        \
    if (pool) hipLaunchKernelGGL((depthwise_kernel<KK, SS, true>), dim3(start), dim3(256), 0, s, b);               \
    else hipLaunchKernelGGL((depthwise_kernel<KK, SS, false>), dim3(start), dim3(256), 0, s, b);                   \
  }
        SNA_DW(3, 1); SNA_DW(3, 2); SNA_DW(5, 1); SNA_DW(5, 2); SNA_DW(7, 1); SNA_DW(7, 2);
#undef SNA_DW
        hipError_t e = hipGetLastError();
        if (e != hipSuccess) return e;
      }
  return hipSuccess;
}

int depthwise_pool_blocks(int Ho, int Wo, int C) {
  const long strips = (Wo + DW_TW - 1) / DW_TW;
  return (int)(((long)Ho * strips * (C / 8) + 255) / 256);
}

// ---------------------------------------------------------------------------------------------
// Squeeze-excite gate:
//   z = mean over pixels of the depthwise output (from the depthwise blocks' partial sums)
//   h = relu(W1[:Q,:C] z + b1[:Q]);  gate = hardsigmoid(W2[:C,:Q] h + b2[:C]);  y = x * gate
// The layer that follows applies the gate where its matrix tile can; pool, h and gate then take one launch for gates of up
// to SE_ONE_MACS weights and two for larger ones (h, then the gate).  Where it cannot, the second launch scales x as well.
// ---------------------------------------------------------------------------------------------
__device__ __forceinline__ SeProblem se_problem(const SeProblem& src) {
  SeProblem p = pinned(src);
  p.x = in_global(p.x); p.y = in_global(p.y); p.w1 = in_global(p.w1); p.b1 = in_global(p.b1); p.w2 = in_global(p.w2);
  p.b2 = in_global(p.b2); p.pooled = in_global(p.pooled); p.gate = in_global(p.gate); p.hidden = in_global(p.hidden);
  return p;
}
// h[n][o] = relu(W1[o, :C] . z[n] + b1[o]).  A block owns one request and 32 outputs.  It first
// builds z in LDS (partial sums added in block order, then scaled by 1 / HW); each of its 4 waves
// then computes 8 outputs together: lanes read 8 consecutive bf16 weights (16 bytes) of each row and
// the matching z, and the wave reduces each output in a fixed order.
template <class Args>
__global__ __launch_bounds__(256) void se_hidden_kernel(const Args args) {
  extern __shared__ __attribute__((aligned(16))) float z[];
  const int g = find_problem(args, blockIdx.x);
  const SeProblem p = se_problem(args.p[g]);
  const int oblocks = (p.Q + 31) / 32;
  const int local = blockIdx.x - p.tile_start;
  const int n = local / oblocks, ob = local % oblocks;
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  // The wave's 8 rows are independent, and none of their weights depends on z: the first loads of all of them (512
  // channels) go out before the pooled sums are read, the next ones before the first are used (one row at a time paid the
  // L2 latency 8 times over, weights after z once more: a lone request's launch 5.5 -> 4.6 us).
  const bf16_t* w = (const bf16_t*)p.w1;
  const int o0 = ob * 32 + wave * 8;
  auto rows = [&](int i8, uint4 (&wq)[8]) {
#pragma unroll
    for (int t = 0; t < 8; ++t)
      wq[t] = i8 < (p.C >> 3) && o0 + t < p.Q ? *(const uint4*)(w + (long)(o0 + t) * p.w1_stride + i8 * 8) : make_uint4(0, 0, 0, 0);
  };
  uint4 cur[8], nxt[8];
  rows(lane, cur);
  const float bias = lane < 8 && o0 + lane < p.Q ? p.b1[o0 + lane] : 0.f;
  const float* part = p.pooled + (long)n * p.pool_segs * p.C;
  for (int c4 = threadIdx.x; c4 < (p.C >> 2); c4 += 256) {
    float4 a = *(const float4*)(part + c4 * 4);
#pragma unroll 8                                    // loads in batches of 8, the additions still in block order
    for (int sgm = 1; sgm < p.pool_segs; ++sgm) {
      const float4 b = *(const float4*)(part + (long)sgm * p.C + c4 * 4);
      a.x += b.x; a.y += b.y; a.z += b.z; a.w += b.w;
    }
    a.x *= p.inv_hw; a.y *= p.inv_hw; a.z *= p.inv_hw; a.w *= p.inv_hw;
    *(float4*)(z + c4 * 4) = a;
  }
  __syncthreads();
  float a[8];
#pragma unroll
  for (int t = 0; t < 8; ++t) a[t] = 0.f;
  for (int i8 = lane; i8 < (p.C >> 3); i8 += 64) {
    const float4 x0 = *(const float4*)(z + i8 * 8), x1 = *(const float4*)(z + i8 * 8 + 4);
    rows(i8 + 64, nxt);
#pragma unroll
    for (int t = 0; t < 8; ++t) {
      float wv[8];
      unpack8(cur[t], wv);
      a[t] = fmaf(wv[0], x0.x, a[t]); a[t] = fmaf(wv[1], x0.y, a[t]); a[t] = fmaf(wv[2], x0.z, a[t]); a[t] = fmaf(wv[3], x0.w, a[t]);
      a[t] = fmaf(wv[4], x1.x, a[t]); a[t] = fmaf(wv[5], x1.y, a[t]); a[t] = fmaf(wv[6], x1.z, a[t]); a[t] = fmaf(wv[7], x1.w, a[t]);
    }
#pragma unroll
    for (int t = 0; t < 8; ++t) cur[t] = nxt[t];
  }
  float mine = 0.f;                          // lane t keeps output t's sum
#pragma unroll
  for (int t = 0; t < 8; ++t) {
    const float sum = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(lane_sum(a[t])), 63));
    mine = lane == t ? sum : mine;
  }
  if (lane < 8 && o0 + lane < p.Q) p.hidden[(long)n * p.Q + o0 + lane] = fmaxf(mine + bias, 0.f);
}

// gate[n][c] = hardsigmoid(W2[c, :Q] . h[n] + b2[c]);  y[n, hw, c] = bf16(x[n, hw, c] * gate[n][c]).
// A block owns one request, 64 channels and SE_PIX pixels: its threads first compute the 64 gate
// values (4 threads per channel, each every fourth octet of Q in order, so that they read a row together, their sums added in
// a fixed order; a quarter of the row each, 64 cache lines per load, took 8.5 us instead of 5.2 for 64 x 960 gates of 240), then
// stream the pixels, 8 lanes per pixel row of 128 bytes.  The gate is recomputed by every pixel
// segment of a request: 64 x Q multiply-adds against one more launch and a round trip through memory.
constexpr int SE_PIX = 256;
constexpr int SE_MAX_Q = 512;       // squeeze channels per gate (host-checked)
template <bool SCALE, class Args>       // SCALE false: the gate goes to p.gate and the layer that follows applies it
__global__ __launch_bounds__(256) void se_gate_kernel(const Args args) {
  __shared__ float gate_s[64];
  __shared__ __attribute__((aligned(16))) float h_s[SE_MAX_Q];
  const int g = find_problem(args, blockIdx.x);
  const SeProblem p = se_problem(args.p[g]);
  const int cgroups = (p.C + 63) / 64, psegs = SCALE ? (p.HW + SE_PIX - 1) / SE_PIX : 1;
  int local = blockIdx.x - p.tile_start;
  const int pseg = local % psegs; local /= psegs;
  const int cg = local % cgroups;
  const int n = local / cgroups;
  // the thread's pixels do not depend on the gate: request them first, so that their latency runs
  // under the gate computation
  const int c8 = cg * 8 + (threadIdx.x & 7);
  const bool live = c8 * 8 < p.C;
  const int h_end = (pseg + 1) * SE_PIX < p.HW ? (pseg + 1) * SE_PIX : p.HW;
  const int h0 = pseg * SE_PIX + (threadIdx.x >> 3);
  const bf16_t* x = (const bf16_t*)p.x + (long)n * p.HW * p.C + c8 * 8;
  uint4 px[SE_PIX / 32];
#pragma unroll
  for (int j = 0; j < SE_PIX / 32; ++j)
    px[j] = (SCALE && live && h0 + 32 * j < h_end) ? *(const uint4*)(x + (long)(h0 + 32 * j) * p.C) : make_uint4(0, 0, 0, 0);
  // so do the gate's weights: a fixed trip count, loads first (a loop over [begin, end) paid the L2 latency once per 8
  // weights), and ahead of the hidden vector, which the barrier waits for
  const int gc = cg * 64 + (threadIdx.x >> 2), quarter = threadIdx.x & 3;
  const int q8n = p.Q >> 3;
  uint4 wq[SE_MAX_Q / 32];
  {
    const bf16_t* w = (const bf16_t*)p.w2 + (long)gc * p.w2_stride;
#pragma unroll
    for (int j = 0; j < SE_MAX_Q / 32; ++j) {
      const int i8 = j * 4 + quarter;
      wq[j] = (gc < p.C && i8 < q8n) ? *(const uint4*)(w + i8 * 8) : make_uint4(0, 0, 0, 0);
    }
  }
  const float b2 = gc < p.C ? p.b2[gc] : 0.f;
  for (int i = threadIdx.x; i < p.Q; i += 256) h_s[i] = p.hidden[(long)n * p.Q + i];
  __syncthreads();
  {
    float a = 0.f;
    if (gc < p.C) {
#pragma unroll
      for (int j = 0; j < SE_MAX_Q / 32; ++j) {
        const int i8 = j * 4 + quarter;
        if (i8 < q8n) {
          float wv[8];
          unpack8(wq[j], wv);
          const float4 x0 = *(const float4*)(h_s + i8 * 8), x1 = *(const float4*)(h_s + i8 * 8 + 4);
          a = fmaf(wv[0], x0.x, a); a = fmaf(wv[1], x0.y, a); a = fmaf(wv[2], x0.z, a); a = fmaf(wv[3], x0.w, a);
          a = fmaf(wv[4], x1.x, a); a = fmaf(wv[5], x1.y, a); a = fmaf(wv[6], x1.z, a); a = fmaf(wv[7], x1.w, a);
        }
      }
    }
    // the channel's four sums sit in adjacent lanes: ((0 + 1) + (2 + 3))
    a += __shfl_xor(a, 1, 64);
    a += __shfl_xor(a, 2, 64);
    const float gate = fminf(fmaxf(a + b2 + 3.f, 0.f), 6.f) * (1.f / 6.f);
    if (!SCALE) {
      if (quarter == 0 && gc < p.C) p.gate[(long)n * p.pool_segs * p.C + gc] = gate;
      return;
    }
    if (quarter == 0 && gc < p.C) gate_s[threadIdx.x >> 2] = gate;
  }
  __syncthreads();
  if (!live) return;
  float gt[8];
#pragma unroll
  for (int e = 0; e < 8; ++e) gt[e] = gate_s[(threadIdx.x & 7) * 8 + e];
  bf16_t* y = (bf16_t*)p.y + (long)n * p.HW * p.C + c8 * 8;
#pragma unroll
  for (int j = 0; j < SE_PIX / 32; ++j) {
    const int h = h0 + 32 * j;
    if (h >= h_end) break;
    float v[8];
    unpack8(px[j], v);
#pragma unroll
    for (int e = 0; e < 8; ++e) v[e] *= gt[e];
    *(uint4*)(y + (long)h * p.C) = pack8(v);
  }
}

// Pool, hidden layer and gate of one request in one launch, for gates that the next layer applies: a block of 16 waves per
// request, with the arithmetic of the two kernels above (same bits).  Taken for layers of up to SE_ONE_MACS weights, which
// one CU reads in about the time that the second launch costs.
constexpr int SE_ONE_NT = 1024, SE_ONE_MACS = 32 * 1024, SE_ONE_Q = 256;
template <class Args>
__global__ __launch_bounds__(SE_ONE_NT) void se_one_kernel(const Args args) {
  extern __shared__ __attribute__((aligned(16))) float z[];
  __shared__ __attribute__((aligned(16))) float h_s[SE_ONE_Q];
  const int g = find_problem(args, blockIdx.x);
  const SeProblem p = se_problem(args.p[g]);
  const int n = blockIdx.x - p.tile_start;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const bf16_t* w1 = (const bf16_t*)p.w1;
  auto rows = [&](int o0, int i8, uint4 (&wq)[8]) {
#pragma unroll
    for (int t = 0; t < 8; ++t)
      wq[t] = i8 < (p.C >> 3) && o0 + t < p.Q ? *(const uint4*)(w1 + (unsigned)((o0 + t) * p.w1_stride + i8 * 8)) : make_uint4(0, 0, 0, 0);
  };
  uint4 cur[8];
  rows(wave * 8, lane, cur);
  // weights of the first 256 gates, four threads a channel
  const int quarter = tid & 3, q8n = p.Q >> 3;
  uint4 wq[SE_ONE_Q / 32];
  float b2 = 0.f;
  auto gate_weights = [&](int c) {
#pragma unroll
    for (int j = 0; j < SE_ONE_Q / 32; ++j) {
      const int i8 = j * 4 + quarter;
      wq[j] = (c < p.C && i8 < q8n) ? *(const uint4*)((const bf16_t*)p.w2 + (unsigned)(c * p.w2_stride + i8 * 8)) : make_uint4(0, 0, 0, 0);
    }
    b2 = c < p.C ? p.b2[c] : 0.f;
  };
  gate_weights(tid >> 2);
  const float* part = p.pooled + (long)n * p.pool_segs * p.C;
  for (unsigned c4 = tid; c4 < (unsigned)(p.C >> 2); c4 += SE_ONE_NT) {
    float4 a = *(const float4*)(part + c4 * 4);
#pragma unroll 8
    for (int sgm = 1; sgm < p.pool_segs; ++sgm) {
      const float4 b = *(const float4*)(part + (long)sgm * p.C + c4 * 4);
      a.x += b.x; a.y += b.y; a.z += b.z; a.w += b.w;
    }
    a.x *= p.inv_hw; a.y *= p.inv_hw; a.z *= p.inv_hw; a.w *= p.inv_hw;
    *(float4*)(z + c4 * 4) = a;
  }
  __syncthreads();                           // from here on nobody reads the pool sums, whose first row takes the gate
  for (int o0 = wave * 8; o0 < p.Q; o0 += SE_ONE_NT / 8) {
    if (o0 != wave * 8) rows(o0, lane, cur);
    const float bias = lane < 8 && o0 + lane < p.Q ? p.b1[o0 + lane] : 0.f;
    float a[8];
#pragma unroll
    for (int t = 0; t < 8; ++t) a[t] = 0.f;
    for (int i8 = lane; i8 < (p.C >> 3); i8 += 64) {
      const float4 x0 = *(const float4*)(z + i8 * 8), x1 = *(const float4*)(z + i8 * 8 + 4);
#pragma unroll
      for (int t = 0; t < 8; ++t) {
        float wv[8];
        unpack8(cur[t], wv);
        a[t] = fmaf(wv[0], x0.x, a[t]); a[t] = fmaf(wv[1], x0.y, a[t]); a[t] = fmaf(wv[2], x0.z, a[t]); a[t] = fmaf(wv[3], x0.w, a[t]);
        a[t] = fmaf(wv[4], x1.x, a[t]); a[t] = fmaf(wv[5], x1.y, a[t]); a[t] = fmaf(wv[6], x1.z, a[t]); a[t] = fmaf(wv[7], x1.w, a[t]);
      }
      // not ahead of the products as in se_hidden_kernel: no register is left for it, and hardly a gate this small has 512 channels
      if (i8 + 64 < (p.C >> 3)) rows(o0, i8 + 64, cur);
    }
    float mine = 0.f;
#pragma unroll
    for (int t = 0; t < 8; ++t) {
      const float sum = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(lane_sum(a[t])), 63));
      mine = lane == t ? sum : mine;
    }
    if (lane < 8 && o0 + lane < p.Q) h_s[o0 + lane] = fmaxf(mine + bias, 0.f);
  }
  __syncthreads();
  for (int c = tid >> 2; c < p.C; c += SE_ONE_NT / 4) {
    if (c != tid >> 2) gate_weights(c);
    float a = 0.f;
#pragma unroll
    for (int j = 0; j < SE_ONE_Q / 32; ++j) {
      const int i8 = j * 4 + quarter;
      if (i8 < q8n) {
        float wv[8];
        unpack8(wq[j], wv);
        const float4 x0 = *(const float4*)(h_s + i8 * 8), x1 = *(const float4*)(h_s + i8 * 8 + 4);
        a = fmaf(wv[0], x0.x, a); a = fmaf(wv[1], x0.y, a); a = fmaf(wv[2], x0.z, a); a = fmaf(wv[3], x0.w, a);
        a = fmaf(wv[4], x1.x, a); a = fmaf(wv[5], x1.y, a); a = fmaf(wv[6], x1.z, a); a = fmaf(wv[7], x1.w, a);
      }
    }
    a += __shfl_xor(a, 1, 64);
    a += __shfl_xor(a, 2, 64);
    if (quarter == 0) p.gate[(long)n * p.pool_segs * p.C + c] = fminf(fmaxf(a + b2 + 3.f, 0.f), 6.f) * (1.f / 6.f);
  }
}

hipError_t launch_se(const SeGroupArgs& a, hipStream_t s) {
  for (int i = 0; i < a.n; ++i) {
    const SeProblem& p = a.p[i];
    if (p.C % 8 || p.Q % 8 || p.Q > SE_MAX_Q || p.w1_stride % 8 || p.w2_stride % 8 || p.pool_segs < 1 || p.C * 4 > 64 * 1024)
      return hipErrorInvalidValue;
  }
  enum { ONE, TWO, SCALED };                 // gate in one launch; in two; in two with the scaling pass
  auto way = [](const SeProblem& p) { return !p.gate ? SCALED : (p.Q <= SE_ONE_Q && p.Q * p.C <= SE_ONE_MACS ? ONE : TWO); };
  // the problems that `take` accepts, `tiles` blocks each
  SeGroupArgs b;
  int blocks = 0, c_max = 0;
  auto gather = [&](auto take, auto tiles) {
    b.n = 0; blocks = 0; c_max = 0;
    for (int i = 0; i < a.n; ++i) {
      if (!take(way(a.p[i]))) continue;
      SeProblem& p = b.p[b.n++];
      p = a.p[i];
      p.tiles = tiles(p);
      p.tile_start = blocks;
      blocks += p.tiles;
      if (p.C > c_max) c_max = p.C;
    }
    return b.n > 0;
  };
  if (gather([](int w) { return w == ONE; }, [](const SeProblem& p) { return p.N; })) {
    if (b.n == 1) hipLaunchKernelGGL(se_one_kernel<Lone<SeProblem>>, dim3(blocks), dim3(SE_ONE_NT), c_max * 4, s, Lone<SeProblem>{{b.p[0]}});
    else hipLaunchKernelGGL(se_one_kernel<SeGroupArgs>, dim3(blocks), dim3(SE_ONE_NT), c_max * 4, s, b);
    const hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
  }
  if (gather([](int w) { return w != ONE; }, [](const SeProblem& p) { return p.N * ((p.Q + 31) / 32); })) {
    if (b.n == 1) hipLaunchKernelGGL(se_hidden_kernel<Lone<SeProblem>>, dim3(blocks), dim3(256), c_max * 4, s, Lone<SeProblem>{{b.p[0]}});
    else hipLaunchKernelGGL(se_hidden_kernel<SeGroupArgs>, dim3(blocks), dim3(256), c_max * 4, s, b);
    const hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
  }
  if (gather([](int w) { return w == TWO; }, [](const SeProblem& p) { return p.N * ((p.C + 63) / 64); })) {
    if (b.n == 1) hipLaunchKernelGGL((se_gate_kernel<false, Lone<SeProblem>>), dim3(blocks), dim3(256), 0, s, Lone<SeProblem>{{b.p[0]}});
    else hipLaunchKernelGGL((se_gate_kernel<false, SeGroupArgs>), dim3(blocks), dim3(256), 0, s, b);
    const hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
  }
  if (gather([](int w) { return w == SCALED; }, [](const SeProblem& p) { return p.N * ((p.C + 63) / 64) * ((p.HW + SE_PIX - 1) / SE_PIX); })) {
    hipLaunchKernelGGL((se_gate_kernel<true, SeGroupArgs>), dim3(blocks), dim3(256), 0, s, b);
    const hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
  }
  return hipSuccess;
}

}  // namespace sna
