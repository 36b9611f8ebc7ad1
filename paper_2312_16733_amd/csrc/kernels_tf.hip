// Transformer pieces that are not plain linear layers: softmax attention over the leading heads
// of a layer (head_dim 64, up to 128 tokens per request) on bf16 MFMA, and LayerNorm.
#include "common.h"

namespace sna {

typedef __attribute__((ext_vector_type(8))) __bf16 bf16x8;
typedef __attribute__((ext_vector_type(16))) float f32x16;
typedef __attribute__((ext_vector_type(4))) unsigned int u32x4;

constexpr int AT_S = 128;          // max tokens per request
constexpr int AT_D = 64;           // head dim
constexpr int AT_LD = AT_S + 8;    // LDS row stride (bf16) for V^T and P

// One block = one (request, head); wave w owns queries [32w, 32w + 32).
//   scores = Q K^T / 8 (fp32) -> softmax over keys (fp32) -> P rounded to bf16 -> ctx = P V -> bf16.
// The scores are computed transposed (K as the row operand, Q as the column operand), so that a lane
// of the accumulator holds one query (column lane % 32) and 16 of the 32 keys of each key block:
// the softmax reduction over keys runs inside a lane plus one exchange with lane ^ 32, and the
// probabilities are already laid out as the column operand of the second product (column = query, 8
// values per K slice) without a trip through LDS.  The slice's 8 values are keys
// {base + 4 hi + 0..3, base + 8 + 4 hi + 0..3} (hi = lane / 32) instead of 8 consecutive keys; a
// sum over keys may take them in any order as long as the V operand uses the same one, and V^T in
// LDS gives each lane its two runs of 4 keys as two 8-byte reads.
// Q and K fragments come straight from global memory (a lane's 8 consecutive head-dim values are
// contiguous); V is transposed through LDS.
__device__ __forceinline__ void attention_block(const AttnProblem p, int local) {
  __shared__ __attribute__((aligned(16))) bf16_t Vt[AT_D * AT_LD];
  const int h = local % p.heads, b = local / p.heads;
  const int S = p.S, ld = p.ld;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const bf16_t* Q = (const bf16_t*)p.q + (long)b * S * ld + h * AT_D;
  const bf16_t* Kp = (const bf16_t*)p.k + (long)b * S * ld + h * AT_D;
  const bf16_t* V = (const bf16_t*)p.v + (long)b * S * ld + h * AT_D;

  // Bound by latency: a load round trip, two short chains of MFMAs and the softmax between them (36 to 384 blocks), so
  // all of a thread's loads go out together, from rows clamped to the last one: a guarded load would be waited for
  // before the next guard.  128 tokens x 3 requests x 12 heads: 9.6 -> 7.1 us a launch, 32 requests 13.4 -> 11.9, with
  // the dword V^T writes and 8-byte output stores below.  Scores of keys >= S are masked below and query rows >= S are not stored, so only V needs zeros.
  const int r32 = lane & 31, hi = lane >> 5;
  const int qrow = wave * 32 + r32;
  const int qld = qrow < S ? qrow : S - 1;
  uint4 qv[4], kv[4][4], vv[2][2];
#pragma unroll
  for (int ks = 0; ks < 4; ++ks) qv[ks] = *(const uint4*)(Q + (long)qld * ld + ks * 16 + hi * 8);
#pragma unroll
  for (int j = 0; j < 4; ++j) {
    const int key = j * 32 + r32 < S ? j * 32 + r32 : S - 1;
#pragma unroll
    for (int ks = 0; ks < 4; ++ks) kv[j][ks] = *(const uint4*)(Kp + (long)key * ld + ks * 16 + hi * 8);
  }
  // V: a lane takes two neighbouring keys of a head-dim octet, so that it writes V^T as whole dwords and a wave's 64
  // lanes write 64 consecutive ones
#pragma unroll
  for (int it = 0; it < 2; ++it)
#pragma unroll
    for (int e = 0; e < 2; ++e) {
      const int key = 2 * lane + e < S ? 2 * lane + e : S - 1;
      vv[it][e] = *(const uint4*)(V + (long)key * ld + (wave + 4 * it) * 8);
    }
  __builtin_amdgcn_sched_barrier(0);     // keep the loads ahead of everything that waits for one of them

  // sc[j][v]: query qrow, key 32 j + 8 (v / 4) + 4 hi + v % 4
  f32x16 sc[4];
#pragma unroll
  for (int j = 0; j < 4; ++j) {
#pragma unroll
    for (int v = 0; v < 16; ++v) sc[j][v] = 0.f;
#pragma unroll
    for (int ks = 0; ks < 4; ++ks)
      sc[j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, kv[j][ks]),
                                                      __builtin_bit_cast(bf16x8, qv[ks]), sc[j], 0, 0, 0);
  }
  // V^T into LDS: Vt[d][key], zero for keys >= S
#pragma unroll
  for (int it = 0; it < 2; ++it) {
    const unsigned lo_ok = 2 * lane < S ? 0xffffffffu : 0u, hi_ok = 2 * lane + 1 < S ? 0xffffffffu : 0u;
    const unsigned a[4] = {vv[it][0].x & lo_ok, vv[it][0].y & lo_ok, vv[it][0].z & lo_ok, vv[it][0].w & lo_ok};
    const unsigned c[4] = {vv[it][1].x & hi_ok, vv[it][1].y & hi_ok, vv[it][1].z & hi_ok, vv[it][1].w & hi_ok};
    bf16_t* col = Vt + (wave + 4 * it) * 8 * AT_LD + 2 * lane;
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      *(unsigned*)(col + (2 * e) * AT_LD) = (a[e] & 0xffffu) | (c[e] << 16);
      *(unsigned*)(col + (2 * e + 1) * AT_LD) = (a[e] >> 16) | (c[e] & 0xffff0000u);
    }
  }
  // softmax over the keys of this lane's query, in base 2: exp(x / 8 - max) = exp2((x - max') * log2(e) / 8)
  const float kScale = 0.125f * 1.44269504088896340736f;
  float m = -3.0e38f;
#pragma unroll
  for (int j = 0; j < 4; ++j)
#pragma unroll
    for (int v = 0; v < 16; ++v) {
      const int key = 32 * j + 8 * (v >> 2) + 4 * hi + (v & 3);
      sc[j][v] = key < S ? sc[j][v] * kScale : -3.0e38f;
      m = fmaxf(m, sc[j][v]);
    }
  m = fmaxf(m, __shfl_xor(m, 32, 64));
  float sum = 0.f;
#pragma unroll
  for (int j = 0; j < 4; ++j)
#pragma unroll
    for (int v = 0; v < 16; ++v) {
      const int key = 32 * j + 8 * (v >> 2) + 4 * hi + (v & 3);
      sc[j][v] = key < S ? __builtin_amdgcn_exp2f(sc[j][v] - m) : 0.f;
      sum += sc[j][v];
    }
  sum += __shfl_xor(sum, 32, 64);
  const float inv = 1.f / sum;
  __syncthreads();                     // V^T complete (all waves)
  f32x16 oc[2];
#pragma unroll
  for (int jd = 0; jd < 2; ++jd)
#pragma unroll
    for (int v = 0; v < 16; ++v) oc[jd][v] = 0.f;
#pragma unroll
  for (int j = 0; j < 4; ++j)
#pragma unroll
    for (int ap = 0; ap < 2; ++ap) {
      // probabilities rounded to bf16: elements 8 ap .. 8 ap + 7 of the key block
      u32x4 pw;
      pw.x = pack_bf16x2(sc[j][8 * ap + 0] * inv, sc[j][8 * ap + 1] * inv);
      pw.y = pack_bf16x2(sc[j][8 * ap + 2] * inv, sc[j][8 * ap + 3] * inv);
      pw.z = pack_bf16x2(sc[j][8 * ap + 4] * inv, sc[j][8 * ap + 5] * inv);
      pw.w = pack_bf16x2(sc[j][8 * ap + 6] * inv, sc[j][8 * ap + 7] * inv);
      const int key0 = 32 * j + 16 * ap + 4 * hi;
#pragma unroll
      for (int jd = 0; jd < 2; ++jd) {
        const bf16_t* vrow = Vt + (jd * 32 + r32) * AT_LD + key0;
        const uint2 v0 = *(const uint2*)vrow, v1 = *(const uint2*)(vrow + 8);
        const u32x4 vw = {v0.x, v0.y, v1.x, v1.y};
        oc[jd] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, vw), __builtin_bit_cast(bf16x8, pw), oc[jd], 0, 0, 0);
      }
    }
  // the second product is transposed as well: oc[jd][v] is query qrow, head dim 32 jd + 8 (v / 4) + 4 hi + v % 4, so a
  // lane stores four neighbouring values at a time
  if (qrow < S) {
    bf16_t* O = (bf16_t*)p.o + (long)b * S * ld + h * AT_D + (long)qrow * ld + 4 * hi;
#pragma unroll
    for (int jd = 0; jd < 2; ++jd)
#pragma unroll
      for (int v4 = 0; v4 < 4; ++v4)
        *(uint2*)(O + jd * 32 + 8 * v4) = make_uint2(pack_bf16x2(oc[jd][4 * v4], oc[jd][4 * v4 + 1]),
                                                     pack_bf16x2(oc[jd][4 * v4 + 2], oc[jd][4 * v4 + 3]));
  }
}

__global__ __launch_bounds__(256) void attention_kernel(const AttnGroupArgs args) {
  const int g = find_problem(args, blockIdx.x);
  attention_block(args.p[g], blockIdx.x - args.p[g].tile_start);
}
// One problem: its descriptor comes in scalar arguments, which the dispatch puts into registers
__global__ __launch_bounds__(256) void attention_lone_kernel(const void* q, const void* k, const void* v, void* o, int S, int heads, int ld) {
  attention_block(AttnProblem{q, k, v, o, 0, S, heads, ld, 0, 0}, blockIdx.x);
}

hipError_t launch_attention(const AttnGroupArgs& a, hipStream_t s) {
  if (a.n == 0) return hipSuccess;
  AttnGroupArgs b = a;
  int start = 0;
  for (int i = 0; i < b.n; ++i) {
    if (b.p[i].S > AT_S || b.p[i].S < 1 || b.p[i].ld % 8) return hipErrorInvalidValue;
    b.p[i].tile_start = start;
    b.p[i].tiles = b.p[i].B * b.p[i].heads;
    start += b.p[i].tiles;
  }
  const AttnProblem& p = b.p[0];
  if (b.n == 1) hipLaunchKernelGGL(attention_lone_kernel, dim3(start), dim3(256), 0, s, p.q, p.k, p.v, p.o, p.S, p.heads, p.ld);
  else hipLaunchKernelGGL(attention_kernel, dim3(start), dim3(256), 0, s, b);
  return hipGetLastError();
}

// ---------------------------------------------------------------------------------------------
// LayerNorm over the last dimension, one wave per row; the row stays in registers between the
// mean, variance and normalise passes.  cols is a multiple of 8 and at most 2048.
// ---------------------------------------------------------------------------------------------
constexpr int LN_MAX_OCT = 4;      // octets per lane -> cols <= 2048

__device__ __forceinline__ void layernorm_block(const LnProblem p, int local) {
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const long row = (long)local * 4 + wave;
  if (row >= p.rows) return;
  const int octs = p.cols >> 3;
  const bf16_t* x = (const bf16_t*)p.x + row * p.cols;
  // The row, gamma and beta are requested together: the per-column vectors then arrive under the two reductions instead of
  // a round trip after them (rows of 768, both sides traced in turn on one card: 384 rows 4.15 -> 4.03 us a launch, 4096
  // rows 5.83 -> 5.41).  An octet past the row reads the last one and is left out of the sums and the store.
  uint4 u[LN_MAX_OCT];
  float v[LN_MAX_OCT][8], ga[LN_MAX_OCT][8], be[LN_MAX_OCT][8];
#pragma unroll
  for (int i = 0; i < LN_MAX_OCT; ++i)
    if (64 * i < octs) {                                   // uniform
      const int o = lane + 64 * i < octs ? lane + 64 * i : octs - 1;
      u[i] = *(const uint4*)(x + o * 8);
    }
#pragma unroll
  for (int i = 0; i < LN_MAX_OCT; ++i)
    if (64 * i < octs) {
      const int o = lane + 64 * i < octs ? lane + 64 * i : octs - 1;
#pragma unroll
      for (int e = 0; e < 8; ++e) { ga[i][e] = p.gamma[o * 8 + e]; be[i][e] = p.beta[o * 8 + e]; }
    }
  float sum = 0.f;
#pragma unroll
  for (int i = 0; i < LN_MAX_OCT; ++i) {
    if (lane + 64 * i < octs) {
      const unsigned w[4] = {u[i].x, u[i].y, u[i].z, u[i].w};
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        v[i][2 * e] = __uint_as_float(w[e] << 16);
        v[i][2 * e + 1] = __uint_as_float(w[e] & 0xffff0000u);
      }
#pragma unroll
      for (int e = 0; e < 8; ++e) sum += v[i][e];
    }
  }
#pragma unroll
  for (int off = 32; off >= 1; off >>= 1) sum += __shfl_xor(sum, off, 64);
  const float mean = sum / (float)p.cols;
  float sq = 0.f;
#pragma unroll
  for (int i = 0; i < LN_MAX_OCT; ++i)
    if (lane + 64 * i < octs) {
#pragma unroll
      for (int e = 0; e < 8; ++e) { const float d = v[i][e] - mean; sq = fmaf(d, d, sq); }
    }
#pragma unroll
  for (int off = 32; off >= 1; off >>= 1) sq += __shfl_xor(sq, off, 64);
  const float rstd = 1.f / sqrtf(sq / (float)p.cols + 1e-5f);
  bf16_t* y = (bf16_t*)p.y + row * p.cols;
#pragma unroll
  for (int i = 0; i < LN_MAX_OCT; ++i) {
    const int o = lane + 64 * i;
    if (o < octs) {
      float r[8];
#pragma unroll
      for (int e = 0; e < 8; ++e) r[e] = fmaf((v[i][e] - mean) * rstd, ga[i][e], be[i][e]);
      uint4 out;
      out.x = pack_bf16x2(r[0], r[1]);
      out.y = pack_bf16x2(r[2], r[3]);
      out.z = pack_bf16x2(r[4], r[5]);
      out.w = pack_bf16x2(r[6], r[7]);
      *(uint4*)(y + o * 8) = out;
    }
  }
}

__global__ __launch_bounds__(256) void layernorm_kernel(const LnGroupArgs args) {
  const int g = find_problem(args, blockIdx.x);
  layernorm_block(args.p[g], blockIdx.x - args.p[g].tile_start);
}
__global__ __launch_bounds__(256) void layernorm_lone_kernel(const void* x, const float* gamma, const float* beta, void* y, int rows, int cols) {
  layernorm_block(LnProblem{x, gamma, beta, y, rows, cols, 0, 0}, blockIdx.x);
}

hipError_t launch_layernorm(const LnGroupArgs& a, hipStream_t s) {
  if (a.n == 0) return hipSuccess;
  LnGroupArgs b = a;
  int start = 0;
  for (int i = 0; i < b.n; ++i) {
    if (b.p[i].cols % 8 || b.p[i].cols > 8 * 64 * LN_MAX_OCT) return hipErrorInvalidValue;
    b.p[i].tile_start = start;
    b.p[i].tiles = (b.p[i].rows + 3) / 4;
    start += b.p[i].tiles;
  }
  const LnProblem& p = b.p[0];
  if (b.n == 1) hipLaunchKernelGGL(layernorm_lone_kernel, dim3(start), dim3(256), 0, s, p.x, p.gamma, p.beta, p.y, p.rows, p.cols);
  else hipLaunchKernelGGL(layernorm_kernel, dim3(start), dim3(256), 0, s, b);
  return hipGetLastError();
}

}  // namespace sna
