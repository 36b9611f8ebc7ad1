// Transformer pieces that are not plain linear layers: softmax attention over the leading heads
// of a layer (head_dim 64, up to 128 tokens per request) on bf16 MFMA, and LayerNorm.
#include "common.h"

namespace sna {

typedef __attribute__((ext_vector_type(8))) __bf16 bf16x8;
typedef __attribute__((ext_vector_type(4))) float f32x4;
typedef __attribute__((ext_vector_type(4))) unsigned int u32x4;

constexpr int AT_S = 128;          // max tokens per request
constexpr int AT_D = 64;           // head dim
constexpr int AT_LD = AT_S + 8;    // LDS row stride (bf16) of V^T
constexpr int AT_KD = AT_D + 8;    // and of K

constexpr int AT_Q = 64;           // queries per block
constexpr int AT_NT = 64 * (AT_Q / 16);      // threads: a wave per 16 queries

// One block = 64 queries of one (request, head); wave w owns 16 of them, from 16w on.
//   scores = Q K^T / 8 (fp32) -> softmax over keys (fp32) -> P rounded to bf16 -> ctx = P V -> bf16.
// The scores are computed transposed (K as the row operand, Q as the column operand), so that a lane
// of the accumulator holds one query (column lane % 16) and 4 of the 16 keys of each key block:
// the softmax reduction over keys runs inside a lane plus exchanges with lanes ^ 16 and ^ 32, and the
// probabilities are already laid out as the column operand of the second product (column = query, 8
// values per slice of 32 keys) without a trip through LDS.  The slice's 8 values are keys
// {base + 4 hi + 0..3, base + 16 + 4 hi + 0..3} (hi = lane / 16) instead of 8 consecutive keys; a
// sum over keys may take them in any order as long as the V operand uses the same one, and V^T in
// LDS gives each lane its two runs of 4 keys as two 8-byte reads.
// K and V^T lie in LDS: read by each wave from global memory, K came in as many times over as there are waves, and the CU's
// fetch of it was half of the launch (3 requests of 128 tokens x 12 heads 7.1 -> 5.8 us, 32 requests 12.0 -> 9.9, with 16
// queries a wave instead of 32).  Two blocks a head rather than one of eight waves: 5.8 -> 4.9 and 9.9 -> 9.2, since two
// thirds of the CUs had one block and the others two, and a few heads occupy twice the CUs.
__device__ __forceinline__ void attention_block(const AttnProblem p, int local) {
  __shared__ __attribute__((aligned(16))) bf16_t Vt[AT_D * AT_LD];
  __shared__ __attribute__((aligned(16))) bf16_t Ks[AT_S * AT_KD];
  const int pairs = p.B * p.heads, part = local / pairs;
  local -= part * pairs;
  const int h = local % p.heads, b = local / p.heads;
  const int S = p.S, ld = p.ld;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const bf16_t* Q = (const bf16_t*)p.q + (long)b * S * ld + h * AT_D;
  const bf16_t* Kp = (const bf16_t*)p.k + (long)b * S * ld + h * AT_D;
  const bf16_t* V = (const bf16_t*)p.v + (long)b * S * ld + h * AT_D;

  // All of a thread's loads go out together, from rows clamped to the last one: a guarded load would be waited for
  // before the next guard.  Scores of keys >= S are masked below and query rows >= S are not stored, so only V needs zeros.
  const int l16 = lane & 15, hi = lane >> 4;
  const int qrow = part * AT_Q + wave * 16 + l16;
  const int qld = qrow < S ? qrow : S - 1;
  u32x4 qv[2], kv[AT_S * AT_D / 8 / AT_NT], vv[2][2];
#pragma unroll
  for (int i = 0; i < AT_S * AT_D / 8 / AT_NT; ++i) {
    const int key = i * (AT_NT / 8) + (tid >> 3);
    kv[i] = *(const u32x4*)(Kp + (long)(key < S ? key : S - 1) * ld + (tid & 7) * 8);
  }
#pragma unroll
  for (int ks = 0; ks < 2; ++ks) qv[ks] = *(const u32x4*)(Q + (long)qld * ld + ks * 32 + hi * 8);
  // V: a lane takes two neighbouring keys of a head-dim octet, so that it writes V^T as whole dwords and a wave's 64
  // lanes write 64 consecutive ones
  static_assert(AT_NT == 64 * (AT_D / 16) && AT_S == 128, "two octets a wave, two keys a lane");
#pragma unroll
  for (int it = 0; it < 2; ++it)
#pragma unroll
    for (int e = 0; e < 2; ++e) {
      const int key = 2 * lane + e < S ? 2 * lane + e : S - 1;
      vv[it][e] = *(const u32x4*)(V + (long)key * ld + (wave + 4 * it) * 8);
    }
  __builtin_amdgcn_sched_barrier(0);     // keep the loads ahead of everything that waits for one of them

#pragma unroll
  for (int i = 0; i < AT_S * AT_D / 8 / AT_NT; ++i) *(u32x4*)(Ks + (i * (AT_NT / 8) + (tid >> 3)) * AT_KD + (tid & 7) * 8) = kv[i];
  // V^T into LDS: Vt[d][key], zero for keys >= S
#pragma unroll
  for (int it = 0; it < 2; ++it) {
    const unsigned lo_ok = 2 * lane < S ? 0xffffffffu : 0u, hi_ok = 2 * lane + 1 < S ? 0xffffffffu : 0u;
    bf16_t* col = Vt + (wave + 4 * it) * 8 * AT_LD + 2 * lane;
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      const unsigned a = vv[it][0][e] & lo_ok, c = vv[it][1][e] & hi_ok;
      *(unsigned*)(col + (2 * e) * AT_LD) = (a & 0xffffu) | (c << 16);
      *(unsigned*)(col + (2 * e + 1) * AT_LD) = (a >> 16) | (c & 0xffff0000u);
    }
  }
  __syncthreads();
  // sc[j][v]: query qrow, key 16 j + 4 hi + v
  f32x4 sc[AT_S / 16];
#pragma unroll
  for (int j = 0; j < AT_S / 16; ++j) {
    sc[j] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int ks = 0; ks < 2; ++ks)
      sc[j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(*(const bf16x8*)(Ks + (16 * j + l16) * AT_KD + ks * 32 + hi * 8),
                                                      __builtin_bit_cast(bf16x8, qv[ks]), sc[j], 0, 0, 0);
  }
  // softmax over the keys of this lane's query, in base 2: exp(x / 8 - max) = exp2((x - max') * log2(e) / 8)
  const float kScale = 0.125f * 1.44269504088896340736f;
  float m = -3.0e38f;
#pragma unroll
  for (int j = 0; j < AT_S / 16; ++j)
#pragma unroll
    for (int v = 0; v < 4; ++v) {
      const int key = 16 * j + 4 * hi + v;
      sc[j][v] = key < S ? sc[j][v] * kScale : -3.0e38f;
      m = fmaxf(m, sc[j][v]);
    }
  m = fmaxf(m, __shfl_xor(m, 16, 64));
  m = fmaxf(m, __shfl_xor(m, 32, 64));
  float sum = 0.f;
#pragma unroll
  for (int j = 0; j < AT_S / 16; ++j)
#pragma unroll
    for (int v = 0; v < 4; ++v) {
      const int key = 16 * j + 4 * hi + v;
      sc[j][v] = key < S ? __builtin_amdgcn_exp2f(sc[j][v] - m) : 0.f;
      sum += sc[j][v];
    }
  sum += __shfl_xor(sum, 16, 64);
  sum += __shfl_xor(sum, 32, 64);
  const float inv = 1.f / sum;
  f32x4 oc[AT_D / 16];
#pragma unroll
  for (int jd = 0; jd < AT_D / 16; ++jd) oc[jd] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
  for (int ks = 0; ks < AT_S / 32; ++ks) {
    // probabilities rounded to bf16: key blocks 2 ks and 2 ks + 1
    u32x4 pw;
    pw.x = pack_bf16x2(sc[2 * ks][0] * inv, sc[2 * ks][1] * inv);
    pw.y = pack_bf16x2(sc[2 * ks][2] * inv, sc[2 * ks][3] * inv);
    pw.z = pack_bf16x2(sc[2 * ks + 1][0] * inv, sc[2 * ks + 1][1] * inv);
    pw.w = pack_bf16x2(sc[2 * ks + 1][2] * inv, sc[2 * ks + 1][3] * inv);
#pragma unroll
    for (int jd = 0; jd < AT_D / 16; ++jd) {
      const bf16_t* vrow = Vt + (jd * 16 + l16) * AT_LD + 32 * ks + 4 * hi;
      const uint2 v0 = *(const uint2*)vrow, v1 = *(const uint2*)(vrow + 16);
      const u32x4 vw = {v0.x, v0.y, v1.x, v1.y};
      oc[jd] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, vw), __builtin_bit_cast(bf16x8, pw), oc[jd], 0, 0, 0);
    }
  }
  // the second product is transposed as well: oc[jd][v] is query qrow, head dim 16 jd + 4 hi + v, so a
  // lane stores four neighbouring values at a time
  if (qrow < S) {
    bf16_t* O = (bf16_t*)p.o + (long)b * S * ld + h * AT_D + (long)qrow * ld + 4 * hi;
#pragma unroll
    for (int jd = 0; jd < AT_D / 16; ++jd)
      *(uint2*)(O + jd * 16) = make_uint2(pack_bf16x2(oc[jd][0], oc[jd][1]), pack_bf16x2(oc[jd][2], oc[jd][3]));
  }
}

__global__ __launch_bounds__(AT_NT, 4) void attention_kernel(const AttnGroupArgs args) {
  const int g = find_problem(args, blockIdx.x);
  attention_block(args.p[g], blockIdx.x - args.p[g].tile_start);
}
// One problem: its descriptor comes in scalar arguments, which the dispatch puts into registers
__global__ __launch_bounds__(AT_NT, 4) void attention_lone_kernel(const void* q, const void* k, const void* v, void* o, int B, int S, int heads, int ld) {
  attention_block(AttnProblem{q, k, v, o, B, S, heads, ld, 0, 0}, blockIdx.x);
}

hipError_t launch_attention(const AttnGroupArgs& a, hipStream_t s) {
  if (a.n == 0) return hipSuccess;
  AttnGroupArgs b = a;
  int start = 0;
  for (int i = 0; i < b.n; ++i) {
    if (b.p[i].S > AT_S || b.p[i].S < 1 || b.p[i].ld % 8) return hipErrorInvalidValue;
    b.p[i].tile_start = start;
    b.p[i].tiles = b.p[i].B * b.p[i].heads * ((b.p[i].S + AT_Q - 1) / AT_Q);
    start += b.p[i].tiles;
  }
  const AttnProblem& p = b.p[0];
  if (b.n == 1) hipLaunchKernelGGL(attention_lone_kernel, dim3(start), dim3(AT_NT), 0, s, p.q, p.k, p.v, p.o, p.B, p.S, p.heads, p.ld);
  else hipLaunchKernelGGL(attention_kernel, dim3(start), dim3(AT_NT), 0, s, b);
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
