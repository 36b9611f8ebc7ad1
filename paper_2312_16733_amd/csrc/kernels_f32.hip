// WeightSlice convolution / linear of the fp32 family on the fp32 matrix instruction (gfx950).
//
//   Y[m, k] = sum_{r,s,c} X[n, p*st + r - pad, q*st + s - pad, c] * W[k, r, s, c]
//
// These layers are short (at 4 images of 32 x 32: 4096 output pixels of 16 channels down to 64 of 128) and what bounds them is the
// serial chain of one output's reduction: with one thread per pixel and 16 channels a layer of 1152 terms took 150 us
// on 8 CUs.  Here an output tile is 16 pixels x 16 channels of v_mfma_f32_16x16x4_f32 (fp32 products and sums), and a
// long reduction is spread over the 8 waves of a block, which add their sums through LDS: the chain becomes 1/8 as long
// and there are 32 .. 256 tiles where there were 4 .. 16 blocks.  Operands go from global memory (the whole net stays in L2)
// straight to registers: a lane loads 4 consecutive reduction elements of its pixel and of its channel with one
// 16-byte bounds-checked load each, which four MFMAs take element by element; the loads of five steps are requested
// together, ahead of the MFMAs that use the five before.
//
// Measured on the largest tiny subnet (thread per pixel -> here, event-bracketed): 4 images, 64 x 128 x 1152 (pixels x
// channels x reduction) 153 -> 10.1 us, 256 x 64 x 576 96 -> 8.2, 1024 x 32 x 288 63 -> 8.1, the whole forward
// 514 -> 51 us, where an empty launch takes 6; 64 images, 1024 x 128 x 1152 166 -> 12.6, 16384 x 32 x 288 62 -> 14.3
// (with one block a CU instead of two, 13.8 and 17.0).
//
// The reduction order depends on the layer's reduction length alone (wave w sums its run of steps in order, the waves'
// sums are added in wave order), so a request's result does not depend on what it is batched with.
#include "common.h"

namespace sna {

typedef __attribute__((ext_vector_type(4))) float f32x4;
typedef __attribute__((ext_vector_type(4))) unsigned int u32x4_t;

constexpr int F32_WAVES = 8;          // waves per block
constexpr int F32_TILE = 16;
constexpr int F32_STEP = 16;          // reduction elements per step: 4 lanes groups x 4 elements
// Steps whose loads are requested together, twice that many in flight: a wave's share of 18, 36 and 72 steps is 5, 5 and 9.
// Without fours of channels a step is eight loads with an address each, and the layers are images' first ones, of two steps.
constexpr int f32_ahead(bool vec) { return vec ? 5 : 2; }

// Waves that share one output tile: with fewer than 4 steps each, adding up through LDS costs more than it saves.
__host__ __device__ __forceinline__ int f32_k_waves(int steps) {
  return steps >= 32 ? 8 : (steps >= 16 ? 4 : (steps >= 8 ? 2 : 1));
}

// What the kernel takes of a descriptor
struct F32Problem {
  const void* x; const void* w; const float* scale; const float* shift; const void* res; void* y;
  int H, W, C, Ho, Wo, K, R, S, stride, pad, wk, wr, ws, M;
  unsigned magic_wo, magic_ho;
  int inv_s, tiles_n, tile_start, act, y_stride, res_stride;
  unsigned x_bytes, w_bytes;
  int res_after_act, unused;
};
__device__ __forceinline__ F32Problem f32_problem(const ConvProblem& q) {
  return {q.x, q.w, q.scale, q.shift, q.res, q.y, q.H, q.W, q.C, q.Ho, q.Wo, q.K, q.R, q.S, q.stride, q.pad, q.wk, q.wr, q.ws, q.M,
          q.magic_wo, q.magic_ho, q.inv_s, q.tiles_n, q.tile_start, q.act, q.y_stride, q.res_stride, q.x_bytes, q.w_bytes, q.res_after_act, 0};
}

// VEC: the input channels come in fours, so that a lane's 4 elements lie inside one tap
// Four waves a SIMD, which is two blocks a CU; at 130 registers it was one.
template <bool VEC, class Args>
__global__ __launch_bounds__(64 * F32_WAVES, 4) void conv_f32_kernel(const Args args) {
#if defined(__HIP_DEVICE_COMPILE__)
  constexpr int F32_AHEAD = f32_ahead(VEC);
  __shared__ float red[F32_WAVES][F32_TILE * F32_TILE];
  const int g = find_problem(args, blockIdx.x);
  F32Problem p = pinned(f32_problem(args.p[g]));
  p.scale = in_global(p.scale); p.shift = in_global(p.shift); p.res = in_global(p.res); p.y = in_global(p.y);
  const int local = blockIdx.x - p.tile_start;
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int RSC = p.R * p.S * p.C;
  const int steps = (RSC + F32_STEP - 1) / F32_STEP;
  const int kw = f32_k_waves(steps);                       // waves per tile
  const int tiles_b = F32_WAVES / kw;                      // pixel tiles per block
  const int tn = local % p.tiles_n, tmb = local / p.tiles_n;
  const int tile = tmb * tiles_b + wave / kw, part = wave % kw;
  const int l16 = lane & 15, grp = lane >> 4;
  const int m = tile * F32_TILE + l16, k = tn * F32_TILE + l16;

  constexpr unsigned OOB = 0x80000000u;
  const __amdgpu_buffer_rsrc_t rsrc_x = __builtin_amdgcn_make_buffer_rsrc((void*)p.x, 0, (int)p.x_bytes, 0x00020000);
  const __amdgpu_buffer_rsrc_t rsrc_w = __builtin_amdgcn_make_buffer_rsrc((void*)p.w, 0, (int)p.w_bytes, 0x00020000);
  const bool m_ok = m < p.M, k_ok = k < p.K;
  const int t = p.Wo == 1 ? m : (int)__umulhi((unsigned)m, p.magic_wo);
  const int q = m - t * p.Wo;
  const int n = p.Ho == 1 ? t : (int)__umulhi((unsigned)t, p.magic_ho);
  const int pp = t - n * p.Ho;
  const int ih0 = pp * p.stride - p.pad, iw0 = q * p.stride - p.pad;
  const int xbase = ((n * p.H + ih0) * p.W + iw0) * p.C, wbase = k * p.wk;
  // x / C = mulhi(x, magic) for x < 2^32 / C; a reduction is far shorter
  const unsigned magic_c = p.C > 1 ? 0xFFFFFFFFu / (unsigned)p.C + 1u : 0u;

  // byte offsets of reduction element e (of its run of 4, if VEC) in this lane's pixel window and weight row
  auto locate = [&](int e, int e_end, unsigned& ox, unsigned& ow) {
    const int rs = p.C > 1 ? (int)__umulhi((unsigned)e, magic_c) : e;
    const int c = e - rs * p.C;
    const int r = (rs * p.inv_s) >> 16, s = rs - r * p.S;
    const int ih = ih0 + r, iw = iw0 + s;
    const bool in = e < e_end;
    ox = in && m_ok && (unsigned)ih < (unsigned)p.H && (unsigned)iw < (unsigned)p.W
             ? (unsigned)(xbase + (r * p.W + s) * p.C + c) * 4u : OOB;
    ow = in && k_ok ? (unsigned)(wbase + r * p.wr + s * p.ws + c) * 4u : OOB;
  };
  struct Operands { f32x4 a, b; };
  auto load = [&](int step, int e_end) {
    Operands o;
    if constexpr (VEC) {
      unsigned ox, ow;
      locate(step * F32_STEP + grp * 4, e_end, ox, ow);
      o.a = __builtin_bit_cast(f32x4, __builtin_amdgcn_raw_buffer_load_b128(rsrc_x, ox, 0, 0));
      o.b = __builtin_bit_cast(f32x4, __builtin_amdgcn_raw_buffer_load_b128(rsrc_w, ow, 0, 0));
    } else {
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        unsigned ox, ow;
        locate(step * F32_STEP + grp * 4 + j, e_end, ox, ow);
        o.a[j] = __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(rsrc_x, ox, 0, 0));
        o.b[j] = __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(rsrc_w, ow, 0, 0));
      }
    }
    return o;
  };

  const int s0 = part * steps / kw, s1 = (part + 1) * steps / kw;
  const int e_end = s1 * F32_STEP < RSC ? s1 * F32_STEP : RSC;
  f32x4 acc = {0.f, 0.f, 0.f, 0.f};
  Operands cur[F32_AHEAD];
#pragma unroll
  for (int i = 0; i < F32_AHEAD; ++i) cur[i] = load(s0 + i, e_end);
  // What the outputs of this thread need at the end, requested here so that no second round trip follows the sums
  constexpr int EPI = F32_TILE * F32_TILE / 64;            // outputs per thread, at most: one tile per wave
  float e_sc[EPI], e_sh[EPI], e_rv[EPI];
#pragma unroll
  for (int it = 0; it < EPI; ++it) {
    const int i = threadIdx.x + it * 64 * F32_WAVES, e = i & 255;
    const int mo = (tmb * tiles_b + (i >> 8)) * F32_TILE + (e >> 4), ko = tn * F32_TILE + (e & 15);
    const bool ok = i < tiles_b * F32_TILE * F32_TILE && mo < p.M && ko < p.K;
    e_sc[it] = ok && p.scale ? p.scale[ko] : 1.f;
    e_sh[it] = ok && p.shift ? p.shift[ko] : 0.f;
    e_rv[it] = ok && p.res ? ((const float*)p.res)[(long)mo * p.res_stride + ko] : 0.f;
  }
  for (int s = s0; s < s1; s += F32_AHEAD) {
    Operands nxt[F32_AHEAD];
    if (s + F32_AHEAD < s1) {
#pragma unroll
      for (int i = 0; i < F32_AHEAD; ++i) nxt[i] = load(s + F32_AHEAD + i, e_end);
    }
#pragma unroll
    for (int i = 0; i < F32_AHEAD; ++i)                    // a step past the end multiplies zeros
#pragma unroll
      for (int j = 0; j < 4; ++j) acc = __builtin_amdgcn_mfma_f32_16x16x4f32(cur[i].a[j], cur[i].b[j], acc, 0, 0, 0);
#pragma unroll
    for (int i = 0; i < F32_AHEAD; ++i) cur[i] = nxt[i];
  }

  // A sum that is not finite, taken again over the output's in-image taps in order: at the border the MFMAs multiplied
  // padding zeros by weights, and an infinite or NaN weight makes NaN of that (which ReLU then makes 0).  The layer is
  // looked up by an index that the compiler cannot see through, so that nothing of this is computed ahead (the check
  // costs 1 % of a nine-launch forward, 51.3 -> 51.9 us; with the set-up hoisted it was 2.4 %).
  auto own_taps = [&](int mo, int ko) {
    int go = g;
    asm volatile("" : "+s"(go));
    const ConvProblem& o = args.p[go];
    const int to = mo / o.Wo, no = to / o.Ho;
    const int ih = (to - no * o.Ho) * o.stride - o.pad, iw = (mo - to * o.Wo) * o.stride - o.pad;
    float sum = 0.f;
#pragma unroll 1
    for (int r = 0; r < o.R; ++r)
#pragma unroll 1
      for (int s = 0; s < o.S; ++s) {
        if ((unsigned)(ih + r) >= (unsigned)o.H || (unsigned)(iw + s) >= (unsigned)o.W) continue;
        const float* x = (const float*)o.x + ((long)(no * o.H + ih + r) * o.W + iw + s) * o.C;
        const float* w = (const float*)o.w + (long)ko * o.wk + r * o.wr + s * o.ws;
#pragma unroll 1
        for (int c = 0; c < o.C; ++c) sum = fmaf(x[c], w[c], sum);
      }
    return sum;
  };
  // accumulator element v of lane l: pixel 4 (l / 16) + v, channel l % 16 of the tile
#pragma unroll
  for (int v = 0; v < 4; ++v) red[wave][(4 * grp + v) * F32_TILE + l16] = acc[v];
  __syncthreads();
#pragma unroll
  for (int it = 0; it < EPI; ++it) {
    const int i = threadIdx.x + it * 64 * F32_WAVES, tl = i >> 8, e = i & 255;
    const int mo = (tmb * tiles_b + tl) * F32_TILE + (e >> 4), ko = tn * F32_TILE + (e & 15);
    if (i >= tiles_b * F32_TILE * F32_TILE || mo >= p.M || ko >= p.K) continue;
    float v = red[tl * kw][e];
    for (int w = 1; w < kw; ++w) v += red[tl * kw + w][e];
    if (__builtin_expect(!(fabsf(v) < __builtin_inff()), 0)) v = own_taps(mo, ko);
    v = fmaf(v, e_sc[it], e_sh[it]);
    if (p.res && !p.res_after_act) v += e_rv[it];
    v = apply_act(v, p.act);
    if (p.res && p.res_after_act) v += e_rv[it];
    ((float*)p.y)[(long)mo * p.y_stride + ko] = v;
  }
#endif
}

void conv_f32_tiles(ConvProblem& p) {
  const int steps = (p.R * p.S * p.C + F32_STEP - 1) / F32_STEP;
  const int rows_b = F32_TILE * F32_WAVES / f32_k_waves(steps);
  p.tiles_n = (p.K + F32_TILE - 1) / F32_TILE;
  p.tiles = (p.M + rows_b - 1) / rows_b * p.tiles_n;
}

hipError_t launch_conv_f32(const ConvGroupArgs& a, hipStream_t s) {
  if (a.n == 0) return hipSuccess;
  bool vec = true;
  for (int i = 0; i < a.n; ++i) vec = vec && a.p[i].C % 4 == 0;
  const dim3 grid(a.total_tiles), block(64 * F32_WAVES);
  typedef Lone<ConvProblem> One;
  if (a.n == 1) {
    if (vec) hipLaunchKernelGGL((conv_f32_kernel<true, One>), grid, block, 0, s, One{{a.p[0]}});
    else hipLaunchKernelGGL((conv_f32_kernel<false, One>), grid, block, 0, s, One{{a.p[0]}});
  } else {
    if (vec) hipLaunchKernelGGL((conv_f32_kernel<true, ConvGroupArgs>), grid, block, 0, s, a);
    else hipLaunchKernelGGL((conv_f32_kernel<false, ConvGroupArgs>), grid, block, 0, s, a);
  }
  return hipGetLastError();
}

}  // namespace sna
