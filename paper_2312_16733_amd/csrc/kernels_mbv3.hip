// Head of the MBV3-shaped SuperNet as one kernel: 3x3 stride-2 stem conv + SubnetNorm + hardswish, then the
// fixed first block (depthwise 3x3 + SubnetNorm + ReLU, pointwise 1x1 + SubnetNorm, residual), 3 -> 16 -> 16
// channels.  As separate launches this is four kernels (channel-padding copy, stem, depthwise, pointwise)
// that move the full-resolution 16-channel tensor through memory three times and each pay a launch's fixed
// cost.  Here a block owns a 14 x 14 tile of the block's output: it stages the 33 x 33 x 3 input patch in LDS,
// computes the stem for the tile plus the depthwise conv's one-pixel halo (16 x 16 pixels; zeros outside the
// image, which is the depthwise conv's padding), keeps it in LDS rounded to bf16 exactly as the stored
// activation would be, and finishes the tile from there.
// Stem and pointwise are products on the matrix pipe, with 16 channels as rows and 16 pixels of a row as
// columns, so that a lane holds 4 channels of one pixel throughout, and takes the depthwise conv in between for
// those four out of registers.  With all of it in vector fp32, every thread a pixel with its 16 channels, a wave
// read 208 broadcast vectors of weights from LDS per 64 pixels, which is what bounded it.
// The stem's 27 products are one MFMA of 32: a lane group takes a window row's first 8 values (2 columns of 3
// channels and 2 of the third's, contiguous in the patch), the fourth group the ninth values of the three rows.
// Every activation is rounded to bf16 where the unfused layers store it, sums are fp32 in a fixed order, so a
// request's values do not depend on its batch mates.
#include "common.h"

namespace sna {

constexpr int MH_T = 14;             // output tile side
constexpr int MH_G = MH_T + 2;       // with the halo: 16 x 16 stem pixels
constexpr int MH_P = 2 * MH_G + 1;   // input patch side (stride 2, 3 taps): 33
constexpr int MH_C = 16;             // channels of the stem and of the first block
constexpr int MH_NT = 256;
constexpr int MH_ROW = 100;          // patch row in LDS, bf16 values: 33 x 3 and one that makes the windows' starts 4-byte aligned
static_assert(MH_P * 3 < MH_ROW && MH_G == 16 && MH_C == 16, "MFMA tiles of 16 channels x 16 pixels");

typedef __attribute__((ext_vector_type(8))) __bf16 mh_bf16x8;
typedef __attribute__((ext_vector_type(4))) short mh_s16x4;
typedef __attribute__((ext_vector_type(4))) float mh_f32x4;
typedef __attribute__((ext_vector_type(4))) unsigned int mh_u32x4;

__device__ __forceinline__ void mh_unpack4(const uint2 v, float* f) {
  f[0] = __uint_as_float(v.x << 16); f[1] = __uint_as_float(v.x & 0xffff0000u);
  f[2] = __uint_as_float(v.y << 16); f[3] = __uint_as_float(v.y & 0xffff0000u);
}

template <class Args>
__global__ __launch_bounds__(MH_NT, 4) void mbv3_head_kernel(const Args args) {
#if defined(__HIP_DEVICE_COMPILE__)        // the host pass needs the symbol only, not the body
  __shared__ __attribute__((aligned(16))) bf16_t patch[(MH_P + 1) * MH_ROW];
  __shared__ uint2 stem[MH_G * MH_G + 2][4];       // stem output of the tile and its halo, bf16; columns 16 and 17 of the last row are read, for pixels that are not stored

  const int g = find_problem(args, blockIdx.x);
  Mbv3HeadProblem p = pinned(args.p[g]);
  p.x = in_global(p.x); p.y = in_global(p.y); p.w_stem = in_global(p.w_stem); p.w_dw = in_global(p.w_dw); p.w_pw = in_global(p.w_pw);
  p.sc0 = in_global(p.sc0); p.sh0 = in_global(p.sh0); p.sc1 = in_global(p.sc1); p.sh1 = in_global(p.sh1); p.sc2 = in_global(p.sc2); p.sh2 = in_global(p.sh2);
  int local = blockIdx.x - p.tile_start;
  const int tx = local % p.tiles_x; local /= p.tiles_x;
  const int ty = local % p.tiles_y;
  const int n = local / p.tiles_y;
  const int oh0 = ty * MH_T, ow0 = tx * MH_T;
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int l16 = lane & 15, kg = lane >> 4;       // pixel (or weight row) of a 16 x 16 tile, and which four channels

  // ---- everything from memory is requested before any of it is used.  Patch: a thread takes one value of every second
  // row, so that rows are uniform over a wave; from addresses clamped into the image, and zeroed outside of it ----
  constexpr int ROWS = (MH_P + 1) / 2;
  const int ce = tid & 127, row0 = wave >> 1;      // value of a patch row, first row
  const int W = p.W, H = p.H, pix_e = p.pix_e;
  const int iy0 = 2 * oh0 - 3 + row0, iw = 2 * ow0 - 3 + ce / 3;
  const int col_e = (iw < 0 ? 0 : (iw < W ? iw : W - 1)) * pix_e + ce % 3;
  const bool col_ok = (ce < MH_P * 3) & ((unsigned)iw < (unsigned)W);
  const bf16_t* const img = (const bf16_t*)p.x + (long)n * H * W * pix_e;
  bf16_t pv[ROWS];
#pragma unroll
  for (int i = 0; i < ROWS; ++i) {
    const int ih = iy0 + 2 * i;
    pv[i] = img[(long)(ih < 0 ? 0 : (ih < H ? ih : H - 1)) * W * pix_e + col_e];
  }
  bf16_t ws[8], wd[9][4], wp[4];
  {
    const bf16_t* w = (const bf16_t*)p.w_stem + (long)l16 * p.wk0;
#pragma unroll
    for (int j = 0; j < 8; ++j) {
      const int r = kg < 3 ? kg : (j < 3 ? j : 0), sc = kg < 3 ? j : 8;
      ws[j] = w[r * p.wr0 + (sc / 3) * p.ws0 + sc % 3];
    }
#pragma unroll
    for (int t = 0; t < 9; ++t)
#pragma unroll
      for (int e = 0; e < 4; ++e) wd[t][e] = ((const bf16_t*)p.w_dw)[(t / 3) * p.wr1 + (t % 3) * p.ws1 + 4 * kg + e];
#pragma unroll
    for (int e = 0; e < 4; ++e) wp[e] = ((const bf16_t*)p.w_pw)[(long)l16 * p.wk2 + 4 * kg + e];
  }
  float sc0[4], sh0[4], sc1[4], sh1[4], sc2[4], sh2[4];
#pragma unroll
  for (int e = 0; e < 4; ++e) {
    const int c = 4 * kg + e;
    sc0[e] = p.sc0[c]; sh0[e] = p.sh0[c]; sc1[e] = p.sc1[c]; sh1[e] = p.sh1[c]; sc2[e] = p.sc2[c]; sh2[e] = p.sh2[c];
  }
  if (ce < MH_ROW) {
#pragma unroll
    for (int i = 0; i < ROWS; ++i) {
      const bool ok = col_ok & ((unsigned)(iy0 + 2 * i) < (unsigned)H);
      patch[(2 * i + row0) * MH_ROW + ce] = ok ? pv[i] : (bf16_t)0;
    }
  }
  mh_u32x4 wa;                                     // stem weights of channel l16, as the patch values lie in a lane
#pragma unroll
  for (int j = 0; j < 4; ++j) wa[j] = (kg < 3 || 2 * j < 3 ? (unsigned)ws[2 * j] : 0u) | (kg < 3 || 2 * j + 1 < 3 ? (unsigned)ws[2 * j + 1] << 16 : 0u);
  const mh_s16x4 wq = {(short)wp[0], (short)wp[1], (short)wp[2], (short)wp[3]};
  __syncthreads();

  // ---- stem for the 16 pixels of grid row gy ----
  int at[4];
#pragma unroll
  for (int j = 0; j < 4; ++j) at[j] = 12 * l16 + (kg < 3 ? 2 * MH_ROW * kg + 4 * j : 2 * MH_ROW * (j < 3 ? j : 2) + 16);
#pragma unroll
  for (int i = 0; i < MH_G / 4; ++i) {
    const int gy = wave * (MH_G / 4) + i;
    unsigned u[4];
#pragma unroll
    for (int j = 0; j < 4; ++j) u[j] = *(const unsigned*)((const char*)patch + 4 * MH_ROW * gy + at[j]);
    mh_u32x4 xb;
    xb[0] = kg < 3 ? u[0] : (u[0] & 0xffffu) | (u[1] << 16);
    xb[1] = kg < 3 ? u[1] : u[2] & 0xffffu;
    xb[2] = kg < 3 ? u[2] : 0u;
    xb[3] = kg < 3 ? u[3] : 0u;
    const mh_f32x4 zero = {0.f, 0.f, 0.f, 0.f};
    const mh_f32x4 acc = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(mh_bf16x8, wa), __builtin_bit_cast(mh_bf16x8, xb), zero, 0, 0, 0);
    const bool inside = ((unsigned)(oh0 - 1 + gy) < (unsigned)p.Ho) & ((unsigned)(ow0 - 1 + l16) < (unsigned)p.Wo);
    float v[4];
#pragma unroll
    for (int e = 0; e < 4; ++e) v[e] = apply_act(fmaf(acc[e], sc0[e], sh0[e]), SNA_ACT_HSWISH);
    stem[gy * MH_G + l16][kg] = inside ? make_uint2(pack_bf16x2(v[0], v[1]), pack_bf16x2(v[2], v[3])) : make_uint2(0u, 0u);
  }
  __syncthreads();

  // ---- depthwise 3x3 + SubnetNorm + ReLU, pointwise + SubnetNorm + residual for output row oh0 + oy (grid row + 1) ----
  float w1[9][4];
#pragma unroll
  for (int t = 0; t < 9; ++t)
#pragma unroll
    for (int e = 0; e < 4; ++e) w1[t][e] = bf16_to_f32(wd[t][e]);
  const bool col_out = (l16 < MH_T) & (ow0 + l16 < p.Wo);
  for (int oy = wave; oy < MH_T && oh0 + oy < p.Ho; oy += 4) {     // uniform over the wave: the MFMA wants all lanes
    uint2 x[9];
#pragma unroll
    for (int t = 0; t < 9; ++t) x[t] = stem[(oy + t / 3) * MH_G + l16 + t % 3][kg];
    float a[4] = {0.f, 0.f, 0.f, 0.f}, centre[4];
#pragma unroll
    for (int t = 0; t < 9; ++t) {
      float f[4];
      mh_unpack4(x[t], f);
#pragma unroll
      for (int e = 0; e < 4; ++e) a[e] = fmaf(f[e], w1[t][e], a[e]);
    }
    mh_unpack4(x[4], centre);
#pragma unroll
    for (int e = 0; e < 4; ++e) a[e] = fmaxf(fmaf(a[e], sc1[e], sh1[e]), 0.f);
    const uint2 d = make_uint2(pack_bf16x2(a[0], a[1]), pack_bf16x2(a[2], a[3]));
    const mh_f32x4 zero = {0.f, 0.f, 0.f, 0.f};
    const mh_f32x4 acc = __builtin_amdgcn_mfma_f32_16x16x16bf16_1k(wq, __builtin_bit_cast(mh_s16x4, d), zero, 0, 0, 0);
    float o[4];
#pragma unroll
    for (int e = 0; e < 4; ++e) o[e] = fmaf(acc[e], sc2[e], sh2[e]) + centre[e];
    if (col_out)
      *(uint2*)((bf16_t*)p.y + (((long)n * p.Ho + oh0 + oy) * p.Wo + ow0 + l16) * MH_C + 4 * kg) =
          make_uint2(pack_bf16x2(o[0], o[1]), pack_bf16x2(o[2], o[3]));
  }
#endif
}

int mbv3_head_channels() { return MH_C; }

hipError_t launch_mbv3_head(const Mbv3HeadArgs& a, hipStream_t s) {
  if (a.n == 0) return hipSuccess;
  Mbv3HeadArgs b = a;
  long start = 0;
  for (int i = 0; i < b.n; ++i) {
    Mbv3HeadProblem& p = b.p[i];
    if (p.N < 1 || p.H < 1 || p.W < 1 || p.Ho != (p.H - 1) / 2 + 1 || p.Wo != (p.W - 1) / 2 + 1 || p.pix_e < 3 ||
        !p.x || !p.y || !p.w_stem || !p.w_dw || !p.w_pw || !p.sc0 || !p.sh0 || !p.sc1 || !p.sh1 || !p.sc2 || !p.sh2)
      return hipErrorInvalidValue;
    p.tiles_x = (p.Wo + MH_T - 1) / MH_T; p.tiles_y = (p.Ho + MH_T - 1) / MH_T;
    p.tile_start = (int)start;
    p.tiles = p.N * p.tiles_x * p.tiles_y;
    start += p.tiles;
    if (start > 0x7fffffff) return hipErrorInvalidValue;
  }
  if (b.n == 1) hipLaunchKernelGGL(mbv3_head_kernel<Lone<Mbv3HeadProblem>>, dim3((unsigned)start), dim3(MH_NT), 0, s, Lone<Mbv3HeadProblem>{{b.p[0]}});
  else hipLaunchKernelGGL(mbv3_head_kernel<Mbv3HeadArgs>, dim3((unsigned)start), dim3(MH_NT), 0, s, b);
  return hipGetLastError();
}

}  // namespace sna
