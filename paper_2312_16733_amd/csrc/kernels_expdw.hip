// First half of an inverted-residual block in one launch: pointwise expand + SubnetNorm + activation, and the depthwise
// k x k convolution on its output + SubnetNorm + activation, with the squeeze-excite pool's partial sums; both
// convolutions on bf16 MFMA.
//
// The expanded tensor is the widest of the network (3 to 6 times the block's input); as two launches it was written to
// memory and fetched back (3 + k) / 4 * k times per element by a depthwise kernel bound by the texture path and by
// instruction issue (95 VALU instructions per output at k = 7).  Here a block owns a spatial tile (of one request, or of
// the same small image in several) and 16 expanded channels:
//   A  the in-image input pixels the tile needs, halo included, go through v_mfma_f32_16x16x32_bf16 16 pixels at a time
//      (pixels as rows, channels as columns: a lane ends up with 4 pixels of one channel), are normalised, activated and
//      rounded to bf16 as a stored activation would be, and go to LDS channel by channel, [channel][row][column], with
//      zeros outside the image;
//   B  the depthwise convolution is a contraction per channel and kernel row r: 16 output columns q of a row are
//      Y[q] += sum_j X[j] T_r[j][q] with the band matrix T_r[j][q] = w[r][j - q], so that one MFMA takes 16 row segments
//      of 16 outputs (its rows: any 16 segments of the tile, each reading 32 consecutive columns of its row at one
//      16-byte LDS read per lane), 7 MFMAs a 7 x 7 kernel.  A lane's part of T_r is a window of the kernel row shifted
//      by the lane's place in the band: the rows lie in LDS between zeros, once at even and once at odd alignment, so
//      that it is four aligned words.  The zeros of the band are 78 % of the products at k = 7, and it is still 5 times
//      the rate of the dot-product instructions.  The tile's output rows are dealt out to the MFMA groups in turn (group g
//      has rows g, g + ng, g + 2 ng ..), so that what group g reads for kernel row r is what group g + 1 reads for kernel
//      row r - stride: a row fragment is read once for all groups, 10 reads for the 28 MFMAs of four groups at k = 7.
// The pool's sums are taken from the registers (a wave holds all outputs of its channels).  The results wait there until
// the block is done with the planes, are turned channel-fastest through LDS and stored, 16 bytes per lane.
//
// Measured, batch 64, expand + depthwise as two launches -> here (event-bracketed): 56^2, 24 -> 144, 7 x 7: 23.7 + 91.5 ->
// 42.7 us; 28^2, 40 -> 240: 12.6 + 47.9 -> 24.2; 14^2, 112 -> 672: 12.3 + 42.7 -> 31.6; 7^2, 160 -> 960: 8.5 + 21.1 -> 23.0;
// 112^2, stride 2, 16 -> 96: 44.8 + 90.4 -> 93.1; 14^2, stride 2, 112 -> 672, the one layer of the largest and the smallest
// subnet that loses: 12.3 + 22.5 -> 36.3; one request, 12^2, 80 -> 320: 8.2.  In the first version of this kernel, where the
// first of these layers took 55.6 us: 4 waves per block instead of 8 71.6 us (waves wait for each other's phases), half the
// LDS per block, 3 blocks per CU and more halo 82; the same design with v_dot2_f32_bf16 in B (56 VGPRs of weight pairs)
// 87.8 us and 15.7 us for a lone 6^2 x 960 layer against 8.7.
//
// The tile depends on the layer's shape alone, and every sum is taken in a fixed order, so a request's result does not
// depend on what it is batched with.
#include "igemm_common.h"

namespace sna {

constexpr int XD_CH = 16;           // expanded channels per block
constexpr int XD_NT = 512;          // threads: with the LDS two blocks fit on a CU, 4 waves per SIMD
constexpr int XD_SEG = 16;          // outputs per row segment
constexpr int XD_GROUPS = 4;        // MFMA groups of 16 segments per block, at most
constexpr int XD_OUT_PX = XD_CH / 2 + 2;                 // staged output: words per pixel, padded against bank conflicts
constexpr int XD_OUT_SEG = XD_SEG * XD_OUT_PX + 2;       // words per segment
constexpr int XD_TROW = 16;         // words per kernel row of the band table: 4 even-aligned, 4 zeros, 4 odd-aligned, 4 zeros

typedef __attribute__((ext_vector_type(4))) float f32x4;
typedef unsigned u32x4w __attribute__((ext_vector_type(4), aligned(4)));

// LDS layout and tile of one problem, the same on host and device
struct XdGeom {
  int th, ntx, rq;                  // output rows, 16-wide segments per row, requests per block
  int ng, na;                       // MFMA groups, rows of a request in one (group g has rows g, g + ng, ..)
  int seg;                          // segments of a request in a group, na ntx and those that are left empty: rq seg <= 16
  int tiles_y, tiles_x;
  int IH, CW;                       // rows and columns (elements) of a channel plane; column 0 is input column x0 * stride - 4
  int plane, req_plane;             // bytes per channel plane (an odd number of 16-byte units) and per request
};

// i / d for 0 <= i < 2^20, with inv = rcp(d): (i + 1/2) / d lies 1/(2 d) or more from an integer, the product within
// (i + 1/2) / d * 2^-22 of it
__device__ __forceinline__ int xd_div(int i, float inv) { return (int)(((float)i + 0.5f) * inv); }
__device__ __forceinline__ float xd_rcp(int d) { return __builtin_amdgcn_rcpf((float)d); }
__device__ __forceinline__ bool xd_finite(float v) { return fabsf(v) < __builtin_inff(); }

template <int K, int STRIDE>
__global__ __launch_bounds__(XD_NT, 4) void expand_dw_kernel(const ExpDwArgs args) {
#if defined(__HIP_DEVICE_COMPILE__)
  extern __shared__ __attribute__((aligned(16))) char smem[];
  ExpDwProblem p = args.p[0];
  int local;
  if (args.n > 1) {
    const TilePlace at = place_of_block(args, blockIdx.x);
    if (at.problem > 0) p = args.p[at.problem];
    local = at.tile;
  } else {
    local = tile_of_block(p);
  }                           // the channel groups of a tile, which read the same input, on one XCD
  if (local < 0) return;
  const int t1 = p.by_chunks.div(local), t2 = p.by_tiles_x.div(t1), t3 = p.by_tiles_y.div(t2);
  const int chunk = local - t1 * p.chunks, tx = t1 - t2 * p.tiles_x, ty = t2 - t3 * p.tiles_y;
  const int n0 = t3 * p.rq;                                     // first request of the block
  const int rq = p.N - n0 < p.rq ? p.N - n0 : p.rq;
  constexpr int PAD = K / 2, OFF = 4 - PAD;                     // output column q reads plane columns q * STRIDE + OFF + s
  constexpr int KB = ((XD_SEG - 1) * STRIDE + OFF + K + 31) / 32;     // MFMAs per kernel row
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int l16 = lane & 15, grp = lane >> 4;
  const int Cin = p.Cin, C = p.C, KS = (Cin + 31) >> 5, c0 = chunk * XD_CH;
  const int py0 = ty * p.th, qx0 = tx * p.ntx * XD_SEG;         // first output of the tile
  const int iy0 = py0 * STRIDE - PAD, ix0 = qx0 * STRIDE - 4;   // input pixel behind plane cell (0, 0)
  const int th_v = p.Ho - py0 < p.th ? p.Ho - py0 : p.th;
  const int tw_v = p.Wo - qx0 < p.ntx * XD_SEG ? p.Wo - qx0 : p.ntx * XD_SEG;

  char* const planes = smem;
  unsigned* const ttab = (unsigned*)(smem + p.x_lds);           // [4 zeros][XD_CH][K][XD_TROW]
  char* const wfrag = (char*)(ttab + 4 + XD_CH * K * XD_TROW);  // [KS][64 lanes][16 bytes]: expand weights as MFMA columns
  uint4* const qtab = (uint4*)(wfrag + KS * 1024);              // per quad of pixels: plane offset, masks, input offset

  // in-image rectangle of input pixels that valid outputs of this tile read, in quads of 4 columns
  const int y0 = iy0 < 0 ? 0 : iy0, y_need = iy0 + (th_v - 1) * STRIDE + K, y1 = y_need < p.H ? y_need : p.H;
  const int xa = ix0 < 0 ? 0 : ix0, x_need = ix0 + OFF + (tw_v - 1) * STRIDE + K, x1 = x_need < p.W ? x_need : p.W;
  const int rh = y1 - y0, nq = (x1 - xa + 3) >> 2, quads = rq * rh * nq, ngroups = (quads + 3) >> 2;

  constexpr unsigned OOB = 0x80000000u;
  const __amdgpu_buffer_rsrc_t rsrc_x = __builtin_amdgcn_make_buffer_rsrc((void*)p.x, 0, (int)p.x_bytes, 0x00020000);
  const __amdgpu_buffer_rsrc_t rsrc_we = __builtin_amdgcn_make_buffer_rsrc((void*)p.w_e, 0, (int)p.we_bytes, 0x00020000);
  const __amdgpu_buffer_rsrc_t rsrc_y = __builtin_amdgcn_make_buffer_rsrc(p.y, 0, p.N * p.Ho * p.Wo * C * 2, 0x00020000);

  // ---- set-up: every load goes out before its first use ----------------------------------------
  constexpr int WF_U = 1;                                       // 64 KS fragments: up to 256 input channels without a loop
  auto we_off = [&](int i) {                                    // fragment i: channel i % 16, elements 8 (i / 16) ..
    const int c = c0 + (i & 15), k = (i >> 4) * 8;
    return c < C && k < Cin ? (unsigned)((c * p.we_k + k) * 2) : OOB;
  };
  u32x4 wf[WF_U];
#pragma unroll
  for (int u = 0; u < WF_U; ++u) wf[u] = __builtin_bit_cast(u32x4, __builtin_amdgcn_raw_buffer_load_b128(rsrc_we, we_off(tid + u * XD_NT), 0, 0));
  // thread (r, c) fetches kernel row r of channel c
  static_assert(K * XD_CH <= XD_NT, "one thread per kernel row");
  unsigned wrow[8];
  {
    const int c = c0 + (tid & 15), r = tid >> 4;
    const bf16_t* w = (const bf16_t*)p.w_d + (long)r * p.wd_r + c;
#pragma unroll
    for (int s = 0; s < 8; ++s) wrow[s] = s < K && r < K && c < C ? (unsigned)w[s * p.wd_s] : 0u;
  }
  const int ce = c0 + l16;                                      // this lane's expanded channel
  const float se = ce < C ? p.sc_e[ce] : 0.f, he = ce < C ? p.sh_e[ce] : 0.f;

  const float inv_nq = xd_rcp(nq), inv_rh = xd_rcp(rh);
  for (int i = tid; i < ngroups * 4; i += XD_NT) {
    const int t = xd_div(i, inv_nq), cq = i - t * nq;
    const int rr = xd_div(t, inv_rh), ry = t - rr * rh;
    const int x = xa + 4 * cq, left = x1 - x;
    uint4 e;
    e.x = (unsigned)(rr * p.req_plane + ((y0 - iy0 + ry) * p.CW + x - ix0) * 2);
    e.y = left >= 2 ? 0xffffffffu : 0xffffu;
    e.z = left >= 4 ? 0xffffffffu : (left == 3 ? 0xffffu : 0u);
    e.w = (unsigned)((((n0 + rr) * p.H + y0 + ry) * p.W + x) * Cin * 2);
    if (i >= quads) { e.x = 0xffffffffu; e.w = OOB; }
    qtab[i] = e;
  }
  // (the planes, and behind them what the last segments of a tile whose rows ng does not divide read, and drop)
  for (int i = tid; i < p.x_lds / 16; i += XD_NT) *(uint4*)(planes + i * 16) = make_uint4(0, 0, 0, 0);
  __syncthreads();

  // what the loads above brought goes to LDS
  auto finish_setup = [&] {
#pragma unroll
    for (int u = 0; u < WF_U; ++u)
      if (tid + u * XD_NT < KS * 64) *(u32x4*)(wfrag + (tid + u * XD_NT) * 16) = wf[u];
    for (int i = tid + WF_U * XD_NT; i < KS * 64; i += XD_NT)
      *(u32x4*)(wfrag + i * 16) = __builtin_bit_cast(u32x4, __builtin_amdgcn_raw_buffer_load_b128(rsrc_we, we_off(i), 0, 0));
    if (tid < K * XD_CH) {
      unsigned* const row = ttab + 4 + ((tid & 15) * K + (tid >> 4)) * XD_TROW;
      *(uint4*)row = make_uint4(wrow[0] | (wrow[1] << 16), wrow[2] | (wrow[3] << 16), wrow[4] | (wrow[5] << 16), wrow[6]);
      *(uint4*)(row + 4) = make_uint4(0, 0, 0, 0);
      *(uint4*)(row + 8) = make_uint4(wrow[0] << 16, wrow[1] | (wrow[2] << 16), wrow[3] | (wrow[4] << 16), wrow[5] | (wrow[6] << 16));
      *(uint4*)(row + 12) = make_uint4(0, 0, 0, 0);
    }
    if (tid == 0) *(uint4*)ttab = make_uint4(0, 0, 0, 0);
    __syncthreads();
  };

  // ---- A: expand ------------------------------------------------------------------------------
  constexpr int NW = XD_NT / 64;
  // Pixel loads: lane (l16, grp) takes channels 8 grp .. of 32 of pixel l16 of a group; past Cin it reads zeros
  const unsigned px_lane = (unsigned)((l16 & 3) * Cin * 2 + grp * 16);
  const unsigned px_tail = (KS - 1) * 32 + grp * 8 < Cin ? 0u : OOB;        // of the last 32 channels
  char* const px_dst = planes + l16 * p.plane;
  // rows 4 grp .. 4 grp + 3 of a group's 16 pixels, one quad, of channel l16
  auto store_quad = [&](auto act_c, const f32x4& acc, const uint4& e) {
    constexpr int ACT = decltype(act_c)::value;
    float v[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) v[i] = apply_act(fmaf(acc[i], se, he), ACT);
    if (e.x != 0xffffffffu) *(uint2*)(px_dst + e.x) = make_uint2(pack_bf16x2(v[0], v[1]) & e.y, pack_bf16x2(v[2], v[3]) & e.z);
  };
  // Up to 5 steps of 32 input channels: a wave has the loads of its next PF groups of 16 pixels in flight (one group ahead,
  // waited for before the epilogue, a group took 2000 cycles, a load's round trip; 14^2, 112 -> 672, 7 x 7, four groups a
  // wave: 9900 cycles for this phase), the first ones under the rest of the set-up.  Loads past the last group are
  // out of range and cost no memory traffic; no branch stands between a load and its wait.
  auto expand = [&](auto act_c, auto ku_c) {
    constexpr int KU = decltype(ku_c)::value, PF = KU == 1 ? 8 : (KU == 2 ? 6 : (KU == 3 ? 4 : 3));
    u32x4 px[PF][KU];
    auto offset_of = [&](int pg) { return qtab[(pg < ngroups ? pg : 0) * 4 + (l16 >> 2)].w; };
    auto request = [&](int pg, unsigned off, u32x4 (&v)[KU]) {
      const unsigned base = (off + px_lane) | (pg < ngroups ? 0u : OOB);
#pragma unroll
      for (int j = 0; j < KU; ++j)
        v[j] = __builtin_bit_cast(u32x4, __builtin_amdgcn_raw_buffer_load_b128(rsrc_x, (j + 1 < KU ? base : base | px_tail) + j * 64, 0, 0));
    };
#pragma unroll
    for (int s = 0; s < PF; ++s) request(wave + s * NW, offset_of(wave + s * NW), px[s]);
    finish_setup();
    bf16x8 w[KU];
#pragma unroll
    for (int j = 0; j < KU; ++j) w[j] = *(const bf16x8*)(wfrag + (j * 64 + lane) * 16);
    for (int pg = wave;;) {
#pragma unroll
      for (int s = 0; s < PF; ++s, pg += NW) {
        if (pg >= ngroups) return;
        uint4 e = qtab[pg * 4 + grp];
        const unsigned off = offset_of(pg + PF * NW);
        f32x4 acc = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int j = 0; j < KU; ++j) acc = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, px[s][j]), w[j], acc, 0, 0, 0);
        request(pg + PF * NW, off, px[s]);
        asm volatile("" : "+v"(e.x), "+v"(e.y), "+v"(e.z));     // read up there, not behind the test of e.x
        store_quad(act_c, acc, e);
      }
    }
  };
  // More than 160 input channels: a group's steps in runs of five, the loads of the next run (or of the wave's next group) in
  // flight under the MFMAs of this one, the first run's under the rest of the set-up (twelve layers of 168 to 640 channels, 3 x 3:
  // 569 -> 542 us at 32 requests and 230 -> 217 at one, against loading and multiplying in turn).
  auto expand_wide = [&](auto act_c) {
    constexpr int KU = 5;
    auto request = [&](unsigned base, int ks0, u32x4 (&v)[KU]) {
#pragma unroll
      for (int j = 0; j < KU; ++j) {
        const int ks = ks0 + j;
        v[j] = __builtin_bit_cast(u32x4, __builtin_amdgcn_raw_buffer_load_b128(rsrc_x, ks < KS ? (ks < KS - 1 ? base : base | px_tail) + ks * 64 : OOB, 0, 0));
      }
    };
    auto base_of = [&](int pg) { return pg < ngroups ? qtab[pg * 4 + (l16 >> 2)].w + px_lane : OOB; };
    u32x4 cur[KU], nxt[KU];
    unsigned base = base_of(wave);
    request(base, 0, cur);
    finish_setup();
    for (int pg = wave; pg < ngroups; pg += NW) {
      const unsigned base_next = base_of(pg + NW);
      f32x4 acc = {0.f, 0.f, 0.f, 0.f};
      for (int ks0 = 0; ks0 < KS; ks0 += KU) {
        const bool more = ks0 + KU < KS;
        request(more ? base : base_next, more ? ks0 + KU : 0, nxt);
#pragma unroll
        for (int j = 0; j < KU; ++j)
          if (ks0 + j < KS)
            acc = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, cur[j]), *(const bf16x8*)(wfrag + ((ks0 + j) * 64 + lane) * 16), acc, 0, 0, 0);
#pragma unroll
        for (int j = 0; j < KU; ++j) cur[j] = nxt[j];
      }
      base = base_next;
      store_quad(act_c, acc, qtab[pg * 4 + grp]);
    }
  };
  auto expand_k = [&](auto act_c) {
    if (KS == 1) expand(act_c, std::integral_constant<int, 1>{});
    else if (KS == 2) expand(act_c, std::integral_constant<int, 2>{});
    else if (KS == 3) expand(act_c, std::integral_constant<int, 3>{});
    else if (KS == 4) expand(act_c, std::integral_constant<int, 4>{});
    else if (KS == 5) expand(act_c, std::integral_constant<int, 5>{});
    else expand_wide(act_c);
  };
  if (p.act == SNA_ACT_RELU) expand_k(std::integral_constant<int, SNA_ACT_RELU>{});
  else expand_k(std::integral_constant<int, SNA_ACT_HSWISH>{});
  __syncthreads();

  // ---- B: depthwise ---------------------------------------------------------------------------
  // Row l of every MFMA group is a segment (request rr, rows ng aa + g, column segment tt); of an empty one the row is th or more
  const int ng = p.ng;
  const float inv_ntx = xd_rcp(p.ntx), inv_sr = xd_rcp(p.seg);
  struct Seg { int rr, row, tt; };                              // row: of group 0
  auto segment = [&](int l) {
    const int rr = xd_div(l, inv_sr), ii = l - rr * p.seg;
    const int aa = xd_div(ii, inv_ntx);
    return Seg{rr, aa * ng, ii - aa * p.ntx};
  };
  int seg_off;                                                  // plane offset of this lane's segment, MFMA row l16
  {
    const Seg s = segment(l16);
    const int off = s.rr * p.req_plane + (s.row * STRIDE * p.CW + s.tt * XD_SEG * STRIDE) * 2;
    seg_off = (s.rr < p.rq) & (s.row < p.th) ? off : 0;
  }
  // this lane's 8 elements of the band: columns 32 kb + 8 grp .. + 7 against output l16
  int col_off[KB], t_off[KB];
#pragma unroll
  for (int kb = 0; kb < KB; ++kb) {
    const int j0 = 32 * kb + 8 * grp, sh = l16 * STRIDE + OFF - j0;
    col_off[kb] = j0 < (XD_SEG - 1) * STRIDE + OFF + K ? j0 * 2 : 0;      // past the band every weight is 0: read any column
    int b = -(sh >> 1);                                         // floor
    b = b < -4 ? -4 : (b > 4 ? 4 : b);
    t_off[kb] = ((sh & 1) ? 8 : 0) + b;
  }
  // A sum that is not finite, taken again over the output's own in-image taps in order: the band's zeros make NaN of an Inf
  // or NaN pixel for all 16 outputs of its row segment, and ReLU then makes 0 of that.  The check on every sum costs 0.6 %
  // of a forward (64 requests of the largest subnet 1249 -> 1256 us, a lone one 334 -> 336); one check after all groups,
  // which keeps their sums alive until then, costs 2.5 % (1283).
  auto own_taps = [&](f32x4 acc, int cl, int g) {
#pragma unroll 1
    for (int v = 0; v < 4; ++v) {
      const float a = v == 0 ? acc[0] : (v == 1 ? acc[1] : (v == 2 ? acc[2] : acc[3]));
      if (xd_finite(a)) continue;
      const Seg sg = segment(4 * grp + v);
      const int rr = sg.rr, pr = sg.row + g, q = sg.tt * XD_SEG + l16;
      if (rr >= rq || pr >= p.th) continue;                     // no output of the tile
      const int iy = (py0 + pr) * STRIDE - PAD, ix = (qx0 + q) * STRIDE - PAD;
      const bf16_t* x = (const bf16_t*)(planes + cl * p.plane + rr * p.req_plane) + pr * STRIDE * p.CW + q * STRIDE + OFF;
      const bf16_t* w = (const bf16_t*)(ttab + 4 + cl * K * XD_TROW);
      float sum = 0.f;
#pragma unroll 1
      for (int r = 0; r < K; ++r, x += p.CW, w += XD_TROW * 2)
#pragma unroll 1
        for (int s = 0; s < K; ++s)
          if ((unsigned)(iy + r) < (unsigned)p.H && (unsigned)(ix + s) < (unsigned)p.W) sum = fmaf(bf16_to_f32(x[s]), bf16_to_f32(w[s]), sum);
      acc[0] = v == 0 ? sum : acc[0]; acc[1] = v == 1 ? sum : acc[1]; acc[2] = v == 2 ? sum : acc[2]; acc[3] = v == 3 ? sum : acc[3];
    }
    return acc;
  };
  static_assert(XD_CH == 2 * (XD_NT / 64), "a wave has one pair of channels");
  unsigned packed[XD_GROUPS][4];                                // outputs of the pair: group g, segment 4 grp + v, column l16
  auto depthwise = [&](auto act_c, auto ng_c) {
    constexpr int ACT = decltype(act_c)::value, NG = decltype(ng_c)::value;
    float first[NG][4];
#pragma unroll
    for (int h = 0; h < 2; ++h) {
      const int cl = wave * 2 + h, c = c0 + cl;
      const float sc = c < C ? p.sc_d[c] : 0.f, sh = c < C ? p.sh_d[c] : 0.f;
      u32x4 band[K][KB];
#pragma unroll
      for (int r = 0; r < K; ++r)
#pragma unroll
        for (int kb = 0; kb < KB; ++kb) band[r][kb] = *(const u32x4w*)(ttab + 4 + (cl * K + r) * XD_TROW + t_off[kb]);
      const char* src = planes + cl * p.plane + seg_off;
      f32x4 acc[NG];
#pragma unroll
      for (int g = 0; g < NG; ++g) acc[g] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
      for (int d = 0; d < (NG - 1) * STRIDE + K; ++d) {         // plane rows from the segment's own on, kernel row d - g stride of group g
#pragma unroll
        for (int kb = 0; kb < KB; ++kb) {
          const uint4 a = *(const uint4*)(src + col_off[kb]);
#pragma unroll
          for (int g = 0; g < NG; ++g)
            if (d >= g * STRIDE && d - g * STRIDE < K)
              acc[g] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, a), __builtin_bit_cast(bf16x8, band[d - g * STRIDE][kb]), acc[g], 0, 0, 0);
        }
        src += p.CW * 2;
      }
#pragma unroll
      for (int g = 0; g < NG; ++g) {
        if (__builtin_expect(__any(!xd_finite((acc[g][0] + acc[g][1]) + (acc[g][2] + acc[g][3]))), 0)) acc[g] = own_taps(acc[g], cl, g);
#pragma unroll
        for (int v = 0; v < 4; ++v) {
          const float y = apply_act(fmaf(acc[g][v], sc, sh), ACT);
          if (h == 0) first[g][v] = y;
          else packed[g][v] = pack_bf16x2(first[g][v], y);
        }
      }
    }
#pragma unroll
    for (int g = NG; g < XD_GROUPS; ++g)
#pragma unroll
      for (int v = 0; v < 4; ++v) packed[g][v] = 0;
  };
  auto depthwise_act = [&](auto act_c) {
    if (ng == 4) depthwise(act_c, std::integral_constant<int, 4>{});
    else if (ng == 3) depthwise(act_c, std::integral_constant<int, 3>{});
    else if (ng == 2) depthwise(act_c, std::integral_constant<int, 2>{});
    else depthwise(act_c, std::integral_constant<int, 1>{});
  };
  if (p.act == SNA_ACT_RELU) depthwise_act(std::integral_constant<int, SNA_ACT_RELU>{});
  else depthwise_act(std::integral_constant<int, SNA_ACT_HSWISH>{});

  // ---- pool: this wave's two channels, per request; a lane over its outputs in order, the lanes by a fixed tree, in an order
  // that does not depend on the request's place in the block ------------------------------------------
  if (p.pool_part) {
    float s0[4], s1[4];
    int req[4];
#pragma unroll
    for (int v = 0; v < 4; ++v) {                               // the groups' rows of a segment belong to one request
      const Seg sg = segment(4 * grp + v);
      const int rows = sg.rr < rq && sg.tt * XD_SEG + l16 < tw_v ? th_v - sg.row : 0;     // valid rows g = 0 ..
      req[v] = sg.rr;
      s0[v] = s1[v] = 0.f;
#pragma unroll
      for (int g = 0; g < XD_GROUPS; ++g) {
        const unsigned w = g < rows && g < ng ? packed[g][v] : 0u;
        s0[v] += __uint_as_float(w << 16);
        s1[v] += __uint_as_float(w & 0xffff0000u);
      }
    }
    const int c = c0 + wave * 2;
    auto out = [&](int rr) { return p.pool_part + ((long)((n0 + rr) * p.tiles_y + ty) * p.tiles_x + tx) * C + c; };
    if (__builtin_expect(p.rq > 1 && p.seg > 2 && (p.seg & 3) != 0, 0)) {
      // A lane's four segments are not all of one request, and in which way depends on the request's place in the block.  So
      // each segment's columns first, and a lane for each request and channel adds that request's segments in order, from where
      // the expand weights lay.
      float* const tot = (float*)wfrag + wave * 32;             // 16 segments of the first channel, then of the second
#pragma unroll
      for (int v = 0; v < 4; ++v) { s0[v] = row_sum(s0[v]); s1[v] = row_sum(s1[v]); }
      if (l16 == 15) {
        *(float4*)(tot + 4 * grp) = make_float4(s0[0], s0[1], s0[2], s0[3]);
        *(float4*)(tot + 16 + 4 * grp) = make_float4(s1[0], s1[1], s1[2], s1[3]);
      }
      asm volatile("" ::: "memory");
      __builtin_amdgcn_wave_barrier();
      const int rr = lane >> 1, ch = lane & 1;
      if (rr < rq && c < C) {
        float a = 0.f;
#pragma unroll
        for (int i = 0; i < 8; ++i) {                           // two requests or more: 8 segments at most
          const float t = tot[ch * 16 + rr * p.seg + (i < p.seg ? i : 0)];
          a += i < p.seg ? t : 0.f;
        }
        out(rr)[ch] = a;
      }
    } else {
      for (int rr = 0; rr < rq; ++rr) {
        float a0 = 0.f, a1 = 0.f;
#pragma unroll
        for (int v = 0; v < 4; ++v) {
          a0 += req[v] == rr ? s0[v] : 0.f;
          a1 += req[v] == rr ? s1[v] : 0.f;
        }
        a0 = lane_sum(a0); a1 = lane_sum(a1);
        if (lane == 63 && c < C) *(float2*)out(rr) = make_float2(a0, a1);
      }
    }
  }
  __syncthreads();                                              // every wave is done with the planes

  // ---- output: [group][segment][16 columns][channel pairs] through LDS -------------------------
  unsigned* const outs = (unsigned*)smem;
#pragma unroll
  for (int g = 0; g < XD_GROUPS; ++g) {
    if (g >= ng) continue;
#pragma unroll
    for (int v = 0; v < 4; ++v) outs[(g * 16 + 4 * grp + v) * XD_OUT_SEG + l16 * XD_OUT_PX + wave] = packed[g][v];
  }
  __syncthreads();
  // a thread stores 8 channels of one pixel per group: segment tid / 32, column tid / 2 % 16
  static_assert(XD_NT == 16 * XD_SEG * 2 && XD_CH == 16, "one thread per 8 channels of a group's pixels");
  const int oh = tid & 1, oq = (tid >> 1) & 15, ol = tid >> 5;
  const Seg so = segment(ol);
  const int qq = so.tt * XD_SEG + oq, c = c0 + oh * 8;
  if (so.rr < rq && qq < tw_v && c < C) {
    const unsigned* src = outs + ol * XD_OUT_SEG + oq * XD_OUT_PX + oh * 4;
    const unsigned off = (unsigned)(((((n0 + so.rr) * p.Ho + py0 + so.row) * p.Wo + qx0 + qq) * C + c) * 2);
#pragma unroll
    for (int g = 0; g < XD_GROUPS; ++g)
      if (g < ng && so.row + g < th_v) {
        const uint2 lo = *(const uint2*)(src + g * 16 * XD_OUT_SEG), hi = *(const uint2*)(src + g * 16 * XD_OUT_SEG + 2);
        __builtin_amdgcn_raw_buffer_store_b128(u32x4{lo.x, lo.y, hi.x, hi.y}, rsrc_y, off + (unsigned)(g * p.Wo * C * 2), 0, 0);
      }
  }
#endif
}

// Tile of a layer, from its shape alone.  Stride 1: whole rows up to 64 columns and as many rows as leave two blocks per
// CU their LDS (halo rows are computed twice, so tall tiles), small images several requests to a block, which share the
// band fragments.  Stride 2: 16 columns (twice the input columns, two MFMAs a kernel row) and 16 rows.
constexpr size_t XD_PLANES_MAX = 52 * 1024;
static XdGeom xd_geometry(int Ho, int Wo, int k, int stride) {
  XdGeom g;
  const int segs = (Wo + XD_SEG - 1) / XD_SEG, off = 4 - k / 2;
  const int max_x = stride == 1 ? 4 : 1;
  g.tiles_x = (segs + max_x - 1) / max_x;
  g.ntx = (segs + g.tiles_x - 1) / g.tiles_x;
  g.tiles_x = (segs + g.ntx - 1) / g.ntx;
  int units = ((g.ntx - 1) * XD_SEG * stride + (XD_SEG - 1) * stride + off + k + 7) / 8;
  units |= 1;                                                   // odd: 16 rows then start on 16 different bank groups
  g.CW = units * 8;
  auto plane = [&](int th) { return ((((th - 1) * stride + k) * units) | 1) * 16; };
  int th = XD_GROUPS * (16 / g.ntx);
  if (stride == 2 && th > 16) th = 16;
  if (th > Ho) th = Ho;
  while (th > 1 && (size_t)plane(th) * XD_CH > XD_PLANES_MAX) --th;
  g.tiles_y = (Ho + th - 1) / th;
  g.th = (Ho + g.tiles_y - 1) / g.tiles_y;
  g.tiles_y = (Ho + g.th - 1) / g.th;
  g.IH = (g.th - 1) * stride + k;
  g.plane = plane(g.th);
  g.req_plane = g.plane * XD_CH;
  g.rq = 1;
  if (g.tiles_x == 1 && g.tiles_y == 1)
    while (g.rq < 4 && (g.rq + 1) * g.th * g.ntx <= 32 && (size_t)(g.rq + 1) * g.req_plane <= XD_PLANES_MAX) ++g.rq;
  // as few groups as hold the segments; four always do (th <= 4 floor(16 / ntx); with several requests, at most 32 segments)
  for (g.ng = 1; g.ng < XD_GROUPS && g.rq * ((g.th + g.ng - 1) / g.ng) * g.ntx > 16; ++g.ng) {}
  g.na = (g.th + g.ng - 1) / g.ng;
  // Of several requests, each begins with a lane's first segment, or fits into half a lane, where there is room for it: then
  // the pool's sums are as if it were alone in the block.  (There is not for three requests of 5 segments, 9 or 10 rows: with
  // two requests 64 of them took 2.6 % of a forward longer, with one group more 1 to 2 % at any batch.)
  g.seg = g.na * g.ntx;
  const int whole = (g.seg + 3) / 4 * 4;
  if (g.rq > 1 && g.seg > 2 && g.rq * whole <= 16) g.seg = whole;
  return g;
}
static size_t xd_planes(const XdGeom& g, int stride) {          // with the rows past the tile that B reads; also holds the staged output
  const size_t x = (size_t)g.rq * g.req_plane + (size_t)(g.na * g.ng - g.th) * stride * g.CW * 2, o = (size_t)g.ng * 16 * XD_OUT_SEG * 4;
  return ((x > o ? x : o) + 15) / 16 * 16;
}
static size_t xd_lds(const XdGeom& g, int k, int stride, int Cin) {
  return xd_planes(g, stride) + (size_t)(4 + XD_CH * k * XD_TROW) * 4 + (size_t)((Cin + 31) / 32) * 1024 +
         (size_t)(g.rq * g.IH * (g.CW / 4) + 3) / 4 * 4 * 16;
}
constexpr size_t XD_LDS_MAX = 160 * 1024;

int expand_dw_pool_parts(int Ho, int Wo, int k, int stride) {
  const XdGeom g = xd_geometry(Ho, Wo, k, stride);
  return g.tiles_x * g.tiles_y;
}
// Each tile column has at least one 16-wide segment, and there are at most ceil(Ho / 16) tile rows: before the rows are
// spread evenly a tile has min(16, Ho) at least (four groups of 16 segments over at most 4 a row, and the planes of 17 rows fit for
// every k and stride), and spreading them adds no tile.
int expand_dw_pool_parts_max(int side) { return ((side + 15) / 16) * ((side + 15) / 16); }

bool expand_dw_ok(const ExpDwProblem& p) {
  if ((p.k != 3 && p.k != 5 && p.k != 7) || (p.stride != 1 && p.stride != 2) || p.Cin % 8 || p.C % 8) return false;
  if (p.act != SNA_ACT_RELU && p.act != SNA_ACT_HSWISH) return false;
  const XdGeom g = xd_geometry(p.Ho, p.Wo, p.k, p.stride);
  return xd_lds(g, p.k, p.stride, p.Cin) <= XD_LDS_MAX && g.tiles_x * g.tiles_y <= expand_dw_pool_parts_max(p.Ho > p.Wo ? p.Ho : p.Wo);
}

hipError_t launch_expand_dw(const ExpDwArgs& a, hipStream_t s) {
  // one launch per (kernel size, stride) present among the problems
  for (int k = 3; k <= 7; k += 2)
    for (int st = 1; st <= 2; ++st) {
      ExpDwArgs b;
      b.n = 0;
      int start = 0;
      size_t lds = 0;
      for (int i = 0; i < a.n; ++i) {
        if (a.p[i].k != k || a.p[i].stride != st) continue;
        if (!expand_dw_ok(a.p[i])) return hipErrorInvalidValue;
        ExpDwProblem& p = b.p[b.n++];
        p = a.p[i];
        if ((double)p.N * p.H * p.W * p.Cin * 2 >= 2147483648.0 || (double)p.N * p.Ho * p.Wo * p.C * 2 >= 2147483648.0)
          return hipErrorInvalidValue;                          // 32-bit buffer offsets; slice_conv has refused such a call
        const XdGeom g = xd_geometry(p.Ho, p.Wo, k, st);
        p.th = g.th; p.ntx = g.ntx; p.rq = g.rq; p.ng = g.ng; p.seg = g.seg; p.tiles_x = g.tiles_x; p.tiles_y = g.tiles_y;
        p.CW = g.CW; p.plane = g.plane; p.req_plane = g.req_plane; p.x_lds = (int)xd_planes(g, st);
        p.chunks = (p.C + XD_CH - 1) / XD_CH;
        p.by_chunks = FastDiv::by(p.chunks); p.by_tiles_x = FastDiv::by(p.tiles_x); p.by_tiles_y = FastDiv::by(p.tiles_y);
        p.tile_start = start;
        p.tiles = (p.N + g.rq - 1) / g.rq * g.tiles_x * g.tiles_y * p.chunks;
        start += tile_rows(p.tiles);
        const size_t l = xd_lds(g, k, st, p.Cin);
        if (l > lds) lds = l;
      }
      if (!b.n) continue;
      b.total_tiles = launch_blocks(b);
      const int blocks = b.total_tiles;
      hipError_t e = hipSuccess;
#define SNA_XD(KK, SS)                                                                                                \
  if (k == KK && st == SS) {                                                                                          \
    e = hipFuncSetAttribute((const void*)expand_dw_kernel<KK, SS>, hipFuncAttributeMaxDynamicSharedMemorySize, (int)XD_LDS_MAX); \
    if (e != hipSuccess) return e;                                                                                    \
    hipLaunchKernelGGL((expand_dw_kernel<KK, SS>), dim3(blocks), dim3(XD_NT), lds, s, b);                             \
  }
      SNA_XD(3, 1); SNA_XD(5, 1); SNA_XD(7, 1); SNA_XD(3, 2); SNA_XD(5, 2); SNA_XD(7, 2);
#undef SNA_XD
      e = hipGetLastError();
      if (e != hipSuccess) return e;
    }
  return hipSuccess;
}

}  // namespace sna
