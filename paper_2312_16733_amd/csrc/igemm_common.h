// Pieces shared by the implicit-GEMM kernels: LDS row format, tile geometry, the inline LDS read.
#pragma once
#include "common.h"

#include <type_traits>

namespace sna {
typedef __attribute__((ext_vector_type(8))) __bf16 bf16x8;
typedef __attribute__((ext_vector_type(16))) float f32x16;
typedef __attribute__((ext_vector_type(4))) unsigned int u32x4;
typedef __attribute__((address_space(3))) char lds_char;

constexpr int BK = 64;             // reduction elements per LDS stage
static_assert(BK == 64, "one LDS row holds one K step");
constexpr int ROW_B = 128;         // bytes per LDS row (one K step of one tile row)

// s_waitcnt immediate that waits until at most n vector-memory operations are outstanding
// (vmcnt is split over bits [3:0] and [15:14]; expcnt and lgkmcnt fields left at "no wait").
constexpr int vmcnt_imm(int n) { return 0x0F70 | (n & 15) | ((n >> 4) << 14); }

// FW: waves that only fetch, beside the computing ones (0: every wave does both)
template <int BM, int BN, int WARPS_M, int WARPS_N, int NS, int FW = 0>
struct IgemmCfg {
  static constexpr int NWAVES = WARPS_M * WARPS_N, NTHREADS = 64 * (FW ? FW : NWAVES);   // computing waves, fetching threads
  static constexpr int WTM = BM / WARPS_M, WTN = BN / WARPS_N;
  static constexpr int TM = WTM < 32 ? 1 : WTM / 32, TN = WTN / 32;      // 32x32 tiles of a wave (half of one: see the small deep rings)
  static constexpr int PASS_ROWS = NTHREADS / 8;                 // tile rows fetched per pass of the block
  static constexpr int A_IT = (BM + PASS_ROWS - 1) / PASS_ROWS, B_IT = (BN + PASS_ROWS - 1) / PASS_ROWS;
  static constexpr int STAGE_B = (BM + BN) * ROW_B;
  static constexpr int EPI_STRIDE = WTN + 4;                     // floats per staged row
  static constexpr int TILE_BYTES = NS * STAGE_B;
  static constexpr int EPI_BYTES = NWAVES * 32 * EPI_STRIDE * 4;
  static constexpr int SMEM = TILE_BYTES > EPI_BYTES ? TILE_BYTES : EPI_BYTES;
};

__device__ __forceinline__ unsigned long long low_bits(int n) { return n >= 64 ? ~0ull : (1ull << n) - 1ull; }   // n >= 0

__device__ __forceinline__ u32x4 lds_read_b128(unsigned addr, int imm) {
  u32x4 v;
#if defined(__HIP_DEVICE_COMPILE__)
  asm volatile("ds_read_b128 %0, %1 offset:%2" : "=v"(v) : "v"(addr), "n"(imm));
#else
  v = u32x4{addr, (unsigned)imm, 0u, 0u};      // host pass only parses this file
#endif
  return v;
}

__device__ __forceinline__ void lds_write_b128(unsigned addr, u32x4 v) {
#if defined(__HIP_DEVICE_COMPILE__)
  asm volatile("ds_write_b128 %0, %1" :: "v"(addr), "v"(v) : "memory");
#endif
}

// N such reads and the wait for them in one block, so that nothing can come between: no copy of a register whose data is
// still on its way, and no address in a register that a read returns to.
template <int N>
__device__ __forceinline__ void lds_read_b128_now(u32x4 (&v)[N], const unsigned (&addr)[N]) {
#if defined(__HIP_DEVICE_COMPILE__)
  if constexpr (N == 1) {
    asm volatile("ds_read_b128 %0, %1\n\ts_waitcnt lgkmcnt(0)" : "=&v"(v[0]) : "v"(addr[0]) : "memory");
  } else if constexpr (N == 2) {
    asm volatile("ds_read_b128 %0, %2\n\tds_read_b128 %1, %3\n\ts_waitcnt lgkmcnt(0)"
                 : "=&v"(v[0]), "=&v"(v[1]) : "v"(addr[0]), "v"(addr[1]) : "memory");
  } else if constexpr (N == 5) {
    asm volatile("ds_read_b128 %0, %5\n\tds_read_b128 %1, %6\n\tds_read_b128 %2, %7\n\tds_read_b128 %3, %8\n\t"
                 "ds_read_b128 %4, %9\n\ts_waitcnt lgkmcnt(0)"
                 : "=&v"(v[0]), "=&v"(v[1]), "=&v"(v[2]), "=&v"(v[3]), "=&v"(v[4])
                 : "v"(addr[0]), "v"(addr[1]), "v"(addr[2]), "v"(addr[3]), "v"(addr[4]) : "memory");
  } else if constexpr (N == 6) {
    asm volatile("ds_read_b128 %0, %6\n\tds_read_b128 %1, %7\n\tds_read_b128 %2, %8\n\tds_read_b128 %3, %9\n\t"
                 "ds_read_b128 %4, %10\n\tds_read_b128 %5, %11\n\ts_waitcnt lgkmcnt(0)"
                 : "=&v"(v[0]), "=&v"(v[1]), "=&v"(v[2]), "=&v"(v[3]), "=&v"(v[4]), "=&v"(v[5])
                 : "v"(addr[0]), "v"(addr[1]), "v"(addr[2]), "v"(addr[3]), "v"(addr[4]), "v"(addr[5]) : "memory");
  } else {
    static_assert(N == 8, "as many as the rings ask for");
    asm volatile("ds_read_b128 %0, %8\n\tds_read_b128 %1, %9\n\tds_read_b128 %2, %10\n\tds_read_b128 %3, %11\n\t"
                 "ds_read_b128 %4, %12\n\tds_read_b128 %5, %13\n\tds_read_b128 %6, %14\n\tds_read_b128 %7, %15\n\t"
                 "s_waitcnt lgkmcnt(0)"
                 : "=&v"(v[0]), "=&v"(v[1]), "=&v"(v[2]), "=&v"(v[3]), "=&v"(v[4]), "=&v"(v[5]), "=&v"(v[6]), "=&v"(v[7])
                 : "v"(addr[0]), "v"(addr[1]), "v"(addr[2]), "v"(addr[3]), "v"(addr[4]), "v"(addr[5]), "v"(addr[6]), "v"(addr[7])
                 : "memory");
  }
#endif
}

}  // namespace sna
