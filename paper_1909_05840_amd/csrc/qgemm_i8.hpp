// Pieces that the int8 forward kernels share: copies into LDS, packed slots out of LDS, the order of tiles.
#pragma once
#include "qb_common.hpp"
#include <type_traits>

namespace qb {
namespace {

// a*b + c for |a|, |b| < 2^23 (full-rate 24-bit multiplier instead of the quarter-rate 32-bit one)
__device__ __forceinline__ int qb_mad24(int a, int b, int c) { return __mul24(a, b) + c; }

// A4 = 4*acc + corr.  The result fits int32 for every K the library accepts, but 4*acc alone can reach 2^31 at
// K = 32768 with end-of-range operands: the sum is formed modulo 2^32 in unsigned arithmetic.
__device__ __forceinline__ int qb_a4(int acc, int corr) { return (int)(4u * (uint32_t)acc + (uint32_t)corr); }

typedef int v4i __attribute__((ext_vector_type(4)));
typedef int v16i __attribute__((ext_vector_type(16)));
typedef unsigned int v4u __attribute__((ext_vector_type(4)));

// Asymmetric group ranges (weights Delta*u + q0, u = 0..L): with R = sum_j (2x'+1) = 2*rs_x + K and
// S = sum_j (2x'+1)*u = (A4 + L*R)/2 the output is h_x*(Delta*S + q0*R).  A4 and R are even (K is), and
// S = A4/2 + L*(R/2) stays inside int32 for every K the library accepts.  rh = R/2 = rs_x + K/2.
__device__ __forceinline__ float asym_value(int a4, int rh, int L, float hx, float delta, float q0)
{
    const int S = (a4 >> 1) + L * rh;
    return hx * (delta * (float)S + q0 * (float)(2 * rh));
}

// global -> LDS copy by the load unit: the global address of a lane is a wavefront-uniform base (in SGPRs) plus
// the lane's 32-bit byte offset, the data of lane l lands at LDS address m0 + BYTES*l (16*l also for the 12-byte form).
// Written as inline assembly on purpose: the compiler then keeps no book on these copies, and the kernel states
// itself, with wait_vmcnt, which of them must have landed before a barrier.  The compiler may have written the base with
// a VALU instruction (v_readlane of a spilled value, v_readfirstlane) right in front, which a vector memory instruction may
// read five wait states later only; it counts them for its own instructions, not into an asm block.  So the block moves the
// base into registers of its own: a scalar instruction may read what a VALU instruction wrote at any time, the copy what a
// scalar one wrote; and the move is the wait state that m0 asks for in front of the copy.
// (qgemm_i8_dma_kernel at 2 bits, 16384 x 2304 x 768: 41.2 us, with five wait states in front of every copy 41.8, with one 40.6.)
template <int BYTES>
__device__ __forceinline__ void copy_to_lds(const void *base, uint32_t off, uint32_t lds_addr)
{
    static_assert(BYTES == 4 || BYTES == 12 || BYTES == 16, "");
    const void *own;
    if constexpr (BYTES == 16)
        asm volatile("s_mov_b32 m0, %3\n\ts_mov_b64 %0, %1\n\tglobal_load_lds_dwordx4 %2, %0" : "=&s"(own) : "s"(base), "v"(off), "s"(lds_addr) : "memory", "m0");
    else if constexpr (BYTES == 12)
        asm volatile("s_mov_b32 m0, %3\n\ts_mov_b64 %0, %1\n\tglobal_load_lds_dwordx3 %2, %0" : "=&s"(own) : "s"(base), "v"(off), "s"(lds_addr) : "memory", "m0");
    else
        asm volatile("s_mov_b32 m0, %3\n\ts_mov_b64 %0, %1\n\tglobal_load_lds_dword %2, %0" : "=&s"(own) : "s"(base), "v"(off), "s"(lds_addr) : "memory", "m0");
}

template <int BITS> struct SlotRead;  // one lane's slot (32 codes) out of LDS
template <> struct SlotRead<2> {
    static __device__ __forceinline__ void get(const uint8_t *p, uint32_t (&o)[2])
    {
        const uint2 v = *reinterpret_cast<const uint2 *>(p);
        o[0] = v.x; o[1] = v.y;
    }
};
template <> struct SlotRead<3> {
    typedef unsigned int v3u __attribute__((ext_vector_type(3)));
    static __device__ __forceinline__ void get(const uint8_t *p, uint32_t (&o)[3])
    {
        const v3u v = *reinterpret_cast<const v3u *>(p);
        o[0] = v[0]; o[1] = v[1]; o[2] = v[2];
    }
};
template <> struct SlotRead<4> {
    static __device__ __forceinline__ void get(const uint8_t *p, uint32_t (&o)[4])
    {
        const v4u v = *reinterpret_cast<const v4u *>(p);
        o[0] = v[0]; o[1] = v[1]; o[2] = v[2]; o[3] = v[3];
    }
};
template <> struct SlotRead<8> {
    static __device__ __forceinline__ void get(const uint8_t *p, uint32_t (&o)[8])
    {
        const v4u a = *reinterpret_cast<const v4u *>(p), b = *reinterpret_cast<const v4u *>(p + 16);
        o[0] = a[0]; o[1] = a[1]; o[2] = a[2]; o[3] = a[3];
        o[4] = b[0]; o[5] = b[1]; o[6] = b[2]; o[7] = b[3];
    }
};

// vmcnt(N) with the other counters left alone (gfx9 encoding of s_waitcnt's immediate)
template <int N>
__device__ __forceinline__ void wait_vmcnt()
{
    static_assert(N >= 0 && N < 64, "vmcnt has six bits");
    __builtin_amdgcn_s_waitcnt((N & 0xF) | ((N >> 4) << 14) | 0x0070 | 0x0F00);
}

// Tile `local` of a problem with nwg = tiles_m*tiles_n tiles -> its number in row-major order, or -1 for a padding
// slot.  Workgroups are dealt to the 8 XCDs in turn; XCD x gets a contiguous range of tiles (n fastest), so that a
// token panel is fetched into one L2 only.
__device__ __forceinline__ int logical_tile(int local, int nwg)
{
    const int xcd = local & 7, idx = local >> 3;
    const int q = nwg >> 3, r = nwg & 7;
    if (idx >= q + (xcd < r ? 1 : 0)) return -1;
    return xcd * q + (xcd < r ? xcd : r) + idx;
}

}  // namespace

// 128 x 256 tiles, two independent workgroups per CU (qgemm_i8_list.hip).  A single call; and at most QB_MAX_BATCH linears (checked) of any
// widths in one launch.
template <int BITS>
void launch_fwd_general(const int8_t *Xq, const int32_t *rs_x, const uint8_t *packed, const float *h, const int32_t *rs_w, const float *bias, float *Y,
                    int32_t *A4, int T, int N, int K, int rpg, float hx, hipStream_t st, const float *hx_rows, const float *q0);
void launch_fwd_list(const qb_fwd_job *jobs, int n_jobs, hipStream_t st);
}  // namespace qb
