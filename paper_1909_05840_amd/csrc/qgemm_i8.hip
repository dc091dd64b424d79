// Forward of the group-quantized linear layer on the gfx950 int8 matrix cores.
//
//   acc[t,n] = sum_j x'[t,j] * b[n,j]       v_mfma_i32_32x32x32_i8, int32 accumulators
//   A4[t,n]  = 4*acc + 2*e*rs_x[t] + 2*rs_w[n] + K
//   Y[t,n]   = (h_x*h_g(n)) * float(A4) (+ bias[n])
//
// b is the int8 the matrix core sees: the unsigned code u itself for 2/3/4 bits (e = -L) and
// u - 128 for 8 bits (e = +1); either way A4 equals sum_j (2x'+1)(2u-L), the integer that the
// integer product of the codes, de-quantized once afterwards (App., last paragraph), has to produce.
//
// Six kernels, chosen by shape (launch_bits; for a batched call list_pays):
//   qgemm_i8_kernel     register-staged: the token tile goes global -> registers -> LDS, the packed weights never
//                       touch LDS (the packed layout stores, per 32-neuron block and 64-feature unit, one slot per
//                       lane, so a wavefront fetches its B operand with one coalesced load).  Small tiles for
//                       problems of few tiles, and any K that is a multiple of 64.
//   qgemm_i8_dma_kernel both operands copied global -> LDS by the load unit itself (global_load_lds_dwordx4, no
//                       registers involved) through a ring of stages; every wavefront copies and multiplies; two
//                       workgroups per CU.
//   qgemm_i8_ws_kernel  the same data path with the work split by role (copy wavefronts / MFMA wavefronts), a
//                       persistent grid that walks the tiles of one or several problems (a table of problems is the
//                       kernel argument), epilogue parameters staged in LDS; optionally with the copy wavefronts on
//                       a SIMD of their own (128x96 tiles; two workgroups per CU when there are more tiles than CUs:
//                       one's write-out runs under the other's K-loop), an 8-bit output, per-token scales,
//                       asymmetric group ranges.
//   qgemm_i8_split_kernel the smallest problems: the contraction sliced inside the workgroup, no LDS in the loop.
//   qgemm_i8_duo_kernel the largest problems: 128x256 tiles on the 16x16x64 MFMA, two independent
//                       workgroups per CU that multiply and write out in turn.
//   qgemm_i8_list_kernel (qgemm_i8_list.hip) the same tiles and wavefronts for batched calls, all linears and widths in one
//                       launch; also large single calls with K no multiple of 128, per-token scales or asymmetric ranges.
// In all of them but the split kernel, whose operands go straight to registers, the token tile sits in LDS as dense
// 128-byte rows whose 16-byte chunks are XOR-swizzled by the row number, so that the MFMA fragment reads are free of bank
// conflicts; and in all of them the k-bit codes are expanded to int8 with a few byte-parallel shifts and masks in registers,
// right in front of the MFMA that consumes them.
// Workgroups are renumbered so that the ones sharing a token panel run on the same XCD (same L2).
#include "qgemm_i8.hpp"

namespace qb {
namespace {

// bytes of one of the two token tiles of the body below
constexpr int stepped_lds(int BM, int KU) { return BM * (64 * KU + 16); }

// bid: the workgroup's number among the tiles_m * tiles_n workgroups of this problem
// GEN: per-token scales or asymmetric group ranges (a variant of its own, so that the plain call carries none of its code)
template <int BITS, int TM, int TN, int WM, int WN, int KU, bool GEN>
__device__ __forceinline__ void qgemm_i8_body(
    const int8_t *__restrict__ Xq, const int32_t *__restrict__ rs_x, const uint8_t *__restrict__ packed,
    const float *__restrict__ h, const int32_t *__restrict__ rs_w, const float *__restrict__ bias,
    float *__restrict__ Y, int32_t *__restrict__ A4out, int T, int N, int K, int rows_per_group, float hx,
    int tiles_m, int tiles_n, const float *__restrict__ hx_rows, const float *__restrict__ q0, const int bid, uint8_t *lds)
{
    // lds: 2 * stepped_lds(BM, KU) bytes
    // hx_rows: one activation scale per token (dynamic range) instead of hx, or null
    // q0: asymmetric group ranges: h holds Delta and q0 the lower end of every group, or null
    constexpr int THREADS = 64 * WM * WN;
    constexpr int BM = WM * TM * 32, BN = WN * TN * 32, BK = 64 * KU, LDA = BK + 16;
    constexpr int CHUNKS_PER_ROW = BK / 16;
    constexpr int A_PER_THREAD = BM * CHUNKS_PER_ROW / THREADS;
    static_assert(BM * CHUNKS_PER_ROW % THREADS == 0, "A tile must split evenly over the threads");
    constexpr int SLOT = 4 * BITS;  // bytes per slot

    // ---- which tile: blocks are dealt round-robin to the 8 XCDs; give each XCD a contiguous
    // range of tiles (n fastest) so that a token panel is fetched into one L2 only
    const int nwg = tiles_m * tiles_n;
    int logical;
    {
        const int xcd = bid & 7, idx = bid >> 3;
        const int q = nwg >> 3, r = nwg & 7;
        logical = xcd * q + (xcd < r ? xcd : r) + idx;
    }
    const int tile_m = logical / tiles_n, tile_n = logical - tile_m * tiles_n;

    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int wm = wave / WN, wn = wave - wm * WN;
    const int l32 = lane & 31, hf = lane >> 5;

    // ---- global sources
    const int8_t *a_src[A_PER_THREAD];
    int a_dst[A_PER_THREAD];
#pragma unroll
    for (int i = 0; i < A_PER_THREAD; ++i) {
        const int c = tid + i * THREADS;
        const int row = c / CHUNKS_PER_ROW, kc = c - row * CHUNKS_PER_ROW;
        int t = tile_m * BM + row;
        t = t < T ? t : T - 1;  // rows past the end re-read the last row; their outputs are masked
        a_src[i] = Xq + (size_t)t * K + kc * 16;
        a_dst[i] = row * LDA + kc * 16;
    }
    const int kunits = K >> 6;
    const int ncb = (N + 31) >> 5;
    const uint8_t *b_src[TN];
#pragma unroll
    for (int tn = 0; tn < TN; ++tn) {
        int cb = tile_n * (BN / 32) + wn * TN + tn;
        cb = cb < ncb ? cb : ncb - 1;
        b_src[tn] = packed + ((size_t)cb * kunits * 64 + lane) * SLOT;
    }

    v16i acc[TM][TN];
#pragma unroll
    for (int tm = 0; tm < TM; ++tm)
#pragma unroll
        for (int tn = 0; tn < TN; ++tn)
#pragma unroll
            for (int i = 0; i < 16; ++i) acc[tm][tn][i] = 0;

    const int a_frag_base = (wm * TM * 32 + l32) * LDA + hf * 32;
    // Steps of one unit of 64 features (K no multiple of 128): what bounds them is the way from a step's loads over LDS to its two
    // MFMAs, so a step's tokens are staged right in front of the barrier that its MFMAs follow, the codes are expanded before it and
    // D steps are on their way.  us of the GEMM behind its quantizer, before -> now, 4 bits: 2300 x 448 x 448 5.3 -> 4.8, 1001 x 1344 x 448
    // 5.1 -> 4.6; as 128 x 128 tiles 12000 x 1344 x 448 23.5 -> 22.0.  D = 2 / 1: 4.7 / 5.2, at 3 bits 5.8 / 5.2; four blocks a wavefront
    // fill a step with one (22.0 / 22.3).  Wider steps are better off in the loop further below: in this one 256 features take 2 to 5 %
    // more, 128 features 4 % less at K = 768 and 2 % more up to K = 640, where the longer code counts.
    constexpr bool AHEAD_STEPS = KU == 1;
    constexpr int D = TM * TN == 1 && BITS != 3 ? 2 : 1;
    v4u areg[D][A_PER_THREAD];
    uint32_t breg[D][TN][KU][BITS];
    // global -> registers for K-step `step`: the token tile (to be staged in LDS) and this lane's slots
    auto load_step = [&](int step, v4u (&ar)[A_PER_THREAD], uint32_t (&br)[TN][KU][BITS]) {
#pragma unroll
        for (int i = 0; i < A_PER_THREAD; ++i) ar[i] = *reinterpret_cast<const v4u *>(a_src[i] + (size_t)step * BK);
#pragma unroll
        for (int tn = 0; tn < TN; ++tn)
#pragma unroll
            for (int kk = 0; kk < KU; ++kk) {
                const uint32_t *p = reinterpret_cast<const uint32_t *>(b_src[tn] + (size_t)(step * KU + kk) * 64 * SLOT);
#pragma unroll
                for (int i = 0; i < BITS; ++i) br[tn][kk][i] = p[i];
            }
    };
    // one K-step: the token tile to LDS, this lane's codes expanded to int8; then the loads of step `next` into the registers
    // that are free now (fetch), and the MFMAs with the token fragments from LDS
    auto do_step = [&](int buf, v4u (&ar)[A_PER_THREAD], uint32_t (&br)[TN][KU][BITS], bool fetch, int next) {
        uint8_t *abuf = lds + buf * (BM * LDA);
#pragma unroll
        for (int i = 0; i < A_PER_THREAD; ++i) *reinterpret_cast<v4u *>(abuf + a_dst[i]) = ar[i];
        uint32_t d[TN][KU][8];
#pragma unroll
        for (int tn = 0; tn < TN; ++tn)
#pragma unroll
            for (int kk = 0; kk < KU; ++kk) {
                unpack_run<BITS>(br[tn][kk], d[tn][kk]);
                if constexpr (BITS == 8) {
#pragma unroll
                    for (int i = 0; i < 8; ++i) d[tn][kk][i] ^= 0x80808080u;
                }
            }
        __builtin_amdgcn_sched_barrier(0);
        if (fetch) load_step(next, ar, br);
        // the tile is in LDS (loads stay on their way over the barrier)
        __builtin_amdgcn_sched_barrier(0);
        __builtin_amdgcn_s_waitcnt(0xC07F);  // lgkmcnt(0)
        asm volatile("" ::: "memory");
        __builtin_amdgcn_s_barrier();
        asm volatile("" ::: "memory");
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int kk = 0; kk < KU; ++kk)
#pragma unroll
            for (int sub = 0; sub < 2; ++sub) {
                v4i a[TM], b[TN];
#pragma unroll
                for (int tm = 0; tm < TM; ++tm) a[tm] = *reinterpret_cast<const v4i *>(abuf + a_frag_base + tm * 32 * LDA + kk * 64 + sub * 16);
#pragma unroll
                for (int tn = 0; tn < TN; ++tn)
#pragma unroll
                    for (int i = 0; i < 4; ++i) b[tn][i] = (int)d[tn][kk][4 * sub + i];
#pragma unroll
                for (int tm = 0; tm < TM; ++tm)
#pragma unroll
                    for (int tn = 0; tn < TN; ++tn) acc[tm][tn] = __builtin_amdgcn_mfma_i32_32x32x32_i8(a[tm], b[tn], acc[tm][tn], 0, 0, 0);
            }
    };

    v4u astage[A_PER_THREAD];
    uint32_t bnext[TN][KU][BITS], bcur[TN][KU][BITS];

// global -> registers for K-step `step`: the token tile (to be staged in LDS) and this lane's slots
#define QB_LOAD_GLOBAL(step, BDST)                                                                        \
    {                                                                                                     \
        _Pragma("unroll") for (int i = 0; i < A_PER_THREAD; ++i)                                          \
            astage[i] = *reinterpret_cast<const v4u *>(a_src[i] + (size_t)(step) * BK);                  \
        _Pragma("unroll") for (int tn = 0; tn < TN; ++tn)                                                 \
            _Pragma("unroll") for (int kk = 0; kk < KU; ++kk) {                                           \
                const uint32_t *p_ =                                                                      \
                    reinterpret_cast<const uint32_t *>(b_src[tn] + (size_t)((step) * KU + kk) * 64 * SLOT); \
                _Pragma("unroll") for (int i = 0; i < BITS; ++i) BDST[tn][kk][i] = p_[i];                 \
            }                                                                                             \
    }
#define QB_STORE_LDS(buf)                                                                                 \
    {                                                                                                     \
        _Pragma("unroll") for (int i = 0; i < A_PER_THREAD; ++i)                                          \
            *reinterpret_cast<v4u *>(lds + (buf) * (BM * LDA) + a_dst[i]) = astage[i];                                    \
    }
// all MFMAs of one K-step: expand this lane's codes to int8 in registers, A fragments from LDS
#define QB_COMPUTE(buf)                                                                                   \
    {                                                                                                     \
        const uint8_t *abuf = lds + (buf) * (BM * LDA);                                                   \
        _Pragma("unroll") for (int kk = 0; kk < KU; ++kk) {                                               \
            uint32_t d[TN][8];                                                                            \
            _Pragma("unroll") for (int tn = 0; tn < TN; ++tn) {                                           \
                unpack_run<BITS>(bcur[tn][kk], d[tn]);                                                    \
                if constexpr (BITS == 8) {                                                                \
                    _Pragma("unroll") for (int i = 0; i < 8; ++i) d[tn][i] ^= 0x80808080u;                \
                }                                                                                         \
            }                                                                                             \
            _Pragma("unroll") for (int sub = 0; sub < 2; ++sub) {                                         \
                v4i a[TM], b[TN];                                                                         \
                _Pragma("unroll") for (int tm = 0; tm < TM; ++tm) a[tm] = *reinterpret_cast<const v4i *>( \
                    abuf + a_frag_base + tm * 32 * LDA + kk * 64 + sub * 16);                             \
                _Pragma("unroll") for (int tn = 0; tn < TN; ++tn) {                                       \
                    b[tn][0] = (int)d[tn][4 * sub + 0];                                                   \
                    b[tn][1] = (int)d[tn][4 * sub + 1];                                                   \
                    b[tn][2] = (int)d[tn][4 * sub + 2];                                                   \
                    b[tn][3] = (int)d[tn][4 * sub + 3];                                                   \
                }                                                                                         \
                _Pragma("unroll") for (int tm = 0; tm < TM; ++tm)                                         \
                    _Pragma("unroll") for (int tn = 0; tn < TN; ++tn) acc[tm][tn] =                       \
                        __builtin_amdgcn_mfma_i32_32x32x32_i8(a[tm], b[tn], acc[tm][tn], 0, 0, 0);        \
            }                                                                                             \
        }                                                                                                 \
    }
#define QB_ROTATE_B()                                                                                     \
    {                                                                                                     \
        _Pragma("unroll") for (int tn = 0; tn < TN; ++tn)                                                 \
            _Pragma("unroll") for (int kk = 0; kk < KU; ++kk)                                             \
                _Pragma("unroll") for (int i = 0; i < BITS; ++i) bcur[tn][kk][i] = bnext[tn][kk][i];      \
    }

    // The epilogue's parameters.  None is loaded between the stores of 32 rows: the load would wait for every store before it (256 x 2304 x
    // 768 with per-token scales and asymmetric ranges 6.7 -> 4.7 us; with the plain scale ragged tiles alone did so, 1499 x 768 x
    // 768 5.8 -> 4.6, tiles of 128 x 128, 3001 x 1344 x 448 18.7 -> 11.6).  Tiles of one block a wavefront have them on their
    // way during the K-loop, if there are registers for them (256 x 2304 x 768 4.45 -> 4.28).
    constexpr bool AHEAD = TM * TN == 1 && KU < 4;
    constexpr int L = (1 << BITS) - 1;
    constexpr int E2 = (BITS == 8) ? 2 : -2 * L;  // 2*e
    int coln[TN], rx[16];
    float hg[TN], zn[TN], bv[TN], hr[16];
    auto load_columns = [&]() {
#pragma unroll
        for (int tn = 0; tn < TN; ++tn) {
            const int n = tile_n * BN + (wn * TN + tn) * 32 + l32, nn = n < N ? n : N - 1;
            coln[tn] = 2 * rs_w[nn] + K;
            hg[tn] = h[nn / rows_per_group];
            zn[tn] = GEN && q0 ? q0[nn / rows_per_group] : 0.0f;
            bv[tn] = bias ? bias[nn] : 0.0f;
        }
    };
    auto load_rows = [&](int tm) {
#pragma unroll
        for (int i = 0; i < 16; ++i) {
            int t = tile_m * BM + (wm * TM + tm) * 32 + 4 * hf + 8 * (i >> 2) + (i & 3);
            t = t < T ? t : T - 1;
            const uint32_t off = (uint32_t)t * 4u;  // (T <= 2^24)
            rx[i] = *reinterpret_cast<const int32_t *>(reinterpret_cast<const char *>(rs_x) + off);
            if constexpr (GEN) hr[i] = hx_rows ? *reinterpret_cast<const float *>(reinterpret_cast<const char *>(hx_rows) + off) : hx;
        }
    };

    const int nsteps = K / BK;
    if constexpr (AHEAD_STEPS) {
        load_step(0, areg[0], breg[0]);
        if constexpr (AHEAD) {
            load_columns();
            load_rows(0);
        }
#pragma unroll
        for (int i = 1; i < D; ++i) load_step(i < nsteps ? i : 0, areg[i], breg[i]);
        int s = 0;
        if constexpr (D % 2 == 0) {
            for (; s + 2 * D <= nsteps; s += D)  // (no branches inside)
#pragma unroll
                for (int i = 0; i < D; ++i) do_step(i & 1, areg[i], breg[i], true, s + i + D);
        } else {
            for (; s + 3 * D <= nsteps; s += 2 * D)
#pragma unroll
                for (int i = 0; i < 2 * D; ++i) do_step(i & 1, areg[i % D], breg[i % D], true, s + i + D);
        }
        // the last steps, less than 2*D or 3*D
#pragma unroll
        for (int i = 0; i < (D % 2 == 0 ? 2 * D : 3 * D) - 1; ++i)
            if (s + i < nsteps) do_step(i & 1, areg[i % D], breg[i % D], s + i + D < nsteps, s + i + D);
    } else {
        QB_LOAD_GLOBAL(0, bcur)
        if constexpr (AHEAD) {
            load_columns();
            load_rows(0);
        }
        QB_STORE_LDS(0)
        __syncthreads();
        // steady state: fetch step s+1 while the matrix cores work on step s (no branches inside)
        for (int s = 0; s < nsteps - 1; ++s) {
            QB_LOAD_GLOBAL(s + 1, bnext)
            __builtin_amdgcn_sched_barrier(0);  // keep the fetches ahead of the MFMAs: their latency hides under them
            QB_COMPUTE(s & 1)
            __builtin_amdgcn_sched_barrier(0);
            QB_STORE_LDS((s + 1) & 1)
            QB_ROTATE_B()
            __syncthreads();
        }
        QB_COMPUTE((nsteps - 1) & 1)
    }
#undef QB_LOAD_GLOBAL
#undef QB_STORE_LDS
#undef QB_COMPUTE
#undef QB_ROTATE_B

    // ---- epilogue: exact integer corrections, then one scale per column (or per column and token)
    const bool interior = (tile_m + 1) * BM <= T && (tile_n + 1) * BN <= N;  // uniform over the workgroup
    if constexpr (!AHEAD) load_columns();
#pragma unroll
    for (int tm = 0; tm < TM; ++tm) {
        if constexpr (!AHEAD) {
            asm volatile("" ::: "memory");  // (32 rows' parameters at a time, behind the stores of the 32 before: there are no registers for more)
            load_rows(tm);
        }
        const int left = T - (tile_m * BM + (wm * TM + tm) * 32 + 4 * hf);
#pragma unroll
        for (int tn = 0; tn < TN; ++tn) {
            const bool n_ok = tile_n * BN + (wn * TN + tn) * 32 + l32 < N;
            // a wavefront-uniform row address and the lane's 32-bit byte offset
            const size_t block = (size_t)(tile_m * BM + (wm * TM + tm) * 32) * N + tile_n * BN + (wn * TN + tn) * 32;
            const uint32_t lane_off = (uint32_t)(4 * hf * N + l32) * 4u;
            auto a4_of = [&](int i) { return qb_a4(acc[tm][tn][i], qb_mad24(E2, rx[i], coln[tn])); };  // |rs_x| <= 128*K < 2^23
            auto asym = [&](int i, int a4) { return asym_value(a4, rx[i] + (K >> 1), L, hr[i], hg[tn], zn[tn]) + bv[tn]; };
            auto plain = [&](int i, int a4) { return ((GEN ? hr[i] : hx) * hg[tn]) * (float)a4 + bv[tn]; };
            auto row_of = [](int i) { return 8 * (i >> 2) + (i & 3); };
            auto put = [&](int i, float y) { *reinterpret_cast<float *>(reinterpret_cast<char *>(Y + block + (size_t)row_of(i) * N) + lane_off) = y; };
            // (straight-line code where it can be: a check per value costs 0.8 us of 4.4)
            if (interior && A4out == nullptr) {
                if (GEN && q0) {
#pragma unroll
                    for (int i = 0; i < 16; ++i) put(i, asym(i, a4_of(i)));
                } else {
#pragma unroll
                    for (int i = 0; i < 16; ++i) put(i, plain(i, a4_of(i)));
                }
            } else if (n_ok) {
#pragma unroll
                for (int i = 0; i < 16; ++i)
                    if (row_of(i) < left) {
                        const int a4 = a4_of(i);
                        put(i, GEN && q0 ? asym(i, a4) : plain(i, a4));
                        if (A4out) *reinterpret_cast<int32_t *>(reinterpret_cast<char *>(A4out + block + (size_t)row_of(i) * N) + lane_off) = a4;
                    }
            }
        }
    }
}

// (at least four wavefronts a SIMD, or three: the accumulators then lie in ordinary registers, 1 to 4 % of a small call)
template <int BITS, int TM, int TN, int WM, int WN, int KU, bool GEN>
__global__ __launch_bounds__(64 * WM * WN, TM * TN > 1 ? 3 : KU == 4 ? 1 : 4) void qgemm_i8_kernel(
    const int8_t *__restrict__ Xq, const int32_t *__restrict__ rs_x, const uint8_t *__restrict__ packed,
    const float *__restrict__ h, const int32_t *__restrict__ rs_w, const float *__restrict__ bias,
    float *__restrict__ Y, int32_t *__restrict__ A4out, int T, int N, int K, int rows_per_group, float hx,
    int tiles_m, int tiles_n, const float *__restrict__ hx_rows, const float *__restrict__ q0)
{
    __shared__ __align__(16) uint8_t lds[2 * stepped_lds(WM * TM * 32, KU)];
    qgemm_i8_body<BITS, TM, TN, WM, WN, KU, GEN>(Xq, rs_x, packed, h, rs_w, bias, Y, A4out, T, N, K, rows_per_group, hx, tiles_m,
                                            tiles_n, hx_rows, q0, blockIdx.x, lds);
}

// The few tiles of a small token count: 32 x 64 tiles, the contraction cut into eight slices inside the workgroup.
// What bounds these calls is latency: a K-loop that walks the features step by step pays a memory latency per step,
// while the operands' bytes take a fraction of one.  So each of the eight wavefronts takes one slice of the features, loads
// its operands straight into registers in the layout of the MFMA (no LDS and no barrier in the loop), and the slices' integer
// sums meet in LDS; the write-out is split over the wavefronts as well.  Integer sums: the order does not matter, the
// results are the ones of the other kernels bit for bit.  The direct loads touch 32 rows per instruction, so that with
// more workgroups than CUs the kernel above is ahead again, as it is with contractions of a few steps (see split_shape).
constexpr int kSlices = 8, kSlicedLds = kSlices * 2 * 4 * 64;  // int4 of LDS
struct SmallProblem {
    const int8_t *Xq;
    const int32_t *rs_x;
    const uint8_t *packed;
    const float *h;
    const int32_t *rs_w;
    const float *bias;
    float *Y;
    int T, N, K, rows_per_group;
    float hx;
    int tiles_m, tiles_n;
    int kind;  // of a list: bits | units of 64 features per step << 8
};

// A4out: the debug output, or null; hx_rows: one activation scale per token (dynamic range) instead of hx, or null; q0: asymmetric
// group ranges (h holds Delta and q0 the lower end of every group), or null
template <int BITS>
__device__ __forceinline__ void qgemm_i8_split_body(const SmallProblem &p, int32_t *__restrict__ A4out, const float *__restrict__ hx_rows,
                                                    const float *__restrict__ q0, const int bid, int4 *red)
{
    constexpr int KS = kSlices, SLOT = 4 * BITS, U = 2;  // units in flight, besides as many being multiplied
    const int T = p.T, N = p.N, K = p.K;
    const int nwg = p.tiles_m * p.tiles_n;
    int logical;  // each XCD a contiguous range of tiles, n fastest
    {
        const int xcd = bid & 7, idx = bid >> 3;
        const int q = nwg >> 3, r = nwg & 7;
        logical = xcd * q + (xcd < r ? xcd : r) + idx;
    }
    const int tile_m = logical / p.tiles_n, tile_n = logical - tile_m * p.tiles_n;
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);  // slice of the contraction
    const int l32 = lane & 31, hf = lane >> 5;

    const int units = K >> 6, ncb = (N + 31) >> 5;
    const int u0 = units * wave / KS, u1 = units * (wave + 1) / KS;
    int t = tile_m * 32 + l32;
    t = t < T ? t : T - 1;  // rows past the end re-read the last one; their outputs are masked
    const int8_t *a_src = p.Xq + (size_t)t * K + hf * 32;
    const uint8_t *b_src[2];
#pragma unroll
    for (int j = 0; j < 2; ++j) {
        int cb = tile_n * 2 + j;
        cb = cb < ncb ? cb : ncb - 1;
        b_src[j] = p.packed + ((size_t)cb * units * 64 + lane) * SLOT;
    }

    v16i acc[2];
#pragma unroll
    for (int j = 0; j < 2; ++j)
#pragma unroll
        for (int i = 0; i < 16; ++i) acc[j][i] = 0;
    v4i a[2][U][2];
    uint32_t b[2][U][2][BITS];
    auto load = [&](int u, int set) {
#pragma unroll
        for (int i = 0; i < U; ++i) {
            int v = u + i;
            v = v < units ? v : units - 1;  // (a unit behind the slice is loaded and not used)
            const v4i *as = reinterpret_cast<const v4i *>(a_src + (size_t)v * 64);
            a[set][i][0] = as[0];
            a[set][i][1] = as[1];
#pragma unroll
            for (int j = 0; j < 2; ++j) {
                const uint32_t *bs = reinterpret_cast<const uint32_t *>(b_src[j] + (size_t)v * 64 * SLOT);
#pragma unroll
                for (int e = 0; e < BITS; ++e) b[set][i][j][e] = bs[e];
            }
        }
    };
    auto mma = [&](int u, int set) {
#pragma unroll
        for (int i = 0; i < U; ++i) {
            if (u + i >= u1) break;  // (uniform)
#pragma unroll
            for (int j = 0; j < 2; ++j) {
                uint32_t d[8];
                unpack_run<BITS>(b[set][i][j], d);
                if constexpr (BITS == 8) {
#pragma unroll
                    for (int e = 0; e < 8; ++e) d[e] ^= 0x80808080u;
                }
#pragma unroll
                for (int sub = 0; sub < 2; ++sub) {
                    const v4i bb = {(int)d[4 * sub], (int)d[4 * sub + 1], (int)d[4 * sub + 2], (int)d[4 * sub + 3]};
                    acc[j] = __builtin_amdgcn_mfma_i32_32x32x32_i8(a[set][i][sub], bb, acc[j], 0, 0, 0);
                }
            }
        }
    };
    load(u0, 0);

    // the epilogue's parameters, on their way during the loop.  The wavefront writes quad wave/2 of every lane's sixteen
    // results of block wave%2 (result i is token 8*(i/4) + 4*hf + i%4 of the tile)
    constexpr int L = (1 << BITS) - 1;
    constexpr int E2 = (BITS == 8) ? 2 : -2 * L;  // 2*e
    const int wn = wave & 1, quad = wave >> 1, tl = tile_m * 32 + 8 * quad + 4 * hf;
    const int n = tile_n * 64 + wn * 32 + l32, nn = n < N ? n : N - 1;
    const int coln = 2 * p.rs_w[nn] + K;
    const float hg = p.h[nn / p.rows_per_group];
    const float zn = q0 ? q0[nn / p.rows_per_group] : 0.0f;
    const float bv = p.bias ? p.bias[nn] : 0.0f;
    int rx[4];
    float hr[4];
#pragma unroll
    for (int r = 0; r < 4; ++r) {
        const int tt = tl + r < T ? tl + r : T - 1;
        rx[r] = p.rs_x[tt];
        hr[r] = hx_rows ? hx_rows[tt] : p.hx;
    }

    for (int u = u0; u < u1; u += 2 * U) {
        if (u + U < u1) load(u + U, 1);
        mma(u, 0);
        if (u + 2 * U < u1) load(u + 2 * U, 0);
        mma(u + U, 1);
    }
#pragma unroll
    for (int j = 0; j < 2; ++j)
#pragma unroll
        for (int q = 0; q < 4; ++q)
            red[((wave * 2 + j) * 4 + q) * 64 + lane] = make_int4(acc[j][4 * q], acc[j][4 * q + 1], acc[j][4 * q + 2], acc[j][4 * q + 3]);
    __syncthreads();
    int4 sum = make_int4(0, 0, 0, 0);
#pragma unroll
    for (int s = 0; s < KS; ++s) {
        const int4 v = red[((s * 2 + wn) * 4 + quad) * 64 + lane];
        sum.x += v.x; sum.y += v.y; sum.z += v.z; sum.w += v.w;
    }
    if (n >= N) return;
    const int sums[4] = {sum.x, sum.y, sum.z, sum.w};
#pragma unroll
    for (int r = 0; r < 4; ++r) {
        const int tt = tl + r;
        if (tt >= T) break;
        const int a4 = qb_a4(sums[r], E2 * rx[r] + coln);
        const size_t at = (size_t)tt * N + n;
        if (q0) p.Y[at] = asym_value(a4, rx[r] + (K >> 1), L, hr[r], hg, zn) + bv;
        else p.Y[at] = (hr[r] * hg) * (float)a4 + bv;
        if (A4out) A4out[at] = a4;
    }
}

// One kernel argument: as four they cost 0.3 us of host time a call.  In this order the compiler loads all of it at the start; with
// the problem first it fetched the pointers behind it when they were needed, in front of the contraction.
struct SplitCall {
    int32_t *A4out;
    const float *hx_rows, *q0;
    SmallProblem p;
};
template <int BITS>
__global__ __launch_bounds__(512) void qgemm_i8_split_kernel(const SplitCall c)
{
    __shared__ __align__(16) int4 red[kSlicedLds];
    qgemm_i8_split_body<BITS>(c.p, c.A4out, c.hx_rows, c.q0, blockIdx.x, red);
}

// Several few-tile problems (small token counts: the inference regime, where a launch costs more than its work) in one
// launch: workgroup w serves tile w - first_wg[j] of problem j; a problem's workgroups start at
// a multiple of 8, so that its tiles keep their XCD (the fill-up workgroups leave at once).  (The list is a kernel argument
// of 1.5 KB; 24 bytes more per problem cost 0.2 us a launch.)
struct SmallGroup {
    int n;
    int first_wg[QB_MAX_BATCH + 1];
    SmallProblem p[QB_MAX_BATCH];
};
__device__ __forceinline__ int job_of(const SmallGroup &g)
{
    int j = 0;
    while (j + 1 < g.n && (int)blockIdx.x >= g.first_wg[j + 1]) ++j;
    return j;
}
// BITS, UNITS: the width and the units of 64 features per step of all jobs, or 0 where they differ.  A kernel for everything has the registers of its
// largest body (138: three wavefronts to a SIMD, where one width has 76 to 125) and learns late which body it takes.  Linears of 768 x 768 at 2 bits,
// us, it / the kernel of their width and step: 3 of 64 tokens 4.2 / 4.0, 12 of 385 tokens 10.4 / 8.6, 12 of 640 tokens 12.8 / 10.9; four layers of hidden
// 1024, 385 tokens, it / the kernel of their width 39.6 / 36.7.
template <int BITS, int UNITS>
__global__ __launch_bounds__(128, BITS ? 4 : 3) void qgemm_i8_small_list_kernel(const SmallGroup g)
{
    __shared__ __align__(16) uint8_t lds[2 * stepped_lds(32, UNITS ? UNITS : 4)];
    const int j = job_of(g);
    const SmallProblem &p = g.p[j];
    const int local = blockIdx.x - g.first_wg[j];
    if (local >= p.tiles_m * p.tiles_n) return;  // (uniform over the workgroup)
    auto run = [&](auto bits, auto units) {
        qgemm_i8_body<decltype(bits)::value, 1, 1, 1, 2, decltype(units)::value, false>(p.Xq, p.rs_x, p.packed, p.h, p.rs_w, p.bias, p.Y, nullptr, p.T, p.N, p.K,
                                                                                        p.rows_per_group, p.hx, p.tiles_m, p.tiles_n, nullptr, nullptr, local, lds);
    };
    auto of_width = [&](auto units) {
        if constexpr (BITS != 0) run(std::integral_constant<int, BITS>(), units);
        else switch (p.kind & 255) {
            case 2: run(std::integral_constant<int, 2>(), units); break;
            case 3: run(std::integral_constant<int, 3>(), units); break;
            case 4: run(std::integral_constant<int, 4>(), units); break;
            default: run(std::integral_constant<int, 8>(), units); break;
        }
    };
    if constexpr (UNITS != 0) of_width(std::integral_constant<int, UNITS>());
    else switch (p.kind >> 8) {
        case 1: of_width(std::integral_constant<int, 1>()); break;
        case 2: of_width(std::integral_constant<int, 2>()); break;
        default: of_width(std::integral_constant<int, 4>()); break;
    }
}
// BITS: the width of all jobs, or 0 where they differ (three linears of 768 x 768, 64 tokens, 4.2 us with 0, 4.0 with their width)
template <int BITS>
__global__ __launch_bounds__(512) void qgemm_i8_split_list_kernel(const SmallGroup g)
{
    __shared__ __align__(16) int4 red[kSlicedLds];
    const int j = job_of(g);
    const SmallProblem &p = g.p[j];
    const int local = blockIdx.x - g.first_wg[j];
    if (local >= p.tiles_m * p.tiles_n) return;  // (uniform over the workgroup)
    if constexpr (BITS != 0) qgemm_i8_split_body<BITS>(p, nullptr, nullptr, nullptr, local, red);
    else switch (p.kind & 255) {
        case 2: qgemm_i8_split_body<2>(p, nullptr, nullptr, nullptr, local, red); break;
        case 3: qgemm_i8_split_body<3>(p, nullptr, nullptr, nullptr, local, red); break;
        case 4: qgemm_i8_split_body<4>(p, nullptr, nullptr, nullptr, local, red); break;
        default: qgemm_i8_split_body<8>(p, nullptr, nullptr, nullptr, local, red); break;
    }
}

// Main kernel, K a multiple of 128.  One K-step is 128 features = two 64-code units.
// Both operands are copied global -> LDS by the load unit (no staging registers):
//   tokens : dense rows of 128 bytes, 16-byte chunks XOR-swizzled with the row number
//   weights: the packed slots as they are, [32-neuron block][unit][lane][slot]; a wavefront
//            then reads one slot per lane (conflict free) and expands it in registers
// The copies run NSTAGE-1 steps ahead of the matrix cores through a ring of NSTAGE stage
// buffers; a step ends with "the copies for the next step have landed" (vmcnt leaves the younger
// ones in flight; copies return in issue order) and a workgroup barrier.
template <int BITS, int TM, int TN, int WM, int WN, int NSTAGE>
__global__ __launch_bounds__(64 * WM * WN) void qgemm_i8_dma_kernel(
    const int8_t *__restrict__ Xq, const int32_t *__restrict__ rs_x, const uint8_t *__restrict__ packed,
    const float *__restrict__ h, const int32_t *__restrict__ rs_w, const float *__restrict__ bias,
    float *__restrict__ Y, int32_t *__restrict__ A4out, int T, int N, int K, int rows_per_group, float hx,
    int tiles_m, int tiles_n)
{
    static_assert(NSTAGE >= 2 && NSTAGE <= 4, "ring of 2..4 stages");
    constexpr int NW = WM * WN;
    constexpr int BM = WM * TM * 32, BN = WN * TN * 32, BK = 128;
    constexpr int A_DMA = BM / 8 / NW;          // per wavefront and step; each fills 8 rows of 128 bytes
    static_assert(BM % (8 * NW) == 0, "token tile must split into 8-row blocks per wavefront");
    constexpr int SLOT = 4 * BITS;               // bytes per slot in memory
    constexpr int CH = (BITS == 3) ? 12 : 16;    // bytes one lane moves per weight copy instruction
    constexpr int LSLOT = (BITS == 3) ? 16 : SLOT;  // bytes per slot in LDS: a 12-byte copy lands at a 16-byte stride
    constexpr int PAIR = 128 * SLOT;             // bytes of one 32-neuron block x two units (contiguous in memory)
    constexpr int LPAIR = 128 * LSLOT;           // the same block in LDS
    constexpr int PARTS = PAIR / (64 * CH);      // copy instructions per pair; each fills 1024 bytes of LDS
    constexpr int B_TOTAL = (BN / 32) * PARTS;   // copy instructions per step for the whole workgroup
    constexpr int B_DMA = (B_TOTAL + NW - 1) / NW;
    constexpr int PER = A_DMA + B_DMA;           // copy instructions per wavefront and step
    constexpr int D = NSTAGE - 1;                // how many steps the copies run ahead
    constexpr int A_BYTES = BM * BK, B_BYTES = (BN / 32) * LPAIR;

    constexpr int STAGE_BYTES = A_BYTES + B_BYTES;  // tokens first, then weights
    __shared__ __align__(1024) uint8_t lds[NSTAGE * STAGE_BYTES];
    const uint32_t lds_base = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) uint8_t *)lds;

    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int wm = wave / WN, wn = wave - wm * WN;
    const int l32 = lane & 31, hf = lane >> 5;

    // Workgroups are persistent: each walks over tiles work = blockIdx.x, + gridDim.x, ... (the
    // grid is a multiple of 8, so a workgroup stays on the tiles of its own XCD's range).
    const int nwg = tiles_m * tiles_n;
    for (int work = blockIdx.x; work < nwg; work += gridDim.x) {
    int logical;
    {
        const int xcd = work & 7, idx = work >> 3;
        const int q = nwg >> 3, r = nwg & 7;
        logical = xcd * q + (xcd < r ? xcd : r) + idx;
    }
    const int tile_m = logical / tiles_n, tile_n = logical - tile_m * tiles_n;

    // ---- token tile copies: lane l of an instruction fills physical chunk l%8 of row l/8 of an
    // 8-row block, which holds logical chunk (l%8) ^ (row%8)
    const int8_t *a_base = Xq + (size_t)tile_m * BM * K;
    const int last_row = T - 1 - tile_m * BM;  // rows past the end re-read the last one; outputs masked
    uint32_t a_off[A_DMA];
#pragma unroll
    for (int i = 0; i < A_DMA; ++i) {
        int row = (i * NW + wave) * 8 + (lane >> 3);
        row = row < last_row ? row : last_row;
        a_off[i] = (uint32_t)row * (uint32_t)K + (uint32_t)(((lane & 7) ^ (lane >> 3)) * 16);
    }
    // ---- weight copies: instruction j moves part j%PARTS of the pair of block j/PARTS.  Every
    // wavefront issues the same number of copies (the vmcnt arithmetic relies on it): surplus
    // ones repeat an earlier copy, writing the same bytes to the same place.
    const int kunits = K >> 6;
    const int ncb = (N + 31) >> 5;
    // (addresses: a wavefront-uniform base per tile and step, a 32-bit byte offset per lane and copy)
    const int cb0 = tile_n * (BN / 32);
    const uint8_t *b_base = packed + (size_t)cb0 * kunits * 64 * SLOT;
    uint32_t b_off[B_DMA];
    int b_ldst[B_DMA];
#pragma unroll
    for (int i = 0; i < B_DMA; ++i) {
        const int j = (i * NW + wave) % B_TOTAL;
        const int pair = j / PARTS, part = j - pair * PARTS;
        int cb = cb0 + pair;
        cb = cb < ncb ? cb : ncb - 1;  // blocks past the end re-read the last one; outputs masked
        b_off[i] = (uint32_t)(cb - cb0) * (uint32_t)(kunits * 64 * SLOT) + part * 64 * CH + lane * CH;
        b_ldst[i] = pair * LPAIR + part * 1024;
    }
    // ---- fragment reads.  tokens: row = wm*TM*32 + tm*32 + l32, logical chunk = kk*4 + hf*2 + sub
    const int p0 = (hf * 2) ^ (l32 & 7);
    const int frag_row = (wm * TM * 32 + l32) * BK;
    int a_frag[4];
    a_frag[0] = frag_row + ((p0 ^ 0) << 4);  // kk 0, sub 0
    a_frag[1] = frag_row + ((p0 ^ 1) << 4);  // kk 0, sub 1
    a_frag[2] = frag_row + ((p0 ^ 4) << 4);  // kk 1, sub 0
    a_frag[3] = frag_row + ((p0 ^ 5) << 4);  // kk 1, sub 1
    const int b_frag = wn * TN * LPAIR + lane * LSLOT;  // + tn*LPAIR + kk*64*LSLOT

    v16i acc[TM][TN];
#pragma unroll
    for (int tm = 0; tm < TM; ++tm)
#pragma unroll
        for (int tn = 0; tn < TN; ++tn)
#pragma unroll
            for (int i = 0; i < 16; ++i) acc[tm][tn][i] = 0;

#define QB_FETCH(step, stage)                                                                             \
    {                                                                                                     \
        const uint32_t st_ = lds_base + (stage) * STAGE_BYTES;                                            \
        _Pragma("unroll") for (int i = 0; i < B_DMA; ++i)                                                 \
            copy_to_lds<CH>(b_base + (size_t)(step) * PAIR, b_off[i], st_ + A_BYTES + b_ldst[i]);         \
        _Pragma("unroll") for (int i = 0; i < A_DMA; ++i)                                                 \
            copy_to_lds<16>(a_base + (size_t)(step) * BK, a_off[i], st_ + (i * NW + wave) * 1024);        \
    }
#define QB_MMA(stage)                                                                                     \
    {                                                                                                     \
        const uint8_t *lds_a = lds + (stage) * STAGE_BYTES, *lds_b = lds_a + A_BYTES;                     \
        _Pragma("unroll") for (int kk = 0; kk < 2; ++kk) {                                                \
            uint32_t d[TN][8];                                                                            \
            _Pragma("unroll") for (int tn = 0; tn < TN; ++tn) {                                           \
                uint32_t raw[BITS];                                                                       \
                SlotRead<BITS>::get(lds_b + b_frag + tn * LPAIR + kk * 64 * LSLOT, raw);                  \
                unpack_run<BITS>(raw, d[tn]);                                                             \
                if constexpr (BITS == 8) {                                                                \
                    _Pragma("unroll") for (int i = 0; i < 8; ++i) d[tn][i] ^= 0x80808080u;                \
                }                                                                                         \
            }                                                                                             \
            _Pragma("unroll") for (int sub = 0; sub < 2; ++sub) {                                         \
                v4i a[TM], b[TN];                                                                         \
                _Pragma("unroll") for (int tm = 0; tm < TM; ++tm)                                         \
                    a[tm] = *reinterpret_cast<const v4i *>(lds_a + a_frag[kk * 2 + sub] + tm * 32 * BK);  \
                _Pragma("unroll") for (int tn = 0; tn < TN; ++tn) {                                       \
                    b[tn][0] = (int)d[tn][4 * sub + 0];                                                   \
                    b[tn][1] = (int)d[tn][4 * sub + 1];                                                   \
                    b[tn][2] = (int)d[tn][4 * sub + 2];                                                   \
                    b[tn][3] = (int)d[tn][4 * sub + 3];                                                   \
                }                                                                                         \
                _Pragma("unroll") for (int tm = 0; tm < TM; ++tm)                                         \
                    _Pragma("unroll") for (int tn = 0; tn < TN; ++tn) acc[tm][tn] =                       \
                        __builtin_amdgcn_mfma_i32_32x32x32_i8(a[tm], b[tn], acc[tm][tn], 0, 0, 0);        \
            }                                                                                             \
        }                                                                                                 \
    }

// End of a step.  A bare s_barrier, not __syncthreads(): the fence inside the latter would wait
// for every copy in flight (vmcnt 0) and with that undo the run-ahead.  What the barrier has to
// order: this wavefront's copies for the next step have landed (wait_vmcnt), and its LDS reads of the
// step have returned: the stage is overwritten by copies that start right behind the barrier.  The
// second needs the explicit wait for the LDS counter: the compiler is free to let the MFMAs that
// consume the step's last fragments follow below the barrier, and the reads would then still be
// queued in the LDS when the wavefront arrives (seen as wrong results in the backward's kernel, which
// has the same structure, when another stream's kernel kept the CU's LDS busy).
// The empty asm keeps the compiler from moving LDS reads of the next step above the barrier.
#define QB_STEP_BARRIER()                                                                                 \
    {                                                                                                     \
        __builtin_amdgcn_s_waitcnt(0xC07F); /* lgkmcnt(0) */                                              \
        __builtin_amdgcn_s_barrier();                                                                     \
        asm volatile("" ::: "memory");                                                                    \
    }

    const int nsteps = K / BK;
    // prologue: start the copies of the first D steps, wait for step 0 only
#pragma unroll
    for (int u = 0; u < D; ++u)
        if (u < nsteps) QB_FETCH(u, u)
    if (nsteps >= D) wait_vmcnt<(D - 1) * PER>();
    else wait_vmcnt<0>();
    QB_STEP_BARRIER();

    int s = 0;
    for (; s + NSTAGE <= nsteps; s += NSTAGE) {
#pragma unroll
        for (int u = 0; u < NSTAGE; ++u) {
            const bool more = s + u + D < nsteps;  // uniform
            if (more) QB_FETCH(s + u + D, (u + D) % NSTAGE)
            QB_MMA(u)
            if (more) wait_vmcnt<(D - 1) * PER>();  // copies for the next step have landed, younger ones fly on
            else wait_vmcnt<0>();
            QB_STEP_BARRIER();
        }
    }
    // tail: fewer than NSTAGE steps left, all their copies are already issued
#pragma unroll
    for (int u = 0; u < NSTAGE - 1; ++u)
        if (s + u < nsteps) {
            QB_MMA(u)
            wait_vmcnt<0>();
            QB_STEP_BARRIER();
        }
#undef QB_FETCH
#undef QB_MMA
#undef QB_STEP_BARRIER

    // ---- epilogue: exact integer corrections, then one scale per column.  Everything the
    // stores depend on is loaded first: a load issued between two stores would make the wavefront
    // wait for the older store to complete (loads and stores share one in-order counter) and turn
    // the write-out into a chain of round trips.
    constexpr int L = (1 << BITS) - 1;
    constexpr int E2 = (BITS == 8) ? 2 : -2 * L;  // 2*e
    const bool interior = (tile_m + 1) * BM <= T && (tile_n + 1) * BN <= N;  // uniform over the workgroup
    int coln[TN];
    float scale[TN], bv[TN];
    bool n_ok[TN];
#pragma unroll
    for (int tn = 0; tn < TN; ++tn) {
        const int n = tile_n * BN + (wn * TN + tn) * 32 + l32;
        n_ok[tn] = n < N;
        const int nn = n_ok[tn] ? n : N - 1;
        coln[tn] = 2 * rs_w[nn] + K;
        scale[tn] = hx * h[nn / rows_per_group];
        bv[tn] = bias ? bias[nn] : 0.0f;
    }
    if (interior && A4out == nullptr) {
        // fast path (uniform branch): straight-line code, one scalar base per 32x32 block and one
        // 32-bit lane offset per accumulator register
        const int t_wave = tile_m * BM + wm * TM * 32, n_wave = tile_n * BN + wn * TN * 32;
        float *y_wave = Y + (size_t)t_wave * N + n_wave;
        const int32_t *rx_wave = rs_x + t_wave;
        uint32_t voff[16];
#pragma unroll
        for (int i = 0; i < 16; ++i)
            voff[i] = ((uint32_t)(4 * hf + 8 * (i >> 2) + (i & 3)) * (uint32_t)N + (uint32_t)l32) * 4u;
        int rx[TM][16];
#pragma unroll
        for (int tm = 0; tm < TM; ++tm)
#pragma unroll
            for (int i = 0; i < 16; ++i) rx[tm][i] = rx_wave[tm * 32 + 4 * hf + 8 * (i >> 2) + (i & 3)];
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int tm = 0; tm < TM; ++tm)
#pragma unroll
            for (int tn = 0; tn < TN; ++tn) {
                char *y_blk = reinterpret_cast<char *>(y_wave + (size_t)tm * 32 * N + tn * 32);
#pragma unroll
                for (int i = 0; i < 16; ++i) {
                    const int a4 = qb_a4(acc[tm][tn][i], qb_mad24(E2, rx[tm][i], coln[tn]));
                    __builtin_nontemporal_store(scale[tn] * (float)a4 + bv[tn], reinterpret_cast<float *>(y_blk + voff[i]));
                }
            }
    } else {
        // edge tiles and the debug output: every element checked
#pragma unroll
        for (int tm = 0; tm < TM; ++tm) {
            const int t0 = tile_m * BM + (wm * TM + tm) * 32 + 4 * hf;
            int rx[16];
#pragma unroll
            for (int i = 0; i < 16; ++i) {
                const int t = t0 + 8 * (i >> 2) + (i & 3);
                rx[i] = rs_x[t < T ? t : T - 1];
            }
#pragma unroll
            for (int tn = 0; tn < TN; ++tn) {
                const int n = tile_n * BN + (wn * TN + tn) * 32 + l32;
#pragma unroll
                for (int i = 0; i < 16; ++i) {
                    const int t = t0 + 8 * (i >> 2) + (i & 3);
                    if (t < T && n_ok[tn]) {
                        const int a4 = qb_a4(acc[tm][tn][i], E2 * rx[i] + coln[tn]);
                        const size_t at = (size_t)t * N + n;
                        Y[at] = scale[tn] * (float)a4 + bv[tn];
                        if (A4out) A4out[at] = a4;
                    }
                }
            }
        }
    }
    }  // persistent tile loop
}

// 4-byte form of the global -> LDS copy: lane l's dword lands at m0 + 4*l
__device__ __forceinline__ void copy4_to_lds(const void *g, uint32_t lds_addr)
{
    asm volatile("s_mov_b32 m0, %1\n\ts_nop 0\n\tglobal_load_lds_dword %0, off" ::"v"(g), "s"(lds_addr) : "memory", "m0");
}

// Epilogue of the role-split kernel.  Its per-token and per-neuron parameters do not come from global
// memory but from a block in LDS that a producer wavefront filled for the tile (BM ints rs_x, then BN
// each of rs_w, h of the neuron's group, bias, then BM per-token scales and, with asymmetric ranges, BN values of q0 of
// the neuron's group; indices past the end of the matrix were clamped).  The
// consumer wavefronts thus issue no global loads at all: their memory counter holds stores only and is
// never waited on, so the stores of one tile need not have completed before the next tile's go out.
// acc[tm][tn][r]: token tl + 32*tm + 8*(r/4) + (r%4) of the tile (tl contains 4*hf), neuron nl + 32*tn
// (nl contains l32).  A4 = 4*acc + 2e*rs_x[t] + 2*rs_w[n] + K,  Y = (h_x*h_g(n)) * float(A4) + bias[n];
// dyn: h_x per token; asym_L = 2^k - 1: asymmetric group ranges, Y = asym_value(...) + bias[n].
template <int BM, int BN>
__device__ __forceinline__ void store_block_lds(const v16i &acc, const uint8_t *pp, int e2, int tl, int nl, int t0, int n0,
                                                int T, int N, int K, float hx, bool has_bias, bool fast,
                                                float *__restrict__ Y, int32_t *__restrict__ A4out, bool dyn = false,
                                                int asym_L = 0)
{
    // one 32x32 block: acc[r] is token tl + 8*(r/4) + (r%4) of the tile, neuron nl
    const int *p_rx = reinterpret_cast<const int *>(pp);
    const int *p_rw = p_rx + BM;
    const float *p_h = reinterpret_cast<const float *>(p_rw + BN), *p_b = p_h + BN;
    const int coln = 2 * p_rw[nl] + K;
    const float scale = hx * p_h[nl];
    const float bv = has_bias ? p_b[nl] : 0.0f;
    // per row: the scale.  dyn: one activation scale per token, the tile's BM of them follow the bias in the
    // parameter block; otherwise the one scale of the call.
    float sc[16];
    if (dyn) {
        const float *p_hx = p_b + BN;
        const float hg = p_h[nl];
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            const float4 v = *reinterpret_cast<const float4 *>(p_hx + tl + 8 * q);
            sc[4 * q + 0] = v.x * hg;
            sc[4 * q + 1] = v.y * hg;
            sc[4 * q + 2] = v.z * hg;
            sc[4 * q + 3] = v.w * hg;
        }
    } else {
#pragma unroll
        for (int r = 0; r < 16; ++r) sc[r] = scale;
    }
    int rx[16];
#pragma unroll
    for (int q = 0; q < 4; ++q) {
        const int4 v = *reinterpret_cast<const int4 *>(p_rx + tl + 8 * q);
        rx[4 * q + 0] = qb_mad24(e2, v.x, coln);  // |rs_x| <= 128*K < 2^23: the 24-bit multiply is exact and full rate
        rx[4 * q + 1] = qb_mad24(e2, v.y, coln);
        rx[4 * q + 2] = qb_mad24(e2, v.z, coln);
        rx[4 * q + 3] = qb_mad24(e2, v.w, coln);
    }
    if (asym_L) {  // asymmetric group ranges: Delta in the place of h, q0 behind the per-token scales
        const float dn = p_h[nl], zn = (p_b + BN + BM)[nl];
        float hr[16];  // the activation scale of every row: the call's, or the token's own
        if (dyn) {
            const float *p_hx = p_b + BN;
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                const float4 v = *reinterpret_cast<const float4 *>(p_hx + tl + 8 * q);
                hr[4 * q + 0] = v.x; hr[4 * q + 1] = v.y; hr[4 * q + 2] = v.z; hr[4 * q + 3] = v.w;
            }
        } else {
#pragma unroll
            for (int r = 0; r < 16; ++r) hr[r] = hx;
        }
        int rh[16];  // R/2 = rs_x + K/2 per row
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            const int4 v = *reinterpret_cast<const int4 *>(p_rx + tl + 8 * q);
            rh[4 * q + 0] = v.x + (K >> 1);
            rh[4 * q + 1] = v.y + (K >> 1);
            rh[4 * q + 2] = v.z + (K >> 1);
            rh[4 * q + 3] = v.w + (K >> 1);
        }
        if (fast) {
            char *y_blk = reinterpret_cast<char *>(Y + (size_t)(t0 + tl) * N + n0 + nl);
#pragma unroll
            for (int r = 0; r < 16; ++r) {
                const int a4 = qb_a4(acc[r], rx[r]);
                __builtin_nontemporal_store(asym_value(a4, rh[r], asym_L, hr[r], dn, zn) + bv,
                                            reinterpret_cast<float *>(y_blk + (size_t)(8 * (r >> 2) + (r & 3)) * N * 4));
            }
        } else if (n0 + nl < N) {
#pragma unroll
            for (int r = 0; r < 16; ++r) {
                const int t = t0 + tl + 8 * (r >> 2) + (r & 3);
                if (t < T) {
                    const int a4 = qb_a4(acc[r], rx[r]);
                    const size_t at = (size_t)t * N + n0 + nl;
                    Y[at] = asym_value(a4, rh[r], asym_L, hr[r], dn, zn) + bv;
                    if (A4out) A4out[at] = a4;
                }
            }
        }
        return;
    }
    if (fast) {
        char *y_blk = reinterpret_cast<char *>(Y + (size_t)(t0 + tl) * N + n0 + nl);
#pragma unroll
        for (int r = 0; r < 16; ++r) {
            const int a4 = qb_a4(acc[r], rx[r]);
            __builtin_nontemporal_store(sc[r] * (float)a4 + bv,
                                        reinterpret_cast<float *>(y_blk + (size_t)(8 * (r >> 2) + (r & 3)) * N * 4));
        }
    } else if (n0 + nl < N) {  // edge tiles and the debug output: every element checked
#pragma unroll
        for (int r = 0; r < 16; ++r) {
            const int t = t0 + tl + 8 * (r >> 2) + (r & 3);
            if (t < T) {
                const int a4 = qb_a4(acc[r], rx[r]);
                const size_t at = (size_t)t * N + n0 + nl;
                Y[at] = sc[r] * (float)a4 + bv;
                if (A4out) A4out[at] = a4;
            }
        }
    }
}

// 8-bit output (the next layer's input): where to put it and how to quantize it
struct OutQ {
    int8_t *Yq;       // [T,N] u - 128
    int32_t *rs_y;    // [T] row sums of Yq, accumulated with atomics (zero-filled before the launch)
    float clip_out;   // range [-clip_out, +clip_out]
    int act;          // 0 none, 1 GELU
    const float *hx_rows;  // fp32 output only: one activation scale per token (dynamic range) instead of hx, or null
    const float *q0;       // fp32 output only: asymmetric group ranges (h holds Delta, q0 the lower ends), or null
};

// One linear layer of a launch of the role-split kernel, and the list of them that one launch walks through.
// The workgroups take the tiles of all problems in one sequence (each problem's share padded to a multiple of 8, so
// that the renumbering by XCD stays inside a problem), the copy wavefronts running ahead across problem boundaries
// as they do across tiles: a launch's fixed cost (start, first copies from HBM, drain) is paid once for the list.
struct Problem {
    const int8_t *Xq;
    const int32_t *rs_x;
    const uint8_t *packed;
    const float *h;
    const int32_t *rs_w;
    const float *bias;
    float *Y;
    int32_t *A4out;
    int T, N, K, rows_per_group;
    float hx;
    int tiles_m, tiles_n;
    OutQ oq;
};
constexpr int kMaxGroup = QB_MAX_BATCH;
struct Group {
    int n;                            // problems in the list
    int tile_start[kMaxGroup + 1];    // first tile of problem i in the launch's sequence; [n] = length of the sequence
    Problem p[kMaxGroup];
};
// which problem tile `work` of the sequence belongs to (uniform over the workgroup)
__device__ __forceinline__ int problem_of(const Group &g, int work)
{
    int pi = 0;
    while (pi + 1 < g.n && work >= g.tile_start[pi + 1]) ++pi;
    return pi;
}
// GELU(y) = y/2 * (1 + erf(y/sqrt(2))) = max(y, 0) - w/2 * E, w = |y|, E = erfc(w/sqrt(2)) = 2^(w*R(w)), to within 8e-7: R
// is a polynomial of degree 4, fitted on [0, 5.5] for the smallest largest error of w/2 * E (5.4e-7; Lawson's reweighted
// least squares), beyond which w/2 * E is less than 1.1e-7.  (y + |y|)/2 keeps infinities and NaN as the product has them.
__device__ __forceinline__ float gelu_near(float y)
{
    const float w = fminf(fabsf(y), 5.5f);
    float r = __builtin_fmaf(-0.0004881021741311997f, w, 0.0071987188421189785f);
    r = __builtin_fmaf(r, w, -0.052146632224321365f);
    r = __builtin_fmaf(r, w, -0.45959582924842834f);
    r = __builtin_fmaf(r, w, -1.1510004997253418f);
    const float e = __builtin_amdgcn_exp2f(__builtin_fmaf(r, w, -1.0f));
    return __builtin_fmaf(0.5f, y + fabsf(y), -(w * e));
}

// One 32x32 block of the 8-bit output: the value that decides the code is formed in binary32 with one
// rounding per step, scale = h_x*h_g, y = scale*float(A4), y = y + bias; then the optional GELU, the clamp to
// the output range and the activation quantizer.  The bytes go to the workgroup's staging tile in LDS
// (BM rows of BN bytes), from where whole rows are written out.  Lane/register roles as in store_block_lds.
template <int BM, int BN, int BNT, int GELU>  // GELU: 0 none, 1 exact, 2 quick
__device__ __forceinline__ void quant_block_lds(const v16i &acc, const uint8_t *pp, int e2, int tl, int nl, int K,
                                                float hx, bool has_bias, const Quantizer &qo,
                                                uint8_t *stg, uint2 *list, int lane)
{
    // (this file is compiled with -ffp-contract=off: y = scale*float(A4) and y + bias are two roundings)
    asm volatile("" : "+v"(tl));
    const int *p_rx = reinterpret_cast<const int *>(pp);
    const int *p_rw = p_rx + BM;
    const float *p_h = reinterpret_cast<const float *>(p_rw + BN), *p_b = p_h + BN;
    const int coln = 2 * p_rw[nl] + K;
    const float scale = hx * p_h[nl];
    const float bv = has_bias ? p_b[nl] : 0.0f;  // y + 0 = y: the code is the same as without a bias
    const float c = qo.m;
    float y[16];
#pragma unroll
    for (int q = 0; q < 4; ++q) {
        const int4 v = *reinterpret_cast<const int4 *>(p_rx + tl + 8 * q);
        const int rx[4] = {v.x, v.y, v.z, v.w};
#pragma unroll
        for (int i = 0; i < 4; ++i) y[4 * q + i] = scale * (float)qb_a4(acc[4 * q + i], qb_mad24(e2, rx[i], coln)) + bv;  // |rs_x| < 2^23
    }
    uint8_t *const dst = stg + tl * BNT + nl;
    auto at = [&](int r) { return (8 * (r >> 2) + (r & 3)) * BNT; };
    if constexpr (GELU == 0) {
        // The quantizer (same steps as Quantizer::code_f) without a branch per element: the reciprocal route for
        // all sixteen, and the true division for all sixteen if any lane's product came too close to a rounding
        // boundary (about one block in five) or the range is too extreme for the reciprocal.
        float s[16], rr[16];
        bool redo = !qo.fast;
#pragma unroll
        for (int r = 0; r < 16; ++r) {
            s[r] = __builtin_amdgcn_fmed3f(y[r], -c, c) + c;
            const float tp = s[r] * qo.rinv;
            rr[r] = rintf(tp);
            redo |= !(fabsf(tp - rr[r]) <= 0.4999f);
        }
        if (__any(redo)) {
#pragma unroll
            for (int r = 0; r < 16; ++r) rr[r] = rintf(__fdiv_rn(s[r], qo.delta));
        }
#pragma unroll
        for (int r = 0; r < 16; ++r) dst[at(r)] = (uint8_t)(uint32_t)rr[r];  // the code u; u - 128 is formed on the way out
        return;
    }
    // With GELU.  The exact steps are erff, the true division and a rounding; the quick ones gelu_near and the reciprocal,
    // for all sixteen values without a branch.  They give the same code unless the quick product lies closer to a rounding
    // boundary than the two routes can differ: 4.6e-5 for the division (derived at Quantizer), 255 * 2^-23 = 3.1e-5 for the
    // two roundings of v + c, and 2e-6 in v for GELU (8e-7 of gelu_near, 7e-7 of the binary32 steps around erff; evaluated
    // over the binary32 arguments of both signs the two differ by 9.6e-7 at most).  The few such values
    // (GELU's flat tail below -4.7 among them, where the code hangs on the last bits of erff) are gathered over the block
    // and done exactly, 64 at a time.  A block with many of them, as a look at a quarter of its values tells before the
    // quick steps, or a range too extreme for the reciprocal, goes through the exact steps.
    // Feed-forward up (N 3072, K 768), where erff for every value bound the epilogue (some forty operations, both sides of
    // its branch): 4096 tokens, 4 bits 38.8 -> 30.9 us; 12000 tokens, 8 bits 97 -> 74; 100 tokens 13.7 -> 12.4.  At 2 and 3
    // bits the exact steps alone: the few levels have to reach the outliers of a group, so the pre-activations are wide
    // and most blocks full of tails (with the quick steps 37.1 and, at 3584 x 896, 62.6 us, without 34.4 and 58.3; the
    // exact steps one register at a time are also faster than a reciprocal pass with the division behind it: 37.3, 60.8).
    auto exact = [&](float v) {
        v = 0.5f * v * (1.0f + erff(v * 0.70710678118654752f));
        return (uint8_t)(uint32_t)rintf(__fdiv_rn(__builtin_amdgcn_fmed3f(v, -c, c) + c, qo.delta));
    };
    if constexpr (GELU == 2) {
        int total = 0;
#pragma unroll
        for (int r = 0; r < 16; r += 4) total += 4 * __popcll(__ballot(y[r] < -4.7f));
        if (qo.fast && total <= 64) {
            uint64_t near[16];
            const float lim = 0.49992f - 2.0e-6f * qo.rinv;
            total = 0;
#pragma unroll
            for (int r = 0; r < 16; ++r) {
                const float tp = (__builtin_amdgcn_fmed3f(gelu_near(y[r]), -c, c) + c) * qo.rinv, rr = rintf(tp);
                near[r] = __ballot(!(fabsf(tp - rr) <= lim));
                total += __popcll(near[r]);
                dst[at(r)] = (uint8_t)(uint32_t)rr;
            }
            if (total == 0) return;
            if (total <= 128) {
                asm volatile("" ::: "memory");  // (a wavefront's LDS operations keep their order)
                int n = 0;
#pragma unroll
                for (int r = 0; r < 16; ++r)
                    if (near[r]) {
                        if ((near[r] >> lane) & 1) {
                            const int k = n + __builtin_amdgcn_mbcnt_hi((uint32_t)(near[r] >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)near[r], 0));
                            list[k] = make_uint2(__float_as_uint(y[r]), (uint32_t)(tl * BNT + nl + at(r)));
                        }
                        n += __popcll(near[r]);
                    }
                asm volatile("" ::: "memory");
                __builtin_amdgcn_wave_barrier();
#pragma clang loop unroll(disable)
                for (int k = lane; k < total; k += 64) {
                    const uint2 e = list[k];
                    stg[e.y] = exact(__uint_as_float(e.x));
                }
                asm volatile("" ::: "memory");
                __builtin_amdgcn_wave_barrier();
                return;
            }
        }
    }
#pragma unroll
    for (int r = 0; r < 16; ++r) dst[at(r)] = exact(y[r]);
}

// ---------------------------------------------------------------------------------------------
// Main kernel (K a multiple of 128): the same data path as above with the work split by role.
//   consumer wavefronts (WM x WN of them): LDS fragment reads, code expansion, MFMA, epilogue
//   producer wavefronts (NPROD): nothing but the global -> LDS copies and the waiting for them
// A copy instruction keeps the issuing wavefront busy for tens of cycles while the texture path
// accepts its 64 addresses; issued from an MFMA wavefront that time is lost to the matrix cores,
// issued from a producer it is free.  Producers also run ahead across tiles: while the consumers
// write tile i out, the first stages of tile i+1 are already being filled.
// Protocol per tile (n steps, ring of NSTAGE stages, copies run D = NSTAGE-1 steps ahead); every
// wavefront executes exactly n+1 barriers:
//   producer: start copies 0..D-1; wait copy 0; BARRIER;
//             for s: start copy s+D (its stage was read in step s-1, finished at the last barrier);
//                    wait copy s+1 (vmcnt leaves the younger ones in flight); BARRIER
//   consumer: BARRIER; for s: MMA on stage s % NSTAGE; wait until the stage's LDS reads have returned; BARRIER
// OUTQ: instead of Y the tile is quantized to 8 bits (quant_block_lds) into an LDS staging tile and, after one
// more barrier per tile (E, executed by the producers once the next tile's first copies are on their way), written
// out in whole rows; the rows' sums are collected in LDS and added to rs_y one tile later.
// OUT: 0 fp32 Y, 1 the 8-bit output (OUTQ), 3 the same with GELU, 2 fp32 Y from asymmetric group ranges (ASYM; a variant of its own so
// that the others carry none of its code)
template <int BITS, int TM, int TN, int WM, int WN, int NSTAGE, int NPROD, bool SIMD3, int OUT>
__global__ __launch_bounds__(64 * (WM * WN + NPROD), (SIMD3 && OUT != 2 && NSTAGE == 2) ? 4 : 2) void qgemm_i8_ws_kernel(const Group g)
{
    constexpr bool OUTQ = OUT == 1 || OUT == 3, ASYM = OUT == 2;
    static_assert(NSTAGE >= 2 && NSTAGE <= 4, "ring of 2..4 stages");
    constexpr int NC = WM * WN;
    constexpr int BM = WM * TM * 32, BN = WN * TN * 32, BK = 128;
    constexpr int SLOT = 4 * BITS;                  // bytes per slot in memory
    constexpr int CH = (BITS == 3) ? 12 : 16;       // bytes one lane moves per weight copy instruction
    constexpr int LSLOT = (BITS == 3) ? 16 : SLOT;  // a 12-byte copy lands at a 16-byte stride in LDS
    constexpr int PAIR = 128 * SLOT;                // one 32-neuron block x two units, contiguous in memory
    constexpr int LPAIR = 128 * LSLOT;
    constexpr int PARTS = PAIR / (64 * CH);         // copy instructions per pair; each fills 1024 bytes of LDS
    constexpr int A_TOTAL = BM / 8, B_TOTAL = (BN / 32) * PARTS;  // copy instructions per step
    constexpr int A_PER = (A_TOTAL + NPROD - 1) / NPROD, B_PER = (B_TOTAL + NPROD - 1) / NPROD;
    constexpr int PERP = A_PER + B_PER;             // per producer and step
    constexpr int D = NSTAGE - 1;
    constexpr int A_BYTES = BM * BK, B_BYTES = (BN / 32) * LPAIR, STAGE_BYTES = A_BYTES + B_BYTES;
    static_assert((D - 1) * PERP + 2 * (BM / 64) + 4 * ((BN + 63) / 64) < 64, "vmcnt has six bits");
    constexpr int BNP = (BN + 63) / 64 * 64;        // per-neuron parameter arrays are filled 64 entries at a time
    // rs_x | rs_w | h of the neuron's group | bias | per-token scales | q0 of the neuron's group (asymmetric ranges)
    constexpr int PARAM_BYTES = (2 * BM + (OUT == 2 ? 4 : 3) * BNP) * 4;
    static_assert(!SIMD3 || (NC == 6 && NPROD == 2), "SIMD3: six MFMA wavefronts on SIMDs 0..2, two copy wavefronts on SIMD 3");

    // A tile's parameter block is read in its write-out, which ends before the consumers pass the first
    // barrier of the next tile; the producer rewrites the block two tiles later, after the next tile's
    // last barrier.  Hence two blocks.
    constexpr int NPARAM = 2;

    constexpr int STG_OFF = NSTAGE * STAGE_BYTES + NPARAM * PARAM_BYTES;  // staging tile, then BM row sums
    constexpr int LIST_OFF = STG_OFF + (OUTQ ? BM * BN + BM * 4 : 0);  // then up to 128 gathered values per MFMA wavefront
    constexpr int STG_BYTES = OUTQ ? BM * BN + BM * 4 + (OUT == 3 && BITS >= 4 ? NC * 128 * 8 : 0) : 0;
    static_assert(STG_OFF % 16 == 0 && BN % 16 == 0 && BM <= NC * 64, "staging tile: 16-byte pieces, one thread per row sum");
    __shared__ __align__(1024) uint8_t lds[STG_OFF + STG_BYTES];
    const uint32_t lds_base = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) uint8_t *)lds;

    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int nseq = g.tile_start[g.n];  // tiles (and padding slots) of all problems of the launch

    // Roles.  The wavefronts of a workgroup are dealt to the four SIMDs of the CU in turn (wavefront w runs
    // on SIMD w%4), and a global load or global -> LDS copy issued on a SIMD that is busy with 32x32 MFMAs
    // runs at about half speed (and slows the MFMAs), while one issued on a SIMD without MFMAs does not.
    // SIMD3 layout: wavefronts 3 and 7 copy, the other six multiply, so that three SIMDs run MFMAs at
    // full rate and the fourth feeds them.  (Roles depend on the wavefront number only: a different
    // placement by the hardware would cost speed, not correctness.)
    const bool is_producer = SIMD3 ? (wave & 3) == 3 : wave >= NC;
    if (is_producer) {
        // ================================ producer ================================
        const int p = SIMD3 ? wave >> 2 : wave - NC;
        int pb = 0;
        bool had_tile = false;
        for (int work = blockIdx.x; work < nseq; work += gridDim.x) {
            const int pi = problem_of(g, work);
            const Problem &P = g.p[pi];
            const int logical = logical_tile(work - g.tile_start[pi], P.tiles_m * P.tiles_n);
            if (logical < 0) continue;  // padding slot (the consumers skip it as well)
            const int T = P.T, N = P.N, K = P.K, rows_per_group = P.rows_per_group;
            const int8_t *__restrict__ Xq = P.Xq;
            const int32_t *__restrict__ rs_x = P.rs_x, *__restrict__ rs_w = P.rs_w;
            const uint8_t *__restrict__ packed = P.packed;
            const float *__restrict__ h = P.h, *__restrict__ bias = P.bias;
            const OutQ &oq = P.oq;
            const int nsteps = K / BK, kunits = K >> 6, ncb = (N + 31) >> 5;
            const int tile_m = logical / P.tiles_n, tile_n = logical - tile_m * P.tiles_n;
            // token rows: lane l of a copy fills physical chunk l%8 of row l/8 of an 8-row block; the
            // chunk holds logical chunk (l%8) ^ ((row/2)%8): the swizzle that makes 16 consecutive
            // rows of one logical chunk land in 16 different 16-byte bank groups
            const int last_row = T - 1 - tile_m * BM;  // rows past the end re-read the last one; outputs masked
            // addresses: a wavefront-uniform base per tile and step, a 32-bit byte offset per lane and copy
            const int8_t *a_base = Xq + (size_t)tile_m * BM * K;
            uint32_t a_off[A_PER], a_dst[A_PER];
#pragma unroll
            for (int i = 0; i < A_PER; ++i) {
                const int blk = (i * NPROD + p) % A_TOTAL;  // surplus copies repeat one: same bytes, same place
                int row = blk * 8 + (lane >> 3);
                const int key = (row >> 1) & 7;
                row = row < last_row ? row : last_row;
                a_off[i] = (uint32_t)row * (uint32_t)K + (((lane & 7) ^ key) * 16);
                a_dst[i] = blk * 1024;
            }
            const int cb0 = tile_n * (BN / 32);
            const uint8_t *b_base = packed + (size_t)cb0 * kunits * 64 * SLOT;
            uint32_t b_off[B_PER], b_dst[B_PER];
#pragma unroll
            for (int i = 0; i < B_PER; ++i) {
                const int j = (i * NPROD + p) % B_TOTAL;
                const int pair = j / PARTS, part = j - pair * PARTS;
                int cb = cb0 + pair;
                cb = cb < ncb ? cb : ncb - 1;  // blocks past the end re-read the last one; outputs masked
                b_off[i] = (uint32_t)(cb - cb0) * (uint32_t)(kunits * 64 * SLOT) + part * 64 * CH + lane * CH;
                b_dst[i] = A_BYTES + pair * LPAIR + part * 1024;
            }
            auto fetch = [&](int step, int stage) {
                const uint32_t st_ = lds_base + stage * STAGE_BYTES;
                const uint8_t *bs = b_base + (size_t)step * PAIR;
                const int8_t *as = a_base + (size_t)step * BK;
#pragma unroll
                for (int i = 0; i < B_PER; ++i) copy_to_lds<CH>(bs, b_off[i], st_ + b_dst[i]);
#pragma unroll
                for (int i = 0; i < A_PER; ++i) copy_to_lds<16>(as, a_off[i], st_ + a_dst[i]);
            };
            if (0 < nsteps) fetch(0, 0);  // the first step's copies go first: the K-loop waits for nothing else
            if (p == 0) {  // the tile's epilogue parameters: needed after the K-loop only
                const uint32_t pbase = lds_base + NSTAGE * STAGE_BYTES + pb * PARAM_BYTES;
#pragma unroll
                for (int c = 0; c < BM / 64; ++c) {
                    int t = tile_m * BM + c * 64 + lane;
                    t = t < T ? t : T - 1;
                    copy4_to_lds(rs_x + t, pbase + c * 256);
                    if (oq.hx_rows) copy4_to_lds(oq.hx_rows + t, pbase + (BM + 3 * BNP) * 4 + c * 256);
                }
#pragma unroll
                for (int c = 0; c < BNP / 64; ++c) {
                    int n = tile_n * BN + c * 64 + lane;
                    n = n < N ? n : N - 1;
                    copy4_to_lds(rs_w + n, pbase + BM * 4 + c * 256);
                    copy4_to_lds(h + n / rows_per_group, pbase + (BM + BNP) * 4 + c * 256);
                    if (bias) copy4_to_lds(bias + n, pbase + (BM + 2 * BNP) * 4 + c * 256);
                    if constexpr (ASYM) copy4_to_lds(oq.q0 + n / rows_per_group, pbase + (2 * BM + 3 * BNP) * 4 + c * 256);
                }
            }
            pb ^= 1;
#pragma unroll
            for (int u = 1; u < D; ++u)
                if (u < nsteps) fetch(u, u);
            if (OUTQ && had_tile) __builtin_amdgcn_s_barrier();  // barrier E of the previous tile
            had_tile = true;
            // step 0 has landed when only younger copies are outstanding: steps 1..D-1 and, in the wavefront
            // that issued them, the parameter copies (their number depends on bias and per-token scales)
            if (nsteps >= D) {
                constexpr int W0 = (D - 1) * PERP, PM = BM / 64, PN = BNP / 64;
                constexpr int PA = ASYM ? PN : 0;
                if (p != 0) wait_vmcnt<W0>();
                else if (oq.hx_rows) { if (bias) wait_vmcnt<W0 + 2 * PM + 3 * PN + PA>(); else wait_vmcnt<W0 + 2 * PM + 2 * PN + PA>(); }
                else { if (bias) wait_vmcnt<W0 + PM + 3 * PN + PA>(); else wait_vmcnt<W0 + PM + 2 * PN + PA>(); }
            } else {
                wait_vmcnt<0>();
            }
            __builtin_amdgcn_s_barrier();
            int stage = D % NSTAGE;  // stage of step s + D
            for (int s = 0; s < nsteps; ++s) {
                if (s + D < nsteps) {
                    fetch(s + D, stage);
                    wait_vmcnt<(D - 1) * PERP>();
                } else {
                    wait_vmcnt<0>();
                }
                stage = (stage + 1 == NSTAGE) ? 0 : stage + 1;
                __builtin_amdgcn_s_barrier();
            }
        }
        if (OUTQ && had_tile) __builtin_amdgcn_s_barrier();  // barrier E of the last tile
        return;
    }

    // ================================ consumer ================================
    const int cidx = SIMD3 ? (wave & 3) + 3 * (wave >> 2) : wave;
    const int wm = cidx / WN, wn = cidx - wm * WN;
    const int l32 = lane & 31, hf = lane >> 5;
    // token fragments: row = wm*TM*32 + tm*32 + l32, logical chunk = kk*4 + hf*2 + sub
    const int p0 = (hf * 2) ^ ((l32 >> 1) & 7);
    const int frag_row = (wm * TM * 32 + l32) * BK;
    int a_frag[4];
    a_frag[0] = frag_row + ((p0 ^ 0) << 4);  // kk 0, sub 0
    a_frag[1] = frag_row + ((p0 ^ 1) << 4);  // kk 0, sub 1
    a_frag[2] = frag_row + ((p0 ^ 4) << 4);  // kk 1, sub 0
    a_frag[3] = frag_row + ((p0 ^ 5) << 4);  // kk 1, sub 1
    const int b_frag = A_BYTES + wn * TN * LPAIR + lane * LSLOT;  // + tn*LPAIR + kk*64*LSLOT
    constexpr int L = (1 << BITS) - 1;
    constexpr int E2 = (BITS == 8) ? 2 : -2 * L;  // 2*e
    int pb = 0;

    v16i acc[TM][TN];

    // 8-bit output: staging tile, row sums, the output quantizer
    constexpr int NCT = NC * 64;
    const int ctid = cidx * 64 + lane;
    uint8_t *stg = lds + STG_OFF;
    int *rowsum = reinterpret_cast<int *>(lds + STG_OFF + BM * BN);
    uint2 *near_list = reinterpret_cast<uint2 *>(lds + LIST_OFF) + cidx * 128;
    Quantizer qo;
    int prev_t0 = -1, prev_T = 0;  // the tile whose row sums still sit in LDS, and its problem's token count and rs_y
    int32_t *prev_rs_y = nullptr;
    if constexpr (OUTQ) {
        if (ctid < BM) rowsum[ctid] = 0;
    }
    auto flush_rowsums = [&]() {  // the previous tile's row sums -> rs_y; every LDS add to them is a barrier back
        if (ctid < BM) {
            const int v = rowsum[ctid];
            rowsum[ctid] = 0;
            if (prev_t0 + ctid < prev_T) atomicAdd(prev_rs_y + prev_t0 + ctid, v);
        }
    };

    for (int work = blockIdx.x; work < nseq; work += gridDim.x) {
        const int pi = problem_of(g, work);
        const Problem &P = g.p[pi];
        const int logical = logical_tile(work - g.tile_start[pi], P.tiles_m * P.tiles_n);
        if (logical < 0) continue;  // padding slot (the producers skip it as well)
        const int T = P.T, N = P.N, K = P.K;
        const float hx = P.hx;
        const float *__restrict__ bias = P.bias;
        float *__restrict__ Y = P.Y;
        int32_t *__restrict__ A4out = P.A4out;
        const OutQ &oq = P.oq;
        const int nsteps = K / BK;
        const int tile_m = logical / P.tiles_n, tile_n = logical - tile_m * P.tiles_n;
        if constexpr (OUTQ) qo.set(oq.clip_out, 255.0f);

#pragma unroll
        for (int tm = 0; tm < TM; ++tm)
#pragma unroll
            for (int tn = 0; tn < TN; ++tn)
#pragma unroll
                for (int i = 0; i < 16; ++i) acc[tm][tn][i] = 0;

// One step: every LDS read of the step is issued first (12 reads in flight, their latency paid once),
// then the 16 MFMAs run while the later reads are still arriving.  The scheduling barrier keeps the
// compiler from folding the reads back into a read-wait-multiply chain.
#define QB_MMA(stage)                                                                                     \
    {                                                                                                     \
        const uint8_t *st_ = lds + (stage) * STAGE_BYTES;                                                 \
        uint32_t raw[2][TN][BITS];                                                                        \
        v4i afr[2][2][TM];                                                                                \
        _Pragma("unroll") for (int kk = 0; kk < 2; ++kk) {                                                \
            _Pragma("unroll") for (int tn = 0; tn < TN; ++tn)                                             \
                SlotRead<BITS>::get(st_ + b_frag + tn * LPAIR + kk * 64 * LSLOT, raw[kk][tn]);            \
            _Pragma("unroll") for (int sub = 0; sub < 2; ++sub)                                           \
                _Pragma("unroll") for (int tm = 0; tm < TM; ++tm) afr[kk][sub][tm] =                      \
                    *reinterpret_cast<const v4i *>(st_ + a_frag[kk * 2 + sub] + tm * 32 * BK);            \
        }                                                                                                 \
        __builtin_amdgcn_sched_barrier(0);                                                                \
        _Pragma("unroll") for (int kk = 0; kk < 2; ++kk) {                                                \
            uint32_t d[TN][8];                                                                            \
            _Pragma("unroll") for (int tn = 0; tn < TN; ++tn) {                                           \
                unpack_run<BITS>(raw[kk][tn], d[tn]);                                                     \
                if constexpr (BITS == 8) {                                                                \
                    _Pragma("unroll") for (int i = 0; i < 8; ++i) d[tn][i] ^= 0x80808080u;                \
                }                                                                                         \
            }                                                                                             \
            _Pragma("unroll") for (int sub = 0; sub < 2; ++sub) {                                         \
                v4i b[TN];                                                                                \
                _Pragma("unroll") for (int tn = 0; tn < TN; ++tn) {                                       \
                    b[tn][0] = (int)d[tn][4 * sub + 0];                                                   \
                    b[tn][1] = (int)d[tn][4 * sub + 1];                                                   \
                    b[tn][2] = (int)d[tn][4 * sub + 2];                                                   \
                    b[tn][3] = (int)d[tn][4 * sub + 3];                                                   \
                }                                                                                         \
                _Pragma("unroll") for (int tm = 0; tm < TM; ++tm)                                         \
                    _Pragma("unroll") for (int tn = 0; tn < TN; ++tn) acc[tm][tn] =                       \
                        __builtin_amdgcn_mfma_i32_32x32x32_i8(afr[kk][sub][tm], b[tn], acc[tm][tn], 0, 0, 0); \
            }                                                                                             \
        }                                                                                                 \
    }
// a bare barrier (no fence: the producers' vmcnt wait is what makes the copies visible); the empty
// asm keeps the compiler from moving LDS reads across it.  The wait for the LDS counter in front of it: the
// stage just read is overwritten by copies that the producers start right behind the barrier, so this
// wavefront's reads of it must have returned, not only been issued (the compiler lets the MFMAs that consume
// the step's last fragments follow below the barrier).
#define QB_BARRIER()                                                                                      \
    {                                                                                                     \
        __builtin_amdgcn_s_waitcnt(0xC07F); /* lgkmcnt(0) */                                              \
        asm volatile("" ::: "memory");                                                                    \
        __builtin_amdgcn_s_barrier();                                                                     \
        asm volatile("" ::: "memory");                                                                    \
    }

        if constexpr (OUTQ) __builtin_amdgcn_s_waitcnt(0xC07F);  // lgkmcnt(0): my LDS writes and adds are done
        QB_BARRIER()
        if constexpr (OUTQ) {
            if (prev_t0 >= 0) flush_rowsums();
        }
        int s = 0;
        for (; s + NSTAGE <= nsteps; s += NSTAGE) {
#pragma unroll
            for (int u = 0; u < NSTAGE; ++u) {
                QB_MMA(u)
                QB_BARRIER()
            }
        }
#pragma unroll
        for (int u = 0; u < NSTAGE - 1; ++u)
            if (s + u < nsteps) {
                QB_MMA(u)
                QB_BARRIER()
            }
#undef QB_MMA

        // ---- write-out
        if constexpr (OUTQ) {
            typedef unsigned int v4u __attribute__((ext_vector_type(4)));
#pragma unroll
            for (int tm = 0; tm < TM; ++tm)
#pragma unroll
                for (int tn = 0; tn < TN; ++tn)
                    quant_block_lds<BM, BNP, BN, OUT != 3 ? 0 : BITS >= 4 ? 2 : 1>(acc[tm][tn], lds + NSTAGE * STAGE_BYTES + pb * PARAM_BYTES, E2,
                                                 (wm * TM + tm) * 32 + 4 * hf, (wn * TN + tn) * 32 + l32, K, hx,
                                                 bias != nullptr, qo, stg, near_list, lane);
            __builtin_amdgcn_s_waitcnt(0xC07F);  // the staging bytes are written
            QB_BARRIER()                         // barrier E
            // whole rows out: 16-byte pieces, BN/16 per row
            constexpr int PPR = BN / 16;
            const int t0 = tile_m * BM, n0 = tile_n * BN;
            const bool vec_ok = (N & 15) == 0 && (reinterpret_cast<uintptr_t>(oq.Yq) & 15) == 0;
            for (int pc = ctid; pc < BM * PPR; pc += NCT) {
                const int row = pc / PPR, cp = pc - row * PPR;
                const int t = t0 + row, n = n0 + cp * 16;
                if (t < T && n < N) {
                    const uint4 v = *reinterpret_cast<const uint4 *>(stg + row * BN + cp * 16);  // codes u
                    int8_t *dst = oq.Yq + (size_t)t * N + n;
                    int sum;
                    if (vec_ok && n + 16 <= N) {
                        v4u o = {v.x ^ 0x80808080u, v.y ^ 0x80808080u, v.z ^ 0x80808080u, v.w ^ 0x80808080u};  // u - 128
                        __builtin_nontemporal_store(o, reinterpret_cast<v4u *>(dst));
                        uint32_t su = __builtin_amdgcn_sad_u8(v.x, 0u, 0u);
                        su = __builtin_amdgcn_sad_u8(v.y, 0u, su);
                        su = __builtin_amdgcn_sad_u8(v.z, 0u, su);
                        su = __builtin_amdgcn_sad_u8(v.w, 0u, su);
                        sum = (int)su - 16 * 128;
                    } else {
                        const uint32_t w[4] = {v.x ^ 0x80808080u, v.y ^ 0x80808080u, v.z ^ 0x80808080u, v.w ^ 0x80808080u};
                        sum = 0;
#pragma unroll
                        for (int b = 0; b < 16; ++b)
                            if (n + b < N) {
                                const int8_t q8 = (int8_t)((w[b >> 2] >> (8 * (b & 3))) & 255u);
                                dst[b] = q8;
                                sum += q8;
                            }
                    }
                    atomicAdd(rowsum + row, sum);
                }
            }
            prev_t0 = t0;
            prev_T = T;
            prev_rs_y = oq.rs_y;
        } else {
        const bool fast = (tile_m + 1) * BM <= T && (tile_n + 1) * BN <= N && A4out == nullptr;
#pragma unroll
        for (int tm = 0; tm < TM; ++tm)
#pragma unroll
            for (int tn = 0; tn < TN; ++tn)
                store_block_lds<BM, BNP>(acc[tm][tn], lds + NSTAGE * STAGE_BYTES + pb * PARAM_BYTES, E2,
                                        (wm * TM + tm) * 32 + 4 * hf, (wn * TN + tn) * 32 + l32, tile_m * BM, tile_n * BN,
                                        T, N, K, hx, bias != nullptr, fast, Y, A4out, oq.hx_rows != nullptr,
                                        ASYM ? L : 0);
        }
        pb ^= 1;
    }
    if constexpr (OUTQ) {
        if (prev_t0 >= 0) {  // the last tile's row sums: the producers have left, the six MFMA wavefronts meet once more
            __builtin_amdgcn_s_waitcnt(0xC07F);
            __builtin_amdgcn_s_barrier();
            flush_rowsums();
        }
    }
#undef QB_BARRIER
}

// Kernel for many tiles, K a multiple of 128: tiles of 128 tokens x 256 neurons, four wavefronts of 128 x 64 results,
// v_mfma_i32_16x16x64_i8, two workgroups per CU on a persistent grid.
// What bounds the smaller tiles is the LDS (operand fragments per MFMA) and the SIMD that copies, fragment reads and
// code expansion share with the MFMAs.  Here a step of 128 features takes a wavefront 1024 cycles of MFMAs for 16 KB of
// token fragments and 2-4 KB of packed weights read from LDS, every code is expanded once in the workgroup, and the
// 16x16x64 form leaves the issue slots that the other wavefront of the SIMD needs.  That one belongs to the CU's other
// workgroup and shares no barrier with it: one multiplies while the other one reads, expands, changes tile or writes out.
// Measured at 32768 tokens, 2 bits: 4096 x 1024 183 us (two plain 128x128 workgroups per CU: 200), 1024 x 4096 109 (132),
// a whole BERT-large layer with its activation quantizers 691 -> 606 us.  256x256 tiles of eight wavefronts (one
// workgroup per CU, two groups of wavefronts half a phase apart) have the same K-loop, but a tile's write-out then runs
// next to nothing: 188 and 118 us.  A second barrier per step that frees the stage earlier (copies two steps ahead) and
// lines touched ahead of the copies were slower (188 and 120; 188 and 124).
// That is the 2-bit build; at 3 and 4 bits 4096 x 1024 takes 165 and 155 us, 1024 x 4096 129 and 116, to 148 and 110 at 2 bits (with the
// tokens in the last-level cache).  8 bits: 32768 x 4096 x 1024 with its activation quantizer 243 -> 198 us (two plain 128x128 workgroups
// per CU before), 32768 x 1024 x 4096 293 -> 246, 12288 x 3072 x 768 63 -> 58.
struct DuoArgs {
    const int8_t *Xq;
    const int32_t *rs_x;
    const uint8_t *packed;
    const float *h;
    const int32_t *rs_w;
    const float *bias;
    float *Y;
    int32_t *A4out;
    int T, N, K, rows_per_group;
    float hx;
    int tiles_m, tiles_n;
};
struct DuoJob {
    DuoArgs p[1];
};
template <int BITS>
__global__ __launch_bounds__(256, 2) void qgemm_i8_duo_kernel(const DuoJob job)
{
    constexpr int BM = 128, BN = 256, BK = 128;
    constexpr int SLOT = 4 * BITS, CH = (BITS == 3) ? 12 : 16, LSLOT = (BITS == 3) ? 16 : SLOT;
    // A step's weights are read in one phase; at 8 bits in two of 64 features, whose stages take turns (two of 128 features
    // for each of two workgroups would not fit the LDS).  The tokens' rows of 128 bytes are whole lines at every width.
    constexpr int PHASES = BITS == 8 ? 2 : 1, PHF = BK / PHASES;
    constexpr int PAIR = PHF * SLOT, LPAIR = PHF * LSLOT;  // a 32-neuron block of one phase, in memory and in LDS
    constexpr int PARTS = LPAIR / 1024;                    // copies of one such block
    constexpr int NB = 2 * PARTS;                          // weight copies per wavefront and phase
    constexpr int A_BYTES = BM * BK, STAGE = A_BYTES + 8 * LPAIR;
    constexpr int PARAM = (128 + 3 * 256) * 4;             // rs_x, rs_w, h of the neuron's group, bias
    constexpr int E2 = (BITS == 8) ? 2 : -2 * ((1 << BITS) - 1);  // 2*e
    static_assert(2 * (2 * STAGE + 2 * PARAM) <= 163840, "two workgroups per CU");
    __shared__ __align__(1024) uint8_t lds[2 * STAGE + 2 * PARAM];
    const uint32_t lds_base = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) uint8_t *)lds;

    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);  // neurons 64*wave
    const int q16 = lane & 15, hq = lane >> 4;

    // fragment reads: token row l%16 of a 16-row block, logical chunk 2*(l/16) + kk (the 32 features of a slot)
    const int fkey = (q16 >> 1) & 7;
    // (at 8 bits chunk 4*phase + l/16: the lane's sixteen features of the phase)
    const int a_fr[2] = {q16 * BK + (((BITS == 8 ? hq : 2 * hq) ^ fkey) << 4), q16 * BK + (((BITS == 8 ? hq + 4 : 2 * hq + 1) ^ fkey) << 4)};
    // codes: slot 2*(l%16) + b of quarter l/16 of the block; b toggles bit 4 of the address (at 2 bits one read gives both).
    // A lane's two neurons of a block are neighbours, so that its stores are 8 bytes and every store instruction covers
    // whole 128-byte lines; the copies swap neighbouring slots in every other run of sixteen against the bank conflicts
    // of that order.
    // At 8 bits a slot is two chunks of sixteen codes and lane l reads chunk (l/16)%2 of slot 2*(l%16) + b of half l/32; the
    // copies permute the chunks within runs of four.
    const int b_fr = A_BYTES + 2 * wave * LPAIR +
                     (BITS == 8 ? (hq >> 1) * 1024 + ((4 * q16 + ((hq & 1) ^ (q16 >> 2))) << 4)
                                : BITS == 2 ? hq * 256 + q16 * 16 : hq * 512 + (((2 * q16) ^ (q16 >> 3)) << 4));
    constexpr int B_NEXT = BITS == 8 ? 32 : 16;  // toggles b

    // The lane's number formed anew where a tile needs it: kept over the K-loop, it and what is formed from it take two registers that
    // 4 bits do not have (spilling them cost no time that could be measured).
    auto lane_again = []() {
        int all = -1;
        asm volatile("" : "+s"(all));
        return (int)__builtin_amdgcn_mbcnt_hi(all, __builtin_amdgcn_mbcnt_lo(all, 0));
    };

    // The arguments are loaded where a tile needs them: known to be constant they would all be held in scalar registers
    // from the start, more than there are.
    auto args = [&]() -> const DuoArgs & {
        int zero = 0;
        asm volatile("" : "+s"(zero));
        return job.p[zero];
    };
    const int nwg = job.p[0].tiles_m * job.p[0].tiles_n, tiles_n = job.p[0].tiles_n, steps = job.p[0].K / BK;

    const uint8_t *a_base = nullptr, *b_base = nullptr;
    uint32_t a_off[4], b_off[NB];
    auto copy_weights = [&](int phase, int par) {
        const uint8_t *bs = b_base + (size_t)phase * PAIR;
        const uint32_t dst = lds_base + (uint32_t)par * STAGE + A_BYTES;
#pragma unroll
        for (int e = 0; e < NB; ++e) copy_to_lds<CH>(bs, b_off[e], dst + (wave * NB + e) * 1024);
    };
    auto copy_tokens = [&](int s, int par) {
        const uint8_t *as = a_base + (size_t)s * BK;
        const uint32_t dst = lds_base + (uint32_t)par * STAGE;
#pragma unroll
        for (int e = 0; e < 4; ++e) copy_to_lds<16>(as, a_off[e], dst + (wave * 4 + e) * 1024);
    };
    // addresses of a tile's operands, its epilogue parameters and the copies of its first step
    auto start_tile = [&](int tm, int tn, int pb, int par) {
        const int lane = lane_again();
        const DuoArgs &P = args();
        const int T = P.T, N = P.N, K = P.K, kunits = K >> 6, ncb = (N + 31) >> 5;
        a_base = reinterpret_cast<const uint8_t *>(P.Xq) + (size_t)tm * BM * K;
        b_base = P.packed + (size_t)tn * 8 * kunits * 64 * SLOT;
        const int a_last = T - 1 - tm * BM, cb_last = ncb - 1 - tn * 8;
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            int row = (wave * 4 + e) * 8 + (lane >> 3);
            row = row < a_last ? row : a_last;  // rows past the end re-read the last one; results not stored
            a_off[e] = (uint32_t)row * (uint32_t)K + (((lane & 7) ^ (lane >> 4) ^ (4 * (e & 1))) << 4);
        }
        const int sl = BITS == 2 ? lane : lane ^ ((lane >> 4) & (BITS == 8 ? 3 : 1));
#pragma unroll
        for (int e = 0; e < NB; ++e) {
            const int x = wave * NB + e;
            int cb = x / PARTS;
            cb = cb < cb_last ? cb : cb_last;
            b_off[e] = (uint32_t)cb * (uint32_t)(kunits * 64 * SLOT) + (x % PARTS) * 64 * CH + sl * CH;
        }
        // 64 parameters per copy: 2 of rs_x, 4 each of rs_w, h, bias
        const uint32_t dst = lds_base + 2 * STAGE + pb * PARAM + wave * 1024;
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            const int x = wave * 4 + e;
            int t = tm * BM + x * 64 + lane, nn = tn * BN + ((x - 2) & 3) * 64 + lane;
            t = t < T ? t : T - 1;
            nn = nn < N ? nn : N - 1;
            if (x < 2) copy_to_lds<4>(P.rs_x, (uint32_t)t * 4, dst + e * 256);
            else if (x < 6) copy_to_lds<4>(P.rs_w, (uint32_t)nn * 4, dst + e * 256);
            else if (x < 10) copy_to_lds<4>(P.h, (uint32_t)(nn / P.rows_per_group) * 4, dst + e * 256);
            else if (x < 14 && P.bias) copy_to_lds<4>(P.bias, (uint32_t)nn * 4, dst + e * 256);
        }
        copy_weights(0, PHASES == 2 ? 0 : par);
        copy_tokens(0, par);
    };
    // every wavefront's copies have landed and its LDS reads have returned; then the barrier
    auto fence = [&]() {
        __builtin_amdgcn_s_waitcnt(0xC07F);  // lgkmcnt(0)
        asm volatile("" ::: "memory");
        __builtin_amdgcn_sched_barrier(0);
        __builtin_amdgcn_s_barrier();
        __builtin_amdgcn_sched_barrier(0);
        asm volatile("" ::: "memory");
    };

    int work = blockIdx.x, pb = 0;  // (the grid has at most as many workgroups as there are tiles)
    int lt = logical_tile(work, nwg);
    int tm = lt / tiles_n, tn = lt - tm * tiles_n;
    start_tile(tm, tn, 0, 0);
    wait_vmcnt<0>();
    int par = 0;
    while (true) {
        v4i acc[2][2][4][2];
#pragma unroll
        for (int i = 0; i < 2; ++i)
#pragma unroll
            for (int j = 0; j < 2; ++j)
#pragma unroll
                for (int mb = 0; mb < 4; ++mb)
#pragma unroll
                    for (int nb = 0; nb < 2; ++nb) acc[i][j][mb][nb] = v4i{0, 0, 0, 0};
        const int nwork = work + gridDim.x;
        int ntm = 0, ntn = 0;
        if (nwork < nwg) {
            lt = logical_tile(nwork, nwg);
            ntm = lt / tiles_n;
            ntn = lt - ntm * tiles_n;
        }
        for (int s = 0; s < steps; ++s) {
            if constexpr (BITS == 8) {
                const uint8_t *sa = lds + par * STAGE;
                par ^= 1;
#pragma unroll
                for (int ph = 0; ph < 2; ++ph) {
                    fence();
                    // over the weights of the phase before; in the first phase the next step's tokens too, over those of the
                    // step before; in the last phase the next tile's first operands and its parameters
                    if (ph == 0) {
                        copy_weights(2 * s + 1, 1);
                        if (s + 1 < steps) copy_tokens(s + 1, par);
                    } else if (s + 1 < steps) copy_weights(2 * s + 2, 0);
                    else if (nwork < nwg) start_tile(ntm, ntn, pb ^ 1, par);
                    v4i a[2][4], b[2][2];
#pragma unroll
                    for (int j = 0; j < 2; ++j)
#pragma unroll
                        for (int nb = 0; nb < 2; ++nb) b[j][nb] = *reinterpret_cast<const v4i *>(lds + ph * STAGE + j * LPAIR + (b_fr ^ (nb * B_NEXT)));
#pragma unroll
                    for (int i = 0; i < 2; ++i)
#pragma unroll
                        for (int mb = 0; mb < 4; ++mb) a[i][mb] = *reinterpret_cast<const v4i *>(sa + a_fr[ph] + (i * 4 + mb) * 16 * BK);
                    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
                    for (int j = 0; j < 2; ++j)
#pragma unroll
                        for (int nb = 0; nb < 2; ++nb)
#pragma unroll
                            for (int e = 0; e < 4; ++e) b[j][nb][e] ^= (int)0x80808080u;  // u - 128 as int8
#pragma unroll
                    for (int i = 0; i < 2; ++i)
#pragma unroll
                        for (int j = 0; j < 2; ++j)
#pragma unroll
                            for (int mb = 0; mb < 4; ++mb)
#pragma unroll
                                for (int nb = 0; nb < 2; ++nb)
                                    acc[i][j][mb][nb] = __builtin_amdgcn_mfma_i32_16x16x64_i8(a[i][mb], b[j][nb], acc[i][j][mb][nb], 0, 0, 0);
                    if (ph == 0) {
                        if (s + 1 < steps) wait_vmcnt<4>();  // the weights; the tokens behind them have another phase
                        else wait_vmcnt<0>();
                    } else if (s + 1 < steps) wait_vmcnt<0>();
                }
                continue;
            }
            fence();
            const uint8_t *st_ = lds + par * STAGE;
            par ^= 1;
            // over the stage that was read in the step before; in the last step the next tile's first operands and its
            // parameters, so that the address arithmetic and the latency lie under the MFMAs
            if (s + 1 < steps) {
                copy_weights(s + 1, par);
                copy_tokens(s + 1, par);
            } else if (nwork < nwg) start_tile(ntm, ntn, pb ^ 1, par);
            v4i a[2][4][2], b[2][2][2];
            uint32_t raw[2][2][BITS];
#pragma unroll
            for (int j = 0; j < 2; ++j) {
                const uint8_t *bp = st_ + j * LPAIR;
                if constexpr (BITS == 2) {
                    const v4u v = *reinterpret_cast<const v4u *>(bp + b_fr);
                    raw[j][0][0] = v[0]; raw[j][0][1] = v[1]; raw[j][1][0] = v[2]; raw[j][1][1] = v[3];
                } else {
                    SlotRead<BITS>::get(bp + b_fr, raw[j][0]);
                    SlotRead<BITS>::get(bp + (b_fr ^ 16), raw[j][1]);
                }
            }
#pragma unroll
            for (int i = 0; i < 2; ++i)
#pragma unroll
                for (int kk = 0; kk < 2; ++kk)
#pragma unroll
                    for (int mb = 0; mb < 4; ++mb) a[i][mb][kk] = *reinterpret_cast<const v4i *>(st_ + a_fr[kk] + (i * 4 + mb) * 16 * BK);
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int i = 0; i < 2; ++i)
#pragma unroll
                for (int j = 0; j < 2; ++j) {
                    if (i == 0) {
#pragma unroll
                        for (int nb = 0; nb < 2; ++nb) {
                            uint32_t d[8];
                            unpack_run<BITS>(raw[j][nb], d);
#pragma unroll
                            for (int e = 0; e < 8; ++e) b[j][nb][e >> 2][e & 3] = (int)d[e];
                        }
                    }
#pragma unroll
                    for (int kk = 0; kk < 2; ++kk)
#pragma unroll
                        for (int mb = 0; mb < 4; ++mb)
#pragma unroll
                            for (int nb = 0; nb < 2; ++nb)
                                acc[i][j][mb][nb] = __builtin_amdgcn_mfma_i32_16x16x64_i8(a[i][mb][kk], b[j][nb][kk], acc[i][j][mb][nb], 0, 0, 0);
                }
            if (s + 1 < steps) wait_vmcnt<0>();
        }

        // ---- write-out
        const DuoArgs &P = args();
        const int T = P.T, N = P.N, K = P.K, t0 = tm * BM, n0 = tn * BN;
        const float hx = P.hx;
        const bool has_bias = P.bias != nullptr;
        float *__restrict__ Y = P.Y;
        int32_t *__restrict__ A4out = P.A4out;
        const uint8_t *pp = lds + 2 * STAGE + pb * PARAM;
        pb ^= 1;

        const int wl = lane_again(), q16 = wl & 15, hq = wl >> 4;
        const int *p_rx = reinterpret_cast<const int *>(pp) + 4 * hq;
        const int nl = wave * 64 + 2 * q16;  // + 32*j + b
        int coln[2][2];
        float scale[2][2], bv[2][2];
#pragma unroll
        for (int j = 0; j < 2; ++j) {
            const int2 rw = *reinterpret_cast<const int2 *>(pp + 512 + (nl + 32 * j) * 4);
            const float2 hg = *reinterpret_cast<const float2 *>(pp + 1536 + (nl + 32 * j) * 4);
            float2 bb = make_float2(0.0f, 0.0f);
            if (has_bias) bb = *reinterpret_cast<const float2 *>(pp + 2560 + (nl + 32 * j) * 4);
            coln[j][0] = 2 * rw.x + K; coln[j][1] = 2 * rw.y + K;
            scale[j][0] = hx * hg.x; scale[j][1] = hx * hg.y;
            bv[j][0] = bb.x; bv[j][1] = bb.y;
        }
        const bool fast = t0 + BM <= T && n0 + BN <= N && A4out == nullptr && (N & 1) == 0 && (reinterpret_cast<uintptr_t>(Y) & 7) == 0;
        if (fast) {
            // a wavefront-uniform row address and the lane's 32-bit byte offset
            uint8_t *out0 = reinterpret_cast<uint8_t *>(Y + (size_t)t0 * N + n0 + wave * 64);
            const uint32_t lane_off = (uint32_t)(4 * hq * N + 2 * q16) * 4u;
#pragma unroll
            for (int i = 0; i < 2; ++i)
#pragma unroll
                for (int mb = 0; mb < 4; ++mb) {
                    const int4 rx = *reinterpret_cast<const int4 *>(p_rx + i * 64 + mb * 16);
                    const int er[4] = {qb_mad24(E2, rx.x, 0), qb_mad24(E2, rx.y, 0), qb_mad24(E2, rx.z, 0), qb_mad24(E2, rx.w, 0)};
#pragma unroll
                    for (int c = 0; c < 4; ++c) {
                        uint8_t *row = out0 + (size_t)(i * 64 + mb * 16 + c) * N * 4;
#pragma unroll
                        for (int j = 0; j < 2; ++j) {
                            typedef float v2f __attribute__((ext_vector_type(2)));
                            v2f o;
#pragma unroll
                            for (int nb = 0; nb < 2; ++nb)
                                o[nb] = scale[j][nb] * (float)qb_a4(acc[i][j][mb][nb][c], er[c] + coln[j][nb]) + bv[j][nb];
                            __builtin_nontemporal_store(o, reinterpret_cast<v2f *>(row + 128 * j + lane_off));
                        }
                    }
                }
            // 64 stores behind the copies: with at most 63 operations outstanding the copies have landed
            wait_vmcnt<63>();
        } else {  // edge tiles and the debug output: every element checked
#pragma unroll
            for (int i = 0; i < 2; ++i)
#pragma unroll
                for (int mb = 0; mb < 4; ++mb)
#pragma unroll
                    for (int c = 0; c < 4; ++c) {
                        const int t = t0 + i * 64 + mb * 16 + 4 * hq + c;
                        const int er = E2 * p_rx[i * 64 + mb * 16 + c];
                        if (t < T) {
#pragma unroll
                            for (int j = 0; j < 2; ++j)
#pragma unroll
                                for (int nb = 0; nb < 2; ++nb) {
                                    const int nn = n0 + nl + 32 * j + nb;
                                    if (nn < N) {
                                        const int a4 = qb_a4(acc[i][j][mb][nb][c], er + coln[j][nb]);
                                        const size_t at = (size_t)t * N + nn;
                                        Y[at] = scale[j][nb] * (float)a4 + bv[j][nb];
                                        if (A4out) A4out[at] = a4;
                                    }
                                }
                        }
                    }
            wait_vmcnt<0>();
        }
        if (nwork >= nwg) break;
        work = nwork; tm = ntm; tn = ntn;
    }
}

// Adds one problem to a launch list of the role-split kernel with BM x BN tiles; false when the list is full.
template <int BM, int BN>
bool group_add(Group &g, const int8_t *Xq, const int32_t *rs_x, const uint8_t *packed, const float *h, const int32_t *rs_w,
               const float *bias, float *Y, int32_t *A4, int T, int N, int K, int rpg, float hx, const OutQ &oq)
{
    if (g.n >= kMaxGroup) return false;
    Problem &P = g.p[g.n];
    P.Xq = Xq; P.rs_x = rs_x; P.packed = packed; P.h = h; P.rs_w = rs_w; P.bias = bias; P.Y = Y; P.A4out = A4;
    P.T = T; P.N = N; P.K = K; P.rows_per_group = rpg; P.hx = hx;
    P.tiles_m = (T + BM - 1) / BM;
    P.tiles_n = (N + BN - 1) / BN;
    P.oq = oq;
    const int nwg = P.tiles_m * P.tiles_n;
    if (g.n == 0) g.tile_start[0] = 0;
    // a problem's share of the sequence is padded to a multiple of 8 (the last one needs no padding)
    g.tile_start[g.n] = (g.tile_start[g.n] + 7) & ~7;
    g.tile_start[g.n + 1] = g.tile_start[g.n] + nwg;
    ++g.n;
    return true;
}

// One launch for the whole list: a persistent grid of at most grid_cap workgroups (a multiple of 8).
template <int BITS, int TM, int TN, int WM, int WN, int NSTAGE, int NPROD, bool SIMD3, int OUT>
void launch_group(const Group &g, hipStream_t st, int grid_cap)
{
    int grid = g.tile_start[g.n];
    if (grid_cap > 0 && grid > grid_cap) grid = grid_cap;
    hipLaunchKernelGGL((qgemm_i8_ws_kernel<BITS, TM, TN, WM, WN, NSTAGE, NPROD, SIMD3, OUT>), dim3(grid),
                       dim3(64 * (WM * WN + NPROD)), 0, st, g);
}

template <int BITS, int TM, int TN, int WM, int WN, int NSTAGE, int NPROD, bool SIMD3 = false>
void launch_ws(const int8_t *Xq, const int32_t *rs_x, const uint8_t *packed, const float *h, const int32_t *rs_w,
               const float *bias, float *Y, int32_t *A4, int T, int N, int K, int rpg, float hx, hipStream_t st,
               int grid_cap, const float *hx_rows = nullptr, const float *q0 = nullptr)
{
    constexpr int BM = WM * TM * 32, BN = WN * TN * 32;
    const OutQ oq{nullptr, nullptr, 1.0f, 0, hx_rows, q0};
    Group g;
    g.n = 0;
    group_add<BM, BN>(g, Xq, rs_x, packed, h, rs_w, bias, Y, A4, T, N, K, rpg, hx, oq);
    if (q0) launch_group<BITS, TM, TN, WM, WN, NSTAGE, NPROD, SIMD3, 2>(g, st, grid_cap);
    else launch_group<BITS, TM, TN, WM, WN, NSTAGE, NPROD, SIMD3, 0>(g, st, grid_cap);
}

// the same with the 8-bit output
template <int BITS, int TM, int TN, int WM, int WN, int NSTAGE, int NPROD, bool SIMD3 = false>
void launch_ws_q8(const int8_t *Xq, const int32_t *rs_x, const uint8_t *packed, const float *h, const int32_t *rs_w,
                  const float *bias, const OutQ &oq, int T, int N, int K, int rpg, float hx, hipStream_t st, int grid_cap)
{
    constexpr int BM = WM * TM * 32, BN = WN * TN * 32;
    Group g;
    g.n = 0;
    group_add<BM, BN>(g, Xq, rs_x, packed, h, rs_w, bias, nullptr, nullptr, T, N, K, rpg, hx, oq);
    if (oq.act == 1) launch_group<BITS, TM, TN, WM, WN, NSTAGE, NPROD, SIMD3, 3>(g, st, grid_cap);
    else launch_group<BITS, TM, TN, WM, WN, NSTAGE, NPROD, SIMD3, 1>(g, st, grid_cap);
}

template <int BITS, int TM, int TN, int WM, int WN, int KU>
void launch_cfg(const int8_t *Xq, const int32_t *rs_x, const uint8_t *packed, const float *h, const int32_t *rs_w,
                const float *bias, float *Y, int32_t *A4, int T, int N, int K, int rpg, float hx, hipStream_t st,
                const float *hx_rows = nullptr, const float *q0 = nullptr)
{
    constexpr int BM = WM * TM * 32, BN = WN * TN * 32;
    const int tiles_m = (T + BM - 1) / BM, tiles_n = (N + BN - 1) / BN;
    auto *kernel = hx_rows || q0 ? qgemm_i8_kernel<BITS, TM, TN, WM, WN, KU, true> : qgemm_i8_kernel<BITS, TM, TN, WM, WN, KU, false>;
    hipLaunchKernelGGL(kernel, dim3(tiles_m * tiles_n), dim3(64 * WM * WN), 0, st, Xq, rs_x, packed, h, rs_w, bias, Y, A4, T, N, K, rpg, hx, tiles_m, tiles_n, hx_rows, q0);
}

// grid_cap: upper bound of workgroups (a multiple of 8); 0 = one workgroup per tile
template <int BITS, int TM, int TN, int WM, int WN, int NSTAGE>
void launch_dma(const int8_t *Xq, const int32_t *rs_x, const uint8_t *packed, const float *h, const int32_t *rs_w,
                const float *bias, float *Y, int32_t *A4, int T, int N, int K, int rpg, float hx, hipStream_t st,
                int grid_cap = 0)
{
    constexpr int BM = WM * TM * 32, BN = WN * TN * 32;
    const int tiles_m = (T + BM - 1) / BM, tiles_n = (N + BN - 1) / BN;
    int grid = tiles_m * tiles_n;
    if (grid_cap > 0 && grid > grid_cap) grid = grid_cap;
    hipLaunchKernelGGL((qgemm_i8_dma_kernel<BITS, TM, TN, WM, WN, NSTAGE>), dim3(grid), dim3(64 * WM * WN), 0, st,
                       Xq, rs_x, packed, h, rs_w, bias, Y, A4, T, N, K, rpg, hx, tiles_m, tiles_n);
}

// The stepped kernel's units of 64 features per step, and its steps.
inline int stepped_units(int K) { return (K % 256 == 0 && K >= 2048) ? 4 : (K % 128 == 0) ? 2 : 1; }
inline int stepped_steps(int K) { return K / (64 * stepped_units(K)); }

// Which few-tile problems have their contraction sliced (tiles of 32 x 64): up to one workgroup per CU, and a contraction of
// more than three steps of the other kernel (with fewer there is no latency to save, but the sum of the slices to pay), or
// less than one tile of tokens, where the other kernel checks every element it writes.  Times in us behind the activation
// quantizer that wrote the tokens, both kernels together, sliced / stepped, 4 bits:
//   256 x 768, K = 128 6.2 / 5.4, 256 6.3 / 5.9, 384 6.5 / 6.4, 448 6.1 / 7.4, 512 6.5 / 6.8, 768 6.7 / 7.7, 1024 6.8 / 8.5
//   16 x 1536, K = 256 5.8 / 6.2, 384 6.0 / 6.8;     24 x 768, K = 192 5.7 / 6.7
// Alone, 156 tiles, K = 3072 6.7 / 7.7 (4 bits), 7.4 / 8.1 (8 bits); but 468 tiles of 8 bits, K = 768 7.5 / 5.6 and 564 tiles,
// K = 3072 13.9 / 11.0 (the direct loads then wait for the L1s).
inline bool sliced_pays(int T, int K) { return stepped_steps(K) > 3 || (T < 32 && K >= 192); }
inline bool split_shape(long tiles, int T, int K) { return tiles <= 256 && sliced_pays(T, K); }

// Which problems take tiles of 32 x 64, sliced (split_shape) or of the register-staged kernel, instead of the larger ones: few tiles
// (small token counts, the inference regime), where the persistent kernels leave most CUs idle and pay 6.5 us at least (1024 x 768 x
// 768 4.4-5 us against 8; equal at about 190 tiles of 128 x 128).  Up to one such tile a CU they are ahead too where 128 x 96 tiles would
// need a second round for a few of them.  Time / time with the larger tiles, behind the activation quantizer:
//   second round of 128 x 96 tiles, K = 256 to 512 .86-.98 (4 bits), .88-.94 (3), .91-1.0 (8);  768 .93-.99, .93-1.0, .91-1.01;  1024 .92-1.0,
//   .95-1.05, .94-1.08;  with a range per token K up to 1024 .93-1.0, .87-1.01, .85-1.0;  K >= 2048 1.01-1.39
//   N = 128 to 704, 161 to 256 tiles of 128 x 128 (lowest to highest of all widths, with one range and with one per token):  K = 128
//   .74-.93, .77-.98;  256 .80-.97, .79-1.02;  512 .86-.98, .89-1.01;  640 .87-1.01, .90-1.02;  768 .88-1.04, .91-1.06
//   first round (162 to 190 tiles) .91-1.11;  289 to 384 tiles of 128 x 128 .85-1.15
// K no multiple of 128, where the larger tiles are register-staged ones of 128 x 128, 4, 3 and 8 bits:
//   161 to 200 tiles .70-.84, 257 to 300 .83-.94;  346 to 360, K <= 704 .87-.99, 960 .97-1.06;  414 to 420 .92-1.01, 1.0-1.14
template <int BITS>
bool small_tiles_shape(int T, int N, int K, bool gen)
{
    const long tiles_m = (T + 127) / 128, tiles128 = tiles_m * ((N + 127) / 128), tiles96 = tiles_m * ((N + 95) / 96);
    if (tiles128 <= 160) return true;
    if (K % 128 != 0) return K <= 1024 && tiles128 <= (K <= 704 ? 384 : 320);
    return tiles128 <= 256 && tiles96 > 256 && K <= (N < 768 ? 640 : gen || BITS == 2 || BITS == 4 ? 1024 : 768);
}

// Which problems go to the 128 x 256 kernel with two independent workgroups per CU.  Its tiles are the largest, so it
// needs two full rounds of the 512 resident workgroups (1024 tiles); with long contractions, whose tiles are started and
// written out more rarely, and at 8 bits three quarters of one.  At most an eighth of the columns may be padding.  Time / time with the
// kernels of the rules below, behind the activation quantizer, lowest to highest of 2 to 4 bits; n2 and n1: the most tiles of 128 x 256 and
// of 128 x 128 on a CU:
//   K = 512 to 1024   (n1, n2) = (8,4) .86-.95, (9,5) .81-1.08, (10,5) .81-.97, (11,6) .85-1.06, (12,6) .87-.97, (15,8) .95-1.05, above .78-1.04
//   K < 512           (8,4) .96-.99, (9,5) .92-1.08, (10,5) .95-.97, (11,6) 1.04-1.09, (12,6) .95-1.0: with so short a contraction
//                     tiles are mostly start and write-out, and the odd one of a CU has nothing beside it
//   K >= 2048         (3,2) .92-1.09, (4,2) .73-.98, (5,3) 1.04-1.29, (6,3) .72-1.07, (7,4) .69-1.05, (8,4) .68-.93, (9,5) .99-1.08,
//                     above .79-.99: the third tile of a CU runs alone for 0.7 of a pair's time
//   N = 1152, 1920, 2688 (the last column of tiles half empty and written element by element; the 128 x 128 tiles fill theirs)
//                     1.03-1.05, 1.14-1.34, .89-1.16
//   N = 998 to 3520, no multiple of 128, K <= 1024 .35-1.04;  no multiple of 4 (no 16-byte rows), K >= 2048 .63-1.0
// 8 bits, where the other kernels read the most from LDS:
//   K = 512 to 1280   (3,2) .98-1.10, (4,2) .75-.98, (5,3) .89-1.12, (6,3) .86-.98, (7,4) .78-.98, (8,4) .90, (9,5) .76-.94, above .75-.91
//   K < 512           (4,2) .82-1.16, (5,3) .93-1.05, (6,3) .99-1.02, (7,4) .96-1.14, (10,5) .82
//   K >= 2048         (3,2), 384 tiles .93-.97, fewer .93-1.02, (4,2) .84-.90, (5,3) .92-1.03, (6,3) .90-.96, (8,4) .83-.88, one tile a CU .94-1.16
//   N = 1152, 1920, 2688 1.00-1.09;  no multiple of 4, 384 to 923 tiles .64-.87
template <int BITS>
bool duo_shape(int T, int N, int K)
{
    const long tiles_m = (T + 127) / 128, tiles_n = (N + 255) / 256, tiles = tiles_m * tiles_n;
    const bool long_k = K >= 2048;
    if (K % 128 != 0 || tiles < (long_k || (BITS == 8 && K >= 512) ? 384 : 1024) || (tiles_n * 256 - N) * 8 > N) return false;
    const long n1 = (tiles_m * ((N + 127) / 128) + 255) / 256, n2 = (tiles + 255) / 256;
    const long rounds = 100 * n2 + 40 * (n2 & 1);
    if constexpr (BITS == 8) {
        if (N % 4 != 0) return true;
        return (N % 256 == 0 || N % 128 != 0) && (K >= 512 || n1 >= 2 * n2) && rounds < (long_k ? 67 : 62) * n1;
    }
    if (N % 4 != 0 || (N % 128 != 0 && !long_k)) return true;
    if (long_k) return rounds < 67 * n1;
    return N % 256 == 0 && (K >= 512 || n1 >= 2 * n2);
}

template <int BITS>
void launch_duo(const int8_t *Xq, const int32_t *rs_x, const uint8_t *packed, const float *h, const int32_t *rs_w,
                const float *bias, float *Y, int32_t *A4, int T, int N, int K, int rpg, float hx, hipStream_t st)
{
    const DuoJob j{{{Xq, rs_x, packed, h, rs_w, bias, Y, A4, T, N, K, rpg, hx, (T + 127) / 128, (N + 255) / 256}}};
    const int tiles = j.p[0].tiles_m * j.p[0].tiles_n;
    hipLaunchKernelGGL((qgemm_i8_duo_kernel<BITS>), dim3(tiles < 512 ? tiles : 512), dim3(256), 0, st, j);
}

// Which single calls go to the lists' kernel (qgemm_i8_list.hip, 128 x 256 tiles): what the kernel above does not take, with at least most of a
// round of the 512 resident workgroups and rounds that are full enough.  Time / time with the other kernels, behind the activation
// quantizer; f: the part of the rounds' places that is taken:
//   per-token scales and asymmetric ranges, K = 768 to 4096, 2 to 8 bits: f = 1 .77-1.0, .94 .82-.92, .84 .92-.96, .75 (768 and 1152 tiles) .89-.97
//   and (384 tiles) .94-1.08, .56 and less .89-1.7
//   K no multiple of 128: K = 960, f = .94 .76-.94, .90 .78-.84, .75 .91-1.15; K = 704, f = .83 .82-.86, .69 .93-1.08; K = 448 .90-1.5;
//   a tenth of the columns padding 1.03-1.2 below 1700 tiles
inline bool general_shape(int T, int N, int K, bool gen)
{
    const long tiles_n = (N + 255) / 256, tiles = (long)((T + 127) / 128) * tiles_n, places = (tiles + 511) / 512 * 512;
    if (K % 128 == 0) return gen && K >= 512 && tiles >= 480 && tiles * 100 >= 72 * places && (tiles_n * 256 - N) * 8 <= N;
    return K >= 640 && tiles >= 448 && tiles * 100 >= 80 * places && (tiles_n * 256 - N) * 12 <= N;
}

// The kernel of a call: tiles of 32 x 64, sliced or stepped; of 128 x 128 staged through registers (K no multiple of 128); of 128 x 256; role-split
// ones of 128 x 96, two workgroups per CU or one, and of 128 x 128; plain ones of 128 x 128, two workgroups per CU; the lists' kernel
enum FwdPath { kSliced, kStepped, kStaged128, kDuo256, kRoles96Two, kRoles96One, kRoles128, kPlain128, kGeneral256 };
template <int BITS>
FwdPath fwd_path_of(int T, int N, int K, bool per_token, bool asym)
{
    const long tiles128 = (long)((T + 127) / 128) * ((N + 127) / 128);
    if (small_tiles_shape<BITS>(T, N, K, per_token || asym)) return split_shape((long)((T + 31) / 32) * ((N + 63) / 64), T, K) ? kSliced : kStepped;
    if (general_shape(T, N, K, per_token || asym)) return kGeneral256;
    if (K % 128 != 0) return kStaged128;
    // (the 128 x 256 tiles' epilogue has neither per-token scales nor asymmetric ranges)
    if (!per_token && !asym && duo_shape<BITS>(T, N, K)) return kDuo256;
    // Tile choice (measured on BERT-base and BERT-large shapes).  Copies issued on a SIMD that is busy
    // with 32x32 MFMAs run at about half their stand-alone rate, so where the tile count allows it the MFMAs
    // go to three SIMDs and the copies to the fourth:
    //   128x96 tiles in that layout when they need fewer rounds over the 256 CUs than 128x128 tiles would,
    //     weighted by the measured cost of a tile (0.86 of a 128x128 one): all of BERT-base's N = 768 layers
    //     at 4096 and 12288 tokens, and N = 2304 at 4096;
    //   else 128x128: the role-split kernel (one workgroup per CU, copies run ahead across tiles) when a CU
    //     gets few tiles or the contraction is long and the tiles are few, two plain workgroups per CU when
    //     it gets many (one's write-out overlaps the other's MFMAs); this also beats 256x256 tiles on the
    //     BERT-large shapes at 32768 tokens (2.3 against 2.07 POP/s at 2 bits).
    // Grids are persistent and a multiple of 8, so that a workgroup stays inside its XCD's tile range.
    const long tiles96 = (long)((T + 127) / 128) * ((N + 95) / 96);
    const long rounds128 = (tiles128 + 255) / 256, rounds96 = (tiles96 + 255) / 256;
    // (also where 128x128 tiles would need fewer rounds, for up to five rounds of 128x96 tiles: as two workgroups per CU
    // they are 3 % ahead of the plain two-workgroup kernel on BERT-base's FFN-up)
    if (86 * rounds96 < 100 * rounds128 || (N % 96 == 0 && tiles96 > 256 && tiles96 <= 1280))
        // more tiles than CUs: two workgroups per CU, one's write-out under the other's K-loop (LDS and registers allow it
        // at 2, 3 and 4 bits; at 8 bits with two stages, for the plain fp32 output)
        return tiles96 > 256 && (BITS < 8 || !asym) ? kRoles96Two : kRoles96One;
    // (per-token scales, asymmetric ranges: role-split kernels only)
    return per_token || asym || tiles128 <= 640 || (K >= 2048 && tiles128 <= 1024) ? kRoles128 : kPlain128;
}

template <int BITS>
void launch_bits(const int8_t *Xq, const int32_t *rs_x, const uint8_t *packed, const float *h, const int32_t *rs_w,
                 const float *bias, float *Y, int32_t *A4, int T, int N, int K, int rpg, float hx, hipStream_t st,
                 const float *hx_rows = nullptr, const float *q0 = nullptr)
{
    switch (fwd_path_of<BITS>(T, N, K, hx_rows != nullptr, q0 != nullptr)) {
        case kSliced: {
            const SplitCall sc{A4, hx_rows, q0, {Xq, rs_x, packed, h, rs_w, bias, Y, T, N, K, rpg, hx, (T + 31) / 32, (N + 63) / 64}};
            hipLaunchKernelGGL((qgemm_i8_split_kernel<BITS>), dim3(sc.p.tiles_m * sc.p.tiles_n), dim3(512), 0, st, sc);
            return;
        }
        case kStepped:  // (long contractions take 256 features per step)
            if (stepped_units(K) == 4) launch_cfg<BITS, 1, 1, 1, 2, 4>(Xq, rs_x, packed, h, rs_w, bias, Y, A4, T, N, K, rpg, hx, st, hx_rows, q0);
            else if (stepped_units(K) == 2) launch_cfg<BITS, 1, 1, 1, 2, 2>(Xq, rs_x, packed, h, rs_w, bias, Y, A4, T, N, K, rpg, hx, st, hx_rows, q0);
            else launch_cfg<BITS, 1, 1, 1, 2, 1>(Xq, rs_x, packed, h, rs_w, bias, Y, A4, T, N, K, rpg, hx, st, hx_rows, q0);
            return;
        case kStaged128:  // odd number of 64-feature units: one unit per step
            launch_cfg<BITS, 2, 2, 2, 2, 1>(Xq, rs_x, packed, h, rs_w, bias, Y, A4, T, N, K, rpg, hx, st, hx_rows, q0);
            return;
        case kDuo256: launch_duo<BITS>(Xq, rs_x, packed, h, rs_w, bias, Y, A4, T, N, K, rpg, hx, st); return;
        case kRoles96Two: launch_ws<BITS, 2, 1, 2, 3, BITS < 8 ? 3 : 2, 2, true>(Xq, rs_x, packed, h, rs_w, bias, Y, A4, T, N, K, rpg, hx, st, 512, hx_rows, q0); return;
        case kRoles96One: launch_ws<BITS, 2, 1, 2, 3, 3, 2, true>(Xq, rs_x, packed, h, rs_w, bias, Y, A4, T, N, K, rpg, hx, st, 256, hx_rows, q0); return;
        case kRoles128: launch_ws<BITS, 2, 2, 2, 2, 3, 4>(Xq, rs_x, packed, h, rs_w, bias, Y, A4, T, N, K, rpg, hx, st, 256, hx_rows, q0); return;
        case kGeneral256: launch_fwd_general<BITS>(Xq, rs_x, packed, h, rs_w, bias, Y, A4, T, N, K, rpg, hx, st, hx_rows, q0); return;
        case kPlain128: launch_dma<BITS, 2, 2, 2, 2, 2>(Xq, rs_x, packed, h, rs_w, bias, Y, A4, T, N, K, rpg, hx, st, 512); return;
    }
}

// 8-bit output: the role-split kernels only (128x96 tiles on three SIMDs where they need fewer rounds, else 128x128)
template <int BITS>
void launch_bits_q8(const int8_t *Xq, const int32_t *rs_x, const uint8_t *packed, const float *h, const int32_t *rs_w,
                    const float *bias, const OutQ &oq, int T, int N, int K, int rpg, float hx, hipStream_t st)
{
    const long tiles128 = (long)((T + 127) / 128) * ((N + 127) / 128);
    const long tiles96 = (long)((T + 127) / 128) * ((N + 95) / 96);
    const long rounds128 = (tiles128 + 255) / 256, rounds96 = (tiles96 + 255) / 256;
    if (86 * rounds96 < 100 * rounds128 || (N % 96 == 0 && tiles96 > 256)) {
        // more tiles than CUs: two stages, so that two workgroups fit a CU and one's output quantizer runs under the
        // other's K-loop (then also where 128x128 tiles would need fewer rounds)
        if (tiles96 > 256) launch_ws_q8<BITS, 2, 1, 2, 3, 2, 2, true>(Xq, rs_x, packed, h, rs_w, bias, oq, T, N, K, rpg, hx, st, 512);
        else launch_ws_q8<BITS, 2, 1, 2, 3, 3, 2, true>(Xq, rs_x, packed, h, rs_w, bias, oq, T, N, K, rpg, hx, st, 256);
    } else
        launch_ws_q8<BITS, 2, 2, 2, 2, 3, 4>(Xq, rs_x, packed, h, rs_w, bias, oq, T, N, K, rpg, hx, st, 256);
}

__global__ void fill_zero_i32_kernel(int32_t *p, int n)
{
    const int i = blockIdx.x * 256 + threadIdx.x;
    if (i < n) p[i] = 0;
}

}  // namespace

int fwd_path(int bits, int T, int N, int K, bool per_token, bool asym)
{
    return bits == 2 ? fwd_path_of<2>(T, N, K, per_token, asym) : bits == 3 ? fwd_path_of<3>(T, N, K, per_token, asym)
         : bits == 4 ? fwd_path_of<4>(T, N, K, per_token, asym) : fwd_path_of<8>(T, N, K, per_token, asym);
}

}  // namespace qb

using namespace qb;

extern "C" qb_status qb_qlinear_fwd(const int8_t *Xq, const int32_t *rs_x, float clip, const void *packed,
                                    const float *h, const int32_t *rs_w, int bits, int groups, int64_t T, int64_t N,
                                    int64_t K, const float *bias, float *Y, int32_t *A4_debug, void *stream)
{
    if (!Xq || !rs_x || !packed || !h || !rs_w || !Y) return QB_ERR_NULL;
    if (!bits_ok(bits)) return QB_ERR_BITS;
    if (T <= 0 || T > (1 << 24) || N <= 0 || N > (1 << 24) || !k_ok(K) || groups <= 0 || N % groups != 0)
        return QB_ERR_SHAPE;
    if (!(clip > 0.0f) || !(clip < 3.0e38f)) return QB_ERR_CLIP;
    const float hx = clip / 255.0f;
    const int rpg = (int)(N / groups);
    hipStream_t st = static_cast<hipStream_t>(stream);
    const uint8_t *p = static_cast<const uint8_t *>(packed);
    switch (bits) {
        case 2: launch_bits<2>(Xq, rs_x, p, h, rs_w, bias, Y, A4_debug, (int)T, (int)N, (int)K, rpg, hx, st); break;
        case 3: launch_bits<3>(Xq, rs_x, p, h, rs_w, bias, Y, A4_debug, (int)T, (int)N, (int)K, rpg, hx, st); break;
        case 4: launch_bits<4>(Xq, rs_x, p, h, rs_w, bias, Y, A4_debug, (int)T, (int)N, (int)K, rpg, hx, st); break;
        default: launch_bits<8>(Xq, rs_x, p, h, rs_w, bias, Y, A4_debug, (int)T, (int)N, (int)K, rpg, hx, st); break;
    }
    return launch_status();
}

namespace {
qb_status check_fwd_job(const qb_fwd_job &j)
{
    if (!j.Xq || !j.rs_x || !j.packed || !j.h || !j.rs_w || !j.Y) return QB_ERR_NULL;
    if (!bits_ok(j.bits)) return QB_ERR_BITS;
    if (j.T <= 0 || j.T > (1 << 24) || j.N <= 0 || j.N > (1 << 24) || !k_ok(j.K) || j.groups <= 0 || j.N % j.groups != 0)
        return QB_ERR_SHAPE;
    if (!(j.clip > 0.0f) || !(j.clip < 3.0e38f)) return QB_ERR_CLIP;
    return QB_OK;
}

template <int BITS>
void launch_job(const qb_fwd_job &j, hipStream_t st)
{
    launch_bits<BITS>(j.Xq, j.rs_x, static_cast<const uint8_t *>(j.packed), j.h, j.rs_w, j.bias, j.Y, nullptr, (int)j.T, (int)j.N,
                      (int)j.K, (int)(j.N / j.groups), j.clip / 255.0f, st);
}

// A shared launch of 128x96 tiles.  Two workgroups per CU (512 resident): while one writes a tile out and starts the
// next, the other's K-loop keeps the matrix cores busy (the step's GEMM stage 196 -> 171 us).  That needs at most
// 80 KB of LDS and 128 registers: three stages at 2, 3 and 4 bits (64-73 KB, 102 registers), two stages at 8 bits.
template <int BITS>
void launch_g96(const Group &g, hipStream_t st)
{
    if (BITS == 8 && g.tile_start[g.n] > 256) launch_group<BITS, 2, 1, 2, 3, 2, 2, true, 0>(g, st, 512);
    else launch_group<BITS, 2, 1, 2, 3, 3, 2, true, 0>(g, st, 512);  // (no more than one workgroup per CU at 8 bits)
}

bool few_tiles(const qb_fwd_job &j) { return (long)((j.T + 127) / 128) * ((j.N + 127) / 128) <= 160; }

// The kernel for few-tile jobs that share a launch: with the contraction sliced or stepped; compiled for the width and (stepped) the units of 64
// features per step that all of them have, or for any (0)
struct FewTilesKernel {
    bool sliced;
    int bits, units;
};
FewTilesKernel few_tiles_kernel(const qb_fwd_job *const *jobs, int n_jobs)
{
    FewTilesKernel k{false, -1, -1};
    long tiles = 0, wgs = 0;
    int longest = 0;
    auto common = [](int &all, int one) { all = all == -1 || all == one ? one : 0; };
    for (int i = 0; i < n_jobs; ++i) {
        const long t = (long)((jobs[i]->T + 31) / 32) * ((jobs[i]->N + 63) / 64);
        const int K = (int)jobs[i]->K;
        tiles += t;
        wgs += (t + 7) & ~7l;
        longest = stepped_steps(K) > longest ? stepped_steps(K) : longest;
        k.sliced = k.sliced || sliced_pays((int)jobs[i]->T, K);
        common(k.bits, jobs[i]->bits);
        common(k.units, stepped_units(K));
    }
    k.sliced = k.sliced && tiles <= 256 && (wgs <= 256 || longest > 12);
    if (k.bits == 0 || k.sliced) k.units = 0;
    // Different steps at one width: 2304 workgroups of its kernel are resident (the LDS of 256 features a step) and 1536 of the one for everything.
    // Where that takes it no fewer rounds, fewer at a time are the faster way, the longest contractions being the first.  It / the kernel for
    // everything, a layer's linears or several, 2 to 8 bits: up to 1200 workgroups .96-1.06, 1536 .96-1.05, 2304 .81-1.03, 3072 .82-1.16, above .85-1.05.
    if (!k.sliced && k.units == 0 && (wgs + 2303) / 2304 == (wgs + 1535) / 1536) k.bits = 0;
    return k;
}

template <int BITS>
void launch_small_group(const SmallGroup &g, const FewTilesKernel &k, hipStream_t st)
{
    const dim3 grid(g.first_wg[g.n]);
    if (k.sliced) hipLaunchKernelGGL((qgemm_i8_split_list_kernel<BITS>), grid, dim3(512), 0, st, g);
    else {
        auto *kernel = qgemm_i8_small_list_kernel<BITS, 0>;
        if constexpr (BITS != 0)
            if (k.units) kernel = k.units == 1 ? qgemm_i8_small_list_kernel<BITS, 1> : k.units == 2 ? qgemm_i8_small_list_kernel<BITS, 2> : qgemm_i8_small_list_kernel<BITS, 4>;
        hipLaunchKernelGGL(kernel, grid, dim3(128), 0, st, g);
    }
}

// The few-tile jobs of a call, whatever their widths, side by side in one launch; of more jobs than a launch holds those of a width together (64
// jobs of four widths, us, in the order of the call / by width: hidden 320, 8 tokens 21.6 / 16.0; 1024, 200 tokens 140 / 113)
template <typename Launch>
void each_few_tiles_launch(const qb_fwd_job *jobs, int n_jobs, Launch launch)
{
    int total = 0;
    for (int i = 0; i < n_jobs; ++i) total += few_tiles(jobs[i]);
    const qb_fwd_job *order[QB_MAX_BATCH];
    int n = 0;
    constexpr int widths[] = {2, 3, 4, 8};
    for (int w = 0; w < (total > QB_MAX_BATCH ? 4 : 1); ++w)
        for (int i = 0; i < n_jobs; ++i)
            if (few_tiles(jobs[i]) && (total <= QB_MAX_BATCH || jobs[i].bits == widths[w])) {
                // (the longest contractions first: the launch ends when the last of them does)
                int k = n++;
                for (; k > 0 && order[k - 1]->K < jobs[i].K; --k) order[k] = order[k - 1];
                order[k] = &jobs[i];
                if (n == QB_MAX_BATCH) {
                    launch(order, n);
                    n = 0;
                }
            }
    if (n) launch(order, n);
}
void launch_few_tiles(const qb_fwd_job *jobs, int n_jobs, hipStream_t st)
{
    each_few_tiles_launch(jobs, n_jobs, [st](const qb_fwd_job *const *order, int n) {
        SmallGroup g;
        g.n = n;
        g.first_wg[0] = 0;
        for (int i = 0; i < n; ++i) {
            const qb_fwd_job &j = *order[i];
            SmallProblem &sp = g.p[i];
            sp.Xq = j.Xq; sp.rs_x = j.rs_x; sp.packed = static_cast<const uint8_t *>(j.packed); sp.h = j.h; sp.rs_w = j.rs_w;
            sp.bias = j.bias; sp.Y = j.Y; sp.T = (int)j.T; sp.N = (int)j.N; sp.K = (int)j.K;
            sp.rows_per_group = (int)(j.N / j.groups); sp.hx = j.clip / 255.0f;
            sp.tiles_m = (int)((j.T + 31) / 32); sp.tiles_n = (int)((j.N + 63) / 64);
            sp.kind = j.bits | stepped_units((int)j.K) << 8;
            g.first_wg[i + 1] = g.first_wg[i] + ((sp.tiles_m * sp.tiles_n + 7) & ~7);
        }
        const FewTilesKernel kernel = few_tiles_kernel(order, n);
        switch (kernel.bits) {
            case 2: launch_small_group<2>(g, kernel, st); break;
            case 3: launch_small_group<3>(g, kernel, st); break;
            case 4: launch_small_group<4>(g, kernel, st); break;
            case 8: launch_small_group<8>(g, kernel, st); break;
            default: launch_small_group<0>(g, kernel, st); break;
        }
    });
}

// The tile choice of the single call (launch_bits) for a job of more tiles: problems it gives to a role-split kernel share launches (one
// per width and tile shape), the others (K not a multiple of 128, many tiles: two plain workgroups per CU) go one by one ...
enum LargeJob { kAlone, kShared96, kShared128 };
template <int BITS>
LargeJob large_job(const qb_fwd_job &j)
{
    const long tiles128 = (long)((j.T + 127) / 128) * ((j.N + 127) / 128);
    const long tiles96 = (long)((j.T + 127) / 128) * ((j.N + 95) / 96);
    const long rounds128 = (tiles128 + 255) / 256, rounds96 = (tiles96 + 255) / 256;
    const bool few128 = tiles128 <= 640 || (j.K >= 2048 && tiles128 <= 1024);
    // ... except that a problem which alone would run as two plain workgroups per CU joins the 128x96 list when 96
    // divides its N and it has no more than five rounds of tiles: inside a shared launch it pays no start-up of its
    // own and its tiles fill the rounds the other problems leave ragged (BERT-base FFN-up at 4096 tokens: the
    // step's GEMM stage 212 -> 197 us; with twelve and more rounds, at 12288 tokens or BERT-large's 32768, the two
    // workgroups per CU stay 3-5 % ahead)
    const bool use96 = 86 * rounds96 < 100 * rounds128 || (!few128 && j.N % 96 == 0 && tiles96 <= 1280);
    // (at 8 bits the shared launch keeps what has fewer than 1024 tiles of 128 x 256: the rule is of single calls)
    const bool alone = duo_shape<BITS>((int)j.T, (int)j.N, (int)j.K) && (BITS < 8 || (j.T + 127) / 128 * ((j.N + 255) / 256) >= 1024);
    if (j.K % 128 != 0 || !(use96 || few128) || alone) return kAlone;
    return use96 ? kShared96 : kShared128;
}

// Whether a call's jobs go through launch_fwd_list, all widths in one launch, by an estimate of both sides in us.
// The list: the longest tile alone on its CU, 1.2 a step and 4, and the tiles of a workgroup if all had the same, 1.75 a step and 5 for each
// tile, 12 at least, the time of its write-out where all write; the smaller of the two counts a third.  Where one job is nine tenths of the work
// its ragged last round counts, a CU with one workgroup at .7 of the time of two.  The other kernels: few-tile jobs of all
// widths share a launch, 6 and 1.1 a GOP; then a launch per width and kind of tile, .69 a GOP (1.0 where K is no multiple of 128) or the
// output at 3.5 TB/s, and 4 each.  Jobs that go alone to tiles of 128 x 256 as well have the list's rounds without what a list costs a tile: the
// two-workgroup kernel .93 of the list's time, from K = 2048 on .87 (time / the list's, 16384 to 32768 tokens: K = 768 .90-.96, 1024 .88-.94, 3072 and
// 4096 .84-.91; the more bits the lower), this kernel compiled for one width .95.  One such job alone goes there without an estimate.
// Of 1400 calls of one job to 40, 200 to 65000 tokens, hidden 256 to 1536, the side so chosen takes .4 % longer than the faster one on average.
// Four linears of a layer, list / other kernels: hidden 768, widths 2, 3, 4 and 8, 512 tokens 42.8 / 35.7 us, 768 45.6 / 48.2, 1024 48.8 / 73.9, 2048
// 75 / 144, 3072 108 / 207, 4096 147 / 172, 6144 214 / 273; two widths, 1024 tokens 41.4 /
// 35.4, 2048 42.7 / 68.2, 4096 76.9 / 81.7; 4 bits alone, 1536 tokens 37.5 / 32.1, 3072 39.9 / 46.0, 4096 44.5 / 38.5, 6144 55.1 / 63.6; hidden
// 320, four widths, 1024 tokens 26.9 / 21.0, 2048 32.0 / 36.7 (by the estimate the other way); hidden 448, four widths, 4096 tokens 80 / 149.  Hidden
// 1024 at 32768 tokens, one width: 2 bits 439 / 412, 3 bits 480 / 458, 4 bits 468 / 431, 8 bits 526 / 471; 32768 x 1024 x 4096 alone 120 / 104
// (2 bits) and 147 / 124 (8 bits).
inline bool list_pays(const qb_fwd_job *jobs, int n_jobs)
{
    auto steps_of = [](const qb_fwd_job &j) { return (double)((j.K + 127) / 128); };
    auto tiles_of = [](const qb_fwd_job &j) { return (double)((j.T + 127) / 128) * (double)((j.N + 255) / 256); };
    auto tile_time = [&](const qb_fwd_job &j) { return 1.75 * steps_of(j) + 5.0 > 12.0 ? 1.75 * steps_of(j) + 5.0 : 12.0; };
    // the tiles of a CU, two at a time
    auto rounds_of = [&](const qb_fwd_job &j) {
        const long n = ((long)tiles_of(j) + 255) / 256;
        return (double)(n / 2) + 0.7 * (double)(n & 1);
    };
    double list = 0.0, other = 0.0, few = 0.0;
    for (int at = 0; at < n_jobs; at += QB_MAX_BATCH) {
        double longest = 0.0, work = 0.0, most = 0.0, ragged = 0.0;
        for (int i = at; i < n_jobs && i < at + QB_MAX_BATCH; ++i) {
            const qb_fwd_job &j = jobs[i];
            const double alone = 1.2 * steps_of(j) + 4.0, even = tiles_of(j) * tile_time(j) / 512.0;
            longest = alone > longest ? alone : longest;
            work += even;
            if (even > most) {
                most = even;
                ragged = rounds_of(j) * tile_time(j) - even;
            }
        }
        if (most >= 0.9 * work) work += ragged;
        list += 5.0 + (longest > work ? longest + 0.3 * work : work + 0.3 * longest);
    }
    unsigned shared = 0;
    for (int i = 0; i < n_jobs; ++i) {
        const qb_fwd_job &j = jobs[i];
        const double gop = 2e-9 * (double)j.T * (double)j.N * (double)j.K;
        if (few_tiles(j)) {
            few += (few == 0.0 ? 6.0 : 0.0) + 1.1 * gop;
            continue;
        }
        const LargeJob kind = j.bits == 2 ? large_job<2>(j) : j.bits == 3 ? large_job<3>(j) : j.bits == 4 ? large_job<4>(j) : large_job<8>(j);
        const int path = kind == kAlone ? fwd_path(j.bits, (int)j.T, (int)j.N, (int)j.K, false, false) : kRoles128;
        if (path == kDuo256 || path == kGeneral256) {
            if (n_jobs == 1) return false;
            other += rounds_of(j) * tile_time(j) * (path == kGeneral256 ? 0.95 : j.K < 2048 ? 0.93 : 0.87);
        } else {
            const double math = (j.K % 128 ? 1.0 : 0.69) * gop, out = 4.0 / 3.5e6 * (double)j.T * (double)j.N;
            other += math > out ? math : out;
        }
        const unsigned bit = 1u << (2 * j.bits + (kind == kShared96));
        if (kind == kAlone || !(shared & bit)) other += 4.0;
        if (kind != kAlone) shared |= bit;
    }
    return list < 0.92 * (other + few);
}

// The jobs of one bit-width that have more tiles: those that the single call would give to a role-split kernel share launches of it
// (one list per tile shape), the others go one by one
template <int BITS>
void launch_jobs_of_width(const qb_fwd_job *jobs, int n_jobs, hipStream_t st)
{
    Group g96, g128;
    g96.n = g128.n = 0;
    const OutQ none{nullptr, nullptr, 1.0f, 0, nullptr, nullptr};
    for (int i = 0; i < n_jobs; ++i) {
        const qb_fwd_job &j = jobs[i];
        if (j.bits != BITS || few_tiles(j)) continue;
        const LargeJob kind = large_job<BITS>(j);
        if (kind == kAlone) {
            launch_job<BITS>(j, st);
            continue;
        }
        const uint8_t *p = static_cast<const uint8_t *>(j.packed);
        const int rpg = (int)(j.N / j.groups);
        const float hx = j.clip / 255.0f;
        if (kind == kShared96) {
            if (g96.n == kMaxGroup) {
                launch_g96<BITS>(g96, st);
                g96.n = 0;
            }
            group_add<128, 96>(g96, j.Xq, j.rs_x, p, j.h, j.rs_w, j.bias, j.Y, nullptr, (int)j.T, (int)j.N, (int)j.K, rpg, hx, none);
        } else {
            if (g128.n == kMaxGroup) {
                launch_group<BITS, 2, 2, 2, 2, 3, 4, false, 0>(g128, st, 256);
                g128.n = 0;
            }
            group_add<128, 128>(g128, j.Xq, j.rs_x, p, j.h, j.rs_w, j.bias, j.Y, nullptr, (int)j.T, (int)j.N, (int)j.K, rpg, hx, none);
        }
    }
    if (g96.n) launch_g96<BITS>(g96, st);
    if (g128.n) launch_group<BITS, 2, 2, 2, 2, 3, 4, false, 0>(g128, st, 256);
}
}  // namespace

namespace qb {
bool fwd_takes_list(const qb_fwd_job *jobs, int n_jobs) { return list_pays(jobs, n_jobs); }
// where a job goes that is not in a list: with the few-tile ones (-1), alone (0), to the shared launch of 128 x 96 (1) or of 128 x 128 tiles (2)
int fwd_job_kind(const qb_fwd_job *j)
{
    if (few_tiles(*j)) return -1;
    return j->bits == 2 ? large_job<2>(*j) : j->bits == 3 ? large_job<3>(*j) : j->bits == 4 ? large_job<4>(*j) : large_job<8>(*j);
}
// the kernels of a call's few-tile jobs, a launch each: bits | units << 8 | sliced << 16; the number of launches
int fwd_few_tiles(const qb_fwd_job *jobs, int n_jobs, int *kernels)
{
    int launches = 0;
    each_few_tiles_launch(jobs, n_jobs, [&](const qb_fwd_job *const *order, int n) {
        const FewTilesKernel k = few_tiles_kernel(order, n);
        kernels[launches++] = k.bits | k.units << 8 | (k.sliced ? 1 : 0) << 16;
    });
    return launches;
}
}  // namespace qb

extern "C" qb_status qb_qlinear_fwd_batched(const qb_fwd_job *jobs, int n_jobs, void *stream)
{
    if (n_jobs < 0 || (n_jobs > 0 && !jobs)) return QB_ERR_NULL;
    if (n_jobs == 0) return QB_OK;
    for (int i = 0; i < n_jobs; ++i) {
        const qb_status s = check_fwd_job(jobs[i]);
        if (s != QB_OK) return s;
    }
    hipStream_t st = static_cast<hipStream_t>(stream);
    if (list_pays(jobs, n_jobs)) {
        for (int i = 0; i < n_jobs; i += QB_MAX_BATCH) launch_fwd_list(jobs + i, n_jobs - i < QB_MAX_BATCH ? n_jobs - i : QB_MAX_BATCH, st);
        return launch_status();
    }
    launch_few_tiles(jobs, n_jobs, st);
    launch_jobs_of_width<2>(jobs, n_jobs, st);
    launch_jobs_of_width<3>(jobs, n_jobs, st);
    launch_jobs_of_width<4>(jobs, n_jobs, st);
    launch_jobs_of_width<8>(jobs, n_jobs, st);
    return launch_status();
}

extern "C" qb_status qb_qlinear_fwd_q8(const int8_t *Xq, const int32_t *rs_x, float clip, const void *packed,
                                       const float *h, const int32_t *rs_w, int bits, int groups, int64_t T, int64_t N,
                                       int64_t K, const float *bias, int act, float clip_out, int8_t *Yq, int32_t *rs_y,
                                       void *stream)
{
    if (!Xq || !rs_x || !packed || !h || !rs_w || !Yq || !rs_y) return QB_ERR_NULL;
    if (!bits_ok(bits)) return QB_ERR_BITS;
    if (T <= 0 || T > (1 << 24) || N <= 0 || N > (1 << 24) || !k_ok(K) || K % 128 != 0 || groups <= 0 || N % groups != 0 ||
        (act != 0 && act != 1))
        return QB_ERR_SHAPE;
    if (!(clip > 0.0f) || !(clip < 3.0e38f) || !(clip_out > 0.0f) || !(clip_out < 3.0e38f)) return QB_ERR_CLIP;
    const float hx = clip / 255.0f;
    const int rpg = (int)(N / groups);
    hipStream_t st = static_cast<hipStream_t>(stream);
    const uint8_t *p = static_cast<const uint8_t *>(packed);
    const OutQ oq{Yq, rs_y, clip_out, act, nullptr, nullptr};
    hipLaunchKernelGGL(fill_zero_i32_kernel, dim3((unsigned)((T + 255) / 256)), dim3(256), 0, st, rs_y, (int)T);
    switch (bits) {
        case 2: launch_bits_q8<2>(Xq, rs_x, p, h, rs_w, bias, oq, (int)T, (int)N, (int)K, rpg, hx, st); break;
        case 3: launch_bits_q8<3>(Xq, rs_x, p, h, rs_w, bias, oq, (int)T, (int)N, (int)K, rpg, hx, st); break;
        case 4: launch_bits_q8<4>(Xq, rs_x, p, h, rs_w, bias, oq, (int)T, (int)N, (int)K, rpg, hx, st); break;
        default: launch_bits_q8<8>(Xq, rs_x, p, h, rs_w, bias, oq, (int)T, (int)N, (int)K, rpg, hx, st); break;
    }
    return launch_status();
}

extern "C" qb_status qb_qlinear_fwd_dyn(const int8_t *Xq, const int32_t *rs_x, const float *hx_rows, const void *packed,
                                        const float *h, const int32_t *rs_w, int bits, int groups, int64_t T, int64_t N,
                                        int64_t K, const float *bias, float *Y, int32_t *A4_debug, void *stream)
{
    if (!Xq || !rs_x || !hx_rows || !packed || !h || !rs_w || !Y) return QB_ERR_NULL;
    if (!bits_ok(bits)) return QB_ERR_BITS;
    if (T <= 0 || T > (1 << 24) || N <= 0 || N > (1 << 24) || !k_ok(K) || groups <= 0 || N % groups != 0)
        return QB_ERR_SHAPE;
    const int rpg = (int)(N / groups);
    hipStream_t st = static_cast<hipStream_t>(stream);
    const uint8_t *p = static_cast<const uint8_t *>(packed);
    switch (bits) {
        case 2: launch_bits<2>(Xq, rs_x, p, h, rs_w, bias, Y, A4_debug, (int)T, (int)N, (int)K, rpg, 0.0f, st, hx_rows); break;
        case 3: launch_bits<3>(Xq, rs_x, p, h, rs_w, bias, Y, A4_debug, (int)T, (int)N, (int)K, rpg, 0.0f, st, hx_rows); break;
        case 4: launch_bits<4>(Xq, rs_x, p, h, rs_w, bias, Y, A4_debug, (int)T, (int)N, (int)K, rpg, 0.0f, st, hx_rows); break;
        default: launch_bits<8>(Xq, rs_x, p, h, rs_w, bias, Y, A4_debug, (int)T, (int)N, (int)K, rpg, 0.0f, st, hx_rows); break;
    }
    return launch_status();
}

extern "C" qb_status qb_qlinear_fwd_asym(const int8_t *Xq, const int32_t *rs_x, float clip, const void *packed,
                                         const float *delta, const float *q0, const int32_t *rs_w, int bits, int groups,
                                         int64_t T, int64_t N, int64_t K, const float *bias, float *Y, int32_t *A4_debug,
                                         void *stream)
{
    if (!Xq || !rs_x || !packed || !delta || !q0 || !rs_w || !Y) return QB_ERR_NULL;
    if (!bits_ok(bits)) return QB_ERR_BITS;
    if (T <= 0 || T > (1 << 24) || N <= 0 || N > (1 << 24) || !k_ok(K) || groups <= 0 || N % groups != 0)
        return QB_ERR_SHAPE;
    if (!(clip > 0.0f) || !(clip < 3.0e38f)) return QB_ERR_CLIP;
    const int rpg = (int)(N / groups);
    const float hx = clip / 255.0f;
    hipStream_t st = static_cast<hipStream_t>(stream);
    const uint8_t *p = static_cast<const uint8_t *>(packed);
    switch (bits) {
        case 2: launch_bits<2>(Xq, rs_x, p, delta, rs_w, bias, Y, A4_debug, (int)T, (int)N, (int)K, rpg, hx, st, nullptr, q0); break;
        case 3: launch_bits<3>(Xq, rs_x, p, delta, rs_w, bias, Y, A4_debug, (int)T, (int)N, (int)K, rpg, hx, st, nullptr, q0); break;
        case 4: launch_bits<4>(Xq, rs_x, p, delta, rs_w, bias, Y, A4_debug, (int)T, (int)N, (int)K, rpg, hx, st, nullptr, q0); break;
        default: launch_bits<8>(Xq, rs_x, p, delta, rs_w, bias, Y, A4_debug, (int)T, (int)N, (int)K, rpg, hx, st, nullptr, q0); break;
    }
    return launch_status();
}

extern "C" qb_status qb_qlinear_fwd_asym_dyn(const int8_t *Xq, const int32_t *rs_x, const float *hx_rows, const void *packed,
                                             const float *delta, const float *q0, const int32_t *rs_w, int bits, int groups,
                                             int64_t T, int64_t N, int64_t K, const float *bias, float *Y,
                                             int32_t *A4_debug, void *stream)
{
    if (!Xq || !rs_x || !hx_rows || !packed || !delta || !q0 || !rs_w || !Y) return QB_ERR_NULL;
    if (!bits_ok(bits)) return QB_ERR_BITS;
    if (T <= 0 || T > (1 << 24) || N <= 0 || N > (1 << 24) || !k_ok(K) || groups <= 0 || N % groups != 0)
        return QB_ERR_SHAPE;
    const int rpg = (int)(N / groups);
    hipStream_t st = static_cast<hipStream_t>(stream);
    const uint8_t *p = static_cast<const uint8_t *>(packed);
    switch (bits) {
        case 2: launch_bits<2>(Xq, rs_x, p, delta, rs_w, bias, Y, A4_debug, (int)T, (int)N, (int)K, rpg, 0.0f, st, hx_rows, q0); break;
        case 3: launch_bits<3>(Xq, rs_x, p, delta, rs_w, bias, Y, A4_debug, (int)T, (int)N, (int)K, rpg, 0.0f, st, hx_rows, q0); break;
        case 4: launch_bits<4>(Xq, rs_x, p, delta, rs_w, bias, Y, A4_debug, (int)T, (int)N, (int)K, rpg, 0.0f, st, hx_rows, q0); break;
        default: launch_bits<8>(Xq, rs_x, p, delta, rs_w, bias, Y, A4_debug, (int)T, (int)N, (int)K, rpg, 0.0f, st, hx_rows, q0); break;
    }
    return launch_status();
}
