// Forward of many linears of any widths in one launch: tiles of 128 tokens x 256 neurons, four wavefronts of 128 x 64 results,
// v_mfma_i32_16x16x64_i8, two workgroups per CU that share no barrier, as qgemm_i8_duo_kernel has them.  The host deals the tiles of all
// problems to the 512 resident workgroups, the longest contractions first, so that they end together; a workgroup's next tile may be of
// another width.  Single calls that the other large-tile kernels do not take run here too: K no multiple of 128, per-token scales,
// asymmetric ranges.
// What bounds a list: the K-loop (its MFMAs keep the matrix cores busy for 37 % of the time, 60 % at K = 4096; without copies and stores a
// layer's four linears at four widths take 110 us of 150) and the write-out of short contractions (127 us without the stores).  What it gives: the
// launches of the widths and of the tile shapes, their starts and their ragged last rounds.  Four linears at widths 2, 3, 4 and 8, hidden 768:
// 1024 tokens 111 -> 48 us, 2048 144 -> 75, 4096 172 -> 147, 6144 273 -> 214; hidden 448, 4096 tokens 149 -> 80.
// The copies: tokens two steps ahead in a ring of three slots; weights one step ahead over their own place, which a wavefront alone reads.  Measured
// next to it: both one step ahead (4096 tokens 159 for 144 us), copies between the MFMAs (162 for 154), the codes taken out of LDS and expanded at the
// end of the step before (160 for 154), raised wavefront priority around the MFMAs (no difference).  Long contractions of a single call
// stay with qgemm_i8_duo_kernel (32768 x 1024 x 4096, 2 bits 101 us, here 105).
#include "qgemm_i8.hpp"

namespace qb {
namespace {

struct ListArgs {
    const int8_t *Xq;
    const int32_t *rs_x;
    const uint8_t *packed;
    const float *h;
    const int32_t *rs_w;
    const float *bias;
    float *Y;
    int T, N, K, rows_per_group;
    float hx;
    int tiles_n;
};
// Workgroups [first_wg, first_wg + wgs) take the `count` tiles of a problem from first_tile on in turn.  (Whole words: there are no shorter
// scalar loads.)
struct ListRun {
    uint32_t wg;    // first_wg | wgs << 16
    uint32_t what;  // problem | bits << 16
    int32_t first_tile, count;
};
template <int PROBLEMS, int RUNS>
struct ListWork {
    int n_runs;
    ListRun run[RUNS];
    ListArgs p[PROBLEMS];
    // of a single call: the debug output; one activation scale per token instead of hx; asymmetric group ranges (h holds Delta and q0 the
    // lower end of every group); or null
    int32_t *A4out;
    const float *hx_rows, *q0;
};
constexpr int kListRuns = 64, kListWorkgroups = 512;
using ListSingle = ListWork<1, 1>;
using ListFull = ListWork<QB_MAX_BATCH, kListRuns>;

// A step of 128 features of one width: at 8 bits its weights are two halves of 64 features
template <int BITS>
struct ListWidth {
    static constexpr int PHASES = BITS == 8 ? 2 : 1, PHF = 128 / PHASES, SLOT = 4 * BITS;
    static constexpr int CH = (BITS == 3) ? 12 : 16, LSLOT = (BITS == 3) ? 16 : SLOT;
    static constexpr int PAIR = PHF * SLOT, LPAIR = PHF * LSLOT, PARTS = LPAIR / 1024, NB = 2 * PARTS;
};

// The 16-byte chunks of a token row of 128 bytes are swapped by this number of the row.  The LDS serves a 16-byte read in four groups of
// sixteen lanes, the first of them lanes 0-3, 12-15, 20-23 and 24-27: rows 0-3 and 12-15 at one logical chunk, rows 4-11 at another one
// that differs in its lower two bits.  The former have numbers 0-3, the latter 4-7, so that the group meets every bank once.
__device__ __forceinline__ int row_key(int row)
{
    const int pair = row >> 1;
    return ((pair & 1) | ((pair & 2) << 1)) ^ (pair & 4 ? 6 : 0);
}

// The lane's number, formed where it is used: kept over the K-loop, it and what comes of it take registers that there are not.
__device__ __forceinline__ int lane_anew()
{
    int all = -1;
    asm volatile("" : "+s"(all));
    return (int)__builtin_amdgcn_mbcnt_hi(all, __builtin_amdgcn_mbcnt_lo(all, 0));
}

// The packed codes of a step, expanded to int8: b0 and b1 belong to the two MFMAs of a lane's 32 features
template <int BITS>
__device__ __forceinline__ void expand_step(const v4u (&raw)[4], v4i (&b0)[4], v4i (&b1)[4])
{
#pragma unroll
    for (int x = 0; x < 4; ++x) {
        uint32_t in[BITS], d[8];
#pragma unroll
        for (int e = 0; e < BITS; ++e) in[e] = BITS == 2 ? raw[x & 2][2 * (x & 1) + e] : raw[x][e];
        unpack_run<BITS>(in, d);
        b0[x] = v4i{(int)d[0], (int)d[1], (int)d[2], (int)d[3]};
        b1[x] = v4i{(int)d[4], (int)d[5], (int)d[6], (int)d[7]};
    }
}

// BITS 0: a list, each problem with its own width
// GEN: per-token scales or asymmetric group ranges (a variant of its own, so that the plain call carries none of its code)
template <int BITS, bool GEN, typename WORK>
__global__ __launch_bounds__(256, 2) void qgemm_i8_list_kernel(const WORK job)
{
    constexpr int BM = 128, BN = 256, BK = 128;
    constexpr int SLOT = BM * BK, P_OFF = 4 * SLOT;  // four slots of 16 KB, then the tiles' parameters
    // rs_x | rs_w | h of the neuron's group | bias | per-token scales | q0 of the neuron's group
    constexpr int PARAM = (128 + 3 * 256 + (GEN ? 128 + 256 : 0)) * 4;
    static_assert(2 * (P_OFF + 2 * PARAM) <= 163840, "two workgroups per CU");
    __shared__ __align__(1024) uint8_t lds[P_OFF + 2 * PARAM];
    const uint32_t lds_base = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) uint8_t *)lds;

    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);  // neurons 64*wave
    auto args = [&](int i) -> const ListArgs & {
        asm volatile("" : "+s"(i));
        return job.p[i];
    };
    auto fence = [&]() {
        __builtin_amdgcn_s_waitcnt(0xC07F);  // lgkmcnt(0)
        asm volatile("" ::: "memory");
        __builtin_amdgcn_sched_barrier(0);
        __builtin_amdgcn_s_barrier();
        __builtin_amdgcn_sched_barrier(0);
        asm volatile("" ::: "memory");
    };

    auto scalar = [](const uint8_t *p) {
        const uint64_t v = (uint64_t)p;
        return (const uint8_t *)(((uint64_t)(uint32_t)__builtin_amdgcn_readfirstlane((int)(v >> 32)) << 32) | (uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)v));
    };
    // this workgroup's next tile: tile `at` of run r; false behind the last one
    int r = -1, at = 0, tm = 0, tn = 0, pi = 0, bits = BITS;
    auto next_tile = [&](int &r, int &at, int &pi, int &bits, int &tm, int &tn) {
        if (r >= 0) at += (int)(job.run[r].wg >> 16);
        while (r < 0 || at >= job.run[r].count) {
            if (++r >= job.n_runs) return false;
            const uint32_t wg = job.run[r].wg;
            const int w = (int)blockIdx.x - (int)(wg & 0xffffu);
            at = w >= 0 && w < (int)(wg >> 16) ? w : 0x7fffffff;
        }
        const ListRun &R = job.run[r];
        pi = (int)(R.what & 0xffffu);
        bits = BITS ? BITS : (int)(R.what >> 16);
        const int t = R.first_tile + logical_tile(at, R.count), tiles_n = args(pi).tiles_n;
        tm = __builtin_amdgcn_readfirstlane(t / tiles_n);
        tn = t - tm * tiles_n;
        return true;
    };
    if (!next_tile(r, at, pi, bits, tm, tn)) return;

    const uint8_t *a_base = nullptr, *b_base = nullptr;
    uint32_t a_off[4], b_lane = 0, b_blk[2];  // (weights: the wavefront's two blocks of 32 neurons)
    // this wavefront's weights of a step (8 bits: of 64 features, a half of one) and its share of a step's tokens into a slot
    // (half: the step has 64 features, the last one of an odd number of 64-feature units; what lies behind them is neither read nor used)
    auto copy_weights = [&](auto width, int from, int slot, bool half) {
        using W = ListWidth<decltype(width)::value>;
        const uint8_t *bs = b_base + (uint32_t)(from * W::PAIR);
        const uint32_t dst = lds_base + (uint32_t)slot * SLOT + wave * 4096;
        const uint32_t lane_off = W::PARTS == 1 && half ? b_lane & 511u : b_lane;  // (2 bits: a copy has both units)
#pragma unroll
        for (int e = 0; e < W::NB; ++e)
            if (W::PARTS == 1 || W::PHASES == 2 || !half || e % W::PARTS == 0)
                copy_to_lds<W::CH>(bs + b_blk[e / W::PARTS] + (e % W::PARTS) * 64 * W::CH, lane_off, dst + (e / W::PARTS) * 2048 + (e % W::PARTS) * 1024);
    };
    auto weights = [&](int bits, int s, int w, int s2, bool half) {
        if (bits == 2) copy_weights(std::integral_constant<int, 2>(), s, w, half);
        else if (bits == 3) copy_weights(std::integral_constant<int, 3>(), s, w, half);
        else if (bits == 4) copy_weights(std::integral_constant<int, 4>(), s, w, half);
        else {
            copy_weights(std::integral_constant<int, 8>(), 2 * s, w, false);
            if (!half) copy_weights(std::integral_constant<int, 8>(), 2 * s + 1, s2, false);
        }
    };
    auto tokens = [&](int s, int slot, bool half) {
        const uint8_t *as = a_base + (uint32_t)(s * BK);
        const uint32_t dst = lds_base + (uint32_t)slot * SLOT;
        const uint32_t back = half ? (uint32_t)((lane_anew() ^ (lane_anew() >> 3)) & 4) << 4 : 0u;  // the chunks behind the last feature repeat those before it
#pragma unroll
        for (int e = 0; e < 4; ++e) copy_to_lds<16>(as, half ? a_off[e] - (back ^ (64u * (e & 1))) : a_off[e], dst + (wave * 4 + e) * 1024);
    };
    auto start_tile = [&](int pi, int bits, int tm, int tn, int pb, int s1, int s2, int w) {
        const int lane = lane_anew();
        const ListArgs &P = args(pi);
        const int T = P.T, N = P.N, K = P.K, kunits = K >> 6, ncb = (N + 31) >> 5;
        a_base = scalar(reinterpret_cast<const uint8_t *>(P.Xq) + (size_t)tm * BM * K);
        const int unit_bytes = 256 * bits;  // of a 32-neuron block
        b_base = scalar(P.packed + (size_t)tn * 8 * kunits * unit_bytes);
        const int a_last = T - 1 - tm * BM, cb_last = ncb - 1 - tn * 8;
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            int row = (wave * 4 + e) * 8 + (lane >> 3);
            row = row < a_last ? row : a_last;
            a_off[e] = __umul24(row, K) + (((lane & 7) ^ row_key((lane >> 3) + 8 * (e & 1))) << 4);
        }
        const int sl = bits == 2 ? lane : (bits == 8 ? lane ^ (-(lane >> 4) & 3) : lane ^ ((lane >> 4) & 1));
        b_lane = (uint32_t)sl * (bits == 3 ? 12u : 16u);
#pragma unroll
        for (int e = 0; e < 2; ++e) {
            int cb = wave * 2 + e;
            cb = cb < cb_last ? cb : cb_last;
            b_blk[e] = (uint32_t)cb * (uint32_t)(kunits * unit_bytes);
        }
        // parameters: the first wavefront rs_x (and per-token scales, q0), the others rs_w, h of the neurons' groups, bias
        const uint32_t dst = lds_base + P_OFF + pb * PARAM;
        if (wave == 0) {
#pragma unroll
            for (int e = 0; e < 2; ++e) {
                const int t = tm * BM + e * 64 + lane;
                copy_to_lds<4>(P.rs_x, (uint32_t)(t < T ? t : T - 1) * 4, dst + e * 256);
                if (GEN && job.hx_rows) copy_to_lds<4>(job.hx_rows, (uint32_t)(t < T ? t : T - 1) * 4, dst + 3584 + e * 256);
            }
            if (GEN && job.q0) {
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    const int nn = tn * BN + e * 64 + lane;
                    copy_to_lds<4>(job.q0, (uint32_t)((nn < N ? nn : N - 1) / P.rows_per_group) * 4, dst + 4096 + e * 256);
                }
            }
        } else if (wave < 3 || P.bias) {
            const void *src = wave == 1 ? (const void *)P.rs_w : wave == 2 ? P.h : P.bias;
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                int nn = tn * BN + e * 64 + lane;
                nn = nn < N ? nn : N - 1;
                if (wave == 2) nn /= P.rows_per_group;
                copy_to_lds<4>(src, (uint32_t)nn * 4, dst + 512 + (wave - 1) * 1024 + e * 256);
            }
        }
        weights(bits, 0, w, s2, K == 64);
        tokens(0, s1, K == 64);
    };

    // The slots: s0 this step's tokens, w its weights.  A wavefront alone reads the weights that it copies, so that those of the next step go
    // over them as soon as it has them in registers.  Up to 4 bits s1 holds the next step's tokens and s2 takes those of the step behind
    // it; at 8 bits s1 takes the next step's tokens and s2 belongs to the weights.
    int s0 = 1, s1 = 0, s2 = 2, w = 3, pb = 0;
    start_tile(pi, bits, tm, tn, 0, s1, s2, w);
    s0 = 0; s1 = 1;
    bool late = true;  // the second step's tokens are not on their way yet
    wait_vmcnt<0>();
    while (true) {
        v4i acc[8][4];  // 16 tokens x (block j of 32 neurons, neuron 2*(l%16) + nb): [2*j + nb]
#pragma unroll
        for (int m = 0; m < 8; ++m)
#pragma unroll
            for (int x = 0; x < 4; ++x) acc[m][x] = v4i{0, 0, 0, 0};
        int npi = pi, nbits = bits, ntm = tm, ntn = tn;
        bool more = false;
        const int units = args(pi).K >> 6, steps = (units + 1) >> 1;
        for (int s = 0; s < steps; ++s) {
            fence();
            const int lane = lane_anew(), q16 = lane & 15, hq = lane >> 4;
            v4i a0[8], a1[8], b0[4], b1[4];
            v4u raw[4];
            const uint32_t lo = wave * 4096 + (bits == 8 ? (hq >> 1) * 1024 + ((4 * q16 + ((hq & 1) ^ (-(q16 >> 2) & 3))) << 4)
                                               : bits == 2 ? hq * 256 + q16 * 16 : hq * 512 + (((2 * q16) ^ (q16 >> 3)) << 4));
            raw[0] = *reinterpret_cast<const v4u *>(lds + w * SLOT + lo);
            raw[2] = *reinterpret_cast<const v4u *>(lds + w * SLOT + lo + 2048);
            if (bits != 2) {
                const uint32_t lo1 = lo ^ (bits == 8 ? 32 : 16);
                raw[1] = *reinterpret_cast<const v4u *>(lds + w * SLOT + lo1);
                raw[3] = *reinterpret_cast<const v4u *>(lds + w * SLOT + lo1 + 2048);
                if (bits == 8) {
                    b1[0] = *reinterpret_cast<const v4i *>(lds + s2 * SLOT + lo);
                    b1[2] = *reinterpret_cast<const v4i *>(lds + s2 * SLOT + lo + 2048);
                    b1[1] = *reinterpret_cast<const v4i *>(lds + s2 * SLOT + lo1);
                    b1[3] = *reinterpret_cast<const v4i *>(lds + s2 * SLOT + lo1 + 2048);
                }
            }
            __builtin_amdgcn_sched_barrier(0);
            // tokens: 16-byte chunks 2*(l/16) and the one behind it; at 8 bits l/16 and l/16 + 4 (the two halves of the features)
            const uint32_t ao = s0 * SLOT + q16 * 128 + (((bits == 8 ? hq : 2 * hq) ^ row_key(q16)) << 4), ao1 = ao ^ (bits == 8 ? 64 : 16);
#pragma unroll
            for (int m = 0; m < 8; ++m) a0[m] = *reinterpret_cast<const v4i *>(lds + ao + m * 2048);
            __builtin_amdgcn_sched_barrier(0);
            __builtin_amdgcn_s_waitcnt(0xC87F);  // lgkmcnt(8): the codes are here
            __builtin_amdgcn_sched_barrier(0);
            bool ahead = false;
            if (s + 1 < steps) {
                const bool half1 = 2 * s + 3 == units;  // (the next step)
                if (bits == 8 || late) tokens(s + 1, s1, half1);
                late = false;
                weights(bits, s + 1, w, s2, half1);
                ahead = bits != 8 && s + 2 < steps;
                if (ahead) tokens(s + 2, s2, 2 * s + 5 == units);
            } else {
                more = next_tile(r, at, npi, nbits, ntm, ntn);
                if (more) {
                    start_tile(npi, nbits, ntm, ntn, pb ^ 1, s1, s2, w);
                    // (s2 may hold weights that other wavefronts still read)
                    const int K = args(npi).K;
                    late = bits == 8 || nbits == 8 || K <= BK;
                    if (!late) tokens(1, s2, K == 192);
                }
            }
            __builtin_amdgcn_sched_barrier(0);
            const bool half = 2 * s + 1 == units;
            if (half && bits != 8) {  // no features behind the first 64: their weights count as zeros
                const uint32_t keep = hq < 2 ? 0xffffffffu : 0u;
#pragma unroll
                for (int x = 0; x < 4; ++x) raw[x] &= v4u{keep, keep, keep, keep};
            }
            if (bits == 2) expand_step<2>(raw, b0, b1);
            else if (bits == 3) expand_step<3>(raw, b0, b1);
            else if (bits == 4) expand_step<4>(raw, b0, b1);
            else {
#pragma unroll
                for (int x = 0; x < 4; ++x)
#pragma unroll
                    for (int e = 0; e < 4; ++e) {
                        b0[x][e] = (int)(raw[x][e] ^ 0x80808080u);
                        b1[x][e] = half ? 0 : b1[x][e] ^ (int)0x80808080u;
                    }
            }
            // four rows of blocks at a time; the tokens of the second MFMAs come into the registers that are free by then
#define QB_MMA4(a, b, m0)                                                                                 \
    _Pragma("unroll") for (int m = m0; m < m0 + 4; ++m)                                                   \
        _Pragma("unroll") for (int x = 0; x < 4; ++x)                                                     \
            acc[m][x] = __builtin_amdgcn_mfma_i32_16x16x64_i8(a[m], b[x], acc[m][x], 0, 0, 0);
#define QB_SECOND(m0)                                                                                     \
    _Pragma("unroll") for (int m = m0; m < m0 + 4; ++m) a1[m] = *reinterpret_cast<const v4i *>(lds + ao1 + m * 2048);
            QB_SECOND(0)
            __builtin_amdgcn_sched_barrier(0);
            QB_MMA4(a0, b0, 0)
            __builtin_amdgcn_sched_barrier(0);
            QB_SECOND(4)
            __builtin_amdgcn_sched_barrier(0);
            QB_MMA4(a0, b0, 4)
            QB_MMA4(a1, b1, 0)
            QB_MMA4(a1, b1, 4)
#undef QB_MMA4
#undef QB_SECOND
            if (s + 1 < steps) {
                if (ahead) wait_vmcnt<4>();  // (the tokens of the step after the next have one more step)
                else wait_vmcnt<0>();
            }
            const int x = s0;
            s0 = s1;
            if (bits == 8 || (s + 1 == steps && late)) s1 = x;
            else { s1 = s2; s2 = x; }
        }

        // ---- write-out
        const ListArgs &P = args(pi);
        const int T = P.T, N = P.N, K = P.K, t0 = tm * BM, n0 = tn * BN;
        const int e2 = bits == 8 ? 2 : -2 * ((1 << bits) - 1);
        const float hx = P.hx;
        const bool has_bias = P.bias != nullptr;
        float *__restrict__ Y = P.Y;
        const uint8_t *pp = lds + P_OFF + pb * PARAM;
        pb ^= 1;
        const int wl = lane_anew(), q16 = wl & 15, hq = wl >> 4;
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
        float zn[2][2];
        const float *hr_rows = GEN && job.hx_rows ? reinterpret_cast<const float *>(pp + 3584) + 4 * hq : nullptr;
        const bool asym = GEN && job.q0 != nullptr;
        if constexpr (GEN) {
#pragma unroll
            for (int j = 0; j < 2; ++j) {
                const float2 hg = *reinterpret_cast<const float2 *>(pp + 1536 + (nl + 32 * j) * 4);
                const float2 q = *reinterpret_cast<const float2 *>(pp + 4096 + (nl + 32 * j) * 4);
                scale[j][0] = hg.x; scale[j][1] = hg.y;  // (the row's scale comes to it)
                zn[j][0] = q.x; zn[j][1] = q.y;
            }
        }
        // one result: rh = R/2 of its row, hr the row's scale (GEN)
        auto value = [&](int a4, int j, int nb, int rh, float hr) {
            if constexpr (!GEN) return scale[j][nb] * (float)a4 + bv[j][nb];
            if (asym) return asym_value(a4, rh, (1 << bits) - 1, hr, scale[j][nb], zn[j][nb]) + bv[j][nb];
            return (hr * scale[j][nb]) * (float)a4 + bv[j][nb];
        };
        int32_t *__restrict__ A4out = BITS ? job.A4out : nullptr;
        const bool fast = t0 + BM <= T && n0 + BN <= N && A4out == nullptr && (N & 1) == 0 && (reinterpret_cast<uintptr_t>(Y) & 7) == 0;
        if (fast) {
            // a wavefront-uniform row address and the lane's 32-bit byte offset
            uint8_t *out0 = reinterpret_cast<uint8_t *>(Y + (size_t)t0 * N + n0 + wave * 64);
            const uint32_t lane_off = (uint32_t)(4 * hq * N + 2 * q16) * 4u;
#pragma unroll
            for (int m = 0; m < 8; ++m) {
                const int4 rx = *reinterpret_cast<const int4 *>(p_rx + m * 16);
                const int rs[4] = {rx.x, rx.y, rx.z, rx.w};
                float hr[4] = {hx, hx, hx, hx};
                if (GEN && hr_rows) {
                    const float4 v = *reinterpret_cast<const float4 *>(hr_rows + m * 16);
                    hr[0] = v.x; hr[1] = v.y; hr[2] = v.z; hr[3] = v.w;
                }
#pragma unroll
                for (int c = 0; c < 4; ++c) {
                    const int er = qb_mad24(e2, rs[c], 0);
                    uint8_t *row = out0 + (size_t)(m * 16 + c) * N * 4;
#pragma unroll
                    for (int j = 0; j < 2; ++j) {
                        typedef float v2f __attribute__((ext_vector_type(2)));
                        v2f o;
#pragma unroll
                        for (int nb = 0; nb < 2; ++nb) o[nb] = value(qb_a4(acc[m][2 * j + nb][c], er + coln[j][nb]), j, nb, rs[c] + (K >> 1), hr[c]);
                        __builtin_nontemporal_store(o, reinterpret_cast<v2f *>(row + 128 * j + lane_off));
                    }
                }
            }
            wait_vmcnt<63>();  // 64 stores behind the copies: with at most 63 operations outstanding the copies have landed
        } else {  // edge tiles and the debug output: every element checked
#pragma unroll
            for (int m = 0; m < 8; ++m)
#pragma unroll
                for (int c = 0; c < 4; ++c) {
                    const int t = t0 + m * 16 + 4 * hq + c;
                    const int rs = p_rx[m * 16 + c], er = e2 * rs;
                    const float hr = GEN && hr_rows ? hr_rows[m * 16 + c] : hx;
                    if (t < T) {
#pragma unroll
                        for (int j = 0; j < 2; ++j)
#pragma unroll
                            for (int nb = 0; nb < 2; ++nb) {
                                const int nn = n0 + nl + 32 * j + nb;
                                if (nn < N) {
                                    const int a4 = qb_a4(acc[m][2 * j + nb][c], er + coln[j][nb]);
                                    const size_t at = (size_t)t * N + nn;
                                    Y[at] = value(a4, j, nb, rs + (K >> 1), hr);
                                    if (A4out) A4out[at] = a4;
                                }
                            }
                    }
                }
            wait_vmcnt<0>();
        }
        if (!more) break;
        pi = npi; bits = nbits; tm = ntm; tn = ntn;
    }
}


// Deals the tiles of a list to the workgroups.  The problems go from the longest contraction to the shortest, each to the workgroups that
// have the least to do so far; a tile counts its steps and, for its start and write-out, 4.5 more.
struct ListDealer {
    struct Range {
        int first, len;
        float load;
    } range[kListRuns + 1];
    int n = 0, grid = 0;
    ListFull list;

    void start()
    {
        range[0] = {0, kListWorkgroups, 0.0f};
        n = 1;
        grid = 0;
        list.n_runs = 0;
    }
    void flush(hipStream_t st)
    {
        if (list.n_runs) hipLaunchKernelGGL((qgemm_i8_list_kernel<0, false, ListFull>), dim3(grid), dim3(256), 0, st, list);
        start();
    }
    void add(int problem, int bits, int tiles, float cost, float least, hipStream_t st)
    {
        for (int done = 0; done < tiles;) {
            if (list.n_runs == kListRuns) flush(st);
            int best = 0;
            for (int i = 1; i < n; ++i)
                if (range[i].load < range[best].load) best = i;
            float next = 3.0e38f;
            for (int i = 0; i < n; ++i)
                if (i != best && range[i].load < next) next = range[i].load;
            const int left = tiles - done, len = range[best].len;
            int wgs = len, count;
            if (left >= len) {
                const float gap = (next - range[best].load) / cost + 0.5f;
                int rounds = left / len;
                if (gap < (float)rounds) rounds = gap < 1.0f ? 1 : (int)gap;
                count = rounds * len;
                range[best].load += (float)rounds * cost;
            } else {
                count = left;
                wgs = (left + 7) & ~7;
                if (wgs < len) {
                    for (int i = n; i > best + 1; --i) range[i] = range[i - 1];
                    ++n;
                    range[best + 1] = {range[best].first + wgs, len - wgs, range[best].load};
                    range[best].len = wgs;
                }
                range[best].load += cost;
            }
            list.run[list.n_runs++] = {(uint32_t)(range[best].first | wgs << 16), (uint32_t)(problem | bits << 16), done, count};
            if (range[best].first + wgs > grid) grid = range[best].first + wgs;
            done += count;
            // neighbours less than half a tile of the shortest problem apart count as one
            for (int i = 0; i + 1 < n;) {
                const float d = range[i].load - range[i + 1].load;
                if (d < 0.5f * least && d > -0.5f * least) {
                    range[i].len += range[i + 1].len;
                    range[i].load = d > 0 ? range[i].load : range[i + 1].load;
                    for (int j = i + 1; j + 1 < n; ++j) range[j] = range[j + 1];
                    --n;
                } else
                    ++i;
            }
        }
    }
};

}  // namespace

void launch_fwd_list(const qb_fwd_job *jobs, int n_jobs, hipStream_t st)
{
    ListDealer d;
    d.start();
    d.list.A4out = nullptr;
    d.list.hx_rows = d.list.q0 = nullptr;
    int order[QB_MAX_BATCH];
    auto cost = [&](int i) { return (float)((jobs[i].K + 127) / 128) + 4.5f; };
    for (int i = 0; i < n_jobs; ++i) {
        const qb_fwd_job &j = jobs[i];
        d.list.p[i] = {j.Xq, j.rs_x, static_cast<const uint8_t *>(j.packed), j.h, j.rs_w, j.bias, j.Y, (int)j.T, (int)j.N, (int)j.K,
                       (int)(j.N / j.groups), j.clip / 255.0f, (int)((j.N + 255) / 256)};
        int k = i;
        for (; k > 0 && jobs[order[k - 1]].K < j.K; --k) order[k] = order[k - 1];
        order[k] = i;
    }
    for (int k = 0; k < n_jobs; ++k) {
        const int i = order[k];
        d.add(i, jobs[i].bits, (int)((jobs[i].T + 127) / 128) * d.list.p[i].tiles_n, cost(i), cost(order[n_jobs - 1]), st);
    }
    d.flush(st);
}

template <int BITS>
void launch_fwd_general(const int8_t *Xq, const int32_t *rs_x, const uint8_t *packed, const float *h, const int32_t *rs_w, const float *bias, float *Y,
                    int32_t *A4, int T, int N, int K, int rpg, float hx, hipStream_t st, const float *hx_rows, const float *q0)
{
    const int tiles_n = (N + 255) / 256, tiles = (T + 127) / 128 * tiles_n;
    const int grid = tiles < kListWorkgroups ? tiles : kListWorkgroups, wgs = (grid + 7) & ~7;
    const ListSingle j{1, {{(uint32_t)wgs << 16, (uint32_t)BITS << 16, 0, tiles}}, {{Xq, rs_x, packed, h, rs_w, bias, Y, T, N, K, rpg, hx, tiles_n}}, A4, hx_rows, q0};
    auto *kernel = hx_rows || q0 ? qgemm_i8_list_kernel<BITS, true, ListSingle> : qgemm_i8_list_kernel<BITS, false, ListSingle>;
    hipLaunchKernelGGL(kernel, dim3(grid), dim3(256), 0, st, j);
}
template void launch_fwd_general<2>(const int8_t *, const int32_t *, const uint8_t *, const float *, const int32_t *, const float *, float *, int32_t *, int, int, int, int, float, hipStream_t, const float *, const float *);
template void launch_fwd_general<3>(const int8_t *, const int32_t *, const uint8_t *, const float *, const int32_t *, const float *, float *, int32_t *, int, int, int, int, float, hipStream_t, const float *, const float *);
template void launch_fwd_general<4>(const int8_t *, const int32_t *, const uint8_t *, const float *, const int32_t *, const float *, float *, int32_t *, int, int, int, int, float, hipStream_t, const float *, const float *);
template void launch_fwd_general<8>(const int8_t *, const int32_t *, const uint8_t *, const float *, const int32_t *, const float *, float *, int32_t *, int, int, int, int, float, hipStream_t, const float *, const float *);

}  // namespace qb
