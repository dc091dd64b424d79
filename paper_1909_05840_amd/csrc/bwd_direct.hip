// Straight-through backward without a staging area: both products of a call from dY, the activation codes and the
// packed weights as they lie in memory, in one launch.
//
//   dX[t,j] = sum_n dY[t,n] * What[n,j]     What[n,j] = bf16(h_g * (2u - L)), or bf16(Delta_g * u + q0_g)
//   dW[n,j] = sum_t dY[t,n] * Xhat[t,j]     Xhat[t,j] = h_x * (2x'+1), h_x applied at the end
//
// What bounds a small call is the chain of latencies: with staged operands a launch that transposes (4 us) and a GEMM whose
// workgroups share tiles and wait for each other's partial sums (16 us at 1001 x 1344 x 448, of which the MFMAs need one).
// Here a workgroup does whole 64 x 64 tiles alone, and its teams cut the contraction's steps, each a chain of LDS reads,
// four MFMAs and the arithmetic that makes the next operands.
// With many tiles the arithmetic bounds it; tiles of 128 x 64 and 128 x 128 do less of it per result but leave CUs empty at these sizes and
// gained nothing.
//
// The MFMA wants eight neighbours of the contraction per lane.  dY has them along a row for dX; for dW (dY and the codes
// along t) and for the weights (codes along j) the rows go to LDS as they come, converted, and are turned by the transposing reads.  1001 tokens, 4
// bits, us a call, staged / turned in the registers (permutes and lane exchanges, 64 instructions a step and wavefront for dW, 86 for dX) / now:
// (N, K) = (1344, 448) 20.0 / 11.5 / 11.1, (448, 448) 17.1 / 7.2 / 6.8, (1792, 448) 20.8 / 13.4 / 12.7, (448, 1792) 22.1 / 11.4 / 10.1; 8 bits, 2000 x
// 1024 x 1024 21.0 before, 18.5 now; 4 bits, 390 x 2304 x 768 15.1 and 14.0.
#include "qb_common.hpp"
#include "bwd_direct.hpp"
#include <algorithm>

namespace qb {
namespace {

typedef __bf16 v8bf __attribute__((ext_vector_type(8)));
typedef float v16f __attribute__((ext_vector_type(16)));
typedef unsigned int v4u __attribute__((ext_vector_type(4)));
typedef unsigned int v2u __attribute__((ext_vector_type(2)));
typedef float v4f __attribute__((ext_vector_type(4)));
typedef short v4s __attribute__((ext_vector_type(4)));

constexpr int kRowBytes = 128;  // an LDS row: 64 bf16 of the contraction
constexpr int kTile = 64;
constexpr int kStage = 2 * kTile * kRowBytes;

// Rows are dense; their 16-byte chunks are XOR-swizzled so that 16 consecutive rows read at one chunk (fragments) and
// rows two or four apart written at one chunk (turned operands) meet different banks.
__device__ __forceinline__ int swizzle_key(int row) { return ((row >> 1) ^ ((row >> 4) & 1)) & 7; }
__device__ __forceinline__ uint32_t lds_at(int row, int chunk) { return (uint32_t)(row * kRowBytes + ((chunk ^ swizzle_key(row)) << 4)); }

// The same for an operand whose LDS rows run along the contraction's steps (row: step, 64 results along it), read turned: 16 lanes read 4 rows of 32
// bytes, so that rows two apart lie in different halves of the row, and 16 consecutive rows written at one chunk meet different banks.
__device__ __forceinline__ int turned_key(int row) { return ((row >> 3) & 1) | ((row >> 1) & 2) | ((row << 1) & 4); }
__device__ __forceinline__ uint32_t turned_at(int row, int chunk) { return (uint32_t)(row * kRowBytes + ((chunk ^ turned_key(row)) << 4)); }
// Where a lane reads to get four contraction steps (part q of eight) of its result: lane l of a group of 16 reads four results of row l / 4 and is
// given the four rows of result l.  Sixteen steps further on lie 16 rows further on.
__device__ __forceinline__ uint32_t turned_fragment(int lane, int q)
{
    return turned_at(8 * (lane >> 5) + 4 * q + ((lane >> 2) & 3), ((lane >> 3) & 2) + ((lane >> 1) & 1)) + 8 * (lane & 1);
}
typedef __attribute__((address_space(3))) v4s *turned_ptr;
__device__ __forceinline__ v8bf turned_read(const uint8_t *first, const uint8_t *second)
{
    const v4s a = __builtin_amdgcn_ds_read_tr16_b64_v4i16((turned_ptr)first), b = __builtin_amdgcn_ds_read_tr16_b64_v4i16((turned_ptr)second);
    return __builtin_bit_cast(v8bf, __builtin_shufflevector(a, b, 0, 1, 2, 3, 4, 5, 6, 7));
}

__device__ __forceinline__ uint32_t lo_halves(uint32_t first, uint32_t second) { return __builtin_amdgcn_perm(second, first, 0x05040100u); }
__device__ __forceinline__ uint32_t hi_halves(uint32_t first, uint32_t second) { return __builtin_amdgcn_perm(second, first, 0x07060302u); }
__device__ __forceinline__ uint32_t lane_xor1(uint32_t v) { return (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0xB1, 0xF, 0xF, true); }
__device__ __forceinline__ uint32_t lane_xor2(uint32_t v) { return (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x4E, 0xF, 0xF, true); }
// two floats rounded to nearest even, the first in the low half
__device__ __forceinline__ uint32_t bf16_pair(float lo, float hi)
{
    typedef float f2 __attribute__((ext_vector_type(2)));
    typedef __bf16 b2 __attribute__((ext_vector_type(2)));
    return __builtin_bit_cast(uint32_t, __builtin_convertvector(f2{lo, hi}, b2));
}
// byte i of v as a float.  (In asm, for the compiler turns the arithmetic behind a conversion into whole-number
// instructions in front of it, five for two.)
__device__ __forceinline__ float byte_f(uint32_t v, int i)
{
    float f;
    switch (i) {
        case 0: asm("v_cvt_f32_ubyte0 %0, %1" : "=v"(f) : "v"(v)); break;
        case 1: asm("v_cvt_f32_ubyte1 %0, %1" : "=v"(f) : "v"(v)); break;
        case 2: asm("v_cvt_f32_ubyte2 %0, %1" : "=v"(f) : "v"(v)); break;
        default: asm("v_cvt_f32_ubyte3 %0, %1" : "=v"(f) : "v"(v)); break;
    }
    return f;
}

typedef const __attribute__((address_space(1))) uint8_t *gptr;
// p + offset, kept in scalar registers
template <typename P>
__device__ __forceinline__ gptr scalar(const P *p, size_t offset)
{
    gptr q = (gptr)(const __attribute__((address_space(1))) void *)p + offset;
    asm("" : "+s"(q));
    return q;
}
// (no alignment is asked of p: the load unit takes any address with the same instruction, so where an input lies decides
// neither the path of a call nor its results)
template <typename V>
__device__ __forceinline__ V at(gptr p)
{
    struct __attribute__((packed)) Loose { V v; };
    return ((const __attribute__((address_space(1))) Loose *)p)->v;
}
// dwords of packed codes a thread holds per step: half a slot (16 codes)
template <int BITS>
constexpr int code_words() { return BITS == 8 ? 4 : BITS == 2 ? 1 : 2; }

// One tile of 64 x 64 results by KS teams of four wavefronts, each wavefront 32 x 32 of them; the teams take the
// contraction's steps of 64 in turn and add their sums through LDS at the end.  DW: dW, else dX.
template <int KS, int BITS, bool MASK, bool DW>
__device__ __forceinline__ void direct_tile(const DirectArgs &g, int tile, uint8_t *lds_all)
{
    constexpr int AHEAD = 2;  // steps of a team whose operands are in registers or under way (4: 2 to 10 % slower)
    constexpr int BW = DW ? 4 : code_words<BITS>();
    const int tid = threadIdx.x & 255, lane = tid & 63;
    const int team = KS == 1 ? 0 : __builtin_amdgcn_readfirstlane(threadIdx.x >> 8);
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    uint8_t *const lds = lds_all + team * (2 * kStage);
    const int l32 = lane & 31, hf = lane >> 5;
    const int T = g.T, N = g.N, K = g.K;
    const int tiles_k = K >> 6;
    const int tile_m = tile / tiles_k, tile_n = tile - tile_m * tiles_k;
    const int r0 = tile_m * kTile, c0 = tile_n * kTile;
    const int all_steps = DW ? (T + 63) / 64 : N / 64;
    const int steps = (all_steps + KS - 1) / KS;  // of each team: step s of team t is step s*KS + t of the contraction

    struct Set { uint32_t a[8], b[BW]; float h, z; };  // h, z: the range of this thread's row of the weights (dX)
    Set set[AHEAD];

    // ---- loads
    // dY: rows tid / 8 and 32 further of a step (dW) or of the tile (dX), 16 bytes of each; the activation codes likewise, 8 bytes
    const int rem = T - 64 * ((T + 63) / 64 - 1);
    // dX, weights: wavefront (cb, part): rows 32*cb.. of the step, lane = slot, half `part` of it
    const int cb = wave >> 1, part = wave & 1;
    // Every load is issued whatever the step (no branch around loads: the compiler would wait for all of them where the
    // paths meet): steps past the end repeat the last one.  dW's first step covers the rows that T has beyond a multiple of
    // 64 (rem of them, the others set to zero), so that the loop has no such case.  An address is a wavefront-uniform
    // base and a 32-bit byte offset per lane that stays the same from step to step.
    const uint32_t a_pitch = (uint32_t)N * 2, b_pitch = (uint32_t)K;
    const float *zsrc = g.q0 ? g.q0 : g.h;
    uint32_t a_off[2], b_off[DW ? 2 : 1];
#pragma unroll
    for (int i = 0; i < 2; ++i) {
        const int row = i * 32 + (tid >> 3);
        if constexpr (DW) {
            a_off[i] = (uint32_t)row * a_pitch + 2 * r0 + (tid & 7) * 16;
            b_off[i] = (uint32_t)row * b_pitch + c0 + (tid & 7) * 8;
        } else {
            const int t = r0 + row < T ? r0 + row : T - 1;  // rows past the end re-read the last one; their results are not stored
            a_off[i] = (uint32_t)t * a_pitch + (tid & 7) * 16;
        }
    }
    if constexpr (!DW) b_off[0] = lane * (4 * BITS) + (BITS == 8 ? 16 : BITS == 4 ? 8 : 4) * part;
    const float row_f0 = (float)(32 * cb + l32) + 0.5f;
    auto load = [&](int s, Set &r) {
        // (opaque in every step: else the offsets are widened outside the loop and added to the base by vector arithmetic)
        for (uint32_t &o : a_off) asm("" : "+v"(o));
        for (uint32_t &o : b_off) asm("" : "+v"(o));
        s = s * KS + team;
        s = s < all_steps ? s : all_steps - 1;
        if constexpr (DW) {
            const int t0 = s == 0 ? 0 : rem + 64 * (s - 1);
            const gptr pa = scalar(g.dY, (size_t)t0 * a_pitch), pb = scalar(g.Xq, (size_t)t0 * b_pitch);
#pragma unroll
            for (int i = 0; i < 2; ++i) {
                const v4u q = at<v4u>(pa + a_off[i]);
                r.a[4 * i] = q[0]; r.a[4 * i + 1] = q[1]; r.a[4 * i + 2] = q[2]; r.a[4 * i + 3] = q[3];
                const v2u c = at<v2u>(pb + b_off[i]);
                r.b[2 * i] = c[0]; r.b[2 * i + 1] = c[1];
            }
        } else {
            const gptr pa = scalar(g.dY, (size_t)s * kRowBytes);
#pragma unroll
            for (int i = 0; i < 2; ++i) {
                const v4u q = at<v4u>(pa + a_off[i]);
                r.a[4 * i] = q[0]; r.a[4 * i + 1] = q[1]; r.a[4 * i + 2] = q[2]; r.a[4 * i + 3] = q[3];
            }
            const gptr blk = scalar(g.packed, ((size_t)(2 * s + cb) * tiles_k + tile_n) * (256 * BITS));
            if constexpr (BITS == 8) {
                const v4u q = at<v4u>(blk + b_off[0]);
                r.b[0] = q[0]; r.b[1] = q[1]; r.b[2] = q[2]; r.b[3] = q[3];
            } else if constexpr (BITS == 4) {
                const v2u q = at<v2u>(blk + b_off[0]);
                r.b[0] = q[0]; r.b[1] = q[1];
            } else {
                r.b[0] = at<uint32_t>(blk + b_off[0]);
                if constexpr (BITS == 3) r.b[1] = at<uint32_t>(blk + (uint32_t)(lane * 12 + 8));
            }
            // the row's group: (row + 1/2) / rows lies at least 1/(2 rows) from a whole number, which binary32 keeps apart
            // for rows below 2^20
            const uint32_t gi = (uint32_t)(((float)(s * 64) + row_f0) * g.rcp_rows);
            r.h = g.h[gi];
            r.z = zsrc[gi];
        }
    };

    // ---- registers -> LDS
    auto store = [&](int s, const Set &r) {  // (a step past the end is stored, but not multiplied)
        uint8_t *A = lds + (s & 1) * kStage, *B = A + kTile * kRowBytes;
#pragma unroll
        for (int i = 0; i < 2; ++i) {
            const int row = i * 32 + (tid >> 3);
            *reinterpret_cast<uint4 *>(A + (DW ? turned_at(row, tid & 7) : lds_at(row, tid & 7))) = make_uint4(r.a[4 * i], r.a[4 * i + 1], r.a[4 * i + 2], r.a[4 * i + 3]);
        }
        if constexpr (DW) {
#pragma unroll
            for (int i = 0; i < 2; ++i) {
                uint32_t e[4];
#pragma unroll
                for (int p = 0; p < 4; ++p) {
                    // 2x'+1 = 2(x'+128) - 255: at most eight significant bits, exact in bf16
                    const uint32_t u = r.b[2 * i + (p >> 1)] ^ 0x80808080u;
                    const float f0 = __builtin_fmaf(byte_f(u, 2 * (p & 1)), 2.0f, -255.0f), f1 = __builtin_fmaf(byte_f(u, 2 * (p & 1) + 1), 2.0f, -255.0f);
                    e[p] = hi_halves(__float_as_uint(f0), __float_as_uint(f1));
                }
                *reinterpret_cast<uint4 *>(B + turned_at(i * 32 + (tid >> 3), tid & 7)) = make_uint4(e[0], e[1], e[2], e[3]);
            }
        } else {
            constexpr int L = (1 << BITS) - 1;
            uint32_t d[4];  // sixteen codes
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                if constexpr (BITS == 8) d[i] = r.b[i];
                else if constexpr (BITS == 4) d[i] = (r.b[i >> 1] >> (4 * (i & 1))) & 0x0F0F0F0Fu;
                else if constexpr (BITS == 2) d[i] = (r.b[0] >> (2 * i)) & 0x03030303u;
                else d[i] = ((r.b[0] >> (2 * i)) & 0x03030303u) | (((r.b[1] >> (4 * part) >> i) & 0x01010101u) << 2);
            }
            // h * (2u - L) + 0, or Delta * u + q0; the inner product is exact
            const float um = g.q0 ? 1.0f : 2.0f, uc = g.q0 ? 0.0f : -(float)L, z = g.q0 ? r.z : 0.0f;
            // (the codes belong to one row n of the weights)
            uint32_t w[8];
#pragma unroll
            for (int i = 0; i < 8; ++i) {
                const float u0 = byte_f(d[i >> 1], 2 * (i & 1)), u1 = byte_f(d[i >> 1], 2 * (i & 1) + 1);
                w[i] = bf16_pair(__builtin_fmaf(r.h, __builtin_fmaf(u0, um, uc), z), __builtin_fmaf(r.h, __builtin_fmaf(u1, um, uc), z));
            }
#pragma unroll
            for (int i = 0; i < 2; ++i)
                *reinterpret_cast<uint4 *>(B + turned_at(32 * cb + l32, 4 * hf + 2 * part + i)) = make_uint4(w[4 * i], w[4 * i + 1], w[4 * i + 2], w[4 * i + 3]);
        }
    };

    // ---- fragments: result l32 of 32, contraction steps 16*sub + 8*hf .. +7
    const int wm = wave >> 1, wn = wave & 1;
    uint32_t a_frag[DW ? 2 : 4], b_frag[2];
#pragma unroll
    for (int q = 0; q < 2; ++q) {
        // (32 results further on: the other half of every row)
        if constexpr (DW) a_frag[q] = turned_fragment(lane, q) ^ (64 * wm);
        b_frag[q] = kTile * kRowBytes + (turned_fragment(lane, q) ^ (64 * wn));
    }
    if constexpr (!DW) {
#pragma unroll
        for (int sub = 0; sub < 4; ++sub) a_frag[sub] = wm * 32 * kRowBytes + lds_at(l32, sub * 2 + hf);
    }
    v16f acc;
#pragma unroll
    for (int i = 0; i < 16; ++i) acc[i] = 0.0f;

#pragma unroll
    for (int u = 0; u < AHEAD; ++u) load(u, set[u]);

    // A team finishes UPT of the wavefront's four units of eight rows (lane: rows 4*hf .. +3 of the unit, column l32).
    constexpr int UPT = 4 / KS;
    const int row_base = r0 + wm * 32 + team * UPT * 8 + 4 * hf;
    const int col = c0 + wn * 32 + l32;
    auto fence = [&]() {
        __builtin_amdgcn_s_waitcnt(0xC07F);  // lgkmcnt(0): this wavefront's LDS reads and writes have completed
        asm volatile("" ::: "memory");
        __builtin_amdgcn_s_barrier();
        asm volatile("" ::: "memory");
    };
    auto multiply = [&](int s) {
        const uint8_t *st = lds + (s & 1) * kStage;
        v8bf af[4], bf[4];
#pragma unroll
        for (int sub = 0; sub < 4; ++sub) {
            const uint8_t *rows = st + sub * 16 * kRowBytes;
            bf[sub] = turned_read(rows + b_frag[0], rows + b_frag[1]);
            if constexpr (DW) af[sub] = turned_read(rows + a_frag[0], rows + a_frag[1]);
            else af[sub] = *reinterpret_cast<const v8bf *>(st + a_frag[sub]);
        }
#pragma unroll
        for (int sub = 0; sub < 4; ++sub) acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(af[sub], bf[sub], acc, 0, 0, 0);
    };
    if (DW && team == 0) {
#pragma unroll
        for (int i = 0; i < 8; ++i)
            if ((i >> 2) * 32 + (tid >> 3) >= rem) set[0].a[i] = 0;
    }
    store(0, set[0]);
    fence();
    int s = 0;
    for (; s + AHEAD < steps; s += AHEAD) {
#pragma unroll
        for (int u = 0; u < AHEAD; ++u) {
            load(s + u + AHEAD, set[u]);
            __builtin_amdgcn_sched_barrier(0);
            multiply(s + u);
            store(s + u + 1, set[(u + 1) % AHEAD]);
            fence();
        }
    }
    // The values and limits of the clamp's derivative, on their way while the last operands are multiplied (in front of the first ones they
    // made the tile wait for all of its loads at its start: 1001 tokens, 448 x 1792 11.4 -> 10.5 us, 2000 x 1024 x 1024 19.9 -> 18.9).  Without a mask for this product the same value is read and none is outside.
    float raw[MASK ? UPT * 4 : 1], lim[MASK && DW ? UPT * 4 : 1];
    const float *const mask_src = DW ? g.W : g.X;
    if constexpr (MASK) {
        const float *base = mask_src ? mask_src + col : g.h, *ranges = mask_src ? g.m : g.h;
        const size_t pitch = mask_src ? (size_t)K : 0;
#pragma unroll
        for (int i = 0; i < UPT * 4; ++i) {
            int r = row_base + 8 * (i >> 2) + (i & 3);
            if (!DW) r = r < T ? r : T - 1;
            raw[i] = base[(size_t)r * pitch];
            if constexpr (DW) lim[i] = ranges[(uint32_t)(((float)r + 0.5f) * g.rcp_rows)];
        }
        __builtin_amdgcn_sched_barrier(0);
    }
#pragma unroll
    for (int u = 0; u < AHEAD; ++u) {
        if (s + u < steps && (KS == 1 || s + u < steps - 1 || (s + u) * KS + team < all_steps)) multiply(s + u);
        if (s + u + 1 < steps) {
            store(s + u + 1, set[(u + 1) % AHEAD]);
            fence();
        }
    }

    v4f fin[UPT];
    if constexpr (KS == 1) {
#pragma unroll
        for (int u = 0; u < 4; ++u) fin[u] = v4f{acc[4 * u], acc[4 * u + 1], acc[4 * u + 2], acc[4 * u + 3]};
    } else {
        // every team leaves the units of the others in LDS, then adds its own units in the order of the teams
        fence();
        v4f *ex = reinterpret_cast<v4f *>(lds_all) + wave * 256 + lane;  // [team][wavefront][unit][lane]
#pragma unroll
        for (int u = 0; u < 4; ++u)
            if (u / UPT != team) ex[team * 1024 + u * 64] = v4f{acc[4 * u], acc[4 * u + 1], acc[4 * u + 2], acc[4 * u + 3]};
        fence();
#pragma unroll
        for (int u = 0; u < UPT; ++u)
#pragma unroll
            for (int t = 0; t < KS; ++t) {
                v4f part_sum;
                const int w = 4 * (t * UPT + u);
                if (t == team) part_sum = v4f{acc[w], acc[w + 1], acc[w + 2], acc[w + 3]};
                else part_sum = ex[t * 1024 + (team * UPT + u) * 64];
                fin[u] = t == 0 ? part_sum : fin[u] + part_sum;
            }
    }
    if constexpr (MASK) {
#pragma unroll
        for (int i = 0; i < UPT * 4; ++i) {
            const float limit = !mask_src ? __builtin_huge_valf() : DW ? lim[DW ? i : 0] : g.clip;
            fin[i >> 2][i & 3] = fabsf(raw[i]) > limit ? 0.0f : fin[i >> 2][i & 3];
        }
    }
    if constexpr (DW) {
        float *out = g.dW + (size_t)row_base * K + col;
#pragma unroll
        for (int i = 0; i < UPT * 4; ++i) __builtin_nontemporal_store(fin[i >> 2][i & 3] * g.scale, out + (size_t)(8 * (i >> 2) + (i & 3)) * K);
    } else {
        // four neighbouring lanes exchange words (two butterfly steps) so that each holds one row of four columns
        const int lq = lane & 3, odd = lane & 1, hi2 = (lane >> 1) & 1;
        uint16_t *out = g.dX + (size_t)(row_base + lq) * K + (col - lq);
#pragma unroll
        for (int u = 0; u < UPT; ++u) {
            const uint32_t h01 = bf16_pair(fin[u][0], fin[u][1]), h23 = bf16_pair(fin[u][2], fin[u][3]);
            // this lane's column of rows (0,1), (2,3) -> row odd resp. 2 + odd of the lane pair's two columns
            const uint32_t x01 = lane_xor1(h01), x23 = lane_xor1(h23);
            const uint32_t w0 = odd ? hi_halves(x01, h01) : lo_halves(h01, x01);
            const uint32_t w1 = odd ? hi_halves(x23, h23) : lo_halves(h23, x23);
            const uint32_t rx = lane_xor2(hi2 ? w0 : w1);
            const v2u o = {hi2 ? rx : w0, hi2 ? w1 : rx};
            uint16_t *p = out + (size_t)(8 * u) * K;
            if (row_base + lq + 8 * u < T) {
                if (g.quad_ok) __builtin_nontemporal_store(o, reinterpret_cast<v2u *>(p));
                else { p[0] = (uint16_t)o[0]; p[1] = (uint16_t)(o[0] >> 16); p[2] = (uint16_t)o[1]; p[3] = (uint16_t)(o[1] >> 16); }
            }
        }
    }
}

template <int KS, int BITS, bool MASK>
__global__ __launch_bounds__(256 * KS, 4) void bwd_direct_kernel(const DirectArgs g)
{
    __shared__ __align__(1024) uint8_t lds[KS * 2 * kStage];
    int b = (int)blockIdx.x;
    const int first = g.dw_first ? g.tiles_w : g.tiles_x;
    const bool dw = (b < first) == (g.dw_first != 0);
    if (b >= first) b -= first;
    // workgroups are dealt to the 8 XCDs in turn: each gets a contiguous share of the product's tiles
    const int n = dw ? g.tiles_w : g.tiles_x, x = b & 7, q = n >> 3, r = n & 7;
    const int tile = x * q + (x < r ? x : r) + (b >> 3);
    if (dw) direct_tile<KS, BITS, MASK, true>(g, tile, lds);
    else direct_tile<KS, BITS, MASK, false>(g, tile, lds);
}

template <int KS, bool MASK>
void launch(const DirectArgs &g, int bits, hipStream_t st)
{
    const dim3 grid((unsigned)(g.tiles_w + g.tiles_x)), block(256 * KS);
    switch (bits) {
        case 2: hipLaunchKernelGGL((bwd_direct_kernel<KS, 2, MASK>), grid, block, 0, st, g); break;
        case 3: hipLaunchKernelGGL((bwd_direct_kernel<KS, 3, MASK>), grid, block, 0, st, g); break;
        case 4: hipLaunchKernelGGL((bwd_direct_kernel<KS, 4, MASK>), grid, block, 0, st, g); break;
        default: hipLaunchKernelGGL((bwd_direct_kernel<KS, 8, MASK>), grid, block, 0, st, g); break;
    }
}

template <int KS>
void launch(const DirectArgs &g, int bits, hipStream_t st)
{
    if (g.X || g.W) launch<KS, true>(g, bits, st);
    else launch<KS, false>(g, bits, st);
}

}  // namespace

int bwd_direct_teams(int64_t T, int64_t N, int64_t K, bool dx, bool dw)
{
    if (N % 64 != 0 || T < 64 || N > (1 << 20) || K > (1 << 20) || T * N >= (int64_t)1 << 31) return 0;
    const int64_t tt = (T + 63) / 64, tn = N / 64, tk = K / 64;
    const int64_t tiles = ((dx ? tt : 0) + (dw ? tn : 0)) * tk;  // of 64 x 64 results
    const int64_t chain = std::max(dx ? tn : 0, dw ? tt : 0);    // steps of the longest contraction
    const double share = (double)(((dx ? 1 : 0) + (dw ? 1 : 0)) * tt * tn * tk) / 256;  // steps per CU
    // Microseconds, fitted to some six hundred calls of both paths (64..12000 tokens, N and K 256..4096, 2-8 bits, masked,
    // asymmetric, one output), with operands turned in registers, which took 5 to 15 % longer than the reads that turn them now (of 250 calls of 128 to 8000
    // tokens the choice takes 2 % longer than the best one on average, just beyond the line up to 20 %: 3482 x 768 x 768 26.3 us staged, 22.3 here): a fixed
    // part and the longer of the chain of one workgroup's steps and the CU's share of all steps.  A lone workgroup takes 0.40, 0.57 and 0.85 us for a step of one, two and four teams; the staged path spends two
    // launches, and on long contractions with few tiles a chain of partial sums.  dX alone stages only the weights, so that
    // there the GEMM's tiles (of 128 x 96) show.
    const double staged_share = dw ? 17 + 0.13 * share : 13.7 + 0.13 * share + 1.85 * (double)(((T + 127) / 128) * ((K + 95) / 96)) / 256;
    const double staged = std::max(staged_share, std::min(11 + 0.23 * chain, 37.0));
    const double one = 4.5 + std::max(0.40 * chain, 0.27 * share);
    const double two = 4.5 + std::max(0.57 * ((chain + 1) / 2), 0.32 * share);
    const double four = 4.5 + std::max(0.85 * ((chain + 3) / 4), 0.36 * share + (tiles > 256 ? 2 : 0));
    double best = std::min(one, std::min(two, four));
    const int teams = best == one ? 1 : best == two ? 2 : 4;
    // One team: up to four workgroups share a CU from the start, dealt in the order of the launch (the longer contraction
    // first), and the CU with the most steps decides, which with few workgroups a CU has far more than its share: 3072 x 768 at
    // 2067 tokens, dX alone, 396 workgroups of 48 steps: 29.2 us here, 25.0 staged; 2304 x 768 at 1364: 25.9 and 25.9.
    const int64_t per_cu = (tiles + 255) / 256;
    if (teams == 1 && per_cu <= 4) {
        const double step[4] = {0.40, 0.28, 0.245, 0.22};  // by workgroups on the CU
        const int64_t longer = dx && dw ? (tt >= tn ? tn : tt) * tk : tiles;  // tiles with the longer contraction
        const int64_t n_long = std::min((longer + 255) / 256, per_cu);
        const int64_t steps = n_long * chain + (per_cu - n_long) * std::min(tt, tn);
        best = std::max(best, 4.5 + step[per_cu - 1] * (double)steps);
    }
    // Near the crossover (1024 x 1024 at 2561 tokens: 24.3 us against 29.5; 2099 x 2048 x 512 stays: 25.9 and 25.8) the vector
    // arithmetic that every tile repeats costs what the staging launch does once.
    return best >= 0.97 * staged ? 0 : teams;
}

void bwd_direct_run(DirectArgs g, int teams, int bits, hipStream_t st)
{
    const int tiles_k = g.K / 64;
    g.tiles_x = g.dX ? (g.T + 63) / 64 * tiles_k : 0;
    g.tiles_w = g.dW ? g.N / 64 * tiles_k : 0;
    g.dw_first = (g.T + 63) / 64 >= g.N / 64;  // the longer contraction starts first
    g.rcp_rows = 1.0f / (float)g.rows_per_group;
    g.quad_ok = (reinterpret_cast<uintptr_t>(g.dX) & 7) == 0;
    if (teams == 1) launch<1>(g, bits, st);
    else if (teams == 2) launch<2>(g, bits, st);
    else launch<4>(g, bits, st);
}

}  // namespace qb
