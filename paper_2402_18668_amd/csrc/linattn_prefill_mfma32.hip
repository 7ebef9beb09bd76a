// Causal Taylor linear attention, chunked prefill on the gfx950 matrix cores (bf16 in, fp32
// accumulate), d' = 32.  (Short calls: linattn_prefill_mfma32_short.hip.)
//
// Chunked form of Sec. 4 in blocks of 256 tokens: for a query, the keys of its block come through the masked quadratic
// product 1 + A + A^2 / 2, the tokens before the block through the running state.
//
// Symmetric packing.  One state row per unordered pair of features.  Write a vector as two halves (x, y) of 16 and take indices mod 16.
// Tiles of 32 rows: T = 0 .. 7: x_n x_(n + T), then y_n y_(n + T); T = 8 .. 15: x_n y_(n + T - 8), then y_n x_(n + d), d = 7, 8, 5, 6, 3, 4, 1, 2
// (differences 0 .. 7 and 8 .. 15 of y's index over x's).  Two more: E1 = the linear rows, E2 = x_n x_(n + 8), then y_n y_(n + 8), of which n < 8
// counts.  528 pair rows instead of 1024; the constant's row is kept apart.  Rows are built without the 1 / sqrt(2) of Eq. 4: the readout weighs a
// pair of different features 1 and a square (tile 0) 1/2.  Keys are staged halved, rows hold sum (k_a / 2) (k_b / 2) v, sum (k_a / 2) v, and the outputs
// and denominators are summed as quarters: then nothing inside overflows before the state of Eq. 4 and the kernel's values do.  (Powers of two: no result
// changes by it.  Unhalved and now, us, inputs from memory: 32 units of 16384 tokens 166.0, 166.9, 512 of 2048 236.6, 236.0, 128 of 2048 91.6, 91.3, 16 of 2048
// 36.8, 37.0, 2 of 105 12.5, 12.6.)
//
// Work split.  A workgroup of eight waves takes 64 columns of one (unit, segment).  Wave w owns tiles 2 w, 2 w + 1 (both column tiles of
// 32) and one more product, in accumulators throughout.  A block's phases:
//   operand   every wave writes its tiles, rounded to bf16, to LDS in MFMA operand layout; the rows of K and V go to LDS
//   readout   a wave has 32 queries and all state rows: phi(q) is built from 32 registers, no sum crosses waves
//   intra     the same queries with the key tiles up to their own
//   update    a wave adds the block to its tiles; phi(k) is the product of two rows of K^T, which lies in LDS in fp32.  Of a wave's two tiles
//             the second one's factor is the first one's a lane further within 16 (a DPP operand of the multiplication), so that
//             all waves run the same code and differ in an address
// Two barriers a block; between them waves drift through intra, readout and update.
//
// Denominator.  The K-state is kept as moments: M[a][b] = sum_t k_a k_b, z1[a] = sum_t k_a and the token count.  Per query
// phi(q).z = z0 + sum_a q_a (z1[a] + (M q)[a] / 2); the part from inside the block is the column sum of the masked products.  (M / 4, z1 / 2 are kept.)
//
// Long sequences / few units: G segments; a first launch computes each segment's state increment, segment 0's starting from
// the caller's state, and the main launch starts segment g from the sum of the entries before it (read at full width: all
// loads of an entry in flight together).
//
// What bounds it: per block and SIMD 358 matrix instructions (11,500 cycles) and some 3,300 vector instructions (at 4 cycles each, 13,500), of
// which the hardware overlaps little with two waves to a SIMD: 24,500 cycles in all (phase clocks: operand 3,800, intra 3,500, readout 6,100,
// outputs 1,900, update 8,300, waiting 800), LDS half busy.  What helped on the way (512 units of 2048 tokens, us): the split itself 312 -> 270 (the
// kernel of short calls exchanges 64 KB of partial outputs and rounds the state for every 32 tokens); phi(k) without a branch or an address
// in the slab loop, the matrix instructions at priority 1, 270 -> 249; waves 4 .. 7 ahead in intra and readout, 249 -> 240; half as many LDS writes
// of K^T 240 -> 237.  Tried and not kept: phi(k) from eight code variants with the rotation in the instruction (269), three fp32 rows a slab
// (LDS-bound, 256), two workgroups of four waves in the other kernel's split (300).
// Measured (d_v 64, before and now): 32 units of 16384 tokens 208 -> 168 us, 512 units of 2048 312 -> 237, 128 of 2048 106 -> 85, 192 of 1024
// 78.5 -> 50.6, 64 of 8192 199 -> 160, 16 of 2048 39.2 -> 37.4, of 256 19.5 -> 15.9.
#include "common.h"

#include <cmath>
#include <type_traits>

namespace based {

namespace dp32 {

typedef float f32x2 __attribute__((ext_vector_type(2)));
typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
typedef float f32x16 __attribute__((ext_vector_type(16)));
typedef float f32x8 __attribute__((ext_vector_type(8)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));
typedef short s16x4 __attribute__((ext_vector_type(4)));
typedef short s16x8 __attribute__((ext_vector_type(8)));

constexpr int DP = 32;            // d'
constexpr int NW = 8;             // waves per workgroup
constexpr int NT = NW * 64;
constexpr int QT = 32;            // queries to a wave
constexpr int BLOCK = NW * QT;    // tokens of a block
constexpr int COLS = 64;          // d_v columns per workgroup
constexpr int TILES = 18;
constexpr int SLABS = 35;         // state operands of 16 rows: two to a tile, one of E2
constexpr int KT_LD = BLOCK + 4;  // fp32 rows of K^T (64 banks: the 16-byte reads of 16 consecutive rows fall into different ones)
constexpr int IMG_LD = 40;        // fp32 rows of the state image (the halves of a wave access different banks)

// Workspace entry (one segment's state in accumulator layout): 40 slots of 16 registers x 64 lanes, wave w's from 5 w on: tile 2 w + tt of
// column tile c ^ (w % 2) in slot 2 c + tt, X (below) in slot 4.  Within a slot: [reg / 4][lane][reg % 4].
constexpr int WS_SLOTS = 5 * NW;
constexpr size_t kWsEntryFloats = (size_t)WS_SLOTS * 16 * 64;

struct Kv {   // a block's rows
    float kt[DP][KT_LD];         // K^T / 2
    uint16_t v[BLOCK][COLS];     // 16-byte piece c of row t at c ^ 4 ((t / 2) % 2): the operand reads spread over the banks
};
struct Lds {
    Kv kv;
    uint16_t k[BLOCK][DP];         // K / 2; 16-byte piece c of row t at c ^ (t / 4) % 4
    uint16_t s[SLABS][2][64][8];   // state operands: [slab 2 T + half][column tile][lane][k-slot]
    uint16_t m[2][64][8];          // the same of M
    float cst[COLS], z1[DP];       // a quarter of the constant's row and of the K-state's linear part
};
static_assert(sizeof(Lds) <= 160 * 1024, "one workgroup per CU");
static_assert(sizeof(Lds) >= sizeof(float) * 32 * TILES * IMG_LD, "the state image of one column tile fits the LDS");
struct LdsInc {
    union {
        Kv kv[2];   // block mod 2
        float image[32 * TILES * IMG_LD];
    };
};

__device__ __forceinline__ f32x16 mfma(bf16x8 a, bf16x8 b, f32x16 c)
{
    return __builtin_amdgcn_mfma_f32_32x32x16_bf16(a, b, c, 0, 0, 0);
}

__device__ __forceinline__ bf16x8 pack8(const float *v)
{
    f32x8 f;
#pragma unroll
    for (int e = 0; e < 8; ++e) f[e] = v[e];
    return __builtin_convertvector(f, bf16x8);
}

__device__ __forceinline__ uint32_t pack2(float a, float b)
{
    return __builtin_bit_cast(uint32_t, __builtin_convertvector(f32x2{a, b}, bf16x2));
}

__device__ __forceinline__ bf16x8 as_bf16x8(u32x4 w) { return __builtin_bit_cast(bf16x8, w); }

__device__ __forceinline__ void zero16(f32x16 &a)
{
#pragma unroll
    for (int r = 0; r < 16; ++r) a[r] = 0.f;
}

// Workgroup barrier that orders LDS traffic only (global loads and stores stay in flight).
__device__ __forceinline__ void wg_sync()
{
    asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
}

// MFMA instructions ignore the EXEC mask; an inline-asm statement in a wave-role block makes the
// compiler keep the jump over it (it never runs inline asm with an empty EXEC mask).
__device__ __forceinline__ void role_guard() { asm volatile("; wave-role block: keep the execz branch"); }

__device__ __forceinline__ float bf16lo(uint32_t w) { return __uint_as_float(w << 16); }
__device__ __forceinline__ float bf16hi(uint32_t w) { return __uint_as_float(w & 0xffff0000u); }

// lane i of every 16 gets lane (i + D) % 16
template <int D> __device__ __forceinline__ float rotate16(float x)
{
    return __uint_as_float(__builtin_amdgcn_update_dpp(0u, __float_as_uint(x), 0x120 + 16 - D, 0xf, 0xf, true));
}

// the second factor's index in row fl of tile T < 16
__host__ __device__ constexpr int partner(int T, int fl)
{
    if (T < 8) return (fl & 16) + ((fl + T) & 15);
    return fl < 16 ? 16 + ((fl + T - 8) & 15) : (fl + 7 - (T & 6) + (T & 1)) & 15;
}

// Canonical state rows (Eq. 4 order) of a packed row; a pair row has two (equal for a square).
// With packed_state the buffer is the packed layout (one row per unordered pair: a single row).
struct CanonRows { int r1, r2; };   // r1 < 0: padding
__device__ __forceinline__ CanonRows canon_pair(int a, int b, bool packed_state)
{
    if (packed_state) {
        const int r = packed_pair_row(DP, min(a, b), max(a, b));
        return {r, r};
    }
    return {1 + DP + a * DP + b, 1 + DP + b * DP + a};
}
// row fl of tile T (16: E1; 17: E2)
__device__ __forceinline__ CanonRows canon_rows(int T, int fl, bool packed_state)
{
    if (T == 16) return {1 + fl, 1 + fl};
    if (T < 16) return canon_pair(fl, partner(T, fl), packed_state);
    return fl & 8 ? CanonRows{-1, -1} : canon_pair(fl, fl + 8, packed_state);
}
// what a row is multiplied with on its way out (sum (k_a / 2) (k_b / 2) v to sum k_a k_b v / sqrt(2), sum (k_a / 2) v to sum k_a v)
__device__ __forceinline__ float out_scale(CanonRows c) { return c.r1 > DP ? 4.f * kRsqrt2 : 2.f; }
// and in, and which rows are padding, from the tile: their canonical rows, worked out again, cost a call from a state 1.3 us (7 units of 152 tokens 23.8, 22.4)
__device__ __forceinline__ float in_scale(int T) { return T == 16 ? 0.5f : 0.5f * kRsqrt2; }
__device__ __forceinline__ bool is_padding(int T, int fl) { return T == 17 && (fl & 8) != 0; }

constexpr int kMaxSegments = 16;
struct SegTable { int begin[kMaxSegments + 1]; };

// INC: state increment of piece `seg` of segs only (G - 1 of them, `pieces` to a segment), to workspace entry first_entry + seg; piece 0 starts from the
// caller's state, if any, and also leaves that, converted, in entry 0 (import_only: nothing else).  Otherwise the full prefill of the segment, from
// the sum of the entries of the pieces before it.  A group has `slots` entries.
// init_in_entry: the caller's state is in entry 0 (one workgroup per unit reads it from the buffer itself).
// Slice: columns [64 slice, 64 slice + 64) of v / y.
template <bool INC>
__global__ __launch_bounds__(NT, 2) void prefill_kernel(
    const uint16_t *__restrict__ q, const uint16_t *__restrict__ k, const uint16_t *__restrict__ v,
    uint16_t *__restrict__ y, float *state, int has_init, int import_only, int init_in_entry, float *__restrict__ ws,
    int N, int dv, SegTable segs, int G, int pieces, int first_entry, int slots, int groups, int local)
{
    __shared__ __align__(16) std::conditional_t<INC, LdsInc, Lds> lds;

    // has_init carries three flags: bit 0 an initial state is given, bit 1 the state buffer is packed,
    // bit 2 the outputs are the numerators alone (no division by the denominator)
    const bool packed_state = (has_init & 2) != 0;
    const bool numerator_only = (has_init & 4) != 0;
    has_init &= 1;
    int tid = threadIdx.x;
    const int w = __builtin_amdgcn_readfirstlane(tid >> 6);
    int lane = tid & 63;
    int g = lane >> 5, n = lane & 31;

    const int slices = dv / COLS;
    const int gseg = !INC ? G : import_only ? 1 : G - 1;
    int bid = blockIdx.x;
    // The segments of a group on one XCD (workgroup index mod 8), whose L2 then holds its entries, for the first `local` groups (a
    // multiple of 8; what lies beyond the last group leaves at once); segment by segment over all XCDs for the rest.
    int seg;
    if (bid < local * gseg) {
        seg = (bid >> 3) % gseg;
        bid = ((bid >> 3) / gseg << 3) + (bid & 7);
        if (bid >= groups) return;
    } else {
        bid -= local * gseg;
        seg = bid / (groups - local);
        bid = local + bid % (groups - local);
    }
    seg = __builtin_amdgcn_readfirstlane(seg);
    const int slice = __builtin_amdgcn_readfirstlane(bid % slices);
    const int u = __builtin_amdgcn_readfirstlane(bid / slices);
    const int col0 = slice * COLS;

    const int tok_begin = segs.begin[seg];
    const int tok_end = min(N, segs.begin[seg + 1]);

    const uint16_t *qu = q + (size_t)u * N * DP;
    const uint16_t *ku = k + (size_t)u * N * DP;
    const uint16_t *vu = v + (size_t)u * N * dv + col0;
    uint16_t *yu = y + (size_t)u * N * dv + col0;
    float *Su = state ? state + (size_t)u * (packed_state ? packed_state_stride(DP, dv) : state_stride(DP, dv)) + col0
                      : nullptr;
    float *zu = Su ? Su - col0 + (size_t)(packed_state ? packed_feature_dim(DP) : feature_dim(DP)) * dv : nullptr;
    float *ws_unit = ws + ((size_t)(u * slices + slice) * slots) * kWsEntryFloats;

    // ---- accumulators -------------------------------------------------------------------------
    f32x16 S[2][2];   // [column tile ^ (w % 2)][tile 2 w + tt]
    // wave 0: M; 1: z1 (column b, the same in every row); 2, 3: the constant's row (column c of column tile w - 2, the same in every
    // row); 4, 5: column tile w - 4 of E1; 6, 7: column tile w - 6 of E2
    f32x16 X;
    float z0 = 0.f;   // tokens before this call's first
    zero16(X);
#pragma unroll
    for (int c = 0; c < 2; ++c)
#pragma unroll
        for (int tt = 0; tt < 2; ++tt) zero16(S[c][tt]);

    auto add_entry = [&](int p) {
        const float *e = ws_unit + (size_t)p * kWsEntryFloats;
        const float z = e[4 * 5 * 1024 - 1];
        f32x4 t[5][4];
#pragma unroll
        for (int s = 0; s < 5; ++s)
#pragma unroll
            for (int j = 0; j < 4; ++j) t[s][j] = *reinterpret_cast<const f32x4 *>(e + 5 * 1024 * w + 4 * lane + (s * 4 + j) * 256);
#pragma unroll
        for (int s = 0; s < 5; ++s)
#pragma unroll
            for (int j = 0; j < 4; ++j)
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    if (s < 4) S[s >> 1][s & 1][4 * j + i] += t[s][j][i];
                    else X[4 * j + i] += t[s][j][i];
                }
        z0 += z;
    };
    auto put_entry = [&](int p) {
        float *e = ws_unit + (size_t)p * kWsEntryFloats + 5 * 1024 * w + 4 * lane;
#pragma unroll
        for (int s = 0; s < 5; ++s)
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                f32x4 o;
#pragma unroll
                for (int i = 0; i < 4; ++i) o[i] = s < 4 ? S[s >> 1][s & 1][4 * j + i] : X[4 * j + i];
                if (s == 4 && j == 3 && w == 3) o[3] = lane == 63 ? z0 : o[3];   // (rows hold copies of the constant's)
                *reinterpret_cast<f32x4 *>(e + (s * 4 + j) * 256) = o;
            }
    };

    // The state buffer moves through LDS, one column tile at a time, as an image of its tiles: image[32 T + row][IMG_LD].
    // A wave reaches its registers' places at constant offsets, and the whole workgroup moves 16-byte pieces between the
    // image and the buffer's rows.
    float *image = reinterpret_cast<float *>(&lds);
    constexpr int IMG_Q = 32 * TILES * 8, IMG_STEPS = IMG_Q / NT;   // 16-byte pieces of a column tile: all, per thread
    static_assert(IMG_Q % NT == 0, "");
    auto place = [&](int T, int rr) -> float & { return image[4 * g * IMG_LD + n + (32 * T + 8 * (rr >> 2) + (rr & 3)) * IMG_LD]; };
    auto import_state = [&]() {
#pragma unroll
        for (int cc = 0; cc < 2; ++cc) {
            constexpr int BATCH = 9;
#pragma unroll 1
            for (int s0 = 0; s0 < IMG_STEPS; s0 += BATCH) {
                f32x4 t[BATCH][2];
#pragma unroll
                for (int j = 0; j < BATCH; ++j) {
                    const int i = (s0 + j) * NT + tid, row = i >> 3;
                    const CanonRows cr = canon_rows(row >> 5, row & 31, packed_state);
                    const float *p = Su + 32 * cc + 4 * (i & 7);
                    t[j][0] = *reinterpret_cast<const f32x4 *>(p + (size_t)max(cr.r1, 0) * dv);
                    t[j][1] = *reinterpret_cast<const f32x4 *>(p + (size_t)max(cr.r2, 0) * dv);
                }
#pragma unroll
                for (int j = 0; j < BATCH; ++j) {
                    const int i = (s0 + j) * NT + tid, row = i >> 3;
                    *reinterpret_cast<f32x4 *>(image + row * IMG_LD + 4 * (i & 7)) =
                        is_padding(row >> 5, row & 31) ? f32x4{0.f, 0.f, 0.f, 0.f} : (0.5f * t[j][0] + 0.5f * t[j][1]) * in_scale(row >> 5);   // (halves: the sum may overflow)
                }
            }
            __syncthreads();
#pragma unroll
            for (int rr = 0; rr < 16; ++rr) {
#pragma unroll
                for (int tt = 0; tt < 2; ++tt) {
                    const float t = place(2 * w + tt, rr);
                    S[0][tt][rr] = (w & 1) == cc ? t : S[0][tt][rr];
                    S[1][tt][rr] = (w & 1) == cc ? S[1][tt][rr] : t;
                }
                if (w >= 4 && (w & 1) == cc) X[rr] = place(14 + (w >> 1), rr);
            }
            __syncthreads();
        }
        if (w == 0) {   // M / 4 from the symmetric part of z's pair rows
#pragma unroll
            for (int rr = 0; rr < 16; ++rr) {
                const CanonRows cr = canon_pair(8 * (rr >> 2) + 4 * g + (rr & 3), n, packed_state);
                X[rr] = 0.5f * kRsqrt2 * (0.5f * zu[cr.r1] + 0.5f * zu[cr.r2]);
            }
        }
        if (w > 0 && w < 4) {
            const float t = w == 1 ? 0.5f * zu[1 + n] : Su[32 * (w - 2) + n];
#pragma unroll
            for (int rr = 0; rr < 16; ++rr) X[rr] = t;
        }
        z0 = zu[0];
    };
    auto export_state = [&]() {   // (both rows of a pair; slice 0 writes z)
#pragma unroll
        for (int cc = 0; cc < 2; ++cc) {
            __syncthreads();
#pragma unroll
            for (int rr = 0; rr < 16; ++rr) {
#pragma unroll
                for (int tt = 0; tt < 2; ++tt) {
                    const float t0 = S[0][tt][rr], t1 = S[1][tt][rr];
                    place(2 * w + tt, rr) = (w & 1) == cc ? t0 : t1;
                }
                if (w >= 4 && (w & 1) == cc) place(14 + (w >> 1), rr) = X[rr];
            }
            __syncthreads();
#pragma unroll 3
            for (int st = 0; st < IMG_STEPS; ++st) {
                const int i = st * NT + tid, row = i >> 3;
                const CanonRows cr = canon_rows(row >> 5, row & 31, packed_state);
                if (cr.r1 >= 0) {
                    const f32x4 t = *reinterpret_cast<const f32x4 *>(image + row * IMG_LD + 4 * (i & 7)) * out_scale(cr);
                    float *p = Su + 32 * cc + 4 * (i & 7);
                    *reinterpret_cast<f32x4 *>(p + (size_t)cr.r1 * dv) = t;
                    if (cr.r2 != cr.r1) *reinterpret_cast<f32x4 *>(p + (size_t)cr.r2 * dv) = t;
                }
            }
        }
        if (slice == 0) {
            if (w == 0) {
#pragma unroll
                for (int rr = 0; rr < 16; ++rr) {
                    const int a = 8 * (rr >> 2) + 4 * g + (rr & 3);
                    if (!packed_state || a <= n) zu[canon_pair(a, n, packed_state).r1] = 4.f * kRsqrt2 * X[rr];
                }
            }
            if (w == 1 && g == 0) zu[1 + n] = 2.f * X[0];
            if (tid == 0) zu[0] = z0 + (float)N;
        }
        if ((w == 2 || w == 3) && g == 0) Su[32 * (w - 2) + n] = X[0];
    };

    // The lane's number, worked out anew: what is computed from it in one phase of a block is not kept through the others.
    auto fresh_lane = [&]() {
        asm volatile("v_mbcnt_lo_u32_b32 %0, -1, 0\n\tv_mbcnt_hi_u32_b32 %0, -1, %0" : "=v"(lane));
        tid = 64 * w + lane;
        g = lane >> 5;
        n = lane & 31;
    };

    // ---- a block's rows: global -> registers -> LDS -----------------------------------------------
    // Loads are unconditional (rows past the end re-read the last one, and are zeroed when staged).
    struct Raw { u32x4 k[2], v[4]; } raw;
    auto load_raw = [&](int tok0) {
        const int last = tok_end - 1 - tok0;
        const uint16_t *kb = ku + (size_t)tok0 * DP, *vb = vu + (size_t)tok0 * dv;
#pragma unroll
        for (int h = 0; h < 2; ++h) {
            const uint32_t t = min(2 * (tid >> 2) + h, last);
            raw.k[h] = *reinterpret_cast<const u32x4 *>(kb + (t * DP + 8 * (tid & 3)));
        }
#pragma unroll
        for (int h = 0; h < 4; ++h) {
            const uint32_t t = min((tid >> 3) + 64 * h, last);
            raw.v[h] = *reinterpret_cast<const u32x4 *>(vb + (t * (uint32_t)dv + 8 * (tid & 7)));
        }
    };
    // Queries 32 qt .. + 31 of a block, lane n the n-th.  (Waves w and w + 4 are on one SIMD: nine key tiles for the two.)
    const int qt = w < 4 ? w : 11 - w;
    u32x2 qraw[8];   // elements 16 (b / 4) + 4 ((b + g) % 4) ..
    auto load_q = [&](int tok0) {
        const uint16_t *qb = qu + (size_t)tok0 * DP;
        const uint32_t t = min(QT * qt + n, tok_end - 1 - tok0);
#pragma unroll
        for (int b = 0; b < 8; ++b) qraw[b] = *reinterpret_cast<const u32x2 *>(qb + (t * DP + 16 * (b >> 2) + 4 * ((b + g) & 3)));
    };
    load_raw(tok_begin);
    if (!INC) load_q(tok_begin);

    bool have_state = true;   // (uniform) something to read out before the first block
    if (INC) {
        if (has_init && seg == 0) {
            import_state();
            put_entry(0);
            if (import_only) return;   // uniform
        }
    } else if (seg > 0) {
#pragma unroll 1
        for (int p = 0; p < seg * pieces; ++p) add_entry(first_entry + p);
    } else if (has_init) {
        if (init_in_entry) add_entry(0);
        else import_state();
    } else {
        have_state = false;
    }

    z0 = __uint_as_float(__builtin_amdgcn_readfirstlane(__float_as_uint(z0)));   // (the same in every lane)

    auto stage = [&](int tok0, Kv &kv, uint16_t (*krow)[DP]) {
        const int rows = tok_end - tok0;
        const int t0 = 2 * (tid >> 2), c = tid & 3;
        if (rows < BLOCK) {   // (uniform) rows past the end
            const u32x4 zero = {0u, 0u, 0u, 0u};
#pragma unroll
            for (int h = 0; h < 2; ++h) raw.k[h] = t0 + h < rows ? raw.k[h] : zero;
#pragma unroll
            for (int h = 0; h < 4; ++h) raw.v[h] = (tid >> 3) + 64 * h < rows ? raw.v[h] : zero;
        }
        u32x4 half[2];
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            float lo[2], hi[2];
#pragma unroll
            for (int h = 0; h < 2; ++h) {
                lo[h] = 0.5f * bf16lo(raw.k[h][i]);
                hi[h] = 0.5f * bf16hi(raw.k[h][i]);
                half[h][i] = pack2(lo[h], hi[h]);
            }
            *reinterpret_cast<f32x2 *>(&kv.kt[8 * c + 2 * i][t0]) = f32x2{lo[0], lo[1]};
            *reinterpret_cast<f32x2 *>(&kv.kt[8 * c + 2 * i + 1][t0]) = f32x2{hi[0], hi[1]};
        }
#pragma unroll
        for (int h = 0; h < 2; ++h)
            if (!INC) *reinterpret_cast<u32x4 *>(&krow[t0 + h][8 * (c ^ ((t0 >> 2) & 3))]) = half[h];
#pragma unroll
        for (int h = 0; h < 4; ++h)
            *reinterpret_cast<u32x4 *>(&kv.v[(tid >> 3) + 64 * h][8 * ((tid & 7) ^ (((tid >> 4) & 1) << 2))]) = raw.v[h];
    };

    // ---- operands ---------------------------------------------------------------------------------
    // V^T operand ("8 tokens of one column": lane (g, n): column n of the tile at two runs of 4 tokens) from row-major rows, by the
    // transposing LDS read: in each group of 16 lanes, lane k supplies the address of 4 consecutive columns (4 (k % 4) ..)
    // of row k / 4 of the group's 16-column block and receives column k of that block at the 4 rows.
    // GS: tokens between the runs of g = 0 and 1, RS: between a lane's two runs.
    auto v_place = [&](int GS) {
        return (((lane & 15) >> 2) + GS * g) * COLS + 8 * ((2 * ((lane >> 4) & 1) + ((lane & 3) >> 1)) ^ (((lane >> 3) & 1) << 2)) + 4 * (lane & 1);
    };
    auto read_v = [&](const uint16_t *p, int RS) {   // p: the place in the first row of the 16
        const s16x4 x = __builtin_amdgcn_ds_read_tr16_b64_v4i16((__attribute__((address_space(3))) s16x4 *)p);
        const s16x4 z = __builtin_amdgcn_ds_read_tr16_b64_v4i16((__attribute__((address_space(3))) s16x4 *)(p + RS * COLS));
        s16x8 o;
#pragma unroll
        for (int i = 0; i < 4; ++i) { o[i] = x[i]; o[4 + i] = z[i]; }
        return __builtin_bit_cast(bf16x8, o);
    };

    // ---- state update: S += phi(K)^T V over this wave's tiles; k-slot j of lane (g, n) is token 16 ts + 8 g + j --------
    auto update = [&](const Kv &kv, int slabs) {
        fresh_lane();
        const float *ka = &kv.kt[n][8 * g], *kb = &kv.kt[partner(2 * w, n)][8 * g];
        const uint16_t *v0 = &kv.v[0][0] + (v_place(8) ^ ((w & 1) << 5)), *v1 = &kv.v[0][0] + (v_place(8) ^ ((~w & 1) << 5));
        struct Src { f32x4 a[2], b[2]; bf16x8 v[2]; };
        auto source_k = [&](int ts, Src &s) {
#pragma unroll
            for (int h = 0; h < 2; ++h) {
                s.a[h] = *reinterpret_cast<const f32x4 *>(ka + 16 * ts + 4 * h);
                s.b[h] = *reinterpret_cast<const f32x4 *>(kb + 16 * ts + 4 * h);
            }
        };
        auto source_v = [&](int ts, Src &s) {
            s.v[0] = read_v(v0 + 16 * COLS * ts, 4);   // column tile w % 2
            s.v[1] = read_v(v1 + 16 * COLS * ts, 4);
        };
        // phi(K)^T of the tiles (0, 1), E1 (2), E2 (3)
        auto phi = [&](const Src &s, auto which) {
            constexpr int P = decltype(which)::value;
            float pr[8];
#pragma unroll
            for (int i = 0; i < 8; ++i) {
                const float a = s.a[i >> 2][i & 3], b = s.b[i >> 2][i & 3];
                pr[i] = P == 0 ? a * b : P == 1 ? a * rotate16<1>(b) : P == 2 ? a : a * rotate16<8>(a);
            }
            return pack8(pr);
        };
        constexpr int UNROLL = 4;
        Src src[2];
        source_k(0, src[0]);
        __builtin_amdgcn_sched_barrier(0);   // (in the loop's order, for the count of what is in flight)
        source_v(0, src[0]);
        source_k(1, src[1]);
        __builtin_amdgcn_sched_barrier(0);
        source_v(1, src[1]);
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll 1
        for (int ts = 0; ts < slabs; ts += UNROLL) {   // (past the last token there are zeros, past the end the last ones are read again)
            const int on = ts + UNROLL < slabs ? UNROLL : 0;
#pragma unroll
            for (int i = 0; i < UNROLL; ++i) {
                Src &x = src[i & 1];
                const bf16x8 op0 = phi(x, std::integral_constant<int, 0>{}), op1 = phi(x, std::integral_constant<int, 1>{});
                if (i == UNROLL - 2) {
                    ka += 16 * on, kb += 16 * on;
                    v0 += 16 * COLS * on, v1 += 16 * COLS * on;
                }
                const int next = i < UNROLL - 2 ? i + 2 : i + 2 - UNROLL;
                // (loads stay where they are, two slabs ahead of their use)
                __builtin_amdgcn_sched_barrier(0);
                source_k(next, x);
                __builtin_amdgcn_s_setprio(1);   // (a wave that has its operands goes first: the other one builds its own meanwhile)
                __builtin_amdgcn_sched_barrier(0);
                S[0][0] = mfma(op0, x.v[0], S[0][0]);
                S[1][0] = mfma(op0, x.v[1], S[1][0]);
                S[0][1] = mfma(op1, x.v[0], S[0][1]);
                S[1][1] = mfma(op1, x.v[1], S[1][1]);
                __builtin_amdgcn_sched_barrier(0);
                __builtin_amdgcn_s_setprio(0);
                source_v(next, x);
                __builtin_amdgcn_sched_barrier(0);
            }
            asm volatile("" ::: "memory");
        }
        // X: M / 4 = (K / 2)^T (K / 2), z1 / 2 = 1 (K / 2), the constant 1 V; E1, E2
        const u32x4 one = {0x3F803F80u, 0x3F803F80u, 0x3F803F80u, 0x3F803F80u};
        const float *kx = &kv.kt[n][8 * g];
        const uint16_t *vx = &kv.v[0][0] + (v_place(8) ^ ((w & 1) << 5));
        auto add_x = [&](auto kind) {
            constexpr int P = decltype(kind)::value;
            role_guard();
#pragma unroll 1
            for (int t0 = 0; t0 < slabs; t0 += UNROLL) {
                Src x[UNROLL];
#pragma unroll
                for (int i = 0; i < UNROLL; ++i) {
                    if (P != 2) {
#pragma unroll
                        for (int h = 0; h < 2; ++h) x[i].a[h] = *reinterpret_cast<const f32x4 *>(kx + 16 * i + 4 * h);
                    }
                    if (P >= 2) x[i].v[0] = read_v(vx + 16 * COLS * i, 4);
                }
                kx += 16 * UNROLL, vx += 16 * COLS * UNROLL;
                __builtin_amdgcn_sched_barrier(0);
#pragma unroll
                for (int i = 0; i < UNROLL; ++i) {
                    bf16x8 op = as_bf16x8(one);
                    if (P != 2) op = phi(x[i], std::integral_constant<int, P == 4 ? 3 : 2>{});
                    X = P == 0 ? mfma(op, op, X) : P == 1 ? mfma(as_bf16x8(one), op, X) : mfma(op, x[i].v[0], X);
                }
            }
        };
        if (w == 0) add_x(std::integral_constant<int, 0>{});
        else if (w == 1) add_x(std::integral_constant<int, 1>{});
        else if (w < 4) add_x(std::integral_constant<int, 2>{});
        else if (w < 6) add_x(std::integral_constant<int, 3>{});
        else add_x(std::integral_constant<int, 4>{});
    };
    auto slabs_of = [&](int tok0) { return 2 * min((tok_end - tok0 + QT - 1) / QT, NW); };

    fresh_lane();
    if constexpr (INC) {
        int gen = 0;
#pragma unroll 1
        for (int tok0 = tok_begin; tok0 < tok_end; tok0 += BLOCK, gen ^= 1) {
            fresh_lane();
            stage(tok0, lds.kv[gen], nullptr);
            load_raw(min(tok0 + BLOCK, tok_end - 1));
            wg_sync();
            update(lds.kv[gen], slabs_of(tok0));
        }
        put_entry(first_entry + seg);
        return;
    } else {
    // ---- full pass ----------------------------------------------------------------------------------

#pragma unroll 1
    for (int tok0 = tok_begin; tok0 < tok_end; tok0 += BLOCK) {
        const bool more = tok0 + BLOCK < tok_end;
        // ---- operand
        fresh_lane();
        stage(tok0, lds.kv, lds.k);
        if (have_state) {
            auto put = [&](uint16_t *p, const f32x16 &a, int r0, int r1, float scale = 1.f) {   // registers r0 .. + 3, r1 .. + 3
                f32x8 f;
#pragma unroll
                for (int i = 0; i < 4; ++i) { f[i] = scale * a[r0 + i]; f[4 + i] = scale * a[r1 + i]; }
                *reinterpret_cast<bf16x8 *>(p + 8 * lane) = __builtin_convertvector(f, bf16x8);
            };
#pragma unroll
            for (int tt = 0; tt < 2; ++tt)
#pragma unroll
                for (int c = 0; c < 2; ++c)
#pragma unroll
                    for (int sl = 0; sl < 2; ++sl) {
                        put(lds.s[4 * w + 2 * tt + sl][c ^ (w & 1)][0], S[c][tt], 8 * sl, 8 * sl + 4);
                    }
            if (w == 0) {
                put(lds.m[0][0], X, 0, 4);
                put(lds.m[1][0], X, 8, 12);
            } else if (w < 4) {
                if (g == 0) (w == 1 ? lds.z1 : lds.cst + 32 * (w - 2))[n] = (w == 1 ? 0.5f : 0.25f) * X[0];
            } else if (w < 6) {
                put(lds.s[32][w - 4][0], X, 0, 4, 0.5f);
                put(lds.s[33][w - 4][0], X, 8, 12, 0.5f);
            } else {
                put(lds.s[34][w - 6][0], X, 0, 8);
            }
        }
        wg_sync();

        fresh_lane();
        const bool mine = tok0 + QT * qt < tok_end;   // (uniform) this wave has queries
        f32x16 Y[2];
        float den = 0.f;
        if (mine) {
            role_guard();
            bf16x8 qop[2];   // contraction slots (jj, i): element 16 h + 8 jj + 4 g + i
#pragma unroll
            for (int h = 0; h < 2; ++h) qop[h] = as_bf16x8(u32x4{qraw[4 * h][0], qraw[4 * h][1], qraw[4 * h + 2][0], qraw[4 * h + 2][1]});
            // ---- intra: P^T / 2 = 1 / 4 + (1 / 2 + A^T / 2)^2, masked in the queries' own tile; Y^T / 2 = V^T P^T / 2
            zero16(Y[0]);
            zero16(Y[1]);
            if (w >= 4) __builtin_amdgcn_s_setprio(2);   // (these waves have the most key tiles)
            const int k_row = n * DP + 4 * g, k_sw = (n >> 2) & 3;
            const uint16_t *kr = &lds.k[0][0] + k_row;
            const uint16_t *v0 = &lds.kv.v[0][0] + v_place(4), *v1 = &lds.kv.v[0][0] + (v_place(4) ^ 32);
            u32x2 ko[4];
            bf16x8 va[2][2];
            auto load_k = [&](int kt) {
#pragma unroll
                for (int c = 0; c < 4; ++c) ko[c] = *reinterpret_cast<const u32x2 *>(kr + QT * DP * kt + 8 * (c ^ k_sw));
            };
            auto load_v = [&](int kt) {
#pragma unroll
                for (int sl = 0; sl < 2; ++sl) {
                    va[sl][0] = read_v(v0 + COLS * (QT * kt + 16 * sl), 8);
                    va[sl][1] = read_v(v1 + COLS * (QT * kt + 16 * sl), 8);
                }
            };
            auto scores = [&](f32x16 &P) {   // 1 / 2 + A^T / 2
#pragma unroll
                for (int rr = 0; rr < 16; ++rr) P[rr] = 0.5f;
#pragma unroll
                for (int h = 0; h < 2; ++h)
                    P = mfma(as_bf16x8(u32x4{ko[2 * h][0], ko[2 * h][1], ko[2 * h + 1][0], ko[2 * h + 1][1]}), qop[h], P);
            };
            auto multiply = [&](f32x16 &P, bool own) {
#pragma unroll
                for (int rr = 0; rr < 16; ++rr) P[rr] = fmaf(P[rr], P[rr], 0.25f);
                if (own) {
#pragma unroll
                    for (int rr = 0; rr < 16; ++rr) P[rr] = 8 * (rr >> 2) + (rr & 3) <= n - 4 * g ? P[rr] : 0.f;
                }
                float cs[2] = {0.f, 0.f};
#pragma unroll
                for (int rr = 0; rr < 16; ++rr) cs[rr & 1] += P[rr];
                den += cs[0] + cs[1];
#pragma unroll
                for (int sl = 0; sl < 2; ++sl) {
                    float pr[8];
#pragma unroll
                    for (int e = 0; e < 8; ++e) pr[e] = P[8 * sl + e];
                    const bf16x8 op = pack8(pr);
#pragma unroll
                    for (int c = 0; c < 2; ++c) Y[c] = mfma(va[sl][c], op, Y[c]);
                }
            };
            // (a tile's scores are under way while the one before is multiplied with its values)
            f32x16 P0, P1;
            load_k(0);
            load_v(0);
            scores(P0);
            load_k(min(1, qt));
            int kt = 0;
#pragma unroll 1
            for (; kt + 2 <= qt; kt += 2) {
                auto step = [&](f32x16 &now, f32x16 &next, int kt) {
                    scores(next);
                    load_k(min(kt + 2, qt));
                    __builtin_amdgcn_sched_barrier(0);
                    multiply(now, false);
                    __builtin_amdgcn_sched_barrier(0);
                    load_v(kt + 1);
                    __builtin_amdgcn_sched_barrier(0);
                };
                step(P0, P1, kt);
                step(P1, P0, kt + 1);
            }
            if (kt < qt) {
                scores(P1);
                __builtin_amdgcn_sched_barrier(0);
                multiply(P0, false);
                load_v(kt + 1);
                P0 = P1;
            }
            multiply(P0, true);
            Y[0] *= 0.5f;
            Y[1] *= 0.5f;
            den *= 0.5f;
            if (have_state) {
                // ---- readout: Y^T / 4 += S^T phi(q) / 4
                float r[2][16];   // r[h][m]: element 16 h + (m + 4 g) % 16
#pragma unroll
                for (int b = 0; b < 8; ++b)
#pragma unroll
                    for (int i = 0; i < 2; ++i) {
                        r[b >> 2][4 * (b & 3) + 2 * i] = bf16lo(qraw[b][i]);
                        r[b >> 2][4 * (b & 3) + 2 * i + 1] = bf16hi(qraw[b][i]);
                    }
                // (the state operands are requested AHEAD slabs early; the next slab's phi(q) is built under the matrix instructions)
                constexpr int AHEAD = 4;
                const __attribute__((address_space(3))) bf16x8 *sp[2];   // (an LDS offset reaches 64 KB)
#pragma unroll
                for (int i = 0; i < 2; ++i) {
                    sp[i] = (const __attribute__((address_space(3))) bf16x8 *)&lds.s[18 * i][0][lane][0];
                    asm volatile("" : "+v"(sp[i]));
                }
                bf16x8 ring[AHEAD][2];
                auto request = [&](int s) {
#pragma unroll
                    for (int c = 0; c < 2; ++c) ring[s % AHEAD][c] = sp[s / 18][(2 * (s % 18) + c) * 64];
                };
                auto phi = [&](int s) {   // k-slot (jj, i) = row 16 h + 8 jj + 4 g + i of tile T
                    const int T = s >> 1, h = s & 1;
                    if (T == 16) return qop[h];
                    float pr[8];
#pragma unroll
                    for (int e = 0; e < 8; ++e) {
                        const int m = 8 * (e >> 2) + (e & 3);
                        if (T < 16) {
                            const int to = partner(T, 16 * h + m);
                            pr[e] = (T == 0 ? 0.5f * r[h][m] : r[h][m]) * r[to >> 4][to & 15];
                        } else {   // (the slab's rows are those of E2 that count)
                            pr[e] = r[e >> 2][e & 3] * r[e >> 2][(e & 3) + 8];
                        }
                    }
                    return pack8(pr);
                };
#pragma unroll
                for (int s = 0; s < AHEAD; ++s) request(s);
                bf16x8 op = phi(0);
                __builtin_amdgcn_sched_barrier(0);
#pragma unroll
                for (int s = 0; s < SLABS; ++s) {
                    Y[0] = mfma(ring[s % AHEAD][0], op, Y[0]);
                    Y[1] = mfma(ring[s % AHEAD][1], op, Y[1]);
                    if (s + 1 < SLABS) op = phi(s + 1);
                    __builtin_amdgcn_sched_barrier(0);
                    if (s + AHEAD < SLABS) request(s + AHEAD);
                    __builtin_amdgcn_sched_barrier(0);
                }
                // the constant
#pragma unroll
                for (int c = 0; c < 2; ++c)
#pragma unroll
                    for (int j = 0; j < 4; ++j) {
                        const f32x4 t = *reinterpret_cast<const f32x4 *>(&lds.cst[32 * c + 8 * j + 4 * g]);
#pragma unroll
                        for (int i = 0; i < 4; ++i) Y[c][4 * j + i] += t[i];
                    }
                // denominator: T[a][query] = (M q)[a] / 4, then sum_a q_a (z1[a] / 4 + T[a] / 2)
                f32x16 T;
                zero16(T);
#pragma unroll
                for (int h = 0; h < 2; ++h) T = mfma(*reinterpret_cast<const bf16x8 *>(lds.m[h][lane]), qop[h], T);
#pragma unroll
                for (int j = 0; j < 4; ++j) {
                    const f32x4 t = *reinterpret_cast<const f32x4 *>(&lds.z1[8 * j + 4 * g]);
#pragma unroll
                    for (int i = 0; i < 4; ++i) den = fmaf(r[j >> 1][8 * (j & 1) + i], fmaf(0.5f, T[4 * j + i], t[i]), den);
                }
            }
        }
        if (more) {   // the next block's rows, on their way during the rest of this one
            fresh_lane();
            load_raw(tok0 + BLOCK);
            load_q(min(tok0 + BLOCK, tok_end - 1));
        }
        if (mine) {
            role_guard();
            // ---- outputs: the halves of a wave exchange quads, 16 bytes a lane
            const auto d = __builtin_amdgcn_permlane32_swap(__float_as_uint(den), __float_as_uint(den), false, false);
            const float before = have_state ? 0.25f * (z0 + (float)tok0) : 0.f;   // tokens in the state
            const float inv = numerator_only ? 4.f : 1.f / (before + (__uint_as_float(d[0]) + __uint_as_float(d[1])));
            const int tok = QT * qt + n;
            uint16_t *yb = yu + (size_t)tok0 * dv + (uint32_t)(tok * dv + 8 * g);
#pragma unroll
            for (int c = 0; c < 2; ++c)
#pragma unroll
                for (int j = 0; j < 4; j += 2) {
                    uint32_t p[2][2];
#pragma unroll
                    for (int jj = 0; jj < 2; ++jj)
#pragma unroll
                        for (int i = 0; i < 2; ++i)
                            p[jj][i] = pack2(Y[c][4 * (j + jj) + 2 * i] * inv, Y[c][4 * (j + jj) + 2 * i + 1] * inv);
                    const auto x = __builtin_amdgcn_permlane32_swap(p[0][0], p[1][0], false, false);
                    const auto z = __builtin_amdgcn_permlane32_swap(p[0][1], p[1][1], false, false);
                    if (tok0 + tok < tok_end) *reinterpret_cast<u32x4 *>(yb + 32 * c + 8 * j) = u32x4{x[0], z[0], x[1], z[1]};
                }
        }
        // ---- update
        __builtin_amdgcn_s_setprio(0);
        if (more || (Su && seg == G - 1)) update(lds.kv, slabs_of(tok0));
        have_state = true;
        wg_sync();
    }
    if (Su && seg == G - 1) {
        fresh_lane();
        export_state();
    }
    }
}

// Segments: at most one round of the chip (one workgroup per CU).  With few units the chain of an increment, up to G - 1 entries to sum and
// the main pass is shortest at segments of about 5 tiles of 32 tokens, from some 10 segments on of more (16 units, us: N 777 3 segments 32.5,
// 4 28.4, 5 30.4; N 1024 4 33.7, 6 32.2, 8 34.9; N 2048 6 39.4, 8 40.8, 10 39.3, 16 48.7; N 4096 8 56.9, 10 48.3, 16 51.6; N 16384 10 119.7, 16
// 103.1).  With more units there is room for fewer, and one block after the other is the shorter chain for longer (1 segment and what there is room
// for: 16 units N 512 25.6, 26.1; 32 units N 512 26.3, 28.9, N 1024 45, 34; 64 units N 512 27.9, 32.9, N 1024 47.8, 40.4; 66 units N 769 42.7, 36.0, from a state 52.0, 46.4; 85
// units N 769 42.9, 39.1, N 833 44.1, 40.2, from a state 53.6, 51.1; 96 units N 2048 86.6, 80.2; 128 units N
// 1024 48.6, 54.2, N 4096 178, 156).  Two segments whose increment two workgroups share (without a state) are the shorter chain from 41 tiles on with up to 104 groups
// (one and two: 87 units N 1000 47.4, 47.7, N 1400 63.4, 58.3, N 1664 73.0, 64.5; 100 units N 1280 57.3, 57.8, N 1400 63.7, 60.8, N 1664 73.4, 67.6; 128
// units N 1400 64.1, 67.3, N 1664 73.7, 76.0).  At d_v 128 a state goes through a launch of its own anyhow, which increments can share: room for three is used from 9
// tiles on (one and three: 33 units N 384 40.1, 38.2, N 513 48.4, 40.3, N 769 58.3, 46.1; 42 units N 289 40.1, 39.8, N 448 43.8, 41.5, N 769 59.5, 48.9; with
// the import of a state as it was, 1 us more for either).
static int pick_segments(int U, int N, int dv, int has_init)
{
    const int groups = U * (dv / COLS), tiles = (N + QT - 1) / QT, room = 256 / groups;
    if (has_init && dv == 2 * COLS && room == 3 && tiles >= 9) return 3;
    if (tiles < (room >= 4 ? 17 : room >= 3 ? 25 : groups <= 104 && !has_init ? 41 : 56)) return 1;
    const int chain = (int)(sqrtf((float)tiles) + 0.5f), longest = chain > 10 ? chain : 10;
    int G = 3 * tiles / 16;
    if (G > longest) G = longest;
    if (G > room) G = room;
    if (G > kMaxSegments) G = kMaxSegments;
    return G < 1 ? 1 : G;
}

// Groups whose segments share an XCD each: all of them (the grid has room for a multiple of 8) where the XCD with the most has a CU for
// every segment, else as many as make up a multiple of 8, the others' segments going to all XCDs.  (Segment after segment of a group
// on different XCDs, the entries read from memory: 60 groups of 1024 tokens in 4 segments 45 us instead of 41, of 448 34 instead of 28.
// 41 groups in 6 segments, where one XCD would hold 36: all groups on their XCD 77 us at 2048 tokens and 225 at 8192, as here 50 and 136,
// none 59 and 144.)
static int local_groups(int groups, int G)
{
    const int most = (groups + 7) / 8;
    return most * G <= 32 ? most * 8 : groups / 8 * 8;
}

// Segment g's main pass starts by summing g entries, which takes about as long as 0.75 tiles each, and the last one writes the state (1.5
// tiles): the later a segment, the shorter, but none longer than the blocks that the average takes.  (The last one as long as the rest, and these, us: 16 units
// of 1024 tokens 32.2, 31.2; 32 units 34.4, 33.4.)
static int make_segments(int N, int G, SegTable &t)
{
    const int T = (N + QT - 1) / QT;
    if (G > T) G = T;
    const int most = (T + NW * G - 1) / (NW * G) * NW;
    int len[kMaxSegments], sum = 0;
    for (int g = 0; g < G; ++g) {
        const float off = 0.75f * (0.5f * (G - 1) - g) - (g == G - 1 && G > 1 ? 1.5f : 0.f);
        len[g] = T / G + (int)(off >= 0.f ? off + 0.5f : off - 0.5f);
        if (len[g] < 1) len[g] = 1;
        if (len[g] > most) len[g] = most;
        sum += len[g];
    }
    // the rounding's remainder is handed to (or taken from) the early segments, one tile at a time
    for (int g = 0; sum != T; g = (g + 1) % G) {
        if (sum < T && len[g] < most) { ++len[g]; ++sum; }
        else if (sum > T && len[g] > 1) { --len[g]; --sum; }
    }
    int pos = 0;
    for (int g = 0; g < G; ++g) { t.begin[g] = pos * QT; pos += len[g]; }
    for (int g = G; g <= kMaxSegments; ++g) t.begin[g] = pos * QT;
    return G;
}

// The first segment in two pieces of whole blocks, as many in the second.
static SegTable halves(const SegTable &t)
{
    SegTable o = t;
    const int tiles = t.begin[1] / QT, half = ((tiles + 1) / 2 + NW - 1) / NW * NW;
    o.begin[1] = (half < tiles ? half : tiles - 1) * QT;
    for (int g = 2; g <= kMaxSegments; ++g) o.begin[g] = t.begin[1];
    return o;
}

static size_t entry_bytes(int U, int N, int dv)
{
    const int a = pick_segments(U, N, dv, 0), b = pick_segments(U, N, dv, 1);
    return (size_t)U * (dv / COLS) * (a > b ? a : b) * kWsEntryFloats * sizeof(float);
}

}  // namespace dp32

bool prefill_mfma32_supported(int dp, int dv, int dtype)
{
    return dtype == BASED_BF16 && dp == dp32::DP && (dv == 64 || dv == 128);
}

// Workspace: one entry per (unit, slice, segment), for the kernel that needs more: which one takes a call may depend on whether there is a state to
// start from.  The size never shrinks with N: what was allocated for the longest sequence serves the shorter ones, and those that go to the kernel of
// short calls may be cut into more segments.
size_t prefill_mfma32_workspace_bytes(int U, int N, int dp, int dv)
{
    (void)dp;
    const size_t a = dp32::entry_bytes(U, N, dv), b = prefill_mfma32_short_workspace_bytes(U, N, dv);
    return ((a > b ? a : b) + 255) / 256 * 256;
}

hipError_t launch_prefill_mfma32(const void *q, const void *k, const void *v, void *y, float *state,
                                 int has_init, int packed_state, void *workspace, int U, int N, int dp, int dv,
                                 hipStream_t s)
{
    if (prefill_mfma32_short_takes(U, N, dv, has_init & 1))
        return launch_prefill_mfma32_short(q, k, v, y, state, has_init, packed_state, workspace, U, N, dv, s);
    // the kernels' flag word (has_init arrives with bit 2 set for numerator-only outputs)
    has_init = (has_init & 1) | (packed_state ? 2 : 0) | (has_init & 4);
    using namespace dp32;
    (void)dp;
    const int slices = dv / COLS;
    SegTable segs;
    const int G = make_segments(N, pick_segments(U, N, dv, has_init & 1), segs);
    const uint16_t *q16 = (const uint16_t *)q, *k16 = (const uint16_t *)k, *v16 = (const uint16_t *)v;
    float *ws = static_cast<float *>(workspace);
    const int groups = U * slices, local = local_groups(groups, G), blocks = local > groups ? local : groups;
    if (((long long)groups + 7) * G >= (1ll << 31)) return hipErrorInvalidValue;
    // Several workgroups of a unit read the caller's state and one overwrites it (at d_v = 128 also its K-state): then it goes
    // through entry 0, which the first launch writes.
    const int in_entry = (has_init & 1) && G * slices > 1;
    // The increment of the first of two segments would leave half of the chip idle: two workgroups halve it where entry 0 is free for the second's.  (us,
    // one and two: 128 units N 2048 82.5, 80.5, N 4096 147, 140; 100 units N 2048 76.5, 72.8, N 4096 134.6, 121.9; 88 units N 8192 260, 229; d_v 128, 48 units
    // N 4096 132.5, 119.1.)
    const int pieces = G == 2 && (has_init & 1) == 0 && groups <= 128 ? 2 : 1, first_entry = pieces == 2 ? 0 : 1;
    auto go = [&](auto increment, const SegTable &table, int g, int workgroups) {
        hipLaunchKernelGGL((prefill_kernel<decltype(increment)::value>), dim3((unsigned)(blocks * workgroups)), dim3(NT), 0, s, q16, k16, v16, (uint16_t *)y,
                           state, has_init, decltype(increment)::value && G == 1, in_entry, ws, N, dv, table, g, pieces, first_entry, G, groups, local);
        return hipGetLastError();
    };
    if (G > 1 || in_entry) {
        SegTable inc = segs;
        if (pieces == 2) inc = halves(segs);
        const int n = G > 1 ? (G - 1) * pieces : 1;
        const hipError_t e = go(std::true_type{}, inc, n + 1, n);
        if (e != hipSuccess) return e;
    }
    return go(std::false_type{}, segs, G, G);
}

}  // namespace based
