// Causal Taylor linear attention, chunked prefill on the gfx950 matrix cores (bf16 in, fp32
// accumulate), d' = 32: the kernel of short calls, for which a block of 256 tokens is too coarse (which ones: prefill_mfma32_short_takes).
//
// Same method as the d' = 16 kernel (chunked form of Sec. 4: masked quadratic product inside a
// chunk, running KV-state across chunks, features of Eq. 4 built in registers in MFMA operand layout, k-slots mapped onto
// the rows a lane holds in its accumulators), laid out for the larger state:
//
// Symmetric packing.  One state row per unordered pair {a, b}: row (a, delta) stands for the
// pair {a, (a + delta) mod 32}, delta = 0 .. 15 for every a (16 tiles of exactly 32 rows, one
// delta per tile) and delta = 16 for a < 16.  The k side builds x_a x_b / sqrt(2), the q side
// sqrt(2) x_a x_b (delta != 0) or x_a^2 / sqrt(2) (delta = 0).  528 pair rows instead of 1024.  Two more tiles: E1 = the
// 32 linear rows, E2 = [1, 0 x 15, the 16 rows of delta = 16].
//
// Work split.  A workgroup of eight waves takes 64 columns of one (unit, segment); wave w owns the tiles delta = 2 w and
// 2 w + 1 for both column tiles of 32.  So every feature operand is built once per workgroup and used where it is built: nothing
// of it passes through LDS, only the rows it is made of do.  The eight partial outputs of a chunk meet in LDS and each
// wave finishes four tokens.  Waves 0 .. 3 also have E1 / E2 (one column tile of one of them each) and a 16 x 16 block
// of the K-state, waves 4 .. 7 the intra-chunk block (one half of the keys, one column tile each).
//
// Pipeline.  Chunks of 32 tokens, global -> registers (two chunks ahead) -> LDS (two generations).  Two barriers a chunk: rows
// and partial outputs are there | the previous chunk's partial outputs have been read.
//
// Denominator.  The K-state is kept as moments: M[a][b] = sum_t k_a k_b (an MFMA of the K rows with
// themselves), z1[a] = sum_t k_a (vector adds) and the token count.  Per query
// phi(q).z = z0 + sum_a q_a (z1[a] + (M q)[a] / 2); the part from inside the chunk is the column
// sum of the masked block P.
//
// Long sequences / few units: G segments; a first launch computes each segment's state increment, segment 0's starting from
// the caller's state, and the main launch starts segment g from the sum of the entries before it (read at full width: all
// loads of an entry in flight together).
//
// What bounds it: per chunk and SIMD 44 matrix instructions (1400 cycles) and 600 vector instructions (half of them the products,
// conversions and the state's rounding to bf16), which share the register ports, and 290 KB through LDS, a third of it the
// partial outputs; 5000 cycles in all, because the eight waves do the same things at the same time.  (Operands built by one wave and shared through
// LDS: the same time, more LDS.  Four waves with 512 registers and half the exchange: the same, a lone wave issues a
// vector instruction every 4 cycles instead of 2.  Reading operands' rows a phase ahead: no gain.)
// Measured (d_v 64, us, against blocks of 256 tokens): 16 units from a state, of 64 tokens 17.8, 19.2, of 96 20.1, 20.2.
#include "common.h"

#include <cmath>
#include <type_traits>

namespace based {

namespace dp32s {

typedef float f32x2 __attribute__((ext_vector_type(2)));
typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
typedef float f32x16 __attribute__((ext_vector_type(16)));
typedef float f32x8 __attribute__((ext_vector_type(8)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef __bf16 bf16x4 __attribute__((ext_vector_type(4)));
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));
typedef short s16x4 __attribute__((ext_vector_type(4)));
typedef short s16x8 __attribute__((ext_vector_type(8)));

constexpr int DP = 32;            // d'
constexpr int C = 32;             // chunk length (tokens)
constexpr int NW = 8;             // waves per workgroup
constexpr int NT = NW * 64;
constexpr int PF = 2;             // chunks whose rows are on their way; generations of the rows in LDS
constexpr int COLS = 64;          // d_v columns per workgroup
constexpr int TPW = 2;            // main tiles per wave (and column tile)
constexpr int TILES = 18;         // 16 main tiles, E1, E2
constexpr float kCK = 0.84089641525371454303f;   // 2^(-1/4): (c k_a)(c k_b) = k_a k_b / sqrt(2)
constexpr float kCQ = 1.18920711500272106672f;   // 2^(+1/4): (c q_a)(c q_b) = sqrt(2) q_a q_b

// LDS strides (elements).  (64 banks: the 16-byte reads of 16 consecutive rows fall into different ones.)
constexpr int KTS_LD = C + 4;     // fp32 K^T rows
constexpr int VR_LD = COLS + 16;  // bf16 V rows
constexpr int QS_LD = DP + 4;     // fp32 Q rows
constexpr int KR_LD = 64 + 8;     // bf16 extended K and Q rows (144-byte stride)
constexpr int IMG_LD = 40;        // fp32 rows of the state image (the halves of a wave access different banks)

// Workspace entry (one segment's state in accumulator layout): 40 slots of 16 registers x 64 lanes: column tile c:
// slots 20 c + 2 w + tt = main tile 2 w + tt, 20 c + 16 = E1, 20 c + 17 = E2; 18 = M; 19 = [z1, z0] in the first two
// registers.  Within a slot: [reg / 4][lane][reg % 4].
constexpr int WS_SLOTS = 40;
constexpr size_t kWsEntryFloats = (size_t)WS_SLOTS * 16 * 64;

struct Rows {   // a chunk's rows
    float kts[DP][KTS_LD];     // c_k * K^T
    uint16_t krow[C][KR_LD];   // extended K rows: [k_0..k_31 as given, 1, 0 x 15, k_a k_(a+16) / sqrt(2) for a < 16]
    uint16_t vrow[C][VR_LD];   // V rows of the slice, bf16 as given
    float qs[C][QS_LD];        // c_q * Q
    uint16_t qrow[C][KR_LD];   // extended Q rows: [q as given, 1, 0 x 15, sqrt(2) q_a q_(a+16)]
};
struct Lds {
    Rows rows[PF];                     // generation: chunk mod 2
    float xbuf[NW][2 * 4][64][4];      // partial Y^T: [sender][4 column tile + reg / 4][place of the lane][reg % 4]
    float den[2][C][8];                // denominators: the waves' parts from before the chunk (4) and from inside it (2)
    float z1s[4][16];                  // a wave's z1, for its own broadcast reads
};
static_assert(sizeof(Lds) <= 160 * 1024, "one workgroup per CU");
static_assert(sizeof(Lds) >= sizeof(float) * 32 * TILES * IMG_LD, "the state image of one column tile fits the LDS");

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

__device__ __forceinline__ bf16x8 pack8_acc(const f32x16 &acc, int s)   // registers 8s .. 8s+7
{
    f32x8 f;
#pragma unroll
    for (int e = 0; e < 8; ++e) f[e] = acc[8 * s + e];
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

// Canonical state rows (Eq. 4 order) of a packed row; a pair row has two (equal for delta = 0).
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
__device__ __forceinline__ CanonRows canon_rows_main(int delta, int fl, bool packed_state)
{
    return canon_pair(fl, (fl + delta) & (DP - 1), packed_state);
}
__device__ __forceinline__ CanonRows canon_rows_e1(int fl) { return {1 + fl, 1 + fl}; }
__device__ __forceinline__ CanonRows canon_rows_e2(int fl, bool packed_state)
{
    if (fl == 0) return {0, 0};
    if (fl >= 16) return canon_pair(fl - 16, fl, packed_state);
    return {-1, -1};
}

// row fl of tile T (T < 16: delta = T; 16: E1; 17: E2)
__device__ __forceinline__ CanonRows canon_rows(int T, int fl, bool packed_state)
{
    return T < 16 ? canon_rows_main(T, fl, packed_state) : T == 16 ? canon_rows_e1(fl) : canon_rows_e2(fl, packed_state);
}

constexpr int kMaxSegments = 16;
struct SegTable { int begin[kMaxSegments + 1]; };

// INC: state increment of the segment only, to workspace entry 1 + seg; segment 0 starts from the caller's state, if any,
// and also leaves that, converted, in entry 0 (import_only: nothing else).  Otherwise the full prefill of the segment.
// init_in_entry: the caller's state is in entry 0 (one workgroup per unit reads it from the buffer itself).
// Slice: columns [64 slice, 64 slice + 64) of v / y.
template <bool INC>
__global__ __launch_bounds__(NT, 2) void prefill_kernel(
    const uint16_t *__restrict__ q, const uint16_t *__restrict__ k, const uint16_t *__restrict__ v,
    uint16_t *__restrict__ y, float *state, int has_init, int import_only, int init_in_entry, float *__restrict__ ws,
    int N, int dv, SegTable segs, int G, int groups)
{
    __shared__ __align__(16) Lds lds;

    // has_init carries three flags: bit 0 an initial state is given, bit 1 the state buffer is packed,
    // bit 2 the outputs are the numerators alone (no division by the denominator)
    const bool packed_state = (has_init & 2) != 0;
    const bool numerator_only = (has_init & 4) != 0;
    has_init &= 1;
    int tid = threadIdx.x;
    const int w = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int r = w & 3;   // waves 0 .. 3: E1 / E2 and the K-state; 4 .. 7: the intra-chunk block
    const bool low = w < 4;
    int lane = tid & 63;
    int g = lane >> 5, n = lane & 31, lq = lane >> 4, ln = lane & 15;

    const int slices = dv / COLS;
    const int gseg = !INC ? G : import_only ? 1 : G - 1;
    int bid = blockIdx.x;
    // The segments of a group on one XCD (workgroup index mod 8), whose L2 then holds its entries; what lies beyond the last group leaves at once.
    const int seg = (bid >> 3) % gseg;
    bid = ((bid >> 3) / gseg << 3) + (bid & 7);
    if (bid >= groups) return;
    const int slice = bid % slices;
    const int u = bid / slices;
    const int col0 = slice * COLS;

    const int tok_begin = segs.begin[seg];
    const int tok_end = min(N, segs.begin[seg + 1]);
    const int n_chunks = (tok_end - tok_begin + C - 1) / C;

    const uint16_t *qu = q + (size_t)u * N * DP;
    const uint16_t *ku = k + (size_t)u * N * DP;
    const uint16_t *vu = v + (size_t)u * N * dv + col0;
    uint16_t *yu = y + (size_t)u * N * dv + col0;
    float *Su = state ? state + (size_t)u * (packed_state ? packed_state_stride(DP, dv) : state_stride(DP, dv)) + col0
                      : nullptr;
    float *zu = Su ? Su - col0 + (size_t)(packed_state ? packed_feature_dim(DP) : feature_dim(DP)) * dv : nullptr;
    float *ws_unit = ws + ((size_t)(u * slices + slice) * G) * kWsEntryFloats;

    // ---- accumulators -------------------------------------------------------------------------
    f32x16 S[2][TPW];      // main tiles delta = 2 w + tt, column tile c ^ (r % 2)
    f32x16 X;              // waves 0 .. 3: column tile r % 2 of E1 (r < 2) or E2
    f32x4 M;               // M[16 (r / 2) + 4 (lane / 16) + i][16 (r % 2) + lane % 16]
    float z1 = 0.f, z0 = 0.f;   // z1[16 (r / 2) + lane % 16], tokens before this call's first
    const int xc = r & 1, xe = r >> 1;
    zero16(X);
    M = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int c = 0; c < 2; ++c) {
#pragma unroll
        for (int tt = 0; tt < TPW; ++tt) zero16(S[c][tt]);
    }

    auto add_entry = [&](int p) {
        const float *e = ws_unit + (size_t)p * kWsEntryFloats + 4 * lane;
        f32x4 t[2][TPW][4], tx[4], tm;
        auto fetch = [&](int slot, f32x4 *x) {
#pragma unroll
            for (int j = 0; j < 4; ++j) x[j] = *reinterpret_cast<const f32x4 *>(e + (slot * 4 + j) * 256);
        };
        auto add = [&](const f32x4 *x, f32x16 &a) {
#pragma unroll
            for (int j = 0; j < 4; ++j)
#pragma unroll
                for (int k = 0; k < 4; ++k) a[4 * j + k] += x[j][k];
        };
#pragma unroll
        for (int c = 0; c < 2; ++c)
#pragma unroll
            for (int tt = 0; tt < TPW; ++tt) fetch(20 * (c ^ xc) + 2 * w + tt, t[c][tt]);
        const f32x4 tz = *reinterpret_cast<const f32x4 *>(e + (19 * 4 + r) * 256);
        fetch(20 * xc + 16 + xe, tx);   // (waves 4 .. 7 do not use theirs)
        tm = *reinterpret_cast<const f32x4 *>(e + (18 * 4 + r) * 256);
#pragma unroll
        for (int c = 0; c < 2; ++c)
#pragma unroll
            for (int tt = 0; tt < TPW; ++tt) add(t[c][tt], S[c][tt]);
        add(tx, X);
        M += tm;
        z1 += tz[0];
        z0 += tz[1];
    };
    auto put_entry = [&](int p) {
        float *e = ws_unit + (size_t)p * kWsEntryFloats;
        auto put = [&](int slot, const f32x16 &a) {
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                f32x4 o;
#pragma unroll
                for (int i = 0; i < 4; ++i) o[i] = a[4 * j + i];
                *reinterpret_cast<f32x4 *>(e + (slot * 4 + j) * 256 + 4 * lane) = o;
            }
        };
#pragma unroll
        for (int c = 0; c < 2; ++c) {
#pragma unroll
            for (int tt = 0; tt < TPW; ++tt) put(20 * (c ^ xc) + 2 * w + tt, S[c][tt]);
        }
        if (!low) return;
        put(20 * xc + 16 + xe, X);
        *reinterpret_cast<f32x4 *>(e + (18 * 4 + r) * 256 + 4 * lane) = M;
        *reinterpret_cast<f32x4 *>(e + (19 * 4 + r) * 256 + 4 * lane) = f32x4{z1, z0, 0.f, 0.f};
    };

    // The state buffer moves through LDS, one column tile at a time, as an image of its tiles: image[32 T + row][IMG_LD].
    // A wave reaches its registers' places at constant offsets, and the whole workgroup moves 16-byte pieces between the
    // image and the buffer's rows.
    float *image = reinterpret_cast<float *>(&lds);
    constexpr int IMG_Q = 32 * TILES * 8, IMG_STEPS = IMG_Q / NT;   // 16-byte pieces of a column tile: all, per thread
    static_assert(IMG_Q % NT == 0, "");
    auto import_state = [&]() {
#pragma unroll
        for (int cc = 0; cc < 2; ++cc) {
            constexpr int BATCH = 3;
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
                    const bool zero = canon_rows(row >> 5, row & 31, packed_state).r1 < 0;   // (padding)
                    *reinterpret_cast<f32x4 *>(image + row * IMG_LD + 4 * (i & 7)) =
                        zero ? f32x4{0.f, 0.f, 0.f, 0.f} : 0.5f * t[j][0] + 0.5f * t[j][1];   // (the sum may overflow)
                }
            }
            __syncthreads();
#pragma unroll
            for (int rr = 0; rr < 16; ++rr) {
                const int fl = 8 * (rr >> 2) + (rr & 3);
#pragma unroll
                for (int tt = 0; tt < TPW; ++tt) {
                    const float t = image[4 * g * IMG_LD + n + (32 * (2 * w + tt) + fl) * IMG_LD];
                    S[0][tt][rr] = cc == xc ? t : S[0][tt][rr];
                    S[1][tt][rr] = cc == xc ? S[1][tt][rr] : t;
                }
                if (low && cc == xc) X[rr] = image[4 * g * IMG_LD + n + (32 * (16 + xe) + fl) * IMG_LD];
            }
            __syncthreads();
        }
        // M[a][b] = sqrt(2) x the symmetric part of z's pair rows
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const CanonRows cr = canon_pair(16 * xe + 4 * lq + i, 16 * xc + ln, packed_state);
            M[i] = 2.f * kRsqrt2 * (0.5f * zu[cr.r1] + 0.5f * zu[cr.r2]);
        }
        z1 = zu[1 + 16 * xe + ln];
        z0 = zu[0];
    };
    auto export_state = [&]() {   // (both rows of a pair; slice 0 writes z)
#pragma unroll
        for (int cc = 0; cc < 2; ++cc) {
            __syncthreads();
#pragma unroll
            for (int rr = 0; rr < 16; ++rr) {
                const int fl = 8 * (rr >> 2) + (rr & 3);
#pragma unroll
                for (int tt = 0; tt < TPW; ++tt) {
                    const float t0 = S[0][tt][rr], t1 = S[1][tt][rr];
                    image[4 * g * IMG_LD + n + (32 * (2 * w + tt) + fl) * IMG_LD] = cc == xc ? t0 : t1;
                }
                if (low && cc == xc) image[4 * g * IMG_LD + n + (32 * (16 + xe) + fl) * IMG_LD] = X[rr];
            }
            __syncthreads();
#pragma unroll 3
            for (int st = 0; st < IMG_STEPS; ++st) {
                const int i = st * NT + tid, row = i >> 3;
                const CanonRows cr = canon_rows(row >> 5, row & 31, packed_state);
                if (cr.r1 >= 0) {
                    const f32x4 t = *reinterpret_cast<const f32x4 *>(image + row * IMG_LD + 4 * (i & 7));
                    float *p = Su + 32 * cc + 4 * (i & 7);
                    *reinterpret_cast<f32x4 *>(p + (size_t)cr.r1 * dv) = t;
                    if (cr.r2 != cr.r1) *reinterpret_cast<f32x4 *>(p + (size_t)cr.r2 * dv) = t;
                }
            }
        }
        if (slice == 0 && low) {
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                const int a = 16 * xe + 4 * lq + i, b = 16 * xc + ln;
                if (!packed_state || a <= b) zu[canon_pair(a, b, packed_state).r1] = kRsqrt2 * M[i];
            }
            if (xc == 0 && lq == 0) {
                zu[1 + 16 * xe + ln] = z1;
                if (r == 0 && ln == 0) zu[0] = z0 + (float)N;
            }
        }
    };

    if (INC) {
        if (has_init && seg == 0) {
            import_state();
            put_entry(0);
            if (import_only) return;   // uniform
        }
    } else if (seg > 0) {
#pragma unroll 1
        for (int p = 1; p <= seg; ++p) add_entry(p);
    } else if (has_init) {
        if (init_in_entry) add_entry(0);
        else import_state();
    }

    // What is computed from the lane's place before the loop is not kept through it, and the other way round.
    auto fresh_lane = [&]() {
        asm volatile("" : "+v"(tid));
        lane = tid & 63;
        g = lane >> 5; n = lane & 31; lq = lane >> 4; ln = lane & 15;
    };
    fresh_lane();

    // ---- staging: global -> registers -> LDS ----------------------------------------------------
    // A thread moves elements 2 j, 2 j + 1 of the K and Q rows of a token and 4 columns of its V row (j = tid % 16).  Loads are
    // unconditional (rows past the end re-read the last one, and are zeroed when staged), so that the number in flight is known.
    const int s_tok = tid >> 4, s_j = tid & 15;
    struct Raw { uint32_t k, q; u32x2 v; } raw[PF];   // chunk mod PF
    auto load_raw = [&](int tok0, Raw &x) {
        const int tok = min(tok0 + s_tok, tok_end - 1);
        x.k = *reinterpret_cast<const uint32_t *>(ku + (size_t)tok * DP + 2 * s_j);
        if (!INC) x.q = *reinterpret_cast<const uint32_t *>(qu + (size_t)tok * DP + 2 * s_j);
        x.v = *reinterpret_cast<const u32x2 *>(vu + (size_t)tok * dv + 4 * s_j);
    };
    auto stage = [&](int tok0, const Raw &x, Rows &rows) {
        const bool past = tok0 + s_tok >= tok_end;
        const uint32_t kraw = past ? 0u : x.k;
        const u32x2 vraw = {past ? 0u : x.v[0], past ? 0u : x.v[1]};
        // product of the elements a and a + 16, which is eight lanes to the right (row_shl:8)
        auto pair = [&](float a) {
            return a * __uint_as_float(__builtin_amdgcn_update_dpp(0u, __float_as_uint(a), 0x108, 0xf, 0xf, false));
        };
        const float k0 = bf16lo(kraw) * kCK, k1 = bf16hi(kraw) * kCK;
        rows.kts[2 * s_j][s_tok] = k0;
        rows.kts[2 * s_j + 1][s_tok] = k1;
        *reinterpret_cast<uint32_t *>(&rows.krow[s_tok][2 * s_j]) = kraw;
        const uint32_t kp = pack2(pair(k0), pair(k1));
        uint32_t qp = 0;
        if (!INC) {
            const float q0 = bf16lo(x.q) * kCQ, q1 = bf16hi(x.q) * kCQ;
            *reinterpret_cast<f32x2 *>(&rows.qs[s_tok][2 * s_j]) = f32x2{q0, q1};
            *reinterpret_cast<uint32_t *>(&rows.qrow[s_tok][2 * s_j]) = x.q;
            qp = pack2(pair(q0), pair(q1));
        }
        *reinterpret_cast<u32x2 *>(&rows.vrow[s_tok][4 * s_j]) = vraw;
        if (s_j < 8) {
            *reinterpret_cast<uint32_t *>(&rows.krow[s_tok][48 + 2 * s_j]) = kp;
            if (!INC) *reinterpret_cast<uint32_t *>(&rows.qrow[s_tok][48 + 2 * s_j]) = qp;
        }
    };

    // ---- operands ---------------------------------------------------------------------------------
    // phi(Q)^T operand of slab sl of tile tt: k-slot (jj, i) is row a = 16 sl + 8 jj + 4 g + i, the pair (a, (a + delta) mod 32)
    struct QSrc { float a[8], b[2][6]; };
    auto q_source = [&](const Rows &rows, int sl) {
        const float *row = rows.qs[n];
        QSrc o;
#pragma unroll
        for (int jj = 0; jj < 2; ++jj) {
            const int base = 16 * sl + 8 * jj + 4 * g;
            const f32x4 t = *reinterpret_cast<const f32x4 *>(row + base);
#pragma unroll
            for (int i = 0; i < 4; ++i) o.a[4 * jj + i] = t[i];
#pragma unroll
            for (int h = 0; h < 3; ++h) {
                const f32x2 b = *reinterpret_cast<const f32x2 *>(row + ((base + 2 * w + 2 * h) & 31));
                o.b[jj][2 * h] = b[0];
                o.b[jj][2 * h + 1] = b[1];
            }
        }
        return o;
    };
    // (every wave multiplies: the first one, alone, would be the last to finish)
    const float dw = w == 0 ? 0.5f : 1.f;   // delta = 0: x_a^2 / sqrt(2)
    auto q_op = [&](const QSrc &s, int tt) {
        float pr[8];
#pragma unroll
        for (int jj = 0; jj < 2; ++jj)
#pragma unroll
            for (int i = 0; i < 4; ++i)
                pr[4 * jj + i] = (tt == 0 ? s.a[4 * jj + i] * dw : s.a[4 * jj + i]) * s.b[jj][i + tt];
        return pack8(pr);
    };
    // phi(K)^T operand of token slab ts of tile tt: row n, k-slots the tokens 16 ts + 4 g + {0..3, 8..11}
    struct KSrc { f32x4 a[2], b[TPW][2]; };
    auto k_source = [&](const Rows &rows, int ts) {
        const int tcol = 16 * ts + 4 * g;
        KSrc o;
#pragma unroll
        for (int h = 0; h < 2; ++h) o.a[h] = *reinterpret_cast<const f32x4 *>(&rows.kts[n][tcol + 8 * h]);
#pragma unroll
        for (int tt = 0; tt < TPW; ++tt)
#pragma unroll
            for (int h = 0; h < 2; ++h)
                o.b[tt][h] = *reinterpret_cast<const f32x4 *>(&rows.kts[(n + 2 * w + tt) & 31][tcol + 8 * h]);
        return o;
    };
    auto k_op = [&](const KSrc &s, int tt) {
        float pr[8];
#pragma unroll
        for (int i = 0; i < 4; ++i) { pr[i] = s.a[0][i] * s.b[tt][0][i]; pr[4 + i] = s.a[1][i] * s.b[tt][1][i]; }
        return pack8(pr);
    };
    // V^T operand (lane (g, n): column n of the tile at the 8 tokens of its k-slots, two runs of 4 tokens
    // starting at tok4 and tok4 + 8) from row-major rows, by the transposing LDS read: in each group
    // of 16 lanes, lane k supplies the address of 4 consecutive columns (4 (k % 4) ..) of row k / 4 of
    // the group's 16-column block and receives column k of that block at the 4 rows.
    const int tr_row = ((lane & 15) >> 2) + 4 * g, tr_col = 16 * ((lane >> 4) & 1) + 4 * (lane & 3);
    auto tr_read = [&](const uint16_t *p, int stride) {
        const s16x4 a = __builtin_amdgcn_ds_read_tr16_b64_v4i16((__attribute__((address_space(3))) s16x4 *)p);
        const s16x4 b = __builtin_amdgcn_ds_read_tr16_b64_v4i16((__attribute__((address_space(3))) s16x4 *)(p + 8 * stride));
        s16x8 o;
#pragma unroll
        for (int i = 0; i < 4; ++i) { o[i] = a[i]; o[4 + i] = b[i]; }
        return __builtin_bit_cast(bf16x8, o);
    };
    auto read_v = [&](const Rows &rows, int ts, int c) { return tr_read(&rows.vrow[16 * ts + tr_row][32 * c + tr_col], VR_LD); };
    auto read_k = [&](const Rows &rows, int ts, int col) { return tr_read(&rows.krow[16 * ts + tr_row][col + tr_col], KR_LD); };
    // 16 columns of K at all 32 tokens (operand of the 16 x 16 x 32 product)
    auto read_k16 = [&](const Rows &rows, int col) {
        const uint16_t *p = &rows.krow[(ln >> 2) + 4 * lq][col + 4 * (lane & 3)];
        const s16x4 a = __builtin_amdgcn_ds_read_tr16_b64_v4i16((__attribute__((address_space(3))) s16x4 *)p);
        const s16x4 b = __builtin_amdgcn_ds_read_tr16_b64_v4i16((__attribute__((address_space(3))) s16x4 *)(p + 16 * KR_LD));
        s16x8 o;
#pragma unroll
        for (int i = 0; i < 4; ++i) { o[i] = a[i]; o[4 + i] = b[i]; }
        return __builtin_bit_cast(bf16x8, o);
    };
    // sums over the wave's halves / over the two rows of 16 lanes of each half
    auto add_halves = [&](float a, float b) {   // lanes < 32: a, lanes >= 32: b
        const auto t = __builtin_amdgcn_permlane32_swap(__float_as_uint(a), __float_as_uint(b), false, false);
        return __uint_as_float(t[0]) + __uint_as_float(t[1]);
    };
    auto add_rows = [&](float a) {
        const auto t = __builtin_amdgcn_permlane16_swap(__float_as_uint(a), __float_as_uint(a), false, false);
        return __uint_as_float(t[0]) + __uint_as_float(t[1]);
    };

    struct VSrc { bf16x8 v[2]; };
    auto v_source = [&](const Rows &rows, int ts) {
        VSrc o;
        o.v[0] = read_v(rows, ts, xc);
        o.v[1] = read_v(rows, ts, xc ^ 1);
        return o;
    };
    // S += phi(K)^T V over this wave's tiles
    auto update_slab = [&](const KSrc &src, const VSrc &vs) {
#pragma unroll
        for (int tt = 0; tt < TPW; ++tt) {
            const bf16x8 op = k_op(src, tt);
#pragma unroll
            for (int c = 0; c < 2; ++c) S[c][tt] = mfma(op, vs.v[c], S[c][tt]);
        }
    };
    // waves 0 .. 3: E1 / E2, M += K^T K, z1 += sum of the rows
    auto update_e = [&](const Rows &rows, const VSrc &v0, const VSrc &v1) {
        const bf16x8 e0 = read_k(rows, 0, 32 * xe), e1 = read_k(rows, 1, 32 * xe);
        const bf16x8 ea = read_k16(rows, 16 * xe), eb = read_k16(rows, 16 * xc);
        X = mfma(e0, v0.v[0], X);
        X = mfma(e1, v1.v[0], X);
        M = __builtin_amdgcn_mfma_f32_16x16x32_bf16(ea, eb, M, 0, 0, 0);
        const u32x4 kw = __builtin_bit_cast(u32x4, ea);
        float z1c = 0.f;
#pragma unroll
        for (int i = 0; i < 4; ++i) z1c += bf16lo(kw[i]) + bf16hi(kw[i]);
        z1c = add_halves(z1c, z1c);
        z1 += add_rows(z1c);
        if (!INC) lds.z1s[r][ln] = xe == xc ? z1 : 0.f;
    };

    // columns 32 .. 47 of the K and Q rows: the constant feature (past the end its V row is zero), then zeros
    if (s_j < 8)
#pragma unroll
        for (int gen = 0; gen < 2; ++gen) {
            const uint32_t t = s_j == 0 ? 0x3F80u : 0u;
            *reinterpret_cast<uint32_t *>(&lds.rows[gen].krow[s_tok][32 + 2 * s_j]) = t;
            if (!INC) *reinterpret_cast<uint32_t *>(&lds.rows[gen].qrow[s_tok][32 + 2 * s_j]) = t;
        }
#pragma unroll
    for (int i = 0; i < PF; ++i) load_raw(tok_begin + C * i, raw[i]);
    stage(tok_begin, raw[0], lds.rows[0]);
    load_raw(tok_begin + C * PF, raw[0]);
    // chunk t: f(t mod PF, first token).  (Pairs, and an odd chunk after the loop: with a way out between the two the compiler sees a path on
    // which the first one's loads are the newest, and has the first chunk of every pair wait for all of them.)
    auto for_chunks = [&](auto &&f) {
        int t = 0;
        for (; t + 1 < n_chunks; t += PF) {
            const int tok0 = tok_begin + C * t;
            f(std::integral_constant<int, 0>{}, tok0);
            f(std::integral_constant<int, 1>{}, tok0 + C);
        }
        if (t < n_chunks) f(std::integral_constant<int, 0>{}, tok_begin + C * t);
    };

    if (INC) {
        wg_sync();
        for_chunks([&](auto gen, int tok0) {
            constexpr int p = decltype(gen)::value, p1 = (p + 1) % PF;
            const Rows &rows = lds.rows[p];
            const KSrc k0 = k_source(rows, 0);
            const VSrc v0 = v_source(rows, 0);
            __builtin_amdgcn_sched_barrier(1);   // (only arithmetic crosses)
            const KSrc k1 = k_source(rows, 1);
            const VSrc v1 = v_source(rows, 1);
            __builtin_amdgcn_sched_barrier(1);   // (only arithmetic crosses)
            update_slab(k0, v0);
            stage(tok0 + C, raw[p1], lds.rows[p1]);
            load_raw(tok0 + (PF + 1) * C, raw[p1]);
            update_slab(k1, v1);
            if (low) {
                role_guard();
                update_e(rows, v0, v1);
            }
            wg_sync();
        });
        put_entry(1 + seg);
        return;
    }

    // ---- full pass ----------------------------------------------------------------------------------
    // A chunk's outputs: lane (tk, cq) finishes columns 4 cq .. of token 4 w + tk; the partial sums are read across (the sender's
    // lane l puts its four of column group cj at place l ^ (cj + 8 (l / 32)): 16 consecutive lanes in different banks).
    const int o_tok = 4 * w + (lane >> 4), o_cq = lane & 15;
    const int o_place = (32 * (o_cq & 1) + o_tok) ^ ((o_cq >> 1) + 8 * (o_cq & 1));
    struct Out { f32x4 d4, d2, part[NW]; };
    auto out_source = [&](int g2) {
        Out o;
        o.d4 = *reinterpret_cast<const f32x4 *>(&lds.den[g2][o_tok][0]);
        o.d2 = *reinterpret_cast<const f32x4 *>(&lds.den[g2][o_tok][4]);
#pragma unroll
        for (int sl = 0; sl < NW; ++sl) o.part[sl] = *reinterpret_cast<const f32x4 *>(&lds.xbuf[sl][o_cq >> 1][o_place][0]);
        return o;
    };
    auto output = [&](const Out &x, int tok0) {
        const float den = z0 + (float)tok0 + ((x.d4[0] + x.d4[1]) + (x.d4[2] + x.d4[3])) + (x.d2[0] + x.d2[1]);
        const float inv = numerator_only ? 1.f : 1.f / den;
        const f32x4 sum = ((x.part[0] + x.part[1]) + (x.part[2] + x.part[3])) + ((x.part[4] + x.part[5]) + (x.part[6] + x.part[7]));
        if (tok0 >= tok_begin && tok0 + o_tok < tok_end)
            *reinterpret_cast<u32x2 *>(yu + (ptrdiff_t)(tok0 + o_tok) * dv + 4 * o_cq) =
                __builtin_bit_cast(u32x2, __builtin_convertvector(sum * inv, bf16x4));
    };
    if (low) lds.z1s[r][ln] = xe == xc ? z1 : 0.f;
    wg_sync();
    for_chunks([&](auto gen, int tok0) {
        constexpr int p = decltype(gen)::value, p1 = (p + 1) % PF;
        const Rows &rows = lds.rows[p];
        // the previous chunk's partial outputs, the queries
        const Out prev = out_source(p1);
        __builtin_amdgcn_sched_barrier(1);   // (only arithmetic crosses)
        output(prev, tok0 - C);
        __builtin_amdgcn_sched_barrier(0);
        const QSrc q0 = q_source(rows, 0);
        const QSrc q1 = q_source(rows, 1);
        __builtin_amdgcn_sched_barrier(1);   // (only arithmetic crosses)
        f32x16 Y[2];
        zero16(Y[0]);
        zero16(Y[1]);
        auto readout = [&](const QSrc &src, int sl) {
#pragma unroll
            for (int tt = 0; tt < TPW; ++tt) {
                const bf16x8 op = q_op(src, tt);
#pragma unroll
                for (int c = 0; c < 2; ++c) Y[c] = mfma(pack8_acc(S[c][tt], sl), op, Y[c]);
            }
        };
        readout(q0, 0);
        readout(q1, 1);
        if (low) {
            role_guard();
            // E1 / E2 for column tile xc
            u32x2 qx[2][2], qa[2];
            f32x4 qb[2];
#pragma unroll
            for (int sl = 0; sl < 2; ++sl)
#pragma unroll
                for (int h = 0; h < 2; ++h)
                    qx[sl][h] = *reinterpret_cast<const u32x2 *>(&rows.qrow[n][32 * xe + 4 * g + 16 * sl + 8 * h]);
#pragma unroll
            for (int h = 0; h < 2; ++h) {
                qa[h] = *reinterpret_cast<const u32x2 *>(&rows.qrow[16 * h + ln][16 * xe + 4 * lq]);
                qb[h] = *reinterpret_cast<const f32x4 *>(&rows.qs[16 * h + ln][16 * xc + 4 * lq]);
            }
            const f32x4 zv = *reinterpret_cast<const f32x4 *>(&lds.z1s[r][4 * lq]);
#pragma unroll
            for (int sl = 0; sl < 2; ++sl)
                Y[0] = mfma(pack8_acc(X, sl), as_bf16x8(u32x4{qx[sl][0][0], qx[sl][0][1], qx[sl][1][0], qx[sl][1][1]}), Y[0]);
            // denominator from before the chunk: T[b][query] = sum_a M[a][b] q_a over this wave's a and b, then
            // sum_b q_b (z1[b] + T[b] / 2)
            const s16x4 m4 = __builtin_bit_cast(s16x4, __builtin_convertvector(M, bf16x4));
            float d[2];
#pragma unroll
            for (int h = 0; h < 2; ++h) {
                const f32x4 T = __builtin_amdgcn_mfma_f32_16x16x16bf16_1k(m4, __builtin_bit_cast(s16x4, qa[h]), f32x4{0.f, 0.f, 0.f, 0.f},
                                                                         0, 0, 0);
                d[h] = 0.f;
#pragma unroll
                for (int i = 0; i < 4; ++i) d[h] = fmaf(qb[h][i], fmaf(0.5f, T[i], zv[i]), d[h]);
            }
            lds.den[p][16 * g + ln][r] = add_rows(add_halves(d[0], d[1])) * (1.f / kCQ);
        } else {
            role_guard();
            // intra-chunk block, keys 16 xe .. + 15 and column tile xc: P^T = mask(1 + A^T + A^T^2 / 2), Y^T += V^T P^T
            f32x16 P;
            zero16(P);
#pragma unroll
            for (int ks = 0; ks < 2; ++ks) {   // contraction over d' = 32 in two steps; rows 0 .. 15 of P are used
                const u32x4 kop = *reinterpret_cast<const u32x4 *>(&rows.krow[(n + 16 * xe) & 31][16 * ks + 8 * g]);
                const u32x4 qop = *reinterpret_cast<const u32x4 *>(&rows.qrow[n][16 * ks + 8 * g]);
                P = mfma(as_bf16x8(kop), as_bf16x8(qop), P);
            }
            const bf16x8 vp = read_v(rows, xe, xc);
            float cs = 0.f;
#pragma unroll
            for (int rr = 0; rr < 8; ++rr) {
                const float x = P[rr];
                const float pv = fmaf(x, fmaf(x, 0.5f, 1.f), 1.f);
                P[rr] = 8 * (rr >> 2) + (rr & 3) <= n - 16 * xe - 4 * g ? pv : 0.f;
                cs += P[rr];
            }
            lds.den[p][n][4 + xe] = add_halves(cs, cs);
            Y[0] = mfma(vp, pack8_acc(P, 0), Y[0]);
        }
        wg_sync();   // every wave has the previous chunk's partial outputs
#pragma unroll
        for (int c = 0; c < 2; ++c)
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                f32x4 o;
#pragma unroll
                for (int i = 0; i < 4; ++i) o[i] = Y[c][4 * j + i];
                const int cj = 4 * (c ^ xc) + j;
                *reinterpret_cast<f32x4 *>(&lds.xbuf[w][cj][lane ^ (cj + 8 * g)][0]) = o;
            }
        const KSrc k0 = k_source(rows, 0);
        const VSrc v0 = v_source(rows, 0);
        const KSrc k1 = k_source(rows, 1);
        const VSrc v1 = v_source(rows, 1);
        __builtin_amdgcn_sched_barrier(1);   // (only arithmetic crosses)
        update_slab(k0, v0);
        stage(tok0 + C, raw[p1], lds.rows[p1]);
        load_raw(tok0 + (PF + 1) * C, raw[p1]);
        update_slab(k1, v1);
        if (low) {
            role_guard();
            update_e(rows, v0, v1);
        }
        wg_sync();
    });
    {
        const int last = n_chunks - 1;
        output(last & 1 ? out_source(1) : out_source(0), tok_begin + C * last);
    }
    if (Su && seg == G - 1) {
        fresh_lane();
        export_state();
    }
}

// Segments: the chain of an increment, entries to sum and the main pass is shortest near sqrt(1.5 chunks) of them; no more than the XCD with the most
// groups has CUs for.
static int pick_segments(int groups, int N)
{
    const int chunks = (N + C - 1) / C;
    if (chunks < 8) return 1;
    const int G = (int)(sqrtf(1.5f * chunks) + 0.5f), room = 32 / ((groups + 7) / 8);
    return G < room ? G : room < 1 ? 1 : room;
}

// Segment g's main pass starts by summing g entries, which takes about as long as 0.75 chunks each, and the last one writes the state: the later a
// segment, the shorter.  (Equal ones and these, 16 units of 777 tokens: 33.2, 30.2 us.)
static int make_segments(int N, int G, SegTable &t)
{
    const int T = (N + C - 1) / C;
    if (G > T) G = T;
    int len[kMaxSegments], sum = 0;
    for (int g = 0; g < G; ++g) {
        const float off = 0.75f * (0.5f * (G - 1) - g) - (g == G - 1 && G > 1 ? 0.5f : 0.f);
        len[g] = T / G + (int)(off >= 0.f ? off + 0.5f : off - 0.5f);
        if (len[g] < 1) len[g] = 1;
        sum += len[g];
    }
    // the rounding's remainder is handed to (or taken from) the early segments, one chunk at a time
    for (int g = 0; sum != T; g = (g + 1) % G) {
        if (sum < T) { ++len[g]; ++sum; }
        else if (len[g] > 1) { --len[g]; --sum; }
    }
    int pos = 0;
    for (int g = 0; g < G; ++g) { t.begin[g] = pos * C; pos += len[g]; }
    for (int g = G; g <= kMaxSegments; ++g) t.begin[g] = pos * C;
    return G;
}

}  // namespace dp32s

static constexpr int kLongest[2] = {736, 512};   // without and from a state (there 609 to 672 too: the calls of that length without one need as much)

// Up to 32 tokens, up to 96 from a state (a block's readout is one wave's for 32 queries; here all eight waves have a part).  From 257, 385 or 513
// tokens on, by the number of groups of 64 columns, up to 736 (a last block that is mostly empty, chains of increments of whole blocks).  From a state, which
// blocks read faster, 257 to 512 tokens of up to 24 groups; at d_v 128, where they take it through a launch of their own, 225 to 512 of up to 64; at both widths
// 609 to 672 of up to 28 groups (20 and 21 tiles in three segments of blocks; 22 are four).
// (This kernel and blocks, us: 16 groups N 32 10.0, 11.9, N 33 12.2, 12.0, N 272 20.2, 20.2, N 448 23.9, 25.3, N 768 30.0, 28.2; 200 groups N 32 14.9, 15.2, N 33 17.0,
// 15.3; 512 groups N 32 30.5, 30.4, N 33 34.7, 30.8; 8 groups N 384 21.6, 22.5, N 640 25.9, 28.3; 24 groups N 300 22.1, 21.8, N 416 22.9, 25.4, N 512 25.9,
// 26.4; 32 groups N 300 23.0, 22.2, N 384 23.8, 23.4, N 385 24.0, 25.7, N 416 23.9, 25.7, N 480 25.7, 26.6, N 512 26.8, 26.6, N 704 29.7, 30.7, N 768 32.1,
// 30.9; 48 groups N 384 25.7, 23.9, N 480 28.6, 27.2; 64 groups N 512 30.3, 27.7, N 700 34.1, 34.2.  From a state 16 groups N 300 28.2, 29.3, N 512 33.3, 33.8, N
// 513 33.3, 32.4; 16 groups N 608 32.8, 32.0, N 609 33.0, 34.3, N 656 32.9, 34.3, N 673 32.9, 33.3; 28 groups N 608 35.9, 34.2, N 656 36.1,
// 36.5, N 673 36.1, 35.8; 32 groups N 300 30.8, 30.0, N 640 37.0, 36.8; d_v 128, 8 units N 225 27.4, 29.0, N 400 30.8, 37.8, N 513 33.4, 32.5; 32 units N 225 34.2, 33.0, N 300 36.9, 38.1, N
// 512 40.9, 42.5, N 513 40.2, 39.2.)
bool prefill_mfma32_short_takes(int U, int N, int dv, int has_init)
{
    const int groups = U * (dv / dp32s::COLS);
    if (N <= (has_init ? 96 : 32)) return true;
    const int most = has_init && dv == 64 ? 24 : 64;
    const int from = has_init ? (dv == 64 ? 256 : 224) : groups <= 28 ? 256 : groups <= 40 ? 384 : 512;
    if (has_init && groups <= 28 && N > 608 && N <= 672) return true;
    return groups <= most && N > from && N <= kLongest[has_init];
}

// One entry per (unit, slice, segment), for a call of N tokens and for every shorter one that comes here: segments only get more with N.
size_t prefill_mfma32_short_workspace_bytes(int U, int N, int dv)
{
    const int groups = U * (dv / dp32s::COLS);
    int most = 0;
    for (int has_init = 0; has_init < 2; ++has_init) {
        const int longest = N < kLongest[has_init] ? N : kLongest[has_init];
        if (!prefill_mfma32_short_takes(U, longest, dv, has_init)) continue;   // (up to 96 tokens are one segment, for which blocks need as much)
        const int G = dp32s::pick_segments(groups, longest);
        if (G > most) most = G;
    }
    return (size_t)groups * most * dp32s::kWsEntryFloats * sizeof(float);
}

hipError_t launch_prefill_mfma32_short(const void *q, const void *k, const void *v, void *y, float *state,
                                       int has_init, int packed_state, void *workspace, int U, int N, int dv, hipStream_t s)
{
    // the kernels' flag word (has_init arrives with bit 2 set for numerator-only outputs)
    has_init = (has_init & 1) | (packed_state ? 2 : 0) | (has_init & 4);
    using namespace dp32s;
    const int slices = dv / COLS;
    SegTable segs;
    const int G = make_segments(N, pick_segments(U * slices, N), segs);
    const uint16_t *q16 = (const uint16_t *)q, *k16 = (const uint16_t *)k, *v16 = (const uint16_t *)v;
    float *ws = static_cast<float *>(workspace);
    const int groups = U * slices, blocks = (groups + 7) / 8 * 8;
    if (((long long)groups + 7) * G >= (1ll << 31)) return hipErrorInvalidValue;
    // Several workgroups of a unit read the caller's state and one overwrites it (at d_v = 128 also its K-state): then it goes
    // through entry 0, which the first launch writes.
    const int in_entry = (has_init & 1) && G * slices > 1;
    if (G > 1 || in_entry) {
        hipLaunchKernelGGL((prefill_kernel<true>), dim3((unsigned)(blocks * (G > 1 ? G - 1 : 1))), dim3(NT), 0, s, q16, k16,
                           v16, (uint16_t *)y, state, has_init, G > 1 ? 0 : 1, in_entry, ws, N, dv, segs, G, groups);
        const hipError_t e = hipGetLastError();
        if (e != hipSuccess) return e;
    }
    hipLaunchKernelGGL((prefill_kernel<false>), dim3((unsigned)(blocks * G)), dim3(NT), 0, s, q16, k16, v16, (uint16_t *)y,
                       state, has_init, 0, in_entry, ws, N, dv, segs, G, groups);
    return hipGetLastError();
}

}  // namespace based
