// Causal Taylor linear attention, plain and with decay, chunked prefill of fp32 inputs at d' = 16 on the bf16 matrix instructions,
// at fp32 precision: every operand is cut into three bf16 parts, x = h + m + l, and a product is the sum of the six
// largest products of parts (h h, h m, m h, m m, h l, l h).  What is left out, m l + l m + l l, is 2^-24 of the product at most, one rounding, and
// 2^-27.4 in the root mean square (emulated, uniform mantissas and N(0, 1 / 4): largest 2^-24.0, at mantissas 0x007fc0).
//
// Why: a fp32 matrix instruction occupies the vector ALU (measured with two waves on a SIMD, one of them all 16x16x4 fp32
// products, the other all fused multiply-adds: 583 and 740 cycles alone, 1282 together), so the kernel on those
// (linattn_prefill_f32.h) pays for its products and its vector instructions one after the other, 2816 + 1640 of its 5555
// cycles per wave and 16 tokens.  Six bf16 products take 3/8 of the fp32 one's cycles and run beside the vector ALU
// (667 and 740 cycles alone, 996 together).
//
// Parts.  h = x rounded to bf16, m = x - h rounded to bf16, l = x - h - m: |m| <= 2^-8 and |l| <= 2^-17 for x in 1 .. 2, all exact, 24
// bits together.  (Cutting h off instead of rounding it doubles m and l: 2^-22 left out; 1 % faster.)  Each product's terms enter the accumulator
// smallest first; a chunk's part of the state is summed in an accumulator of its own and added to the state once, so the state is rounded
// once per 32 tokens.  (Values split into narrower parts for exact products: Dekker 1971; for matrix products: Ozaki et al. 2012.)
//
// State rows.  One row per unordered pair, 153 of them in five tiles of 32: tile T < 4 holds the pairs {a, (a + delta) mod 16} for
// delta = 2 T (rows 0 .. 15, a = row) and 2 T + 1; tile 4 the 16 linear rows, the constant row (16), zeros (17 .. 23), and delta = 8
// for a < 8 (24 .. 31).  A row holds the plain sum of k_a k_b v; the readout weighs q_a q_b with 1, with 1/2 for a = b.
//
// Work split.  A workgroup of eight waves takes 64 columns of one (unit, segment), chunks of 32 tokens.  Waves 0 .. 4 own a tile each, for
// both column tiles of 32: a feature is built and cut once per workgroup and used where it is built.  Wave 5 has the
// intra-chunk block P = 1 + A + A^2 / 2.  48 and 30 matrix instructions per chunk.  Waves 6 and 7 help to stage rows and to finish
// outputs (a workgroup of six reserves two waves on every SIMD all the same, and one went to a CU instead of two).  The six partial
// outputs and denominators of a chunk meet in LDS.  K-state: fp32 sums of the features a lane builds.
// Two barriers a chunk: rows staged, partial outputs free | partial outputs written, rows free.
//
// Segments as in linattn_prefill_f32.h: an increment launch, then the main launch, each segment from the sum of the entries before it.  The G - 1
// increments of a unit would leave a part of the chip idle, so without decay G workgroups share their tokens evenly (inc_len each): one whose share
// goes on past the end of a segment leaves an entry there and starts anew.
//
// Decay: as there, in a variant of its own.  The factors are powers of the rate from a table in LDS: on the features of the update,
// the old state, the state's part of the outputs and P.
//
// Values that are not finite: as in linattn_prefill_f32.h (a chunk with one in V is summed key by key).
//
// Range.  Below 2^-103 the third part of a value is not a normal bf16 number and the three hold it to 2^-134 only; a part past the
// largest bf16 number is infinite.  So a segment goes on with the fp32 matrix instructions (32x32x2: the same operands, uncut, and the same
// accumulators) from the first chunk on that holds a value, not 0, outside 2^-38 .. 2^20 in K or Q (their products: 2^-76 .. 2^40) or 2^-60 ..
// 2^40 in V, or from its start if the state it starts from has an entry outside 2^-100 .. 2^100.  Inside, the parts hold all 24 bits of every
// value of the rows and of every feature, and no sum passes 2^112.  An entry of the state may get below 2^-103 (a sum of products of small
// values, or what cancellation leaves): what a query, 2^40 at most per row, then misses is 2^-34 of the smallest value of V at most, for 153 rows 2^-26.
// With decay, where a state shrinks, it is looked at in every chunk, and a rate whose 32nd power is outside 2^-26 .. 2^26 (and
// not 0) has no other instructions.  Of N(0, 1 / 4) values one in 2e11 of K and Q is outside.  All of this takes 3 % of the time, 1 % of it
// the look, by the threads that stage the rows (waves 6 and 7 alone, with loads of their own: 4 %).  128 units of 2048 tokens, d_v 64, uncut: 253 us.
//
// Measured against linattn_prefill_f32.h (us): 128 units of 2048 tokens, d_v 64, 193 -> 144 to 150 (increments 50, main launch 129 in a trace with cold
// inputs); 16 units of 2048 111 -> 57, of 777 43 -> 28; 512 units of 2048 507 -> 403.  Bound by vector instructions, 600 per
// tile, wave and chunk, 350 of them cutting features and state: vector ALU 50 %, matrix pipe 26 % of the cycles, LDS 30 %.  With
// decay and gate: 128 units of 2048, d_v 64, 225 -> 171; 16 of 300 41 -> 31.
// Error against float64 (2-norm; 49 to 8192 tokens, values of scale 1e-3 to 30, both widths): y 0.7e-7 to 1.5e-7, S 0.5e-7 to 2.2e-7; there 0.9e-7 to
// 2.4e-7 and 1.1e-7 to 4.1e-7.  With decay 0.7e-7 to 1.4e-7 and 0.6e-7 to 0.9e-7, there 0.9e-7 to 1.9e-7 and 1.0e-7 to 1.3e-7.
#include "common.h"

#include <limits.h>

#include <utility>

// Sums and products as they are written: at a rate of 1 the decay variant multiplies by ones and gives the plain kernel's bits.
#pragma clang fp contract(off)

namespace based {

namespace f32x3 {

typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef float f32x8 __attribute__((ext_vector_type(8)));
typedef float f32x16 __attribute__((ext_vector_type(16)));
typedef float f32x2 __attribute__((ext_vector_type(2)));
typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
typedef short s16x4 __attribute__((ext_vector_type(4)));

constexpr int DP = 16, C = 32, COLS = 64;
constexpr int TILES = 5, SEND = TILES + 1, NW = 8, NT = 64 * NW;
constexpr int ROWS = 32 * TILES, D = feature_dim(DP);
constexpr int kMaxSegments = 64;
// Workspace entry of one (unit, slice, segment): [tile][column tile][reg / 4][lane][reg % 4], then z [row]
constexpr size_t kEntryFloats = (size_t)ROWS * COLS + ROWS;

constexpr int K_LD = C + 4;            // K^T rows (the 16-byte reads of 16 rows fall into different banks)
constexpr int K_ONE = 16, K_ZERO = 17; // rows of ones (zero past the end) and of zeros
constexpr int K_DECAY = 18;            // row of each token's factor in the state after the chunk
// Q rows, so that both factors of a slab's rows are runs of 16 from one place: q, q again (indices a + delta need no wrap), 1 x 16,
// q_8 .. q_15, [1, 0 x 7], q_0 .. q_7
constexpr int Q_LD = 76, Q_ONES = 32, Q_ONES_HI = 40, Q_UNIT_LO = 56;
constexpr int V_LD = COLS + 16;
constexpr int IMG_LD = COLS + 4;

struct alignas(16) Rows {
    float kt[19][K_LD];
    float q[C][Q_LD];
    uint16_t v[3][C][V_LD];   // the three parts
};
template <bool INC> struct Lds {
    Rows rows[INC ? 2 : 1];   // (the increment has no partial outputs: two generations, one barrier)
    float x[INC ? 1 : SEND][8][2][33][4];   // partial Y^T: [sender][4 column tile + reg / 4][lane / 32][lane % 32][reg % 4]
    float den[SEND][C];
    float z[ROWS];
    int turn;
    int wide_from;            // the first chunk seen with a value in K, Q or V whose parts would not hold it
    int bad[2];               // number of the last even and odd chunk with a value in V that is not finite, plus one
    float power[C + 1];       // of the decay rate
};
static_assert(2 * sizeof(Lds<false>) <= 160 * 1024, "two workgroups to a CU");
static_assert(sizeof(Lds<true>) <= 80 * 1024, "");

template <typename F, int... I> __device__ __forceinline__ void for_seq(F &&f, std::integer_sequence<int, I...>)
{
    (f(std::integral_constant<int, I>{}), ...);
}
template <int N, typename F> __device__ __forceinline__ void for_n(F &&f) { for_seq(f, std::make_integer_sequence<int, N>{}); }

__device__ __forceinline__ f32x16 mfma(bf16x8 a, bf16x8 b, f32x16 c) { return __builtin_amdgcn_mfma_f32_32x32x16_bf16(a, b, c, 0, 0, 0); }
__device__ __forceinline__ f32x16 zero16()
{
    f32x16 a;
    for_n<16>([&](auto i) { a[i.value] = 0.f; });
    return a;
}
// orders LDS traffic only
__device__ __forceinline__ void wg_sync() { asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory"); }
// matrix instructions ignore the EXEC mask: an asm statement keeps the jump over a wave's block
__device__ __forceinline__ void role_guard() { asm volatile("; wave-role block: keep the execz branch"); }
__device__ __forceinline__ float bf16lo(uint32_t w) { return __uint_as_float(w << 16); }
__device__ __forceinline__ float bf16hi(uint32_t w) { return __uint_as_float(w & 0xffff0000u); }
__device__ __forceinline__ uint32_t pack2(float a, float b)
{
    return __builtin_bit_cast(uint32_t, __builtin_convertvector(f32x2{a, b}, bf16x2));
}

struct Parts2 { uint32_t h, m, l; };   // of two values
__device__ __forceinline__ Parts2 split2(float a, float b)
{
    Parts2 o;
    o.h = pack2(a, b);
    const float ra = a - bf16lo(o.h), rb = b - bf16hi(o.h);
    o.m = pack2(ra, rb);
    o.l = pack2(ra - bf16lo(o.m), rb - bf16hi(o.m));
    return o;
}
struct Parts { bf16x8 p[3]; };   // of the eight values of an operand
template <typename G> __device__ __forceinline__ Parts split8(G &&x)
{
    u32x4 p[3];
    for_n<4>([&](auto i) {
        const Parts2 t = split2(x(2 * i.value), x(2 * i.value + 1));
        p[0][i.value] = t.h;
        p[1][i.value] = t.m;
        p[2][i.value] = t.l;
    });
    Parts o;
    for_n<3>([&](auto i) { o.p[i.value] = __builtin_bit_cast(bf16x8, p[i.value]); });
    return o;
}
// acc += a b, terms of increasing size
__device__ __forceinline__ void mfma6(const Parts &a, const Parts &b, f32x16 &acc)
{
    constexpr int pa[6] = {2, 0, 1, 1, 0, 0}, pb[6] = {0, 2, 1, 0, 1, 0};
    for_n<6>([&](auto i) { acc = mfma(a.p[pa[i.value]], b.p[pb[i.value]], acc); });
}

// The same of the values themselves, each lane's eight, on the fp32 matrix instruction.
template <typename A, typename B> __device__ __forceinline__ void mfma_f32(A &&a, B &&b, f32x16 &acc)
{
    for_n<8>([&](auto i) { acc = __builtin_amdgcn_mfma_f32_32x32x2f32(a(i.value), b(i.value), acc, 0, 0, 0); });
}
// Largest and smallest magnitude but 0 of the values seen, as their bits without the sign, doubled (less 1 for the smallest: 0 is last).
struct Magnitudes {
    uint32_t most = 0, least = ~0u;
    __device__ __forceinline__ void see(float x)
    {
        const uint32_t u = __float_as_uint(x) << 1;
        most = max(most, u);
        least = min(least, u - 1);
    }
    // one below 2^LO, or above 2^HI or not finite
    template <int LO, int HI> __device__ __forceinline__ bool outside() const
    {
        return least < ((127u + LO) << 24) - 1 || most > (127u + HI) << 24;
    }
};

// Canonical rows (Eq. 4 order) of a state row, and what a stored value is multiplied by to give the canonical one; r1 < 0: zeros.
struct Canon { int r1, r2; float scale; };
__device__ __forceinline__ Canon canon(int row)
{
    const int T = row >> 5, fl = row & 31;
    const bool pair = T < 4 || fl >= 24;
    const int a = T < 4 ? fl & 15 : fl - 24, b = (a + (T < 4 ? 2 * T + (fl >> 4) : 8)) & 15;
    if (pair) return {1 + DP + a * DP + b, 1 + DP + b * DP + a, kRsqrt2};
    if (fl < 16) return {1 + fl, 1 + fl, 1.f};
    return {fl == 16 ? 0 : -1, fl == 16 ? 0 : -1, 1.f};
}

struct DecayArg {
    const float *gamma, *gate;   // [H] (null: 1); [B][N][H], factors of the rows of y (null: 1)
    int H;
};

// The launch covers `slices` slices of 64 columns from first_slice on.  has_init: bit 0 an initial state is given, bit 2 the outputs are
// the numerators alone.  INC: state increments only.  A unit's slice has `slots` entries: entry 0 is the caller's state, if there is one (segment 0 also
// converts it), then come the increments in the order of their tokens, one to a segment.
// SHARED: the increments are shared out over `shares` workgroups of inc_len tokens (else one to a segment); a share that starts inside a segment has an entry
// of its own.
template <int DV, bool INC, bool DECAY, bool SHARED>
__global__ __launch_bounds__(NT, 4) void prefill_kernel(const float *__restrict__ q, const float *__restrict__ k,
                                                        const float *__restrict__ v, float *__restrict__ y, float *state, int has_init,
                                                        int N, float *ws, int seg_len, int inc_len, int shares, int G, int slots, int first_slice, int slices, int local,
                                                        DecayArg dec)
{
    constexpr int SL = DV / COLS;
    __shared__ __align__(16) Lds<INC> lds;
    const bool numerator_only = (has_init & 4) != 0, init = (has_init & 1) != 0;
    static_assert(!(DECAY && SHARED), "an entry is scaled by the decay of a whole segment");
    const int gseg = !INC ? G : SHARED ? shares : G - 1;
    // The workgroups of a unit's slice run on one XCD (workgroup index mod 8), whose L2 then holds the entries that they write and sum, for the first `local`
    // slices, a multiple of 8; the rest's run on all XCDs.  (All on all XCDs, and this, us: 16 units N 777 31.2, 26.5, N 2048 59.5, 47.1, 32 units
    // N 2048 66.5, 54.5, 60 units N 1500 69.8, 61.0, 128 units N 2048 141.2, 138.4; d_v 128, 8 units N 1024 36.1, 26.0.)  Fewer than 8 slices have a row of the grid each:
    // dealt out with them 4 units of 777 tokens took 27.0 us instead of 26.8, 2 of 2000 at d_v 128 35.9 instead of 35.4.
    int seg = blockIdx.x, us = blockIdx.y;
    if (local > 0) {
        const uint32_t bid = blockIdx.x, here = local * gseg;
        const bool on_one = bid < here;
        const uint32_t idx = on_one ? bid / 8 : bid - here, at = idx / (uint32_t)gseg;
        seg = idx - at * gseg;
        us = on_one ? at * 8 + bid % 8 : local + at;
    }
    const int u = slices == 1 ? us : (uint32_t)us / SL, slice = first_slice + (slices == 1 ? 0 : (uint32_t)us % SL), col0 = slice * COLS;   // (slices: 1 or SL)
    const int tid = threadIdx.x, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    int lane = tid & 63, g = lane >> 5, n = lane & 31;
    const int len = INC && SHARED ? inc_len : seg_len, begin = seg * len, end = min(INC && SHARED ? (G - 1) * seg_len : N, begin + len), chunks = (end - begin + C - 1) / C;
    // Six of the eight waves have matrix work, five of them a tile, and consecutive waves sit on SIMDs 0, 2, 1, 3, 0, .. from any of them on.
    // The roles are dealt out from the first wave's SIMD, and from two places further in the workgroup whose LDS does not start at 0:
    // the two workgroups on a CU then put two or three tiles on every SIMD.  (Any turn gives the same result.)
    if (tid == 0) {
        const unsigned simd = __builtin_amdgcn_s_getreg(4 | 4 << 6 | 1 << 11), lds_base = __builtin_amdgcn_s_getreg(6 | 7 << 11);
        lds.turn = (0x3120 >> 4 * simd & 3) + (lds_base ? 2 : 0);
    }
    __syncthreads();
    const int w = (wave + __builtin_amdgcn_readfirstlane(lds.turn)) & (NW - 1);
    __syncthreads();
    const bool tile = w < TILES;

    const float *qu = q + (size_t)u * N * DP, *ku = k + (size_t)u * N * DP, *vu = v + (size_t)u * N * DV + col0;
    float *yu = y + (size_t)u * N * DV + col0;
    float *Su = state ? state + (size_t)u * state_stride(DP, DV) + col0 : nullptr;
    float *zu = state ? state + (size_t)u * state_stride(DP, DV) + (size_t)D * DV : nullptr;
    float *entries = ws ? ws + ((size_t)u * SL + slice) * slots * kEntryFloats : nullptr;

    const float gm = DECAY && dec.gamma ? dec.gamma[u % dec.H] : 1.f;
    const float *gate = DECAY && dec.gate ? dec.gate + (size_t)(u / dec.H) * N * dec.H + u % dec.H : nullptr;
    auto tokens = [&](int t) { return min(C, end - begin - C * t); };   // of chunk t

    // waves 0 .. 4: S[c][r] = row 8 (r / 4) + 4 g + r % 4 of the tile, column 32 c + n; z: row n of the tile, summed over the halves
    f32x16 S[2];
    float z = 0.f;
    for_n<2>([&](auto c) { S[c.value] = zero16(); });
    auto add_halves = [&](float a) {
        const auto t = __builtin_amdgcn_permlane32_swap(__float_as_uint(a), __float_as_uint(a), false, false);
        return __uint_as_float(t[0]) + __uint_as_float(t[1]);
    };

    // The state buffer moves through LDS as an image of the tiles' rows, 16 bytes a thread.
    float (*image)[IMG_LD] = reinterpret_cast<float (*)[IMG_LD]>(&lds);
    static_assert(sizeof(Lds<INC>) >= sizeof(float) * ROWS * IMG_LD + sizeof(float) * ROWS, "");
    float *image_z = reinterpret_cast<float *>(&lds) + ROWS * IMG_LD;
    constexpr int PIECES = ROWS * COLS / 4;
    auto import_state = [&]() {
        constexpr int BATCH = 4;
#pragma unroll 1
        for (int i0 = tid; i0 < PIECES; i0 += BATCH * NT) {
            f32x4 x[BATCH][2];
            for_n<BATCH>([&](auto s) {
                const int i = min(i0 + s.value * NT, PIECES - 1);
                const Canon c = canon(i >> 4);
                x[s.value][0] = *reinterpret_cast<const f32x4 *>(Su + (size_t)max(c.r1, 0) * DV + 4 * (i & 15));
                x[s.value][1] = *reinterpret_cast<const f32x4 *>(Su + (size_t)max(c.r2, 0) * DV + 4 * (i & 15));
            });
            for_n<BATCH>([&](auto s) {
                const int i = min(i0 + s.value * NT, PIECES - 1);
                const Canon c = canon(i >> 4);
                const f32x4 t = (x[s.value][0] + x[s.value][1]) * (0.5f / c.scale);
                *reinterpret_cast<f32x4 *>(&image[i >> 4][4 * (i & 15)]) = c.r1 < 0 ? f32x4{0.f, 0.f, 0.f, 0.f} : t;
            });
        }
        if (tid < ROWS) {
            const Canon c = canon(tid);
            image_z[tid] = c.r1 < 0 ? 0.f : (0.5f / c.scale) * (zu[max(c.r1, 0)] + zu[max(c.r2, 0)]);
        }
        __syncthreads();
        if (tile) {
            for_n<2>([&](auto c) {
                for_n<16>([&](auto r) { S[c.value][r.value] = image[32 * w + 8 * (r.value >> 2) + 4 * g + (r.value & 3)][32 * c.value + n]; });
            });
            z = g == 0 ? image_z[32 * w + n] : 0.f;
        }
        __syncthreads();
    };
    // Both rows of a pair.  A state that is not symmetric (none of this recurrence is) keeps its antisymmetric part.
    auto put_image = [&]() {   // waves 0 .. 4
        for_n<2>([&](auto c) {
            for_n<16>([&](auto r) { image[32 * w + 8 * (r.value >> 2) + 4 * g + (r.value & 3)][32 * c.value + n] = S[c.value][r.value]; });
        });
        const float zt = add_halves(z);
        if (g == 0) image_z[32 * w + n] = zt;
    };
    auto export_image = [&]() {
        const float g_all = DECAY ? powf(gm, (float)N) : 1.f;
        auto half_difference = [&](float a, float b) { return a == b ? 0.f : 0.5f * (a - b) * g_all; };   // (equal infinities: none)
        __syncthreads();
#pragma unroll 1
        for (int i = tid; i < PIECES; i += NT) {
            const Canon c = canon(i >> 4);
            if (c.r1 < 0) continue;
            float *p1 = Su + (size_t)c.r1 * DV + 4 * (i & 15), *p2 = Su + (size_t)c.r2 * DV + 4 * (i & 15);
            const f32x4 x = *reinterpret_cast<const f32x4 *>(&image[i >> 4][4 * (i & 15)]) * c.scale;
            f32x4 d = {0.f, 0.f, 0.f, 0.f};
            if (init) {
                const f32x4 x1 = *reinterpret_cast<const f32x4 *>(p1), x2 = *reinterpret_cast<const f32x4 *>(p2);
                for_n<4>([&](auto j) { d[j.value] = half_difference(x1[j.value], x2[j.value]); });
            }
            *reinterpret_cast<f32x4 *>(p1) = x + d;
            *reinterpret_cast<f32x4 *>(p2) = x - d;
        }
        if (col0 != 0 || tid >= ROWS) return;
        const Canon c = canon(tid);
        if (c.r1 < 0) return;
        const float s = image_z[tid] * c.scale, d = init ? half_difference(zu[c.r1], zu[c.r2]) : 0.f;
        zu[c.r1] = s + d;
        if (c.r2 != c.r1) zu[c.r2] = s - d;
    };
    auto entry_s = [&](int e) { return entries + (size_t)e * kEntryFloats + (size_t)w * 2048 + 4 * lane; };
    auto entry_z = [&](int e) { return entries + (size_t)e * kEntryFloats + ROWS * COLS + 32 * w + n; };
    // of the tokens that share i of the increments has in segment k (entry 0: the caller's state, if any).  In order without a gap: the launcher's
    // shares end with no segment but the last one.
    auto entry_at = [&](int i, int k) { return init + k + (SHARED ? i : 0); };
    auto store_entry = [&](int e) {
        if (!tile) return;
        float *p = entry_s(e);
        for_n<2>([&](auto c) {
            for_n<4>([&](auto j) {
                f32x4 t;
                for_n<4>([&](auto i) { t[i.value] = S[c.value][4 * j.value + i.value]; });
                *reinterpret_cast<f32x4 *>(p + (4 * c.value + j.value) * 256) = t;
            });
        });
        const float zt = add_halves(z);
        if (g == 0) *entry_z(e) = zt;
    };
    if (INC) {
        if (init && seg == 0) {
            import_state();
            store_entry(0);
            for_n<2>([&](auto c) { S[c.value] = zero16(); });
            z = 0.f;
        }
    } else if (G > 1) {
        if (tile) {
            // the sum of the entries before the segment, two at a time
            int e = 0;
            const int count = init + seg + (SHARED && seg > 0 ? (seg * seg_len - 1) / inc_len : 0);
            const float g_seg = DECAY ? powf(gm, (float)seg_len) : 1.f;
            auto add = [&](auto of) {
                constexpr int E = decltype(of)::value;
                f32x4 x[E][8];
                float xz[E];
                for_n<E>([&](auto i) {
                    for_n<8>([&](auto j) { x[i.value][j.value] = *reinterpret_cast<const f32x4 *>(entry_s(e + i.value) + j.value * 256); });
                    xz[i.value] = *entry_z(e + i.value);
                });
                for_n<E>([&](auto i) {
                    for_n<32>([&](auto r) {
                        float &a = reinterpret_cast<float *>(&S[r.value / 16])[r.value % 16];
                        if (DECAY) a *= g_seg;
                        a += x[i.value][r.value / 4][r.value % 4];
                    });
                    if (DECAY) z *= g_seg;
                    z += g == 0 ? xz[i.value] : 0.f;
                });
                e += E;
            };
            if (count & 1) add(std::integral_constant<int, 1>{});
            while (e < count) add(std::integral_constant<int, 2>{});
        }
    } else if (init) {
        import_state();
    }

    bool wide = false;   // something but the rows keeps this wave from cutting its operands: the state (waves 0 .. 4), the rate's powers
    auto state_outside = [&]() {
        Magnitudes m;
        for_n<32>([&](auto r) { m.see(S[r.value / 16][r.value % 16]); });
        return __any(m.outside<-100, 100>()) != 0;
    };
    if (!INC && tile && (init || G > 1)) wide = state_outside();

    // What is computed from the lane's place is not kept past a call of this.
    auto fresh_lane = [&]() {
        asm volatile("" : "+v"(lane));
        g = lane >> 5;
        n = lane & 31;
    };

    // ---- operands -----------------------------------------------------------------------------
    // key side: row n of the tile is the product of two K^T rows
    auto key_rows = [&](int &ka, int &kb) {
        if (w < 4) {
            ka = n & 15;
            kb = (ka + 2 * w + (n >> 4)) & 15;
        } else {
            ka = n < 16 ? n : n == 16 ? K_ONE : n < 24 ? K_ZERO : n - 24;
            kb = n < 16 ? K_ONE : n == 16 ? K_ONE : n < 24 ? K_ZERO : n - 16;
        }
    };
    // query side: k-slot (jj, i) of slab s is row 16 s + 8 jj + 4 g + i, the product of entries 8 jj + 4 g + i of two runs of the Q row
    const int qa[2] = {0, w < 4 ? 0 : Q_UNIT_LO}, qb[2] = {w < 4 ? 2 * w : Q_ONES, w < 4 ? 2 * w + 1 : Q_ONES_HI};
    const float half = w == 0 ? 0.5f : 1.f;   // delta = 0
    // part p of V^T, tokens 16 s + 4 g + {0 .. 3, 8 .. 11} of column 32 c + n, by the transposing LDS read
    auto read_v = [&](const Rows &rows, int p, int s, int c) {
        const int tr_row = ((lane & 15) >> 2) + 4 * g, tr_col = 16 * ((lane >> 4) & 1) + 4 * (lane & 3);
        const uint16_t *a = &rows.v[p][16 * s + tr_row][32 * c + tr_col];
        const u32x2 x = __builtin_bit_cast(u32x2, __builtin_amdgcn_ds_read_tr16_b64_v4i16((__attribute__((address_space(3))) s16x4 *)a));
        const u32x2 x8 = __builtin_bit_cast(u32x2, __builtin_amdgcn_ds_read_tr16_b64_v4i16((__attribute__((address_space(3))) s16x4 *)(a + 8 * V_LD)));
        return __builtin_bit_cast(bf16x8, u32x4{x[0], x[1], x8[0], x8[1]});
    };
    // the values themselves, from memory
    auto read_v_f32 = [&](int tok0, int s, int c) {
        f32x8 x;
        for_n<8>([&](auto i) {
            const int tok = tok0 + 16 * s + 4 * g + (i.value & 3) + 8 * (i.value >> 2);
            const float t = vu[(size_t)min(tok, end - 1) * DV + 32 * c + n];
            x[i.value] = tok < end ? t : 0.f;
        });
        return x;
    };
    auto v_parts = [&](const Rows &rows, int s, int c) {
        Parts o;
        for_n<3>([&](auto p) { o.p[p.value] = read_v(rows, p.value, s, c); });
        return o;
    };

    // ---- staging: global -> registers -> LDS --------------------------------------------------
    // A thread has one of the 512 pieces of four floats of V; waves 4 and 5 have the 128 of K, 6 and 7 those of Q (the others load one
    // too: every load is unconditional, so that the number in flight is known).
    struct Place { int v, cv, k, ck; };   // token and column of the piece of V, of K or Q
    auto place = [&]() {
        int t = tid;
        asm volatile("" : "+v"(t));   // (what is computed from it is not kept through the loop)
        return Place{t >> 4, 4 * (t & 15), t >> 2 & 31, 4 * (t & 3)};
    };
    const bool k_piece = wave == 4 || wave == 5, q_piece = wave >= 6;
    f32x4 raw[2];
    auto load_raw = [&](int tok0, const Place &p) {   // (rows past the end: the last one again)
        const int base = min(tok0, end - 1), last = end - 1 - base;
        const float *vb = vu + (size_t)base * DV, *kb = (!INC && q_piece ? qu : ku) + (size_t)base * DP;
        raw[0] = *reinterpret_cast<const f32x4 *>(vb + (unsigned)(min(p.v, last) * DV + p.cv));
        raw[1] = *reinterpret_cast<const f32x4 *>(kb + (unsigned)(min(p.k, last) * DP + p.ck));
    };
    auto stage = [&](int t, Rows &rows, const Place &p) {
        const int tok0 = begin + C * t;
        {
            const bool past = tok0 + p.v >= end;
            f32x4 x = raw[0];
            if (past) x = f32x4{0.f, 0.f, 0.f, 0.f};
            const Parts2 a = split2(x[0], x[1]), b = split2(x[2], x[3]);
            *reinterpret_cast<u32x2 *>(&rows.v[0][p.v][p.cv]) = u32x2{a.h, b.h};
            *reinterpret_cast<u32x2 *>(&rows.v[1][p.v][p.cv]) = u32x2{a.m, b.m};
            *reinterpret_cast<u32x2 *>(&rows.v[2][p.v][p.cv]) = u32x2{a.l, b.l};
        }
        if (k_piece) {
            const bool past = tok0 + p.k >= end;
            for_n<4>([&](auto i) { rows.kt[p.ck + i.value][p.k] = past ? 0.f : raw[1][i.value]; });
            if (p.ck == 0) rows.kt[K_ONE][p.k] = past ? 0.f : 1.f;
            if (DECAY && p.ck == 4) rows.kt[K_DECAY][p.k] = lds.power[max(tokens(t) - 1 - p.k, 0)];
        }
        if (!INC && q_piece) {
            *reinterpret_cast<f32x4 *>(&rows.q[p.k][p.ck]) = raw[1];
            *reinterpret_cast<f32x4 *>(&rows.q[p.k][16 + p.ck]) = raw[1];
            *reinterpret_cast<f32x4 *>(&rows.q[p.k][p.ck < 8 ? Q_UNIT_LO + 8 + p.ck : Q_ONES_HI + p.ck]) = raw[1];
        }
    };

    // A look at the pieces of chunk t, in registers.
    auto look = [&](int t) {
        // (0 is inside too, but rare enough to be looked for separately; minimum and maximum keep a NaN, which no comparison lets pass)
        auto least = [](f32x4 x) {
            return __builtin_elementwise_minimum(__builtin_elementwise_minimum(__builtin_elementwise_minimum(fabsf(x[0]), fabsf(x[1])), fabsf(x[2])), fabsf(x[3]));
        };
        auto most = [](f32x4 x) {
            return __builtin_elementwise_maximum(__builtin_elementwise_maximum(__builtin_elementwise_maximum(fabsf(x[0]), fabsf(x[1])), fabsf(x[2])), fabsf(x[3]));
        };
        if (!(least(raw[0]) >= 0x1p-60f && most(raw[0]) <= 0x1p40f)) {
            Magnitudes m;
            for_n<4>([&](auto j) { m.see(raw[0][j.value]); });
            if (m.outside<-60, 40>()) atomicMin(&lds.wide_from, t);
            if (m.most >= 0xff000000u) lds.bad[t & 1] = t + 1;
        }
        if ((k_piece || (!INC && q_piece)) && !(least(raw[1]) >= 0x1p-38f && most(raw[1]) <= 0x1p20f)) {
            Magnitudes m;
            for_n<4>([&](auto j) { m.see(raw[1][j.value]); });
            if (m.outside<-38, 20>()) atomicMin(&lds.wide_from, t);
        }
    };

    // S += phi(K)^T V of a chunk (uncut: on the fp32 matrix instructions)
    auto update = [&](const Rows &rows, int t, auto uncut) {
        f32x16 d[2];
        float zc = 0.f;
        int ka, kb;
        key_rows(ka, kb);
        for_n<2>([&](auto c) { d[c.value] = zero16(); });
        for_n<2>([&](auto s) {
            float f[8];
            for_n<2>([&](auto h) {
                const int tok = 16 * s.value + 4 * g + 8 * h.value;
                const f32x4 a = *reinterpret_cast<const f32x4 *>(&rows.kt[ka][tok]), b = *reinterpret_cast<const f32x4 *>(&rows.kt[kb][tok]);
                for_n<4>([&](auto i) { f[4 * h.value + i.value] = a[i.value] * b[i.value]; });
                if (DECAY) {
                    const f32x4 x = *reinterpret_cast<const f32x4 *>(&rows.kt[K_DECAY][tok]);
                    for_n<4>([&](auto i) { f[4 * h.value + i.value] *= x[i.value]; });
                }
            });
            zc += ((f[0] + f[1]) + (f[2] + f[3])) + ((f[4] + f[5]) + (f[6] + f[7]));
            if constexpr (decltype(uncut)::value) {
                for_n<2>([&](auto c) {
                    const f32x8 x = read_v_f32(begin + C * t, s.value, c.value);
                    mfma_f32([&](int i) { return f[i]; }, [&](int i) { return x[i]; }, d[c.value]);
                });
            } else {
                const Parts op = split8([&](int i) { return f[i]; });
                for_n<2>([&](auto c) {
                    mfma6(op, v_parts(rows, s.value, c.value), d[c.value]);
                    __builtin_amdgcn_sched_barrier(0);   // (bounds what is in flight at a time)
                });
            }
        });
        if (DECAY) {
            const float g_s = lds.power[tokens(t)];
            z *= g_s;
            for_n<32>([&](auto r) { S[r.value / 16][r.value % 16] *= g_s; });
        }
        z += zc;
        // (value by value: as vectors the compiler spills them, with a second copy of this in the kernel)
        for_n<32>([&](auto r) { S[r.value / 16][r.value % 16] += d[r.value / 16][r.value % 16]; });
    };

    for (int i = tid; i < (INC ? 2 : 1) * C; i += NT) {
        Rows &rows = lds.rows[i / C];
        rows.kt[K_ZERO][i % C] = 0.f;
        for_n<16>([&](auto j) { rows.q[i % C][Q_ONES + j.value] = 1.f; });
        for_n<8>([&](auto j) { rows.q[i % C][Q_UNIT_LO + j.value] = j.value == 0 ? 1.f : 0.f; });
    }
    if (tid == 0) {
        lds.bad[0] = lds.bad[1] = 0;
        lds.wide_from = INT_MAX;
    }
    if (DECAY && tid <= C) lds.power[tid] = powf(gm, (float)tid);
    __syncthreads();
    load_raw(begin, place());
    look(0);
    stage(0, lds.rows[0], place());
    load_raw(begin + C, place());
    wg_sync();
    // wide_from as read for a chunk: it has that one, and may have the next, which is told by its number
    int wide_from = __builtin_amdgcn_readfirstlane(lds.wide_from);
    if (DECAY) {
        const float g_c = fabsf(lds.power[C]);
        wide = wide || !(gm == 0.f || (g_c >= 0x1p-26f && g_c <= 0x1p26f));
    }
    auto is_wide = [&](int t) { return wide || t >= wide_from; };
    if (INC) {
        auto next_chunk = [&](int t) {
            const Place p = place();
            look(t + 1);
            stage(t + 1, lds.rows[(t + 1) & 1], p);
            load_raw(begin + C * (t + 2), p);
            wg_sync();
            wide_from = __builtin_amdgcn_readfirstlane(lds.wide_from);
        };
        if (tile) {
            role_guard();
            int k = begin / seg_len, boundary = (k + 1) * seg_len;   // (SHARED)
            for (int t = 0; t < chunks; ++t) {
                fresh_lane();
                if (__builtin_expect(is_wide(t), 0)) update(lds.rows[t & 1], t, std::true_type{});
                else update(lds.rows[t & 1], t, std::false_type{});
                const int next = begin + C * (t + 1);
                if (SHARED && next == boundary && next < end) {
                    store_entry(entry_at(seg, k++));
                    boundary += seg_len;
                    for_n<32>([&](auto r) { S[r.value / 16][r.value % 16] = 0.f; });
                    z = 0.f;
                }
                next_chunk(t);
            }
        } else {
            for (int t = 0; t < chunks; ++t) next_chunk(t);
        }
        store_entry(entry_at(seg, SHARED ? (end - 1) / seg_len : seg));
        return;
    }
    Rows &rows = lds.rows[0];
    // a chunk's outputs: this thread finishes columns 4 (tid % 16) .. of token tid / 16 (rows of 33: 16 consecutive readers in
    // different banks)
    auto output = [&](int tok0, const Place &p) {
        const int tok = p.v, cq = p.cv / 4;
        f32x4 x[SEND];
        float d[SEND];
        for_n<SEND>([&](auto s) {
            x[s.value] = *reinterpret_cast<const f32x4 *>(&lds.x[s.value][cq >> 1][cq & 1][tok][0]);
            d[s.value] = lds.den[s.value][tok];
        });
        const float den = ((d[0] + d[1]) + (d[2] + d[3])) + (d[4] + d[5]);
        float inv = numerator_only ? 1.f : 1.f / den;
        if (gate && tok0 + tok < end) inv *= gate[(size_t)(tok0 + tok) * dec.H];
        const f32x4 sum = ((x[0] + x[1]) + (x[2] + x[3])) + (x[4] + x[5]);
        if (tok0 + tok < end) *reinterpret_cast<f32x4 *>(yu + (size_t)tok0 * DV + (unsigned)(tok * DV + 4 * cq)) = sum * inv;
    };
    auto put_partial = [&](const f32x16 (&Y)[2]) {
        for_n<8>([&](auto cj) {
            f32x4 o;
            for_n<4>([&](auto i) { o[i.value] = Y[cj.value / 4][4 * (cj.value % 4) + i.value]; });
            *reinterpret_cast<f32x4 *>(&lds.x[w][cj.value][g][n][0]) = o;
        });
    };
    auto next_chunk = [&](int t) {
        look(t + 1);
        wg_sync();
        const Place p = place();
        const int from = lds.wide_from;
        output(begin + C * t, p);
        stage(t + 1, rows, p);
        wide_from = __builtin_amdgcn_readfirstlane(from);
        load_raw(begin + C * (t + 2), p);
        wg_sync();
    };
    const bool writes_state = state && seg == G - 1;
    // (a loop for each role: what one keeps in registers is not kept by the others)
    if (tile) {
        role_guard();
        auto chunk = [&](int t, auto uncut) {
            fresh_lane();
            f32x16 Y[2];
            for_n<2>([&](auto c) { Y[c.value] = zero16(); });
            const float zt = add_halves(z);
            if (g == 0) lds.z[32 * w + n] = zt;
            float dsum = 0.f;
            for_n<2>([&](auto s) {
                float f[8];
                for_n<2>([&](auto jj) {
                    const f32x4 a = *reinterpret_cast<const f32x4 *>(&rows.q[n][4 * g + qa[s.value] + 8 * jj.value]);
                    const float *b = &rows.q[n][4 * g + qb[s.value] + 8 * jj.value];
                    for_n<4>([&](auto i) {
                        f[4 * jj.value + i.value] = (s.value == 0 ? a[i.value] * half : a[i.value]) * b[i.value];
                    });
                });
                for_n<2>([&](auto jj) {
                    const f32x4 zv = *reinterpret_cast<const f32x4 *>(&lds.z[32 * w + 16 * s.value + 8 * jj.value + 4 * g]);
                    for_n<4>([&](auto i) { dsum = fmaf(f[4 * jj.value + i.value], zv[i.value], dsum); });
                });
                if constexpr (decltype(uncut)::value) {
                    for_n<2>([&](auto c) {
                        mfma_f32([&](int i) { return S[c.value][8 * s.value + i]; }, [&](int i) { return f[i]; }, Y[c.value]);
                    });
                } else {
                    const Parts op = split8([&](int i) { return f[i]; });
                    __builtin_amdgcn_sched_barrier(0);
                    for_n<2>([&](auto c) {
                        mfma6(split8([&](int i) { return S[c.value][8 * s.value + i]; }), op, Y[c.value]);
                        __builtin_amdgcn_sched_barrier(0);
                    });
                }
                __builtin_amdgcn_sched_barrier(0);   // (bounds what is in flight at a time)
            });
            if (DECAY) {   // the state before the chunk, at query n
                const float g_q = lds.power[n + 1];
                for_n<2>([&](auto c) { Y[c.value] *= g_q; });
                dsum *= g_q;
            }
            dsum = add_halves(dsum);
            if (g == 0) lds.den[w][n] = dsum;
            put_partial(Y);
            fresh_lane();
            __builtin_amdgcn_sched_barrier(0);
            update(rows, t, uncut);
        };
        for (int t = 0; t < chunks; ++t) {
            if (DECAY && gm != 1.f) wide = wide || state_outside();
            if (__builtin_expect(is_wide(t), 0)) chunk(t, std::true_type{});
            else chunk(t, std::false_type{});
            next_chunk(t);
        }
        if (writes_state) put_image();
    } else if (w == TILES) {
        role_guard();
        for (int t = 0; t < chunks; ++t) {
            const int tok0 = begin + C * t;
            fresh_lane();
            const bool uncut = is_wide(t);
            f32x16 Y[2];
            for_n<2>([&](auto c) { Y[c.value] = zero16(); });
            // P^T: register r is key 8 (r / 4) + 4 g + r % 4, lane n the query
            f32x16 P;
            {
                auto key = [&](int i) { return rows.kt[8 * g + i][n]; };
                const f32x4 q0 = *reinterpret_cast<const f32x4 *>(&rows.q[n][8 * g]), q1 = *reinterpret_cast<const f32x4 *>(&rows.q[n][8 * g + 4]);
                auto query = [&](int i) { return i < 4 ? q0[i & 3] : q1[i & 3]; };
                P = zero16();
                if (__builtin_expect(uncut, 0)) mfma_f32(key, query, P);
                else mfma6(split8(key), split8(query), P);
            }
            float dsum = 0.f;
            for_n<16>([&](auto r) {
                const int key = 8 * (r.value >> 2) + 4 * g + (r.value & 3);
                const float x = P[r.value];
                float p = fmaf(x, fmaf(x, 0.5f, 1.f), 1.f);
                if (DECAY) p *= lds.power[max(n - key, 0)];
                P[r.value] = key <= n ? p : 0.f;
                dsum += P[r.value];
            });
            dsum = add_halves(dsum);
            if (g == 0) lds.den[w][n] = dsum;
            // A key that a query cannot see stands in the product as 0 V, which is not 0 where V is not finite: a chunk with such a value is
            // summed key by key, V from memory, without the hidden ones.
            if (__builtin_expect(!uncut, 1)) {
                for_n<2>([&](auto s) {
                    const Parts op = split8([&](int i) { return P[8 * s.value + i]; });
                    for_n<2>([&](auto c) { mfma6(v_parts(rows, s.value, c.value), op, Y[c.value]); });
                });
            } else if (__builtin_amdgcn_readfirstlane(lds.bad[t & 1]) != t + 1) {
                for_n<4>([&](auto sc) {
                    constexpr int s = sc.value / 2, c = sc.value % 2;
                    const f32x8 x = read_v_f32(tok0, s, c);
                    mfma_f32([&](int i) { return x[i]; }, [&](int i) { return P[8 * s + i]; }, Y[c]);
                });
            } else {
                float *pb = &lds.x[w][0][0][0][0];   // P^T [key][query] (this wave's own partial outputs come here afterwards)
                for_n<16>([&](auto r) { pb[32 * (8 * (r.value >> 2) + 4 * g + (r.value & 3)) + n] = P[r.value]; });
                __builtin_amdgcn_wave_barrier();
#pragma unroll 1
                for (int key = 0; key < min(C, end - tok0); ++key) {
                    const float p = pb[32 * key + n];
                    const float *row = vu + (size_t)(tok0 + key) * DV + 4 * g;
                    for_n<8>([&](auto cj) {
                        const f32x4 x = *reinterpret_cast<const f32x4 *>(row + 8 * cj.value);
                        for_n<4>([&](auto i) {
                            float &o = reinterpret_cast<float *>(&Y[cj.value / 4])[4 * (cj.value % 4) + i.value];
                            if (key <= n) o = fmaf(p, x[i.value], o);
                        });
                    });
                }
                __builtin_amdgcn_wave_barrier();
            }
            put_partial(Y);
            next_chunk(t);
        }
    } else {
        for (int t = 0; t < chunks; ++t) next_chunk(t);
    }
    if (writes_state) export_image();
}

inline int segment_len(int N, int G) { return ((N + G - 1) / G + C - 1) / C * C; }

// Segments of at least 64 tokens, at most 64 of them, in one round of the chip.  Two workgroups to a CU take 1.35 times as long for a token of theirs as one does
// (0.235 us for a token of a segment, its increment included, against 0.174) and have twice the entries to sum, about 1 us for each of the first 16 more.  So
// one to a CU while its segments (rounded up to chunks) have up to 15 tokens for an entry more.  (us, d_v 64, one and two to a CU: 16 units N 2048 38.1, 46.8, N 6000 81.2, 75.8; 8
// units N 2048 30.6 with one, there are no more segments, N 6000 51.8, 58.5; 32 units N 777 32.6, 32.4, N 2048 58.9, 54.1, N 6000 144.8, 113.6; 64 units N 777 49.0, 43.4, N 2048
// 101.6, 80.9.)  But not where rounding makes it leave a fifth of the CUs idle and hardly a CU would get two: 24 units N 974, 8 segments of 128 tokens and 11 of 96, 32.8, 29.0.
inline int segments(int U, int N, int dv)
{
    const long groups = (long)U * (dv / COLS);
    struct Cut { int G, len; long workgroups; };
    auto cut = [&](long G) {
        if (G > N / 64) G = N / 64;
        if (G > kMaxSegments) G = kMaxSegments;
        if (G < 1) G = 1;
        const int len = segment_len(N, (int)G);
        return Cut{(int)G, len, groups * ((N + len - 1) / len)};
    };
    const long one = 256 / groups, more = one < 16 ? one : 16;
    const Cut few = cut(one), many = cut(512 / groups);
    const bool idle = few.workgroups <= 208 && many.workgroups <= 288 && many.len < few.len;
    return few.len <= 15 * more && !idle ? few.G : many.G;
}

template <int DV, bool DECAY>
hipError_t launch(const void *q, const void *k, const void *v, void *y, float *state, int has_init, void *workspace, int U, int N,
                  DecayArg dec, hipStream_t s)
{
    constexpr int SL = DV / COLS;
    int G = segments(U, N, DV);
    const int len = segment_len(N, G);
    while (G > 1 && (G - 1) * len >= N) --G;   // rounding the length up can empty trailing segments
    if ((long long)U * SL * G >= (1ll << 31)) return hipErrorInvalidValue;
    // (the workspace is sized for the fp32 matrix kernel, which has at least as many segments and entries of this size)
    const size_t room = prefill_f32_workspace_bytes(U, N, DP, DV) / (sizeof(float) * kEntryFloats * U * SL);   // entries
    if (G > 1 && (size_t)G > room) return hipErrorInvalidValue;
    // Shares of the increments: G, where what would be idle is worth the entries that come on top, which take time to write and to sum: two or three
    // segments of 256 tokens or more, four of 1024 (more segments leave little idle), and where the workspace holds two entries a segment.
    // (us, inputs from memory, G - 1 shares and G: 200 units of 400 tokens 60.5, 58.9, of 512 71.1, 69.1, of 768 98.8, 94.7, of 2048 238, 222; 256 of 449 68.8, 67.1, of
    // 512 73.2, 72.5; from a state 200 of 400 65.1, 66.5; 150 of 449 53.3, 54.6, of 700 72.0, 70.5, of 2048 174.7, 165.8; 170 of 768 76.9, 76.8; 128 of 1500 106.9,
    // 106.3, of 2048 142.3, 141.1, on another GPU 144.7, 147.6, of 4100 275.0, 270.3; 110 of 2048 136.2, 131.9.)
    // With G chunks or more to a segment no share ends with a segment but the last: the i-th ends less than i chunks past i - i / G segments.
    int inc_len = len, entries = G;
    const int share = ((G - 1) * (len / C) + G - 1) / G * C, share_entries = 2 * (G - 1) + (has_init & 1);
    const bool shared = !DECAY && G > 1 && G <= 4 && len >= (G < 4 ? 256 : 1024) && (size_t)share_entries <= room;
    if (shared) {
        inc_len = share;
        entries = share_entries;
    }
    const int shares = ((G - 1) * len + inc_len - 1) / inc_len;
    float *ws = static_cast<float *>(workspace);
    auto go = [&](auto increment, int first_slice, int slices) {
        constexpr bool INC = decltype(increment)::value;
        const int parts = INC ? shares : G, all = U * slices, local = all / 8 * 8;
        const dim3 grid = local ? dim3((unsigned)(all * parts)) : dim3(parts, all);
        if constexpr (!DECAY) {
            if (shared) {
                hipLaunchKernelGGL((prefill_kernel<DV, INC, false, true>), grid, dim3(NT), 0, s, (const float *)q, (const float *)k, (const float *)v,
                                   (float *)y, state, has_init, N, ws, len, inc_len, shares, G, entries, first_slice, slices, local, dec);
                return hipGetLastError();
            }
        }
        hipLaunchKernelGGL((prefill_kernel<DV, INC, DECAY, false>), grid, dim3(NT), 0, s, (const float *)q, (const float *)k, (const float *)v, (float *)y,
                           state, has_init, N, ws, len, inc_len, shares, G, entries, first_slice, slices, local, dec);
        return hipGetLastError();
    };
    hipError_t e = hipSuccess;
    if (G > 1) {
        e = go(std::true_type{}, 0, SL);
    } else if ((has_init & 1) && SL > 1) {
        // every slice reads the caller's K-state and the first one overwrites it: the others go before it
        e = go(std::false_type{}, 1, SL - 1);
        return e == hipSuccess ? go(std::false_type{}, 0, 1) : e;
    }
    return e == hipSuccess ? go(std::false_type{}, 0, SL) : e;
}

}  // namespace f32x3

// Up to 48 tokens the fp32 matrix kernel's shorter chunks of 16 are faster.  (us there and here, 1 to 512 units, d_v 64 and 128, with and
// without an initial state: 16 tokens 7.2 to 43 and 8.0 to 46, 40 tokens 12.3 to 59 and 11.3 to 57 but 25 to 28 at worst, 64 tokens
// 15 to 68 and 12 to 59.)
bool prefill_f32x3_supported(int dp, int dtype, int N) { return dtype == BASED_F32 && dp == f32x3::DP && N > 48; }

hipError_t launch_prefill_f32x3(const void *q, const void *k, const void *v, void *y, float *state, int has_init, void *workspace,
                                const float *gamma, const void *gate, int H, int U, int N, int dv, hipStream_t s)
{
    const f32x3::DecayArg dec{gamma, static_cast<const float *>(gate), H};
#define F32X3_LAUNCH(DV, DECAY) f32x3::launch<DV, DECAY>(q, k, v, y, state, has_init, workspace, U, N, dec, s)
    if (gamma || gate) return dv == 64 ? F32X3_LAUNCH(64, true) : F32X3_LAUNCH(128, true);
    return dv == 64 ? F32X3_LAUNCH(64, false) : F32X3_LAUNCH(128, false);
#undef F32X3_LAUNCH
}

}  // namespace based
