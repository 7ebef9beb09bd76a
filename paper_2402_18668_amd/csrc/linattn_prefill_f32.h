// Causal Taylor linear attention, chunked prefill on the fp32 matrix instructions: fp32 inputs at every supported d' (at d' = 16
// calls of up to 48 tokens: linattn_prefill_f32x3.hip has the others), bf16 inputs at the d' that have no bf16 matrix-core
// kernel (8, 24), and the decay variant of both and of every bf16 call.  Every product and sum is fp32.
//
// Chunked form of Sec. 4 with chunks of 16 tokens: inside a chunk the masked quadratic product P = 1 + A + A^2/2,
// A = Q K^T; across chunks the running KV-state S (Eq. 3), read out with phi(Q) and updated with phi(K)^T V.
//
// State rows.  One row per unordered feature pair.  d' is cut into blocks of four; the pair block (A, B), A <= B, is one
// tile of 16 rows: row 4 i + j stands for the pair (4 A + i, 4 B + j).  In a diagonal block the rows with j < i
// would repeat others, and carry the linear rows and the constant row instead (rows (1,0), (2,1), (3,2), (3,0) of
// block A: features 4 A, 4 A + 1, 4 A + 2, 4 A + 3; row (2,0) of block 0: the constant; the rest is zero).  So the
// whole state is nb (nb + 1) / 2 tiles, nb = d' / 4: 160 rows at d' = 16 for the 153 that are needed.  A row holds the
// plain sum of k_a k_b v; the readout weighs q_a q_b with 1, and with 1/2 for a = b (Eq. 4's 1/sqrt(2) on either side).
//
// Registers.  One wave owns 16 columns of d_v and all state rows for them, in accumulators of the 16x16x4 instruction
// (lane = 16 g + n; accumulator register r: row 4 g + r, column n; A operand: row n, k-slot g; B operand: column n,
// k-slot g).  With contraction step r / s visiting index 4 g + r / 4 g + s in k-slot g, everything is register-local:
//   readout  Y^T += S^T phi(Q)^T:   A = state register r as it stands, B = q[4 A + g] q[4 B + r] of the lane's query n
//   P^T      = K Q^T:               A = k_n[4 A + g], B = q_n[4 A + g]
//   intra    Y^T += V^T P^T:        A = V[4 g + s][n], B = P register s as it stands
//   update   S += phi(K)^T V:       A = k[4 A + n / 4] k[4 B + n % 4] of token 4 g + s, B = V[4 g + s][n]
// One multiply feeds one matrix instruction of 32 cycles: the kernel is bound by the matrix pipe (fp32: 157 TFLOP/s).
//
// Work split: a workgroup is four waves, one (unit, slice of 64 columns, segment).  They share the staged K^T and Q^T rows
// (64 tokens at a time, two generations) and the denominator: wave w keeps the K-state z of the tiles t = w mod 4 and
// adds up their share of phi(q).z; the shares meet in LDS at the one barrier of a chunk.
//
// Long sequences / few units: G segments; a first launch computes the segments' increments (update only) and the main
// launch starts segment g from the sum of the entries before it.
//
// Decay (appendix paragraph on decay: a fixed rate gamma per head multiplies the state at every token, an optional gate
// scales the rows of y): key j enters row i with gamma^(i - j), so inside a chunk P is weighed with that, the readout of
// the state before the chunk with gamma^(n + 1), and the state becomes gamma^16 S + sum_t gamma^(15 - t) phi(k_t) v_t^T.
// The factors are constants of the lane, multiplied in under a uniform branch; with gamma = 1 they change no bit.
//
// Values that are not finite.  One in V reaches its own column from its own token on and nothing else; one in K every later token of
// the unit, one in Q its own token.  What they make of the results they reach (Inf or NaN) is not specified: the zero rows of
// the diagonal tiles turn an infinite sum into NaN.
//
// Measured (B 8, H 16, N 2048, d' 16, d_v 64, fp32, a call that linattn_prefill_f32x3.hip has now): 1230 us on vector instructions (273
// unpacked rows, two fused multiply-adds per row and token) -> 193.  The fp32 matrix instructions occupy the vector ALU: per wave and chunk 2816 cycles of them
// and 1640 of vector instructions add up to 4456 of 5555.
#pragma once
#include "common.h"

#include <type_traits>
#include <utility>

namespace based {

namespace pf32 {

typedef float f32x4 __attribute__((ext_vector_type(4)));

constexpr int C = 16;           // tokens per chunk
constexpr int STAGE = 64;       // tokens staged at a time
constexpr int LD = STAGE + 4;   // floats per staged row
constexpr int NW = 4;           // waves of a workgroup: 16 columns each
constexpr int COLS = 16 * NW;
constexpr int kMaxSegments = 64;

__host__ __device__ constexpr int blocks(int dp) { return dp / 4; }
__host__ __device__ constexpr int tiles(int dp) { return blocks(dp) * (blocks(dp) + 1) / 2; }
// tiles of the state that pass through LDS together on their way from and to the state buffer, and the floats of their rows there
__host__ __device__ constexpr int image_tiles(int dp) { return dp == 32 ? 12 : dp == 24 ? 7 : dp == 16 ? 5 : 3; }
constexpr int IMG_LD = COLS + 4;
// of these, tiles whose loads from the state buffer are in flight together
__host__ __device__ constexpr int image_unroll(int dp) { return dp == 32 ? 4 : image_tiles(dp); }
// Workspace entry of one (unit, slice, segment): per wave the tiles' accumulators [tile][lane][4], then z [tile][16].
__host__ __device__ constexpr size_t entry_floats(int dp) { return (size_t)tiles(dp) * (NW * 256 + 16); }

template <typename F, int... I> __device__ __forceinline__ void for_seq(F &&f, std::integer_sequence<int, I...>)
{
    (f(std::integral_constant<int, I>{}), ...);
}
template <int N, typename F> __device__ __forceinline__ void for_n(F &&f) { for_seq(f, std::make_integer_sequence<int, N>{}); }

// f(t, A, B) for every tile, arguments constant
template <int NB, typename F> __device__ __forceinline__ void for_tiles(F &&f)
{
    for_n<NB>([&](auto Ac) {
        constexpr int A = decltype(Ac)::value;
        for_n<NB - A>([&](auto Dc) {
            constexpr int B = A + decltype(Dc)::value;
            f(std::integral_constant<int, A * NB - A * (A - 1) / 2 + (B - A)>{}, std::integral_constant<int, A>{},
              std::integral_constant<int, B>{});
        });
    });
}

__device__ __forceinline__ f32x4 mfma(float a, float b, f32x4 c) { return __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, 0, 0, 0); }
__device__ __forceinline__ f32x4 zero4() { return f32x4{0.f, 0.f, 0.f, 0.f}; }

// Row (i, j) of a diagonal tile is s1 s2 with s1 = m x_i + c and s2 = x_j, or 1 for i >= 2, j = 0.
struct DiagRow { float m, c; bool one; };
__device__ __forceinline__ DiagRow diag_row(int i, int j, float w_eq)   // w_eq: weight of the rows (i, i)
{
    if (j >= i) return {i == j ? w_eq : 1.f, 0.f, false};
    if (i == j + 1) return {0.f, 1.f, false};                    // (1,0), (2,1), (3,2): linear, j
    if (i == 3 && j == 0) return {1.f, 0.f, true};               // linear, 3
    return {0.f, 0.f, i == 2};                                   // (2,0): the constant (block 0 adds c = 1); (3,1): zero
}

// Canonical rows (Eq. 4 order) of row (i, j) of tile (A, B), and what a stored value is multiplied by to give the canonical
// one; r1 < 0: a zero row.
struct Canon { int r1, r2; float scale; };
template <int DP> __device__ __forceinline__ Canon canon(int A, int B, int i, int j)
{
    const int a = 4 * A + i, b = 4 * B + j;
    if (A != B || j >= i) return {1 + DP + a * DP + b, 1 + DP + b * DP + a, kRsqrt2};
    if (i == j + 1) return {1 + b, 1 + b, 1.f};
    if (i == 3 && j == 0) return {1 + a, 1 + a, 1.f};
    if (A == 0 && i == 2) return {0, 0, 1.f};
    return {-1, -1, 0.f};
}

// Workgroups (waves per SIMD) resident on a CU, as the state's registers allow.
__host__ __device__ constexpr int resident(int dp) { return dp == 32 ? 1 : dp == 24 ? 2 : dp == 16 ? 3 : 4; }

struct DecayArg {
    const float *gamma;   // [H], device; null: no decay
    const void *gate;     // [B][N][H] in the dtype of y, device; null: none
    int H;
};

// fp32 calls come here at d' = 16 up to 48 tokens only: one segment.
template <int DP, typename T> constexpr bool HAS_SEGMENTS = DP != 16 || !std::is_same<T, float>::value;

// The launch covers `slices` slices of 64 columns from first_slice on.
// has_init: bit 0 an initial state is given, bit 2 the outputs are the numerators alone.
// A unit's slice has G entries, those of the segments before a segment end with first + seg * pieces - 1.
// INCREMENT: state increment of the segment (or piece; of the first segment's two, the first one is the longer) only, written to entry first + seg (segment 0 also converts the caller's state
// into entry 0: the main launch overwrites that buffer while other segments may still be starting).
template <int DP, int DV, typename T, bool INCREMENT>
__global__ __launch_bounds__(64 * NW, resident(DP)) void prefill_kernel(const T *__restrict__ q, const T *__restrict__ k,
                                                           const T *__restrict__ v, T *__restrict__ y, float *state,
                                                           int has_init, int N, float *ws, int seg_len, int G, int first, int pieces,
                                                           int first_slice, int slices, int local, DecayArg dec)
{
    constexpr int NB = blocks(DP), NT = tiles(DP), SL = DV / COLS, D = feature_dim(DP);
    constexpr int ZS = (NT + NW - 1) / NW;   // K-state tiles of a wave
    constexpr int IT = image_tiles(DP), IU = image_unroll(DP);
    static_assert(NT % IT == 0 && IT % IU == 0, "");
    struct Rows { float kt[2][DP][LD], qt[2][INCREMENT ? 1 : DP][LD]; };
    __shared__ __align__(16) union { Rows rows; float image[IT][16][IMG_LD]; } lds;
    auto &kt = lds.rows.kt;
    auto &qt = lds.rows.qt;
    __shared__ __align__(16) float zl[NW][ZS][16];
    __shared__ float den[2][NW][16];

    const bool numerator_only = (has_init & 4) != 0, init = (has_init & 1) != 0;
    const int gseg = INCREMENT ? (G - 1) * pieces : G;
    // The workgroups of a unit's slice run on one XCD (workgroup index mod 8), whose L2 then holds the entries that they write and sum, for the first `local`
    // slices, a multiple of 8; the rest's run on all XCDs.  (All on all XCDs, and this, us: fp32, 16 units, d' 32 N 777 110.7, 95.2, d' 8 N 1000 20.9,
    // 18.3; bf16, d' 24 16 units N 2048 141.2, 132.5, d' 8 33 units N 4096 66.3, 59.4.)  Fewer than 8 slices have a row of the grid each: dealt out with them
    // 7 units of 500 tokens, d' 8, bf16, took 18.0 us instead of 17.7, one of 16 4.91 instead of 4.78.
    int seg = blockIdx.x, us = blockIdx.y;
    if (local > 0) {
        const uint32_t bid = blockIdx.x, here = local * gseg;
        const bool on_one = bid < here;
        const uint32_t idx = on_one ? bid / 8 : bid - here, at = idx / (uint32_t)gseg;
        seg = idx - at * gseg;
        us = on_one ? at * 8 + bid % 8 : local + at;
    }
    const int u = slices == 1 ? us : (uint32_t)us / SL, slice = first_slice + (slices == 1 ? 0 : (uint32_t)us % SL), col0 = slice * COLS;   // (slices: 1 or SL)
    const int tid = threadIdx.x, w = __builtin_amdgcn_readfirstlane(tid >> 6), lane = tid & 63, g = lane >> 4, n = lane & 15;
    const int len = INCREMENT && pieces == 2 ? (seg_len + 2 * C - 1) / (2 * C) * C : seg_len;
    const int begin = seg * len, end = min(INCREMENT ? (G - 1) * seg_len : N, begin + len);

    const T *qu = q + (size_t)u * N * DP, *ku = k + (size_t)u * N * DP;
    const T *vu = v + (size_t)u * N * DV + col0 + 16 * w + n;
    T *yu = y + (size_t)u * N * DV + col0 + 16 * w;
    float *Su = state ? state + (size_t)u * state_stride(DP, DV) + col0 : nullptr;
    float *zu = state ? state + (size_t)u * state_stride(DP, DV) + (size_t)D * DV : nullptr;
    float *entries = ws ? ws + ((size_t)u * SL + slice) * G * entry_floats(DP) : nullptr;
    auto entry_s = [&](int e) { return entries + (size_t)e * entry_floats(DP) + (size_t)w * NT * 256 + 4 * lane; };
    auto entry_z = [&](int e) { return entries + (size_t)e * entry_floats(DP) + (size_t)NW * NT * 256; };

    const bool decay = dec.gamma != nullptr;
    const float gm = decay ? dec.gamma[u % dec.H] : 1.f;
    const T *gate = dec.gate ? static_cast<const T *>(dec.gate) + (size_t)(u / dec.H) * N * dec.H + u % dec.H : nullptr;
    // decay factors of this lane: of the state before a chunk at query n, of key 4 g + r at query n, of token 4 g + s and of the
    // old state in the state after the chunk (m tokens in it)
    const float g_seg = decay ? powf(gm, (float)seg_len) : 1.f;
    float g_q = 1.f, g_p[4] = {1.f, 1.f, 1.f, 1.f}, g_v[4] = {1.f, 1.f, 1.f, 1.f}, g_s = 1.f;
    auto set_update_factors = [&](int m) {
        g_s = powf(gm, (float)m);
        for_n<4>([&](auto s) { g_v[s.value] = powf(gm, (float)max(m - 1 - 4 * g - s.value, 0)); });
    };
    if (decay) {
        g_q = powf(gm, (float)(n + 1));
        for_n<4>([&](auto r) { g_p[r.value] = powf(gm, (float)max(n - 4 * g - r.value, 0)); });
        set_update_factors(C);
    }

    f32x4 S[NT];
    float z[ZS];   // lane n (any g): row n of tile ZS-th tile w, w + NW, ..
    for_n<NT>([&](auto t) { S[t.value] = zero4(); });
    for_n<ZS>([&](auto i) { z[i.value] = 0.f; });
    // The state buffer moves through LDS, some tiles at a time: a wave reaches its registers' places there at constant offsets, and
    // the workgroup moves 16-byte pieces of rows in short loops: thread (w, j, c) row (w, j) of a tile, columns 4 c .. 4 c + 3.  (Element
    // by element from the registers it was unrolled code, which a short call runs once and waits for while it is fetched: 64 units
    // from a state, d' 32, d_v 64, 1 token 52 -> 31 us; d' 24, d_v 128, 16 tokens 62 -> 34.)
    const int s_j = lane >> 4, s_c = 4 * (lane & 15);
    auto next_tile = [](int &A, int &B) {
        if (++B == NB) B = ++A;
    };
    auto z_canon = [&](int p) {   // row p of the K-state's tiles
        int A = 0, B = p >> 4;
        while (B >= NB - A) B -= NB - A++;
        return canon<DP>(A, A + B, (p >> 2) & 3, p & 3);
    };
    // the caller's state, symmetric part, into S and z
    auto import_state = [&]() {
        for (int p = tid; p < 16 * NT; p += 64 * NW) {
            const Canon c = z_canon(p);
            zl[(p >> 4) % NW][(p >> 4) / NW][p & 15] = c.r1 < 0 ? 0.f : (0.5f / c.scale) * (zu[c.r1] + zu[c.r2]);
        }
        int A = 0, B = 0;
        for_n<NT / IT>([&](auto part) {
#pragma unroll 1
            for (int i0 = 0; i0 < IT; i0 += IU) {
                f32x4 x[IU][2];
                float scale[IU];
                for_n<IU>([&](auto i) {
                    const Canon c = canon<DP>(A, B, w, s_j);
                    x[i.value][0] = *reinterpret_cast<const f32x4 *>(Su + (size_t)max(c.r1, 0) * DV + s_c);
                    x[i.value][1] = *reinterpret_cast<const f32x4 *>(Su + (size_t)max(c.r2, 0) * DV + s_c);
                    scale[i.value] = c.r1 < 0 ? 0.f : 0.5f / c.scale;
                    next_tile(A, B);
                });
                for_n<IU>([&](auto i) {
                    const f32x4 sum = (x[i.value][0] + x[i.value][1]) * scale[i.value];
                    *reinterpret_cast<f32x4 *>(&lds.image[i0 + i.value][4 * w + s_j][s_c]) = scale[i.value] == 0.f ? zero4() : sum;
                });
            }
            __syncthreads();
            for_n<IT>([&](auto i) {
                for_n<4>([&](auto r) { S[part.value * IT + i.value][r.value] = lds.image[i.value][4 * g + r.value][16 * w + n]; });
            });
            __syncthreads();
        });
        for_n<ZS>([&](auto i) { z[i.value] = NW * i.value + w < NT ? zl[w][i.value][n] : 0.f; });
    };
    // Both rows of a pair.  A state that is not symmetric (none of this recurrence is) keeps its antisymmetric part, which
    // decays like the rest: nothing is added to it, so over the N tokens of the call by gamma^N.
    auto export_state = [&]() {
        const float g_all = decay ? powf(gm, (float)N) : 1.f;
        auto half_difference = [&](float a, float b) { return a == b ? 0.f : 0.5f * (a - b) * g_all; };   // (equal infinities: none)
        int A = 0, B = 0;
        for_n<NT / IT>([&](auto part) {
            for_n<IT>([&](auto i) {
                for_n<4>([&](auto r) { lds.image[i.value][4 * g + r.value][16 * w + n] = S[part.value * IT + i.value][r.value]; });
            });
            __syncthreads();
#pragma unroll 1
            for (int i0 = 0; i0 < IT; i0 += IU) {
                f32x4 d[IU];
                float *p[IU][2];
                float scale[IU];
                for_n<IU>([&](auto i) {
                    const Canon c = canon<DP>(A, B, w, s_j);
                    p[i.value][0] = Su + (size_t)max(c.r1, 0) * DV + s_c;
                    p[i.value][1] = Su + (size_t)max(c.r2, 0) * DV + s_c;
                    scale[i.value] = c.r1 < 0 ? 0.f : c.scale;
                    d[i.value] = zero4();
                    next_tile(A, B);
                });
                if (init)
                    for_n<IU>([&](auto i) {
                        const f32x4 x1 = *reinterpret_cast<const f32x4 *>(p[i.value][0]), x2 = *reinterpret_cast<const f32x4 *>(p[i.value][1]);
                        for_n<4>([&](auto k) { d[i.value][k.value] = half_difference(x1[k.value], x2[k.value]); });
                    });
                for_n<IU>([&](auto i) {
                    if (scale[i.value] == 0.f) return;   // (a zero row; a row of its own is written twice)
                    const f32x4 x = *reinterpret_cast<const f32x4 *>(&lds.image[i0 + i.value][4 * w + s_j][s_c]) * scale[i.value];
                    *reinterpret_cast<f32x4 *>(p[i.value][0]) = x + d[i.value];
                    *reinterpret_cast<f32x4 *>(p[i.value][1]) = x - d[i.value];
                });
            }
            __syncthreads();
        });
        if (col0 != 0) return;
        for_n<ZS>([&](auto i) {
            if (g == 0) zl[w][i.value][n] = z[i.value];
        });
        __syncthreads();
        for (int p = tid; p < 16 * NT; p += 64 * NW) {
            const Canon c = z_canon(p);
            if (c.r1 < 0) continue;
            const float s = zl[(p >> 4) % NW][(p >> 4) / NW][p & 15] * c.scale, d = init ? half_difference(zu[c.r1], zu[c.r2]) : 0.f;
            zu[c.r1] = s + d;
            if (c.r2 != c.r1) zu[c.r2] = s - d;
        }
    };
    auto store_entry = [&](int e) {
        float *p = entry_s(e), *pz = entry_z(e);
        for_n<NT>([&](auto t) {
            *reinterpret_cast<f32x4 *>(p + (size_t)t.value * 256) = S[t.value];
            if (t.value % NW == w && g == 0) pz[16 * t.value + n] = z[t.value / NW];
        });
    };
    if (INCREMENT) {
        if (init && seg == 0) {
            import_state();
            store_entry(0);
            for_n<NT>([&](auto t) { S[t.value] = zero4(); });
            for_n<ZS>([&](auto i) { z[i.value] = 0.f; });
        }
    } else if (HAS_SEGMENTS<DP, T> && G > 1) {
        // the sum of the entries before the segment (up to 64 of them), some at a time with their loads in flight together
        constexpr int EB = NT <= 3 ? 8 : NT <= 10 ? 4 : 1;
        int e = init ? 0 : first;
        const int last = first + seg * pieces;
        auto add_entries = [&](auto count) {
            constexpr int n_e = decltype(count)::value;
            f32x4 x[n_e][NT];
            float xz[n_e][ZS];
            for_n<n_e>([&](auto i) {
                const float *p = entry_s(e + i.value), *pz = entry_z(e + i.value);
                for_n<NT>([&](auto t) { x[i.value][t.value] = *reinterpret_cast<const f32x4 *>(p + (size_t)t.value * 256); });
                for_n<ZS>([&](auto j) { xz[i.value][j.value] = NW * j.value + w < NT ? pz[16 * (NW * j.value + w) + n] : 0.f; });
            });
            for_n<n_e>([&](auto i) {
                for_n<NT>([&](auto t) { S[t.value] = S[t.value] * g_seg + x[i.value][t.value]; });
                for_n<ZS>([&](auto j) { z[j.value] = z[j.value] * g_seg + xz[i.value][j.value]; });
            });
            e += n_e;
        };
        if constexpr (EB == 1) {
            for (; e < last; ++e) {
                const float *p = entry_s(e), *pz = entry_z(e);
                for_n<NT>([&](auto t) {
                    S[t.value] = S[t.value] * g_seg + *reinterpret_cast<const f32x4 *>(p + (size_t)t.value * 256);
                    if (t.value % NW == w) z[t.value / NW] = z[t.value / NW] * g_seg + pz[16 * t.value + n];
                    if constexpr (t.value % 8 == 7) __builtin_amdgcn_sched_barrier(0);
                });
            }
        } else {
            for (int rest = (last - e) % EB; rest > 0; --rest) add_entries(std::integral_constant<int, 1>{});
            while (e < last) add_entries(std::integral_constant<int, EB>{});
        }
    } else if (init) {
        import_state();
    }

    // this lane's rows of the diagonal tiles: query side (i = g, j = r) and key side (i = n / 4, j = n % 4)
    DiagRow dq[4];
    for_n<4>([&](auto r) { dq[r.value] = diag_row(g, r.value, 0.5f); });
    const DiagRow dk = diag_row(n >> 2, n & 3, 1.f);
    const float q_const = g == 2 ? 1.f : 0.f, k_const = n == 8 ? 1.f : 0.f;   // the constant row of block 0: (2, 0)

    // ---- staging: 64 tokens of K (and Q) into registers, then transposed into LDS ----------------------------
    constexpr int PT = STAGE * DP / (64 * NW);   // elements of a tensor per thread: token tid % 64, features (tid / 64) PT ..
    static_assert(DP % PT == 0 && PT >= 1, "");
    float rk[PT], rq[PT];
    const int s_tok = tid & 63, s_f = (tid >> 6) * PT;
    auto load_stage = [&](int tok0) {
        const int tok = min(tok0 + s_tok, end - 1);
        for_n<PT>([&](auto i) {
            rk[i.value] = to_f32(ku[(size_t)tok * DP + s_f + i.value]);
            if (!INCREMENT) rq[i.value] = to_f32(qu[(size_t)tok * DP + s_f + i.value]);
        });
    };
    auto store_stage = [&](int tok0, int b) {
        const bool ok = tok0 + s_tok < end;   // tokens past the end must not touch the state
        for_n<PT>([&](auto i) {
            kt[b][s_f + i.value][s_tok] = ok ? rk[i.value] : 0.f;
            if constexpr (!INCREMENT) qt[b][s_f + i.value][s_tok] = rq[i.value];
        });
    };
    float vr[4];   // V[4 g + s][16 w + n] of the chunk
    auto load_v = [&](int tok0, float (&dst)[4]) {
        for_n<4>([&](auto s) {
            const int tok = tok0 + 4 * g + s.value;
            const float x = to_f32(vu[(size_t)min(tok, end - 1) * DV]);
            dst[s.value] = tok < end ? x : 0.f;
        });
    };

    load_stage(begin);
    store_stage(begin, 0);
    load_v(begin, vr);
    __syncthreads();
    const int chunks = (end - begin + C - 1) / C;
    for (int c = 0; c < chunks; ++c) {
        const int tok0 = begin + C * c, b = (c >> 2) & 1, sub = (c & 3) * C;   // four chunks to a stage
        if ((c & 3) == 0 && c + 4 < chunks) load_stage(tok0 + STAGE);
        float vn[4];
        load_v(min(tok0 + C, end - 1), vn);
        f32x4 Y = zero4();
        if constexpr (!INCREMENT) {
            float qv[DP], qa[NB], kr[NB];
            for_n<NB>([&](auto A) {
                qa[A.value] = qt[b][4 * A.value + g][sub + n];
                kr[A.value] = kt[b][4 * A.value + g][sub + n];
            });
            for_n<DP>([&](auto i) { qv[i.value] = qt[b][i.value][sub + n]; });
            // P^T: register r is key 4 g + r, column = query n; cut by the diagonal
            f32x4 P = zero4();
            for_n<NB>([&](auto A) { P = mfma(kr[A.value], qa[A.value], P); });
            // the K-state of this wave's tiles, [tile][row], for the lanes' rows 4 g + r
            if (g == 0)
                for_n<ZS>([&](auto i) { zl[w][i.value][n] = z[i.value]; });
            float dsum = 0.f;
            __builtin_amdgcn_wave_barrier();
            f32x4 Y2 = zero4();   // two chains, so that a matrix instruction does not wait for the one before it
            for_tiles<NB>([&](auto t, auto A, auto B) {
                float f[4];
                for_n<4>([&](auto r) {
                    if constexpr (A.value == B.value) {
                        const DiagRow &d = dq[r.value];
                        const float s1 = fmaf(qa[A.value], d.m, A.value == 0 && r.value == 0 ? d.c + q_const : d.c);
                        f[r.value] = s1 * (r.value == 0 && d.one ? 1.f : qv[4 * A.value + r.value]);
                    } else {
                        f[r.value] = qa[A.value] * qv[4 * B.value + r.value];
                    }
                    if (r.value & 1) Y2 = mfma(S[t.value][r.value], f[r.value], Y2);
                    else Y = mfma(S[t.value][r.value], f[r.value], Y);
                });
                if (t.value % NW == w) {
                    const f32x4 zv = *reinterpret_cast<const f32x4 *>(&zl[w][t.value / NW][4 * g]);
                    for_n<4>([&](auto r) { dsum = fmaf(f[r.value], zv[r.value], dsum); });
                }
                if constexpr (B.value == NB - 1) __builtin_amdgcn_sched_barrier(0);   // (bounds what is in flight at a time)
            });
            if (decay) {
                Y *= g_q;
                Y2 *= g_q;
                dsum *= g_q;
            }
            for_n<4>([&](auto r) {
                const float x = P[r.value];
                float p = fmaf(x, fmaf(x, 0.5f, 1.f), 1.f);
                if (decay) p *= g_p[r.value];
                P[r.value] = 4 * g + r.value <= n ? p : 0.f;
                if (w == 0) dsum += P[r.value];
            });
            // A key that a query cannot see stands in the product as 0 V, which is not 0 where V is not finite: a block with such a
            // value is summed key by key, without the hidden ones.
            const float probe = fmaf(0.f, vr[0], fmaf(0.f, vr[1], fmaf(0.f, vr[2], 0.f * vr[3])));
            if (__builtin_expect(__builtin_amdgcn_ballot_w64(probe != 0.f) == 0, 1)) {
                for_n<4>([&](auto s) {
                    if (s.value & 1) Y2 = mfma(vr[s.value], P[s.value], Y2);
                    else Y = mfma(vr[s.value], P[s.value], Y);
                });
            } else {
#pragma unroll 1
                for (int j = 0; j < 4; ++j)
                    for_n<4>([&](auto s) {
                        const float p = __shfl(P[s.value], 16 * j + n, 64);
                        for_n<4>([&](auto r) {
                            const float x = __shfl(vr[s.value], 16 * j + 4 * g + r.value, 64);
                            if (4 * j + s.value <= n) Y[r.value] = fmaf(p, x, Y[r.value]);
                        });
                    });
            }
            Y += Y2;
            dsum += __shfl_xor(dsum, 16, 64);
            dsum += __shfl_xor(dsum, 32, 64);
            if (g == 0) den[c & 1][w][n] = dsum;
        }
        // ---- update ------------------------------------------------------------------------------------------
        if (decay) {
            if (c + 1 == chunks) set_update_factors(end - tok0);
            for_n<4>([&](auto s) { vr[s.value] *= g_v[s.value]; });
            for_n<NT>([&](auto t) { S[t.value] *= g_s; });
            for_n<ZS>([&](auto i) { z[i.value] *= g_s; });
        }
        {
            f32x4 kb[NB];
            for_n<NB>([&](auto B) { kb[B.value] = *reinterpret_cast<const f32x4 *>(&kt[b][4 * B.value + (n & 3)][sub + 4 * g]); });
            f32x4 ka = zero4();
            for_tiles<NB>([&](auto t, auto A, auto B) {
                if constexpr (A.value == B.value) ka = *reinterpret_cast<const f32x4 *>(&kt[b][4 * A.value + (n >> 2)][sub + 4 * g]);
                float f[4];
                for_n<4>([&](auto s) {
                    if constexpr (A.value == B.value) {
                        const float s1 = fmaf(ka[s.value], dk.m, A.value == 0 ? dk.c + k_const : dk.c);
                        f[s.value] = s1 * (dk.one ? 1.f : kb[B.value][s.value]);
                    } else {
                        f[s.value] = ka[s.value] * kb[B.value][s.value];
                    }
                    S[t.value] = mfma(f[s.value], vr[s.value], S[t.value]);
                });
                if (t.value % NW == w) {
                    if (decay)
                        for_n<4>([&](auto s) { f[s.value] *= g_v[s.value]; });
                    float zs = (f[0] + f[1]) + (f[2] + f[3]);
                    zs += __shfl_xor(zs, 16, 64);
                    zs += __shfl_xor(zs, 32, 64);
                    z[t.value / NW] += zs;
                }
                if constexpr (B.value == NB - 1) __builtin_amdgcn_sched_barrier(0);
            });
        }
        if ((c & 3) == 3 && c + 1 < chunks) store_stage(tok0 + C, b ^ 1);
        __syncthreads();   // the denominators' shares, and at the end of a stage the rows of the next one
        if constexpr (!INCREMENT) {
            float inv = 1.f;
            if (!numerator_only) {
                float d = 0.f;
                for_n<NW>([&](auto i) { d += den[c & 1][i.value][n]; });
                inv = 1.f / d;
            }
            if (tok0 + n < end) {
                if (gate) inv *= to_f32(gate[(size_t)(tok0 + n) * dec.H]);
                T *p = yu + (size_t)(tok0 + n) * DV + 4 * g;
                if constexpr (std::is_same_v<T, float>) {
                    *reinterpret_cast<f32x4 *>(p) = Y * inv;
                } else {
                    uint2 o;
                    o.x = (uint32_t)f32_to_bf16_bits(Y[0] * inv) | ((uint32_t)f32_to_bf16_bits(Y[1] * inv) << 16);
                    o.y = (uint32_t)f32_to_bf16_bits(Y[2] * inv) | ((uint32_t)f32_to_bf16_bits(Y[3] * inv) << 16);
                    *reinterpret_cast<uint2 *>(p) = o;
                }
            }
        }
        for_n<4>([&](auto s) { vr[s.value] = vn[s.value]; });
    }
    // the tokens that fill up the last chunk are in the count (row (2, 0) of block 0) and nowhere else
    if (w == 0 && n == 8) z[0] -= (float)(chunks * C - (end - begin));

    if (INCREMENT) {
        store_entry(first + seg);
    } else if (state && seg == G - 1) {
        export_state();
    }
}

// Segments: one round of what the chip holds, segments of at least 64 tokens (below that the increment launch and the sum
// over the entries cost what the shorter chain gives), at most 64.  (d' 16, d_v 64, bf16 with decay: 128 units of 2048 tokens 2
// segments 315 us, 4 237, 6 = a full round 226, 8 275; 16 units: 300 tokens 1 segment 66, 2 61, 4 41; 777 tokens 6 66, 12 59, 24 76.
// fp32, 16 units: 777 tokens at d' 32 6 segments 137, 12 109; d' 8, 500 tokens 1 segment 51, 4 23, 8 17, 16 18; 14926 tokens 16
// segments 145, 32 103, 64 99.  All from before a unit's segments shared an XCD.  The scratch of fp32 calls at d' 16 is sized by this rule too.)
inline int segments(int U, int N, int dp, int dv)
{
    const long groups = (long)U * (dv / COLS);
    long G = 256 * resident(dp) / groups;
    if (G > N / 64) G = N / 64;
    if (G > kMaxSegments) G = kMaxSegments;
    return G < 1 ? 1 : (int)G;
}
inline int segment_len(int N, int G) { return ((N + G - 1) / G + C - 1) / C * C; }

template <int DP, int DV, typename T>
hipError_t launch(const void *q, const void *k, const void *v, void *y, float *state, int has_init, void *workspace, int U,
                  int N, DecayArg dec, hipStream_t s)
{
    constexpr int SL = DV / COLS;
    int G = HAS_SEGMENTS<DP, T> ? segments(U, N, DP, DV) : 1;
    // The increment of the first of two segments is shared by two workgroups where entry 0 is free for the second's: one to a unit's slice left half of
    // the chip idle.  Where the rest of the sequence is an odd number of chunks the first segment takes one more: its pieces are no longer for it.  (us, one
    // and two: d' 32, fp32, 100 units N 160 83.2, 73.1, N 512 210, 183, 90 units N 1024 395, 335, d_v 128, 60 units N 700 280, 242; d' 24, bf16, 200 units N
    // 160 66.8, 66.2, N 200 78.9, 78.7, N 224 85.9, 83.4, N 512 172, 165, 256 units N 200 80.2, 80.6, N 1024 328, 310; d' 8, fp32, 350 units N 512 61.4, 58.1, N
    // 1000 110.7, 102.6, bf16, 400 units N 320 50.0, 50.0, N 512 73.5, 72.6, N 1000 136.1, 130.8.  Without the one more, d' 32, 100 units N 160 79.8, N 224 98.8;
    // with the first segment rounded up to two equal pieces, d' 24, bf16, 200 units N 200 83.6, N 336 119.5 instead of 114.7.  Where it is the number of tokens that allows no third segment there is room for the second piece: d' 24, 16 units
    // N 160 48.6, 41.8, d' 8, fp32, 4 units N 168 17.3, 15.3, bf16, 30 units N 176 19.5, 17.2, but 300 units N 152 27.0, 27.3, 340 27.5, 27.9.)
    const bool room = (DP == 8 ? 4l : 3l) * U * SL <= 256 * resident(DP);
    const bool shared = G == 2 && !(has_init & 1) && !dec.gamma && (room || DP == 32 || N > (DP == 24 ? 208 : 511));
    const int len = segment_len(N, G) + (shared && (N + C - 1) / C % 4 == 2 ? C : 0);
    while (G > 1 && (G - 1) * len >= N) --G;   // rounding the length up can empty trailing segments
    if ((long long)U * SL * G >= (1ll << 31)) return hipErrorInvalidValue;
    float *ws = static_cast<float *>(workspace);
    auto go = [&](auto increment, int first_slice, int slices) {
        constexpr bool INC = decltype(increment)::value;
        const int pieces = shared ? 2 : 1, parts = INC ? (G - 1) * pieces : G, all = U * slices, local = all / 8 * 8;
        hipLaunchKernelGGL((prefill_kernel<DP, DV, T, INC>), local ? dim3((unsigned)(all * parts)) : dim3(parts, all), dim3(64 * NW), 0, s, (const T *)q,
                           (const T *)k, (const T *)v, (T *)y, state, has_init, N, ws, len, G, shared ? 0 : 1, pieces,
                           first_slice, slices, local, dec);
        return hipGetLastError();
    };
    hipError_t e = hipSuccess;
    if (G > 1) {
        if constexpr (HAS_SEGMENTS<DP, T>) e = go(std::true_type{}, 0, SL);
    } else if ((has_init & 1) && SL > 1) {
        // every slice reads the caller's K-state and the first one overwrites it: the others go before it
        e = go(std::false_type{}, 1, SL - 1);
        return e == hipSuccess ? go(std::false_type{}, 0, 1) : e;
    }
    return e == hipSuccess ? go(std::false_type{}, 0, SL) : e;
}

template <int DP>
hipError_t launch_dp(const void *q, const void *k, const void *v, void *y, float *state, int has_init, void *workspace, int U,
                     int N, int dv, int dtype, DecayArg dec, hipStream_t s)
{
#define PF32_LAUNCH(DV, T) launch<DP, DV, T>(q, k, v, y, state, has_init, workspace, U, N, dec, s)
    if (dv == 64) return dtype == BASED_F32 ? PF32_LAUNCH(64, float) : PF32_LAUNCH(64, bf16_t);
    return dtype == BASED_F32 ? PF32_LAUNCH(128, float) : PF32_LAUNCH(128, bf16_t);
#undef PF32_LAUNCH
}

}  // namespace pf32

}  // namespace based
