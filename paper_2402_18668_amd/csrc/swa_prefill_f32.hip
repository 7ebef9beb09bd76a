// Sliding-window causal softmax attention over whole sequences (Sec. 3.2 restricting Eq. 1) on the fp32 matrix
// instructions: fp32 inputs at every supported size, bf16 inputs with a scale that is not positive (whose scores the
// bf16 kernels cannot mask and maximise before scaling), and bf16 inputs with rotary encoding at d_h 128, window 128 (whose
// ring leaves the bf16 kernel no room for the rotated queries).  Every product and sum is fp32.
//
// Work split: a workgroup is 64 queries of one unit, a wave 16 of them.  The keys a wave sees are T + 1 tiles of 16 (T = w /
// 16, the first and last cut by the window's edges), and wave w's tiles start w tiles after wave 0's: at step t the
// workgroup works on tiles t .. t + 3 of its w + 64 keys, every wave on one.  So an LDS ring of five tiles is enough:
// tile t + 4 goes into the fifth while step t reads the other four, one barrier a step.  It is loaded into registers a
// step earlier.  First all K tiles go through the ring, then, after the softmax, all V tiles.
//
// Registers (16x16x4 instruction, lane = 16 g + n; accumulator register r: row 4 g + r, column n; A operand: row n,
// k-slot g; B operand: column n, k-slot g).  The scores are computed transposed and kept whole, at most nine tiles:
//   S^T = K Q^T:      contraction step (c, r) visits column 16 c + 4 g + r in k-slot g: both operands are 16 contiguous bytes
//   Y^T += V^T P^T:   step s visits key 4 g + s: A = V[4 g + s][16 c + n], B = score register s as it stands
// Row stride of the ring: d_h + 4 floats, free of bank conflicts for both reads.  The last w rows of (rotated) K and V
// also go to the decode ring from here.
//
// Bound by memory at w = 16, by the matrix pipe (fp32: 157 TFLOP/s; w + 16 keys a query are multiplied) from w = 64 on.
// Measured against the vector-instruction kernel it replaces (a query to a wave, V out of L2), fp32, 32 units of 2048
// tokens: d_h 128, w 128 965 -> 67 us; w 64 248 -> 45; 64 units at d_h 64, w 16 80 -> 27 (4.9 TB/s); 32 units of 186
// tokens, d_h 64, w 64, rotary 28 -> 9.
#include "common.h"

#include <type_traits>
#include <utility>

namespace based {

namespace swa32 {

typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));

constexpr int QB = 64;     // queries of a workgroup
constexpr int NT = 256;    // threads
constexpr int RING = 5;    // staged tiles of 16 rows

template <int... I, typename F> __device__ __forceinline__ void for_seq(F &&f, std::integer_sequence<int, I...>)
{
    (f(std::integral_constant<int, I>{}), ...);
}
template <int N, typename F> __device__ __forceinline__ void for_n(F &&f) { for_seq(f, std::make_integer_sequence<int, N>{}); }

__device__ __forceinline__ f32x4 mfma(float a, float b, f32x4 c) { return __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, 0, 0, 0); }

// four adjacent elements of a row
__device__ __forceinline__ f32x4 load4(const float *p) { return *reinterpret_cast<const f32x4 *>(p); }
__device__ __forceinline__ f32x4 load4(const bf16_t *p)
{
    const u32x2 w = *reinterpret_cast<const u32x2 *>(p);
    return f32x4{__uint_as_float(w[0] << 16), __uint_as_float(w[0] & 0xffff0000u), __uint_as_float(w[1] << 16),
                 __uint_as_float(w[1] & 0xffff0000u)};
}
__device__ __forceinline__ void store4(float *p, f32x4 x) { *reinterpret_cast<f32x4 *>(p) = x; }
__device__ __forceinline__ void store4(bf16_t *p, f32x4 x)
{
    *reinterpret_cast<u32x2 *>(p) = u32x2{(uint32_t)f32_to_bf16_bits(x[0]) | ((uint32_t)f32_to_bf16_bits(x[1]) << 16),
                                          (uint32_t)f32_to_bf16_bits(x[2]) | ((uint32_t)f32_to_bf16_bits(x[3]) << 16)};
}
// two adjacent pairs rotated by their table entries (cos, sin, cos, sin)
__device__ __forceinline__ f32x4 rotate4(f32x4 x, f32x4 t)
{
    return f32x4{fmaf(x[0], t[0], -x[1] * t[1]), fmaf(x[0], t[1], x[1] * t[0]), fmaf(x[2], t[2], -x[3] * t[3]),
                 fmaf(x[2], t[3], x[3] * t[2])};
}

// workgroups on a CU: what the LDS ring allows and the registers of the window's scores leave room for
constexpr int resident(int dh, int w) { return (dh == 64 ? 4 : 3) - (w == 128 ? 1 : 0); }

template <int DH, int W, typename T, bool ROT>
__global__ __launch_bounds__(NT, resident(DH, W)) void kernel(const T *__restrict__ q, const T *__restrict__ k,
                                                               const T *__restrict__ v, T *__restrict__ y, T *__restrict__ ring,
                                                               const float2 *__restrict__ rot, int N, int blocks, float scale)
{
    constexpr int TL = W / 16;         // steps 0 .. TL
    constexpr int LD = DH + 4;
    constexpr int PT = DH / 64;        // 4-element chunks of a tile per thread
    constexpr int CPR = DH / 4;        // chunks of a row
    constexpr int DC = DH / 16;
    __shared__ __align__(16) float lds[RING][16][LD];

    const int u = blockIdx.x / blocks, i0 = (blockIdx.x % blocks) * QB;
    const int tid = threadIdx.x, wv = __builtin_amdgcn_readfirstlane(tid >> 6), lane = tid & 63, g = lane >> 4, n = lane & 15;
    const size_t base = (size_t)u * N * DH;
    const T *ku = k + base, *vu = v + base;
    T *ring_u = ring ? ring + (size_t)u * 2 * W * DH : nullptr;
    const int qbase = i0 + 16 * wv, query = qbase + n;

    // ---- staging: tile t holds the rows of keys i0 - W + 16 t .. + 15; rows outside the sequence are zero -------------
    const int s_row = tid / CPR, s_col = 4 * (tid % CPR);   // this thread's first chunk; the next is NT / CPR rows on
    struct Tile { f32x4 x[PT]; };
    auto load_tile = [&](const T *src, int t) {
        Tile r;
        for_n<PT>([&](auto i) {
            const int key = min(max(i0 - W + 16 * t + s_row + i.value * (NT / CPR), 0), N - 1);
            r.x[i.value] = load4(src + (size_t)key * DH + s_col);
        });
        return r;
    };
    auto store_tile = [&](Tile r, int t, bool key_rows) {
        for_n<PT>([&](auto i) {
            const int row = s_row + i.value * (NT / CPR), key = i0 - W + 16 * t + row;
            f32x4 x = r.x[i.value];
            if (ROT && key_rows) {
                x = rotate4(x, *reinterpret_cast<const f32x4 *>(rot + (size_t)min(max(key, 0), N - 1) * (DH / 2) + s_col / 2));
                if constexpr (std::is_same_v<T, bf16_t>)   // (the decode ring holds rounded keys: the same ones count here)
                    for_n<4>([&](auto j) { x[j.value] = to_f32(from_f32<bf16_t>(x[j.value])); });
            }
            if (key < 0 || key >= N) x = f32x4{0.f, 0.f, 0.f, 0.f};
            *reinterpret_cast<f32x4 *>(&lds[t % RING][row][s_col]) = x;
            if (ring_u && key >= i0 && key < N && key >= N - W)
                store4(ring_u + (size_t)((key_rows ? 0 : W) + key % W) * DH + s_col, x);
        });
    };
    auto slot = [&](int t) { return (wv + t) % RING; };   // where this wave's tile of step t is

    // The tiles before the start of the sequence are not multiplied: at the largest window they are most of a short call's work (8
    // units of 16 tokens, d_h 128: 17.0 -> 12.2 us; the branches cost longer ones up to 4 % one way or the other, smaller windows
    // have little to skip).
    auto in_sequence = [&](int t) { return W < 128 || qbase - W + 16 * t >= 0; };

    f32x4 Q[DC];
    {
        const int row = min(query, N - 1);
        for_n<DC>([&](auto c) { Q[c.value] = load4(q + base + (size_t)row * DH + 16 * c.value + 4 * g); });
        Tile first[4];
        for_n<4>([&](auto t) { first[t.value] = load_tile(ku, t.value); });
        for_n<DC>([&](auto c) {
            if (ROT) Q[c.value] = rotate4(Q[c.value], *reinterpret_cast<const f32x4 *>(rot + (size_t)row * (DH / 2) + 8 * c.value + 2 * g));
            Q[c.value] *= scale;
        });
        for_n<4>([&](auto t) { store_tile(first[t.value], t.value, true); });
    }
    Tile next = load_tile(ku, 4);
    __syncthreads();

    // ---- scores ------------------------------------------------------------------------------------------------------
    f32x4 P[TL + 1];
    Tile vfirst[4];
    for_n<TL + 1>([&](auto t) {
        Tile after = next;
        if constexpr (t.value < TL - 1) after = load_tile(ku, t.value + 5);
        if constexpr (t.value == TL) for_n<4>([&](auto i) { vfirst[i.value] = load_tile(vu, i.value); });
        const float *row = &lds[slot(t.value)][n][4 * g];
        f32x4 a = {0.f, 0.f, 0.f, 0.f}, b = a;   // two chains
        if (in_sequence(t.value))
            for_n<DC>([&](auto c) {
                const f32x4 kc = *reinterpret_cast<const f32x4 *>(row + 16 * c.value);
                for_n<4>([&](auto r) {
                    if (r.value & 1) b = mfma(kc[r.value], Q[c.value][r.value], b);
                    else a = mfma(kc[r.value], Q[c.value][r.value], a);
                });
            });
        P[t.value] = a + b;
        if constexpr (t.value < TL) store_tile(next, t.value + 4, true);
        next = after;
        __syncthreads();
    });
    for_n<4>([&](auto t) { store_tile(vfirst[t.value], t.value, false); });
    next = load_tile(vu, 4);

    // ---- softmax: a query's keys sit in the registers of the four lanes n, n + 16, .. -----------------------------------
    float m = -INFINITY;
    for_n<TL + 1>([&](auto t) {
        for_n<4>([&](auto r) {
            const int local = 4 * g + r.value;
            bool ok = qbase - W + 16 * t.value + local >= 0;
            if (t.value == 0) ok = ok && local > n;     // key > query - w
            if (t.value == TL) ok = ok && local <= n;   // key <= query
            P[t.value][r.value] = ok ? P[t.value][r.value] : -INFINITY;
            m = fmaxf(m, P[t.value][r.value]);
        });
    });
    m = fmaxf(m, __shfl_xor(m, 16, 64));
    m = fmaxf(m, __shfl_xor(m, 32, 64));   // (finite: the query's own key is visible)
    float sum = 0.f;
    for_n<TL + 1>([&](auto t) {
        for_n<4>([&](auto r) {
            const float p = __builtin_amdgcn_exp2f((P[t.value][r.value] - m) * 1.44269504088896340736f);
            P[t.value][r.value] = p;
            sum += p;
        });
    });
    sum += __shfl_xor(sum, 16, 64);
    sum += __shfl_xor(sum, 32, 64);
    __syncthreads();

    // ---- Y^T += V^T P^T ------------------------------------------------------------------------------------------------
    f32x4 Y[DC];
    for_n<DC>([&](auto c) { Y[c.value] = f32x4{0.f, 0.f, 0.f, 0.f}; });
    for_n<TL + 1>([&](auto t) {
        Tile after = next;
        if constexpr (t.value < TL - 1) after = load_tile(vu, t.value + 5);
        const float *col = &lds[slot(t.value)][4 * g][n];
        if (in_sequence(t.value))
            for_n<4>([&](auto s) {
                for_n<DC>([&](auto c) { Y[c.value] = mfma(col[s.value * LD + 16 * c.value], P[t.value][s.value], Y[c.value]); });
            });
        if constexpr (t.value < TL) {
            store_tile(next, t.value + 4, false);
            next = after;
            __syncthreads();
        }
    });
    // In the window's first and last tile a key that a query cannot see stood in the product as 0 V, which is NaN where V is not
    // finite.  Results that are not finite are summed again, key by key and without the hidden ones, V from memory.
    float probe = 0.f;
    for_n<DC>([&](auto c) { for_n<4>([&](auto r) { probe = fmaf(0.f, Y[c.value][r.value], probe); }); });
    if (__builtin_expect(__builtin_amdgcn_ballot_w64(query < N && probe != 0.f) != 0, 0)) {
        for_n<DC>([&](auto c) { Y[c.value] = f32x4{0.f, 0.f, 0.f, 0.f}; });
        for_n<TL + 1>([&](auto t) {
#pragma unroll 1
            for (int j = 0; j < 4; ++j)
                for_n<4>([&](auto s) {
                    const float p = __shfl(P[t.value][s.value], 16 * j + n, 64);
                    const int key = qbase - W + 16 * t.value + 4 * j + s.value;
                    const bool visible = key >= 0 && key > query - W && key <= query;
                    const T *row = vu + (size_t)min(max(key, 0), N - 1) * DH + 4 * g;
                    for_n<DC>([&](auto c) {
                        const f32x4 x = load4(row + 16 * c.value);
                        for_n<4>([&](auto r) { Y[c.value][r.value] = fmaf(p, visible ? x[r.value] : 0.f, Y[c.value][r.value]); });
                    });
                });
        });
    }
    if (query < N) {
        const float inv = 1.f / sum;
        for_n<DC>([&](auto c) { store4(y + base + (size_t)query * DH + 16 * c.value + 4 * g, Y[c.value] * inv); });
    }
}

template <int DH, int W, typename T>
hipError_t launch(const void *q, const void *k, const void *v, void *y, void *ring, const float *rot, int U, int N, float scale,
                  hipStream_t s)
{
    const int blocks = (N + QB - 1) / QB;
    if ((long long)blocks * U >= (1ll << 31)) return hipErrorInvalidValue;
    auto go = [&](auto rotary) {
        hipLaunchKernelGGL((kernel<DH, W, T, decltype(rotary)::value>), dim3((unsigned)(blocks * U)), dim3(NT), 0, s, (const T *)q,
                           (const T *)k, (const T *)v, (T *)y, (T *)ring, reinterpret_cast<const float2 *>(rot), N, blocks, scale);
    };
    if (rot) go(std::true_type{});
    else go(std::false_type{});
    return hipGetLastError();
}

}  // namespace swa32

hipError_t launch_swa_prefill_f32(const void *q, const void *k, const void *v, void *y, void *ring, const float *rot, int U,
                                  int N, int dh, int w, float scale, int dtype, hipStream_t s)
{
#define SWA_CASE(DH_, W_)                                                                                      \
    if (dh == DH_ && w == W_)                                                                                  \
        return dtype == BASED_F32 ? swa32::launch<DH_, W_, float>(q, k, v, y, ring, rot, U, N, scale, s)       \
                                  : swa32::launch<DH_, W_, bf16_t>(q, k, v, y, ring, rot, U, N, scale, s)
    SWA_CASE(64, 16);
    SWA_CASE(64, 32);
    SWA_CASE(64, 64);
    SWA_CASE(64, 128);
    SWA_CASE(128, 16);
    SWA_CASE(128, 32);
    SWA_CASE(128, 64);
    SWA_CASE(128, 128);
#undef SWA_CASE
    return hipErrorInvalidValue;
}

}  // namespace based
