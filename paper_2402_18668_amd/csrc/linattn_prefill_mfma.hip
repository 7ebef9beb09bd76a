// Causal Taylor linear attention, chunked prefill on the gfx950 matrix cores (bf16 in, fp32
// accumulate), d' = 16.
//
// Chunked form of Sec. 4: inside a chunk of C = 64 tokens the masked quadratic product
// (1 + A + A^2/2 with A = Q K^T, exact closed form of Eq. 4), across chunks the running
// KV-state S (Eq. 3) read out with phi(Q) and updated with phi(K)^T V.  The expanded features
// are produced in registers in MFMA operand layout, pass through LDS once, and never reach HBM.
//
// Symmetric packing of the 2nd-order block.  The state rows (a, b) and (b, a) of Eq. 4 are equal
// (x_a x_b = x_b x_a), so only one row per unordered pair is carried: row (a, delta) stands for
// the pair {a, (a + delta) mod 16} with delta = 0 .. 7 for every a (128 rows) and delta = 8 for
// a < 8 (8 rows), 136 rows instead of 256.  The k side builds x_a x_b / sqrt(2) (the canonical
// state row); the q side builds sqrt(2) x_a x_b for delta != 0 (the pair counts twice in the sum
// over ordered pairs) and x_a^2 / sqrt(2) for delta = 0.  The cyclic enumeration keeps the
// operand construction regular: for a fixed delta the 16 features are x (.) rotate(x, delta).
// The final state is written in the canonical layout (both rows of a pair); an initial state is
// read as its symmetric part, which is all the readout can see.
//
// The 153 rows are laid out as five tiles of 32 (160 rows): tile T < 4 holds delta = 2T (local rows
// 0..15, a = row) and delta = 2T + 1 (rows 16..31); tile 4 holds the 16 linear rows, the constant
// row (16), seven rows of padding and the eight rows of delta = 8 (24..31).
//
// Work split.  One workgroup per (unit, sequence segment): one CONSUMER wave per 32 columns of d_v
// (two at d_v = 64, four at 128) and six or four PRODUCER waves (two waves to a SIMD).  A consumer owns ALL 160 state rows of its
// 32 columns: five 32x32 fp32 accumulator tiles that stay in its registers for the whole segment (the
// paper keeps its 2nd-order state in registers for the same reason), and issues every matrix
// instruction for those columns: readout Y^T = S^T phi(Q)^T, intra-chunk Y^T += V^T P^T, update
// S += phi(K)^T V; then it normalises and stores its piece of y.  With the columns split this way
// nothing of one consumer's accumulators is needed by another: no partial outputs are exchanged.
// What the waves share is the operands, which do not depend on the column: each operand (32 x 16
// bf16, one kilobyte) is built ONCE per chunk by a producer, written to LDS in MFMA operand layout
// (16 bytes per lane), and read by every consumer with one 16-byte LDS load per lane, so that the
// vector-ALU cost of the feature map is paid once per workgroup.  The masked intra-chunk blocks P
// and the denominators are shared the same way.
//
// Pipeline.  The producers run one chunk ahead of the consumers: while the consumers multiply the
// operands of chunk t (LDS generation t % 2), the producers stage the rows of chunk t + 1 (fetched
// into registers during chunk t - 1), and build its operands into the other generation.  Per chunk
// there is one workgroup barrier (chunk t + 1's operands are visible, chunk t's are free).  The staged rows of K and Q exist twice and are staged one chunk
// earlier still, so that nothing else is waited for.
//
// What bounds a chunk: the instruction stream of the waves, two to a SIMD, all about equally long (cycles of a chunk with all CUs at work, d_v 64 / 128: 2850 / 3740, with a few
// 2370 / 3300; each wave up to the barrier, reading the counter included: consumers 2300 / 3460, the one with the moments 3720; producers 2500-2950 / 3200-3520).  Three
// things shortened it, where the consumers set the pace: (1) the outputs are normalised and turned between the update's matrix instructions, and turned in registers (the halves of a wave exchange
// quads) instead of through LDS, which each consumer waited for twice: the second half of its chunk 1950 -> 1150; (2) the rows of K and Q come into
// the registers that an operand is built from as products with 0/1 matrices instead of as staged fp32 copies, whose 4-byte LDS writes and 28 KB of reads the
// producers spent a third of their time on; (3) the moments and denominators at d_v 128 are a consumer's.  256 units of 2048 tokens, d_v 64 58 -> 51.5 us,
// d_v 128 85.7 -> 83.1 (inputs out of cache; 84 -> 77 with three sets of buffers in turn).
//
// MFMA 32x32x16 register layouts used throughout (lane = 32 g + n):
//   A operand: row n, k-slots 8g .. 8g+7;  B operand: column n, k-slots 8g .. 8g+7;
//   accumulator register r: row 8 (r / 4) + 4 g + r % 4, column n.
// Because a contraction may visit its index in any order, k-slot 8g + 4jj + i of "slab" s is
// mapped to index 16 s + 8 jj + 4 g + i: then accumulator registers 8s .. 8s+7 of a lane are
// exactly its 8 k-slots of slab s, and a state tile (or the masked intra-chunk block) becomes
// an MFMA operand with a register-local fp32 -> bf16 conversion and no data movement.
//
// Denominator.  z is kept as moments: M' = K'^T K' with K' = [k, 1] (17 x 17 inside one
// accumulator tile), i.e. sum k_a k_b, sum k_a and the token count; phi(q).z =
// count + q.z1 + q^T M q / 2 is evaluated with two small MFMAs (M' split into bf16 hi + lo).
//
// Long sequences / few units: the sequence is cut into G segments, a workgroup each.  The workgroup of segment g > 0 first computes the state
// increment of segment g - 1; its main pass starts from that and the sum of the increments before, which the other workgroups leave in the workspace
// and for which it waits (bounded) on per-entry ready flags.
#include "common.h"

#include <atomic>
#include <cmath>
#include <type_traits>

namespace based {

namespace {

typedef float f32x16 __attribute__((ext_vector_type(16)));
typedef float f32x8 __attribute__((ext_vector_type(8)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef __bf16 bf16x4 __attribute__((ext_vector_type(4)));
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));
typedef short s16x4 __attribute__((ext_vector_type(4)));
typedef short s16x8 __attribute__((ext_vector_type(8)));

constexpr int DP = 16;            // d'
constexpr int C = 64;             // chunk length (tokens)
constexpr int NTILE = 5;          // state tiles of 32 rows
constexpr int NSLAB = 2 * NTILE;  // feature slabs of 16 rows
constexpr float kCQ = 1.18920711500272106672f;   // 2^(+1/4): (c q_a)(c q_b) = sqrt(2) q_a q_b
constexpr float kSqrt2 = 1.41421356237309504880f;

// LDS strides (elements)
constexpr int RB_LD = DP + 8;     // bf16 row-major Q and K rows as given (48-byte stride)

// Workspace entry (one segment's state in accumulator layout): six slots of 16 registers x 64 lanes
// per column tile: slot 6c + T = state tile T of columns 32c .. 32c+31, slot 6 x_tile + 5 = the
// moment tile (the other sixth slots are never written and their contents are never used).
// Within a slot: [r / 4][lane][r % 4], so one 16-byte access per lane is contiguous
// across the wave.
constexpr int WS_WAVE_SLOTS = 6;
constexpr size_t kSlotFloats = 16 * 64;
__host__ __device__ constexpr size_t entry_floats(int nc) { return (size_t)nc * WS_WAVE_SLOTS * kSlotFloats; }

// Producer waves beside NC consumers, and the wave that has the moments, which travel in the sixth slot of column tile x_tile.
__host__ __device__ constexpr int producers(int nc) { return nc == 2 ? 6 : 4; }
__host__ __device__ constexpr int x_wave(int nc) { return nc == 2 ? 2 : 3; }
__host__ __device__ constexpr int x_tile(int nc) { return nc == 2 ? 0 : 3; }
// Bytes of the state buffer's image in LDS; where the increment's rows lie there and, afterwards, what it leaves to the main pass.
constexpr int IMG_LD = 40;   // (the two rows that the halves of a wave access lie in different banks)
__host__ __device__ constexpr int image_bytes(int nc) { return nc * 32 * NTILE * IMG_LD * 4; }
__host__ __device__ constexpr int hand_at(int nc) { return nc == 2 ? image_bytes(2) : 0; }   // (at d_v 128 where the image was)
template <int NC>
struct Lds {
    // the q and k rows of a chunk, by its parity: building one chunk's operands and staging the next one's rows need nothing but the
    // chunk's barrier
    struct alignas(16) Rows {
        uint16_t qrow[C][RB_LD];        // Q rows, bf16 as given
        uint16_t krow[C][RB_LD];        // K rows, bf16 as given
    } rows[2];
    // everything the consumers read exists twice, indexed by the parity of the chunk: the producers fill
    // one generation while the consumers work on the other
    uint16_t vrow[2][C][32 * NC + 16];  // V rows, bf16 as given (operands are read transposed; the stride
                                        // leaves those reads free of bank conflicts)
    u32x4 phiq[2][2][NSLAB][64];        // phi(Q)^T operands: [parity][query tile][slab][lane]
    u32x4 phik[2][NTILE][4][64];        // phi(K)^T operands: [parity][state tile][16-token slab][lane]
    u32x4 pop[2][3][2][64];             // masked intra-chunk blocks as operands: [parity][block][slab][lane]
    float den[2][3][C];                 // per query: inter-chunk part; row sums of the blocks of key tile 0, 1
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

__device__ __forceinline__ bf16x8 pack8_acc(const f32x16 &acc, int s)   // registers 8s .. 8s+7
{
    f32x8 f;
#pragma unroll
    for (int e = 0; e < 8; ++e) f[e] = acc[8 * s + e];
    return __builtin_convertvector(f, bf16x8);
}

__device__ __forceinline__ bf16x8 as_bf16x8(u32x4 w) { return __builtin_bit_cast(bf16x8, w); }
__device__ __forceinline__ u32x4 as_u32x4(bf16x8 w) { return __builtin_bit_cast(u32x4, w); }

__device__ __forceinline__ void zero16(f32x16 &a)
{
#pragma unroll
    for (int r = 0; r < 16; ++r) a[r] = 0.f;
}

// Workgroup barrier that orders LDS traffic only: this wave's LDS operations have completed
// (lgkmcnt) before it arrives, and the compiler moves no memory access across it.  Global loads
// and stores stay in flight (the waves exchange data through LDS only), which is what lets the
// next chunk's rows stream in underneath the current chunk's arithmetic.
__device__ __forceinline__ void wg_sync()
{
    asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
}

// MFMA instructions ignore the EXEC mask.  A branch on the wave's role is uniform across the wave
// but the compiler lowers it to lane masking and may drop the jump over a short masked block, in
// which case the other waves would execute the MFMAs inside it.  An inline-asm statement in the
// block makes the compiler keep the jump (it never runs inline asm with an empty EXEC mask).
__device__ __forceinline__ void role_guard() { asm volatile("; wave-role block: keep the execz branch"); }

__device__ __forceinline__ float bf16lo(uint32_t w) { return __uint_as_float(w << 16); }
__device__ __forceinline__ float bf16hi(uint32_t w) { return __uint_as_float(w & 0xffff0000u); }

// Canonical state rows (Eq. 4 order: row 0 constant, 1 + a linear, 1 + d' + a d' + b the pair
// (a, b)) of a packed row.  A pair row has two canonical rows (equal for delta = 0).
// With packed_state the buffer is the packed layout (one row per unordered pair), where a pair has a
// single row and the constant and linear rows sit at the same indices.
struct CanonRows { int r1, r2; };   // r1 < 0: the packed row is padding
__device__ __forceinline__ CanonRows canon_pair(int a, int b, bool packed_state)
{
    if (packed_state) {
        const int r = packed_pair_row(DP, min(a, b), max(a, b));
        return {r, r};
    }
    return {1 + DP + a * DP + b, 1 + DP + b * DP + a};
}
// local row fl of tile T: T < 4: delta = 2T + fl / 16, a = fl % 16; T = 4: 0..15 linear, 16 constant,
// 24..31 the delta = 8 pairs
__device__ __forceinline__ CanonRows canon_rows(int T, int fl, bool packed_state)
{
    if (T < 4) {
        const int a = fl & 15;
        return canon_pair(a, (a + 2 * T + (fl >> 4)) & 15, packed_state);
    }
    if (fl < DP) return {1 + fl, 1 + fl};
    if (fl == DP) return {0, 0};
    if (fl >= 24) return canon_pair(fl - 24, fl - 16, packed_state);
    return {-1, -1};
}

// Workspace accesses that cross workgroups inside one launch.  Each XCD has its own L2, and memory
// written by a workgroup on one XCD is only guaranteed to be seen by another XCD's workgroups at a
// kernel boundary, unless the accesses are marked system-coherent (sc0 sc1: written through to, and
// read from, the memory side of the L2s).
// (A store of more than 64 bits reads its data registers a few cycles after it issues, and whatever
// overwrites them in the next two cycles corrupts the stored data.  The compiler keeps that distance for
// stores it emits itself but cannot see inside an asm statement, so the wait states are part of it.)
__device__ __forceinline__ void store16_coherent(float *p, const f32x4 &v)
{
    asm volatile("global_store_dwordx4 %0, %1, off sc0 sc1\n\ts_nop 2" : : "v"(p), "v"(v) : "memory");
}
// The six slots of one wave in one entry: all 24 loads are in flight at once and the wait sits in the
// same statement, so that every output register is valid as far as the compiler can tell.  p1, p3, p5
// point at the lane's 16 bytes of slots 1, 3, 5; the slot before each is reached with negative offsets.
__device__ __forceinline__ void load_wave_slots_coherent(const float *p1, const float *p3, const float *p5,
                                                         f32x4 (&t)[24])
{
    asm volatile(
        "global_load_dwordx4 %0, %24, off offset:-4096 sc0 sc1\n\t"
        "global_load_dwordx4 %1, %24, off offset:-3072 sc0 sc1\n\t"
        "global_load_dwordx4 %2, %24, off offset:-2048 sc0 sc1\n\t"
        "global_load_dwordx4 %3, %24, off offset:-1024 sc0 sc1\n\t"
        "global_load_dwordx4 %4, %24, off offset:0 sc0 sc1\n\t"
        "global_load_dwordx4 %5, %24, off offset:1024 sc0 sc1\n\t"
        "global_load_dwordx4 %6, %24, off offset:2048 sc0 sc1\n\t"
        "global_load_dwordx4 %7, %24, off offset:3072 sc0 sc1\n\t"
        "global_load_dwordx4 %8, %25, off offset:-4096 sc0 sc1\n\t"
        "global_load_dwordx4 %9, %25, off offset:-3072 sc0 sc1\n\t"
        "global_load_dwordx4 %10, %25, off offset:-2048 sc0 sc1\n\t"
        "global_load_dwordx4 %11, %25, off offset:-1024 sc0 sc1\n\t"
        "global_load_dwordx4 %12, %25, off offset:0 sc0 sc1\n\t"
        "global_load_dwordx4 %13, %25, off offset:1024 sc0 sc1\n\t"
        "global_load_dwordx4 %14, %25, off offset:2048 sc0 sc1\n\t"
        "global_load_dwordx4 %15, %25, off offset:3072 sc0 sc1\n\t"
        "global_load_dwordx4 %16, %26, off offset:-4096 sc0 sc1\n\t"
        "global_load_dwordx4 %17, %26, off offset:-3072 sc0 sc1\n\t"
        "global_load_dwordx4 %18, %26, off offset:-2048 sc0 sc1\n\t"
        "global_load_dwordx4 %19, %26, off offset:-1024 sc0 sc1\n\t"
        "global_load_dwordx4 %20, %26, off offset:0 sc0 sc1\n\t"
        "global_load_dwordx4 %21, %26, off offset:1024 sc0 sc1\n\t"
        "global_load_dwordx4 %22, %26, off offset:2048 sc0 sc1\n\t"
        "global_load_dwordx4 %23, %26, off offset:3072 sc0 sc1\n\t"
        "s_waitcnt vmcnt(0)"
        : "=&v"(t[0]), "=&v"(t[1]), "=&v"(t[2]), "=&v"(t[3]), "=&v"(t[4]), "=&v"(t[5]), "=&v"(t[6]),
          "=&v"(t[7]), "=&v"(t[8]), "=&v"(t[9]), "=&v"(t[10]), "=&v"(t[11]), "=&v"(t[12]), "=&v"(t[13]),
          "=&v"(t[14]), "=&v"(t[15]), "=&v"(t[16]), "=&v"(t[17]), "=&v"(t[18]), "=&v"(t[19]), "=&v"(t[20]),
          "=&v"(t[21]), "=&v"(t[22]), "=&v"(t[23])
        : "v"(p1), "v"(p3), "v"(p5)
        : "memory");
}

// Default upper bound on the polls of a segment-ready flag (each poll sleeps ~0.25 us): a workgroup
// never waits forever, whatever happens to the workgroup it waits for.  A workgroup that gives up
// stores the call's epoch into the workspace's status word (a plain vector store) and carries on, so
// that every workgroup of the launch exits normally; its outputs are then wrong, and
// based_prefill_status reports the launch as failed.
constexpr int kMaxFlagPolls = 1 << 20;
std::atomic<int> g_flag_poll_limit{kMaxFlagPolls};

// 16 bytes per lane from base (uniform) + off bytes (per lane) to LDS address `to` (uniform) + 16 lane.  (Inline asm: through the
// builtin the compiler makes every LDS read wait for all of it.  The wait states: a scalar register that a vector instruction has just
// written, a spilled one for instance, reaches the memory pipeline five later, and the compiler does not see this use.)
__device__ __forceinline__ void dma16(const void *base, uint32_t off, uint32_t to)
{
    asm volatile("s_mov_b32 m0, %0\n\ts_nop 4\n\tglobal_load_lds_dwordx4 %1, %2" : : "s"(to), "v"(off), "s"(base) : "memory", "m0");
}

// lane i of a row of 16 gets the value of lane (i + D) % 16 (a DPP operand of the multiplication that uses it)
template <int D> __device__ __forceinline__ float rotate16(float x)
{
    if constexpr (D == 0) return x;
    else return __uint_as_float(__builtin_amdgcn_update_dpp(0u, __float_as_uint(x), 0x120 + 16 - D, 0xf, 0xf, true));
}
// the operand with `one` at element `target` of 16 (k-slot (jj, i) of lane half g: element 8 jj + 4 g + i) and zeros
__device__ __forceinline__ bf16x8 one_at(int g, int target, uint32_t one)
{
    u32x4 o;
#pragma unroll
    for (int p = 0; p < 4; ++p) {
        const int e = 8 * (p >> 1) + 4 * g + 2 * (p & 1);
        o[p] = (e == target ? one : 0u) | (e + 1 == target ? one << 16 : 0u);
    }
    return as_bf16x8(o);
}

__device__ __forceinline__ float bf16_at(const uint16_t *p) { return __uint_as_float((uint32_t)*p << 16); }
// Feature row n of state tile T of a token, from its row of K
__device__ __forceinline__ float phik_element(const uint16_t *kr, int T, int n)
{
    const float a = bf16_at(kr + (n & 15)), b = bf16_at(kr + ((T < 4 ? n + 2 * T + (n >> 4) : n - 24) & 15));
    return T < 4 || n >= 24 ? a * kRsqrt2 * b : n < DP ? a : n == DP ? 1.f : 0.f;
}

// The state buffer moves through LDS (which holds nothing else at either end of a segment), as an image of the consumers'
// tiles: image[column tile][32 T + row][IMG_LD].  A consumer reaches its registers' places at constant offsets from one
// address, and the whole workgroup moves 16-byte pieces between the image and the buffer's rows.  (Read and
// written by the consumers straight from and to memory, 160 four-byte accesses to a lane with an address each, it took
// 12 us to read and 5-6 us to write at 16 units, d_v 64.)
template <int NC> struct Image {
    static constexpr int NTHR = 64 * (NC + producers(NC)), DV = 32 * NC;
    static constexpr int Q = 32 * NTILE * (DV / 4), STEPS = (Q + NTHR - 1) / NTHR;   // 16-byte pieces: all, per thread
    static __device__ __forceinline__ float *piece(float *image, int i)   // columns 4 (i % (DV / 4)) .. of row i / (DV / 4)
    {
        return image + ((i % (DV / 4)) / 8 * 32 * NTILE + i / (DV / 4)) * IMG_LD + 4 * (i % 8);
    }
    static __device__ __forceinline__ CanonRows rows(int i, bool packed_state) { return canon_rows(i / (DV / 4) >> 5, i / (DV / 4) & 31, packed_state); }
};
template <int NC> __device__ __forceinline__ void import_state_image(float *image, const float *Su, bool packed_state, int tid)
{
    using I = Image<NC>;
    constexpr int BATCH = 5, DV = 32 * NC;
    for (int s0 = 0; s0 < I::STEPS; s0 += BATCH) {
        f32x4 t[BATCH][2];
#pragma unroll
        for (int j = 0; j < BATCH; ++j) {
            const int i = min((s0 + j) * I::NTHR + tid, I::Q - 1);
            const CanonRows cr = I::rows(i, packed_state);
            const float *p = Su + 4 * (i % (DV / 4));
            t[j][0] = *reinterpret_cast<const f32x4 *>(p + (size_t)max(cr.r1, 0) * DV);
            t[j][1] = *reinterpret_cast<const f32x4 *>(p + (size_t)max(cr.r2, 0) * DV);
        }
#pragma unroll
        for (int j = 0; j < BATCH; ++j) {
            const int i = (s0 + j) * I::NTHR + tid;
            const float w = I::rows(i, packed_state).r1 < 0 ? 0.f : 0.5f;   // (padding rows are zero)
            if (i < I::Q) *reinterpret_cast<f32x4 *>(I::piece(image, i)) = w == 0.f ? f32x4{0.f, 0.f, 0.f, 0.f} : (t[j][0] + t[j][1]) * w;
        }
    }
}
// M'[fl][n] of the caller's K-state (a place in z for every lane: conditional loads would wait for each other)
__device__ __forceinline__ float initial_moment(const float *zu, int fl, int n, bool packed_state)
{
    const bool in = fl <= DP && n <= DP, pair = fl < DP && n < DP;
    const int at = pair ? canon_pair(fl, n, packed_state).r1 : !in ? 0 : fl < DP ? 1 + fl : n < DP ? 1 + n : 0;
    return zu[at] * (pair ? 1.41421356237309504880f : in ? 1.f : 0.f);
}

constexpr int kLdsBytes = 150 * 1024;   // (one workgroup to a CU)
constexpr int kMaxSegments = 16;
// first token of each segment (multiples of the chunk length), and the end of the last one
struct SegTable { int begin[kMaxSegments + 1]; };

}  // namespace

// Full prefill of the segment (readout + update); starts from what the workgroup's own increment has left in LDS (seg > 0) and the sum of workspace
// entries 1 .. seg - 1.
// The caller's initial state is read by the main pass of segment 0 and by the increment of segment 0, which starts from
// it (so that the other segments get it with their first entry).  The last segment overwrites it with the final state, and
// waits until both have read it.
// Flag word F[unit][p][g] == epoch tells the workgroup of segment g that entry p (the increment of segment p - 1, p < g) of this call is complete (p = 0,
// g = G - 1: that the main pass of segment 0 has read the initial state): every word has one writer and one
// reader, and the reader zeroes it once it has seen it, so the words are clear again when the launch
// ends (a replay of a captured launch, which repeats the same epoch, starts from cleared flags).
// SEG: the launch has several segments.
template <int NC, bool SEG>
__device__ __forceinline__ void prefill_body(
    Lds<NC> &lds, unsigned &anew, const uint16_t *__restrict__ q, const uint16_t *__restrict__ k,
    const uint16_t *__restrict__ v, uint16_t *__restrict__ y, float *__restrict__ state, int has_init,
    float *__restrict__ ws, unsigned *__restrict__ flags, unsigned *__restrict__ status, int max_polls,
    unsigned epoch, int N, const SegTable &segs, int G, int seg, int u)
{
    constexpr int NPW = producers(NC);
    constexpr int NP = 64 * NPW;      // producer threads
    constexpr int DV = 32 * NC;       // d_v
    constexpr int VR_LD = DV + 16;
    // has_init carries three flags: bit 0 an initial state is given, bit 1 the state buffer is packed,
    // bit 2 the outputs are the numerators alone (no division by the denominator)
    const bool packed_state = (has_init & 2) != 0;
    const bool numerator_only = (has_init & 4) != 0;
    has_init &= 1;
    const int tid = threadIdx.x;
    const int w = __builtin_amdgcn_readfirstlane(tid >> 6);
    const bool is_p = w >= NC;            // producer wave; else consumer wave (owns the state tiles)
    const int c = is_p ? w - NC : w;      // consumer: column tile (columns 32c .. 32c+31); producer: its role
    const int lane = tid & 63;
    const int g = lane >> 5, n = lane & 31;

    const int tok_begin = segs.begin[seg];
    const int tok_end = min(N, segs.begin[seg + 1]);
    const int n_chunks = (tok_end - tok_begin + C - 1) / C;

    const uint16_t *qu = q + (size_t)u * N * DP;
    const uint16_t *ku = k + (size_t)u * N * DP;
    const uint16_t *vu = v + (size_t)u * N * DV;
    uint16_t *yu = y + (size_t)u * N * DV;
    float *Su = state ? state + (size_t)u * (packed_state ? packed_state_stride(DP, DV) : state_stride(DP, DV))
                      : nullptr;
    // (entry p = 1 .. G - 1 of the unit starts at (p - 1) entry_floats)
    float *ws_unit = ws ? ws + (size_t)u * (G - 1) * entry_floats(NC) : nullptr;
    unsigned *flags_unit = flags ? flags + (size_t)u * G * G : nullptr;
    // this lane's 16 bytes of register group 0 of slot 0 of column tile c, inside an entry (producers: column tile 0, which at
    // d_v 64, where the moments are one's, is the one whose sixth slot holds them)
    const size_t lane_off = (size_t)(is_p ? 0 : c) * WS_WAVE_SLOTS * kSlotFloats + (size_t)lane * 4;
    // the wave with the moments: at d_v 128 the consumer that builds no intra-chunk block, else producer 0 (the other way round at 128 producer 0 was
    // the one that all others waited for: 4240 cycles a chunk instead of 3700)
    const bool holds_x = w == x_wave(NC);

    // A main pass that starts from entries waits for the increments of this call (the last segment also for the initial state to have been
    // read) while its producers stage the first chunk and build what does not need the sum: 16 units of 777 tokens from a state
    // 18.1 us with the wait at the start, 17.0 with it here; without one, d_v 128 22.0, 19.5.
    const bool handed = SEG && seg > 0, from_entries = SEG && seg > 1, waits = SEG && (seg > 1 || (seg == 1 && has_init && G == 2));
    const float *hand = reinterpret_cast<const float *>(reinterpret_cast<const unsigned char *>(&lds) + hand_at(NC)) + 4 * lane;
    auto handed_tile = [&](int slot) {   // what the workgroup's own increment has left
        f32x16 x;
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            const f32x4 t = *reinterpret_cast<const f32x4 *>(hand + slot * kSlotFloats + j * 256);
#pragma unroll
            for (int i = 0; i < 4; ++i) x[4 * j + i] = t[i];
        }
        return x;
    };
    auto wait_flags = [&]() {   // one thread
        bool gave_up = false;
        for (int p = has_init && seg == G - 1 ? 0 : 1; p < seg; ++p) {
            unsigned *f = flags_unit + p * G + seg;
            int polls = 0;
            while (__hip_atomic_load(f, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM) != epoch) {
                if (polls++ >= max_polls) { gave_up = true; break; }
                __builtin_amdgcn_s_sleep(8);
            }
            __hip_atomic_store(f, 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
        }
        // sticky: stays set until based_prefill_status has reported it
        if (gave_up) __hip_atomic_store(status, epoch, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
    };

    // Intra-chunk block bb of the chunk whose rows are staged, into generation b: 0 = key tile 0 against
    // query tile 0, 1 = key tile 0 against query tile 1, 2 = key tile 1 against query tile 1 (0 and 2 are
    // cut by the diagonal).  P^T = mask(1 + A^T + A^T^2 / 2), A^T = K Q^T: lane (g, n) is query 32 qt + n,
    // register r is key 32 kt + 8 (r / 4) + 4 g + r % 4.  Keys past the end of the segment come after every
    // valid query and fall to the causal mask.  Built by the consumer waves (one block each) at d_v 128, which wait
    // for the producers otherwise, and by the producers at d_v 64, which has only two consumers.
    auto build_block = [&](const int b, const int bb) {
        const int kt = bb == 2 ? 1 : 0, qt = bb == 0 ? 0 : 1;
        const bool diag = bb != 1;
        f32x16 P;
        zero16(P);
        const u32x4 kop = *reinterpret_cast<const u32x4 *>(&lds.rows[b].krow[32 * kt + n][8 * g]);
        const u32x4 qop = *reinterpret_cast<const u32x4 *>(&lds.rows[b].qrow[32 * qt + n][8 * g]);
        P = mfma(as_bf16x8(kop), as_bf16x8(qop), P);
        float dsum = 0.f;
#pragma unroll
        for (int r = 0; r < 16; ++r) {
            const float x = P[r];
            float pv = fmaf(x, fmaf(x, 0.5f, 1.f), 1.f);
            const int key = 8 * (r >> 2) + 4 * g + (r & 3);
            pv = (!diag || key <= n) ? pv : 0.f;
            P[r] = pv;
            dsum += pv;
        }
        lds.pop[b][bb][0][lane] = as_u32x4(pack8_acc(P, 0));
        lds.pop[b][bb][1][lane] = as_u32x4(pack8_acc(P, 1));
        dsum += __shfl_xor(dsum, 32, 64);
        if (g == 0) lds.den[b][1 + kt][32 * qt + n] = dsum;
    };
    // which blocks a consumer builds: of four consumers c = 0..2 one each
    auto build_my_blocks = [&](const int b) {
        if (NC == 4) {
#pragma unroll
            for (int bb = 0; bb < 3; ++bb)
                if (c == bb) build_block(b, bb);
        }
    };

    using I = Image<NC>;
    static_assert(sizeof(Lds<NC>) <= kLdsBytes && sizeof(float) * NC * 32 * NTILE * IMG_LD <= kLdsBytes, "");
    float *image = reinterpret_cast<float *>(&lds);
    float *image_lane = image + c * 32 * NTILE * IMG_LD + 4 * g * IMG_LD + n;   // (consumers)
    auto export_image = [&]() {
#pragma unroll 5
        for (int st = 0; st < I::STEPS; ++st) {
            const int i = st * I::NTHR + tid;
            const CanonRows cr = I::rows(i, packed_state);
            if (i < I::Q && cr.r1 >= 0) {
                const f32x4 t = *reinterpret_cast<const f32x4 *>(I::piece(image, i));
                float *p = Su + 4 * (i % (DV / 4));
                *reinterpret_cast<f32x4 *>(p + (size_t)cr.r1 * DV) = t;
                if (cr.r2 != cr.r1) *reinterpret_cast<f32x4 *>(p + (size_t)cr.r2 * DV) = t;
            }
        }
    };
    float *zu = Su ? Su + (size_t)(packed_state ? packed_feature_dim(DP) : feature_dim(DP)) * DV : nullptr;
    auto row_operand = [&](const uint16_t (*rows)[RB_LD], int t) {   // row 32 t + n
        const uint16_t *p = &rows[32 * t + n][4 * g];
        const u32x2 x = *reinterpret_cast<const u32x2 *>(p), y = *reinterpret_cast<const u32x2 *>(p + 8);
        return as_bf16x8(u32x4{x[0], x[1], y[0], y[1]});
    };
    // Inter-chunk denominators of both query tiles from the moments: count + q.z1 + q^T M q / 2.
    auto build_den = [&](const int b, const f32x16 &X) {
        u32x4 o[2];   // elements 4 g .., 8 + 4 g .. of the queries
#pragma unroll
        for (int qt = 0; qt < 2; ++qt) o[qt] = as_u32x4(row_operand(lds.rows[b].qrow, qt));
        float mres[8];
        const bf16x8 mhi = pack8_acc(X, 0);
        {
            const u32x4 hb = __builtin_bit_cast(u32x4, mhi);
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                mres[2 * i] = X[2 * i] - bf16lo(hb[i]);
                mres[2 * i + 1] = X[2 * i + 1] - bf16hi(hb[i]);
            }
        }
        const bf16x8 mlo = pack8(mres);
        const float cnt_prev = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(X[8]), 16));
        f32x16 T[2];
#pragma unroll
        for (int qt = 0; qt < 2; ++qt) {
            zero16(T[qt]);
            T[qt] = mfma(mhi, as_bf16x8(o[qt]), T[qt]);
            T[qt] = mfma(mlo, as_bf16x8(o[qt]), T[qt]);
        }
#pragma unroll
        for (int qt = 0; qt < 2; ++qt) {
            float d2 = 0.f;
            // row of T[e] = 8 (e / 4) + 4 g + e % 4
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                d2 = fmaf(T[qt][2 * e], bf16lo(o[qt][e]), d2);
                d2 = fmaf(T[qt][2 * e + 1], bf16hi(o[qt][e]), d2);
            }
            const float d = fmaf(d2, 0.5f, T[qt][8]);   // T[8]: row 16 = q.z1 on g = 0, zero on g = 1
            const float tot = d + __shfl_xor(d, 32, 64) + cnt_prev;
            if (g == 0) lds.den[b][0][32 * qt + n] = tot;
        }
    };
    // M' += K'^T K' of a chunk (the operand of tile 4 carries k as given in rows 0..15 and the valid flag in row 16)
    auto add_moments = [&](const int b, f32x16 &X) {
#pragma unroll
        for (int ts = 0; ts < 4; ++ts) {
            const bf16x8 e = as_bf16x8(lds.phik[b][NTILE - 1][ts][lane]);
            X = mfma(e, e, X);
        }
    };
    auto import_moments = [&](f32x16 &X) {
#pragma unroll
        for (int r = 0; r < 16; ++r) X[r] = initial_moment(zu, 8 * (r >> 2) + 4 * g + (r & 3), n, packed_state);
    };
    // where row 8 (r / 4) + 4 g + r % 4 of the moments goes, column n (-1: nowhere), and its value from there
    auto moment_place = [&](int r) {
        const int fl = 8 * (r >> 2) + 4 * g + (r & 3);
        if (fl < DP && n < DP) return !packed_state || fl <= n ? canon_pair(fl, n, packed_state).r1 : -1;
        return fl != DP || n > DP ? -1 : n == DP ? 0 : 1 + n;
    };
    auto export_moment = [&](int place, float m) {
        if (place >= 0) zu[place] = place > DP ? m * kRsqrt2 : m;
    };
    auto moments_lds = [&](int r) -> float & { return reinterpret_cast<float *>(&lds)[image_bytes(NC) / 4 + 64 * r + (threadIdx.x & 63)]; };   // register r
    // A key with an element that is not finite.  Its row comes as products with 0/1 matrices, which makes NaN of all of the token's features, of the count of tokens
    // too.  No output of a token that sees it is finite in any case, but the state's rows without the element are: where the count is NaN at the end of the
    // sequence, the state is computed anew, from the rows in memory, element by element.  (us, not at all, so, and with a look at every tile and increment: 256
    // units of 2048 tokens, d_v 128, 82.0, 82.1, 82.8; 128 of 2048, d_v 64, 35.2, 35.1, 35.2; 16 of 777 from a state 15.55, 15.7, 15.7.)
    auto state_by_element = [&]() {   // a wave takes a tile of 32 rows and 32 columns at a time, or the moments, in the layout of accumulators
        if (has_init) {
            import_state_image<NC>(image, Su, packed_state, tid);
            __syncthreads();
        }
#pragma unroll 1
        for (int i = w; i < NC * NTILE + 1; i += NC + NPW) {
            const bool x = i == NC * NTILE;
            const int T = x ? NTILE - 1 : i % NTILE, col = i / NTILE * 32 + n;
            if (x) {
#pragma unroll 1
                for (int r = 0; r < 16; ++r) moments_lds(r) = has_init ? initial_moment(zu, 8 * (r >> 2) + 4 * g + (r & 3), n, packed_state) : 0.f;
            }
            float *at = x ? &moments_lds(0) : image + i * 32 * IMG_LD + 4 * g * IMG_LD + n;
            f32x16 acc;
#pragma unroll
            for (int r = 0; r < 16; ++r) acc[r] = x || has_init ? at[x ? 64 * r : (8 * (r >> 2) + (r & 3)) * IMG_LD] : 0.f;
#pragma unroll 1
            for (int t = 0; t < N; t += 16) {
                float ke[8], ve[8];
#pragma unroll
                for (int e = 0; e < 8; ++e) {
                    const int tok = t + 8 * (e >> 2) + 4 * g + (e & 3);
                    const size_t row = min(tok, N - 1);
                    const float kx = phik_element(ku + row * DP, T, n), vx = bf16_at(vu + row * DV + (x ? 0 : col));
                    ke[e] = tok < N && !(x && n > DP) ? kx : 0.f;
                    ve[e] = x ? ke[e] : tok < N ? vx : 0.f;
                }
                acc = mfma(pack8(ke), pack8(ve), acc);
            }
#pragma unroll
            for (int r = 0; r < 16; ++r) at[x ? 64 * r : (8 * (r >> 2) + (r & 3)) * IMG_LD] = acc[r];
        }
        __syncthreads();
    };
    // The moments' wave leaves them in LDS; the first four producers, which wait for the end, have worked out where they go.  (us, by that wave itself and so, in a
    // graph: 16 units of 64 tokens, d_v 64 5.9, 5.75, d_v 128, where it is a consumer, 7.5, 7.3; 300 units 13.05, 12.8 and 18.4, 17.85.)
    auto finish_moments = [&](const f32x16 &X) {
        if (X[8] != X[8]) anew = 1u;   // (register 8: the row of the constant)
#pragma unroll
        for (int r = 0; r < 16; ++r) moments_lds(r) = X[r];
    };
    if (tid == 0) anew = 0u;   // (ordered before its use by the barriers of the first chunk)
    if (has_init && seg == 0) {
        import_state_image<NC>(image, Su, packed_state, tid);
        __syncthreads();
    }
    // every wave, once it has what it needs of the image
    auto state_was_read = [&]() {
        // (a barrier does not wait for loads into registers, and the flag lets another workgroup overwrite what they read)
        asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
        __syncthreads();
        if (SEG) {
            if (tid == 0) __hip_atomic_store(flags_unit + (G - 1), epoch, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
        }
    };
    int place[4];   // of the moments that the first four producers write
    if (!is_p) {
        // =================================== consumer waves =========================================
        f32x16 S[NTILE];       // the five state tiles of this wave's 32 columns
#pragma unroll
        for (int T = 0; T < NTILE; ++T) zero16(S[T]);

        f32x16 X;              // the moment tile M' = [k, 1]^T [k, 1], of consumer 3 of four
        zero16(X);
        const bool has_x = NC == 4 && holds_x;
        if (has_init && seg == 0) {   // the caller's state
            if (has_x) import_moments(X);
#pragma unroll
            for (int T = 0; T < NTILE; ++T)
#pragma unroll
                for (int r = 0; r < 16; ++r) S[T][r] = image_lane[(32 * T + 8 * (r >> 2) + (r & 3)) * IMG_LD];
            state_was_read();
        }
        if (handed) {
#pragma unroll
            for (int T = 0; T < NTILE; ++T) S[T] = handed_tile(6 * c + T);
            if (has_x) X = handed_tile(6 * x_tile(NC) + 5);
            wg_sync();
        }

        {
            // V operand of an MFMA (lane (g, n): column 32 c + n at the 8 tokens of its k-slots, two runs of
            // 4 consecutive tokens starting at tok4 and tok4 + 8) from the row-major V rows: the transposing
            // LDS read.  In each group of 16 lanes, lane k supplies the address of 4 consecutive columns
            // (4 (k % 4) ..) of row k / 4 of the group's 16-column block and receives column k of that
            // block at the 4 rows.  The same registers serve as A operand (V^T, output product) and as B
            // operand (update).
            const int tr_kk = lane & 15, tr_grp = (lane >> 4) & 1;
            const uint16_t *tr_base = &lds.vrow[0][(tr_kk >> 2) + 4 * g][32 * c + 16 * tr_grp + 4 * (tr_kk & 3)];
            auto load_v = [&](int b, int ts) {   // tokens 16 ts + 4 g + {0..3, 8..11}
                const uint16_t *p = tr_base + (b * C + 16 * ts) * VR_LD;
                const s16x4 lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((__attribute__((address_space(3))) s16x4 *)p);
                const s16x4 hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((__attribute__((address_space(3))) s16x4 *)(p + 8 * VR_LD));
                s16x8 o;
#pragma unroll
                for (int i = 0; i < 4; ++i) { o[i] = lo[i]; o[4 + i] = hi[i]; }
                return __builtin_bit_cast(bf16x8, o);
            };

            wg_sync();   // the producers have staged the first chunk
            build_my_blocks(0);
            if (has_x && !from_entries) build_den(0, X);
            if (waits && tid == 0) wait_flags();
            wg_sync();   // the operands of the first chunk are visible (but the denominators, where these need the entries)
            if (from_entries) {   // the increments of earlier segments
                for (int p = 1; p < seg; ++p) {
                    const float *e = ws_unit + (size_t)(p - 1) * entry_floats(NC) + lane_off;
                    f32x4 x[24];
                    load_wave_slots_coherent(e + 1 * kSlotFloats, e + 3 * kSlotFloats, e + 5 * kSlotFloats, x);
#pragma unroll
                    for (int T = 0; T < NTILE; ++T)
#pragma unroll
                        for (int r = 0; r < 16; ++r) S[T][r] += x[T * 4 + (r >> 2)][r & 3];
                    if (has_x) {
#pragma unroll
                        for (int r = 0; r < 16; ++r) X[r] += x[20 + (r >> 2)][r & 3];
                    }
                }
                if (has_x) build_den(0, X);
                wg_sync();
            }
            for (int t = 0; t < n_chunks; ++t) {
                const int b = t & 1;
                const int tok0 = tok_begin + C * t;
                bf16x8 vop[4];
#pragma unroll
                for (int ts = 0; ts < 4; ++ts) vop[ts] = load_v(b, ts);
                f32x16 Y[2];
                float dn[2][3];
                // ---- readout: Y^T of query tile qt: lane (g, n) = query 32 qt + n, register r = column
                // 32 c + 8 (r / 4) + 4 g + r % 4.  The bf16 copy of a state tile (a register-local
                // conversion: accumulator registers 8 sl .. 8 sl + 7 are the k-slots of slab 2T + sl) is the
                // A operand.  The LDS loads go out in groups, into registers of their own, ahead of the
                // matrix instructions that consume them.
                constexpr int RG = 5, NG = NSLAB / RG;
                u32x4 o[2][RG][2];
                auto load_group = [&](int gi) {
#pragma unroll
                    for (int sl = 0; sl < RG; ++sl)
#pragma unroll
                        for (int qt = 0; qt < 2; ++qt) o[gi & 1][sl][qt] = lds.phiq[b][qt][RG * gi + sl][lane];
                };
                load_group(0);
                zero16(Y[0]); zero16(Y[1]);
#pragma unroll
                for (int gi = 0; gi < NG; ++gi) {
                    if (gi + 1 < NG) load_group(gi + 1);
                    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
                    for (int sl = 0; sl < RG; ++sl) {
                        const bf16x8 sb = pack8_acc(S[(RG * gi + sl) >> 1], (RG * gi + sl) & 1);
#pragma unroll
                        for (int qt = 0; qt < 2; ++qt) Y[qt] = mfma(sb, as_bf16x8(o[gi & 1][sl][qt]), Y[qt]);
                    }
                }
                u32x4 op[3][2];
#pragma unroll
                for (int bb = 0; bb < 3; ++bb)
#pragma unroll
                    for (int sl = 0; sl < 2; ++sl) op[bb][sl] = lds.pop[b][bb][sl][lane];
                // intra-chunk: Y^T += V^T P^T over the key tiles at or before the query tile
#pragma unroll
                for (int sl = 0; sl < 2; ++sl) {
                    Y[0] = mfma(vop[sl], as_bf16x8(op[0][sl]), Y[0]);
                    Y[1] = mfma(vop[sl], as_bf16x8(op[1][sl]), Y[1]);
                }
#pragma unroll
                for (int sl = 0; sl < 2; ++sl) Y[1] = mfma(vop[2 + sl], as_bf16x8(op[2][sl]), Y[1]);
                if (NC == 4) {
                    const bool has_next = t + 1 < n_chunks;
                    if (has_next) build_my_blocks(b ^ 1);
                    if (has_x) {
                        add_moments(b, X);
                        if (has_next) build_den(b ^ 1, X);
                    }
                }

                // ---- update: S += phi(K)^T V over all 160 rows, the outputs normalised and turned between the matrix instructions
                u32x4 ok[4][NTILE];
#pragma unroll
                for (int qt = 0; qt < 2; ++qt)
#pragma unroll
                    for (int d = 0; d < 3; ++d) dn[qt][d] = lds.den[b][d][32 * qt + n];
#pragma unroll
                for (int ts = 0; ts < 4; ++ts)
#pragma unroll
                    for (int T = 0; T < NTILE; ++T) ok[ts][T] = lds.phik[b][T][ts][lane];
                __builtin_amdgcn_sched_barrier(0);
                // the halves of a wave exchange quads of columns: 16 bytes a lane, columns 32 c + 16 jj + 8 g .. of query 32 qt + n
                u32x4 val[2][2];
#pragma unroll
                for (int qt = 0; qt < 2; ++qt) {
                    const float inv = numerator_only ? 1.f : __builtin_amdgcn_rcpf(dn[qt][0] + dn[qt][1] + dn[qt][2]);
#pragma unroll
                    for (int jj = 0; jj < 2; ++jj) {
                        u32x2 p[2];
#pragma unroll
                        for (int k2 = 0; k2 < 2; ++k2) {
                            f32x4 o;
#pragma unroll
                            for (int i = 0; i < 4; ++i) o[i] = Y[qt][8 * jj + 4 * k2 + i] * inv;
                            p[k2] = __builtin_bit_cast(u32x2, __builtin_convertvector(o, bf16x4));
                        }
                        const auto x = __builtin_amdgcn_permlane32_swap(p[0][0], p[1][0], false, false);
                        const auto z = __builtin_amdgcn_permlane32_swap(p[0][1], p[1][1], false, false);
                        val[qt][jj] = u32x4{x[0], z[0], x[1], z[1]};
                    }
                }
#pragma unroll
                for (int ts = 0; ts < 4; ++ts)
#pragma unroll
                    for (int T = 0; T < NTILE; ++T) S[T] = mfma(as_bf16x8(ok[ts][T]), vop[ts], S[T]);
#pragma unroll
                for (int i = 0; i < 4 * NTILE; ++i) {
                    __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);   // a matrix instruction,
                    __builtin_amdgcn_sched_group_barrier(0x002, 4, 0);   // vector instructions
                }
                __builtin_amdgcn_sched_barrier(0);
                uint16_t *yc = yu + (size_t)tok0 * DV;
                const uint32_t yoff = (uint32_t)n * (uint32_t)DV + (uint32_t)(32 * c + 8 * g);
                if (tok0 + C <= tok_end) {
#pragma unroll
                    for (int qt = 0; qt < 2; ++qt)
#pragma unroll
                        for (int jj = 0; jj < 2; ++jj) *reinterpret_cast<u32x4 *>(yc + yoff + 32 * qt * DV + 16 * jj) = val[qt][jj];
                } else {
#pragma unroll
                    for (int qt = 0; qt < 2; ++qt)
#pragma unroll
                        for (int jj = 0; jj < 2; ++jj)
                            if (tok0 + 32 * qt + n < tok_end) *reinterpret_cast<u32x4 *>(yc + yoff + 32 * qt * DV + 16 * jj) = val[qt][jj];
                }
                wg_sync();   // the next chunk's operands are visible; this chunk's are free
            }
        }

        // ---- end of segment --------------------------------------------------------------------
        if (Su && seg == G - 1) {
#pragma unroll
            for (int T = 0; T < NTILE; ++T)
#pragma unroll
                for (int r = 0; r < 16; ++r) image_lane[(32 * T + 8 * (r >> 2) + (r & 3)) * IMG_LD] = S[T][r];
            if (has_x) finish_moments(X);
        }
    } else {
        // =================================== producer waves =========================================
        const int ptid = tid - 64 * NC;   // thread index among the producers
        f32x16 X;                      // the moment tile, of producer 0 of six
        zero16(X);
        const bool has_m = NC == 2 && holds_x;
        if (has_init && seg == 0 && has_m) import_moments(X);
        if (handed && has_m) X = handed_tile(6 * x_tile(NC) + 5);

        {
            // ---- staging: global -> registers -> LDS --------------------------------------------
            // A chunk of V is one contiguous block of 64 rows x DV columns, in 16-byte pieces: piece p is row p / (DV / 8), columns
            // 8 (p % (DV / 8)) ...  A chunk of K (and of Q) is 128 pieces: piece p holds elements 8 (p % 2) .. of token p / 2.  A wave
            // moves 64 pieces at a time.  Of four producers each has a quarter of V and half of K or Q.  Of six, 0 and 1 stage K, 4 and 5 Q, and
            // 1 three eighths of V, the others one: as much as the builds leave time for (each with its own share of K or Q and of V: a chunk takes 6 % more
            // cycles).
            constexpr int VPR = DV / 8;   // pieces per V row
            constexpr int NVP = NPW == 6 ? 3 : 4;   // V pieces per producer thread, at most
            static_assert(NP == 64 * NPW && VPR * C == (NPW == 6 ? 8 : 16) * 64, "");
            const int first_v = NPW == 4 ? 4 * c : c == 0 ? 0 : c == 1 ? 1 : c + 2;
            const int n_v = NPW == 4 ? 4 : c == 1 ? 3 : 1;
            const bool is_k = c < 2, has_x = NPW == 4 || c < 2 || c > 3;
            const int xp = 64 * (c & 1) + lane, x_tok = xp >> 1, x_h = xp & 1;
            u32x4 raw_x = {0u, 0u, 0u, 0u};   // the thread's piece of K or Q
            u32x4 raw_v[NVP];
            // Loads are not conditional on the lane (rows past the end of the segment re-read its last row and are
            // zeroed when staged): a conditional load would have the compiler pre-zero its destination
            // registers, and before that write it waits for every memory operation still in flight.
            auto v_piece = [&](int j) { return 64 * (first_v + j) + lane; };
            auto load_x = [&](int tok0) {
                if (!has_x) return;
                tok0 = min(tok0, tok_end - 1);
                const uint16_t *src = (is_k ? ku : qu) + (size_t)tok0 * DP;
                raw_x = *reinterpret_cast<const u32x4 *>(src + (uint32_t)(min(x_tok, tok_end - 1 - tok0) * DP + 8 * x_h));
            };
            auto load_v = [&](int tok0) {
                tok0 = min(tok0, tok_end - 1);
                const uint16_t *src = vu + (size_t)tok0 * DV;
#pragma unroll
                for (int j = 0; j < NVP; ++j) {
                    if (j >= n_v) break;
                    const int p = v_piece(j);
                    raw_v[j] = *reinterpret_cast<const u32x4 *>(src + (uint32_t)(min(p / VPR, tok_end - 1 - tok0) * DV + 8 * (p % VPR)));
                }
            };
            auto stage_x = [&](int tok0, int b) {
                if (!has_x) return;
                auto &rows = lds.rows[b];
                u32x4 raw = raw_x;
                if (is_k && tok0 + x_tok >= tok_end) raw = u32x4{0u, 0u, 0u, 0u};
                *reinterpret_cast<u32x4 *>(is_k ? &rows.krow[x_tok][8 * x_h] : &rows.qrow[x_tok][8 * x_h]) = raw;
            };
            auto stage_v = [&](int tok0, int b) {
                const u32x4 zero4 = {0u, 0u, 0u, 0u};
#pragma unroll
                for (int j = 0; j < NVP; ++j) {
                    if (j >= n_v) break;
                    const int p = v_piece(j);
                    const int row = p / VPR;
                    *reinterpret_cast<u32x4 *>(&lds.vrow[b][row][8 * (p % VPR)]) = tok0 + row < tok_end ? raw_v[j] : zero4;
                }
            };

            // ---- builders of the shared operands (b: the generation they write) ------------------
            // A tile of 32 rows multiplied with a 0/1 matrix comes back as accumulators: in fp32, without rounding, transposed and in any order of
            // the elements, in the registers and lanes that an operand is built from.  k-slot (jj, i) of lane half g is element 8 jj + 4 g + i.
            const int m = lane & 15;
            const bf16x8 first_eye = one_at(g, m, 0x3F80u);                       // lane n: element n % 16
            const bf16x8 second_eye = one_at(g, (m + (n >> 4)) & 15, 0x3F80u);    // element (n + n / 16) % 16
            const bf16x8 pair_eye = one_at(g, n >= 24 ? n - 24 : -1, 0x3F80u);    // lanes 24 .. 31: element n - 24
            const bf16x8 turned_eye = one_at(g, (4 * ((n >> 2) & 1) + 4 * (n >> 3) + (n & 3)) & 15, 0x3F80u);   // register j: element (4 g + j) % 16
            // phi(Q)^T operands of query tile qt, all ten slabs: lane (g, n) is query 32 qt + n; k-slot
            // (jj, i) of slab s is feature row 16 s + 8 jj + 4 g + i.  xr[j] = c_q q[(4g + j) % 16] is the
            // lane's query row rotated by 4g, so that the "a side" of k-slot (jj, i) is xr[8 jj + i] and the
            // "b side" of delta is xr[(8 jj + i + delta) % 16]: every product is between two registers known
            // at compile time.
            auto build_phiq = [&](const int b, const int qt) {
                const bf16x8 qr = row_operand(lds.rows[b].qrow, qt);
                f32x16 xr;
                zero16(xr);
                xr = mfma(turned_eye, qr, xr);
                xr *= kCQ;
#pragma unroll
                for (int s = 0; s < 8; ++s) {   // pair slabs: delta = s
                    float pr[8];
#pragma unroll
                    for (int jj = 0; jj < 2; ++jj)
#pragma unroll
                        for (int i = 0; i < 4; ++i) {
                            const int a = 8 * jj + i;
                            const float av = s == 0 ? xr[a] * 0.5f : xr[a];   // delta = 0: x_a^2 / sqrt(2)
                            pr[4 * jj + i] = av * xr[(a + s) & 15];
                        }
                    lds.phiq[b][qt][s][lane] = as_u32x4(pack8(pr));
                }
                lds.phiq[b][qt][8][lane] = as_u32x4(qr);   // slab 8: the linear rows, q itself as given
                {   // slab 9: the constant row (k-slot 0 of g = 0 = row 16 of the tile), padding, and the
                    // delta = 8 rows (k-slots 4 + i = row 24 + 4g + i: sqrt(2) q_a q_(a+8), a = 4g + i)
                    float pr[8];
                    pr[0] = g == 0 ? 1.f : 0.f; pr[1] = 0.f; pr[2] = 0.f; pr[3] = 0.f;
#pragma unroll
                    for (int i = 0; i < 4; ++i) pr[4 + i] = xr[i] * xr[8 + i];
                    lds.phiq[b][qt][9][lane] = as_u32x4(pack8(pr));
                }
            };
            // phi(K)^T operands of the chunk's tokens 32 hh .., all five state tiles: lane (g, n) is feature row n of a
            // tile, its k-slots are the tokens 16 ts + 4 g + {0..3, 8..11}.  Pair rows are k_a k_b / sqrt(2): the first factor is the same
            // (a = n % 16) in four tiles, the second one that of tile 0 from a lane 2T further.  Tile 4: k as given (sqrt(2) k / sqrt(2)
            // differs from k by fp32 rounding only, far below half a bf16 step, so the conversion returns it exactly), the constant 1, pairs.  valid: the
            // chunk's tokens before the end (behind it the constant is 0).
            auto build_phik = [&](const int b, const int hh, const int valid) {
                const bf16x8 kr = row_operand(lds.rows[b].krow, hh);
                f32x16 ka, kb, kp;
                zero16(ka); zero16(kb);
#pragma unroll
                for (int r = 0; r < 16; ++r) kp[r] = n < DP ? kSqrt2 : 0.f;
                ka = mfma(kr, first_eye, ka);
                kb = mfma(kr, second_eye, kb);
                kp = mfma(kr, pair_eye, kp);
                ka *= kRsqrt2;
                float one[16];
#pragma unroll
                for (int r = 0; r < 16; ++r) one[r] = n == DP ? 1.f : 0.f;
                if (valid < C) {   // uniform
#pragma unroll
                    for (int r = 0; r < 16; ++r) one[r] = 32 * hh + 8 * (r >> 2) + 4 * g + (r & 3) < valid ? one[r] : 0.f;
                }
#pragma unroll
                for (int s = 0; s < 2; ++s) {
                    auto tile = [&](auto tag) {
                        constexpr int T = decltype(tag)::value;
                        float pr[8];
#pragma unroll
                        for (int e = 0; e < 8; ++e)
                            pr[e] = T < 4 ? ka[8 * s + e] * rotate16<2 * T>(kb[8 * s + e]) : fmaf(ka[8 * s + e], kp[8 * s + e], one[8 * s + e]);
                        lds.phik[b][T][2 * hh + s][lane] = as_u32x4(pack8(pr));
                    };
                    tile(std::integral_constant<int, 0>{});
                    tile(std::integral_constant<int, 1>{});
                    tile(std::integral_constant<int, 2>{});
                    tile(std::integral_constant<int, 3>{});
                    tile(std::integral_constant<int, 4>{});
                }
            };
            // The producers' share of the operands of the chunk from tok0 on, into generation b (the intra-chunk blocks
            // and the denominators are built by the consumers at d_v 128).  Waves 0, 1: phi(Q) of a query tile;
            // 2, 3: phi(K) of half of the tokens each.  Of six (d_v 64), 0: denominators and the intra-chunk block off the diagonal; 1, 4: phi(K); 2, 3, which share a SIMD with a consumer: phi(Q), the
            // shortest; 5: the blocks on the diagonal.
            auto build = [&](const int b, const bool den, const int tok0) {   // den: the denominators too
                const int valid = tok_end - tok0;
                if (NPW == 6) {
                    if (c == 0) {
                        role_guard();
                        if (den) build_den(b, X);
                        build_block(b, 1);
                    } else if (c == 1 || c == 4) {
                        role_guard();
                        build_phik(b, c >> 2, valid);
                    } else if (c < 4) {
                        role_guard();
                        build_phiq(b, c - 2);
                    } else {
                        role_guard();
                        build_block(b, 0);
                        build_block(b, 2);
                    }
                } else {
                    role_guard();
                    if (c < 2) {
                        build_phiq(b, c);
                    } else {
                        build_phik(b, c - 2, valid);
                    }
                }
            };

            // ---- the producers' loop: operands one chunk ahead of the consumers, rows two ahead of them ----
            // in registers: V of chunk t + 1, K and Q of chunk t + 2
            auto stage_next = [&](int t) {
                const int tok_next = tok_begin + C * (t + 1);
                stage_v(tok_next, (t + 1) & 1);
                stage_x(tok_next + C, t & 1);
            };
            auto load_next = [&](int t) {   // for stage_next(t)
                const int tok_next = tok_begin + C * (t + 1);
                load_v(tok_next);
                load_x(tok_next + C);
            };
            load_x(tok_begin);
            load_v(tok_begin);
            if (has_init && seg == 0) state_was_read();
            if (handed) wg_sync();   // what the increment has left has been read
            // once: the row sums of a block that does not exist (key tile 1 against query tile 0)
            // (only the first 32 queries of den[.][2]: the other half belongs to block 2, whose builder does
            // not wait for this wave)
            if (ptid < 32) {
                lds.den[0][2][ptid] = 0.f;
                lds.den[1][2][ptid] = 0.f;
            }
            stage_x(tok_begin, 0);
            load_x(tok_begin + C);
            wg_sync();   // the first chunk's rows are staged
            stage_next(-1);
            load_next(0);
            build(0, !from_entries, tok_begin);
            wg_sync();   // the first chunk's operands are visible
            if (from_entries) {
                if (has_m) {
                    role_guard();
                    for (int p = 1; p < seg; ++p) {
                        const float *e = ws_unit + (size_t)(p - 1) * entry_floats(NC) + lane_off;
                        f32x4 x[24];
                        load_wave_slots_coherent(e + 1 * kSlotFloats, e + 3 * kSlotFloats, e + 5 * kSlotFloats, x);
#pragma unroll
                        for (int r = 0; r < 16; ++r) X[r] += x[20 + (r >> 2)][r & 3];
                    }
                    build_den(0, X);
                }
                wg_sync();
            }
            for (int t = 0; t < n_chunks; ++t) {
                const int b = t & 1;
                const bool has_next = t + 1 < n_chunks;
                if (has_next) stage_next(t);
                if (has_next) load_next(t + 1);   // (rows past the end: the last one again)
                if (has_m) {   // of the chunk the consumers are working on; the denominators of the next chunk need it
                    role_guard();
                    add_moments(b, X);
                }
                if (has_next) build(b ^ 1, true, tok_begin + C * (t + 1));
                wg_sync();   // the next chunk's operands are visible
            }
        }

        // ---- end of segment: the moments ----------------------------------------------------------
        if (has_m && Su && seg == G - 1) finish_moments(X);
        if (c < 4) {
#pragma unroll
            for (int j = 0; j < 4; ++j) place[j] = moment_place(4 * c + j);
        }
    }
    if (Su && seg == G - 1) {
        __syncthreads();
        if (__builtin_expect(__builtin_amdgcn_readfirstlane(anew) != 0u, 0)) state_by_element();
        if (is_p && c < 4) {
#pragma unroll
            for (int j = 0; j < 4; ++j) export_moment(place[j], moments_lds(4 * c + j));
        }
        export_image();
    }
}

// State increment of segment `seg`, left in LDS for the main pass of the next segment and, where a later one needs it too, in workspace entry 1 + seg.
//
// The eight waves need no operand from each other here, so nothing but the rows passes through LDS, and a step has one barrier.  Wave r = w % 4
// owns tile r for two column tiles (waves 2 and 3 also tile 4, for one of them; wave 1 the moments), and a feature is a product of two
// values in its registers: multiplied with 0/1 matrices a tile of 32 rows of K comes back as accumulators, in fp32 and without rounding, with lane
// n holding k_a / sqrt(2) or the k_b of its row and the registers going over the tokens in the order of an operand's k-slots.  At d_v 64 the waves 0-3
// and 4-7 take alternate tiles of 32 tokens and are added up at the end; at d_v 128 they own 64 columns each.  The rows come by the 16-byte LDS
// DMA (a V row's pieces permuted, so that the transposing reads spread over the banks), three to four steps ahead.  The features are the main pass's to
// the bit: rounded as k_a k_b / 2, the sums scaled at the end, they left the state 0.2 to 0.5 % further from float64 (128 units of 2048 tokens, d_v 64 36.8 us either way, d_v 128
// 57.0, now 58.6; 16 of 777 from a state 16.0, now 15.6; figures of several segments at d_v 128 further down are mostly from before, 2 % less).
//
// Bound: memory, with half of the chip at increments and half at main passes (128 units: 1530 cycles a chunk at d_v 64, 2570 at 128, its start and the
// hand-over included); the matrix pipe would take 600 and 960.  As a producer / consumer pipeline like the main pass's, 2200 at d_v 64.
template <int NC>
__device__ __forceinline__ void increment_body(
    unsigned char *lds, const uint16_t *__restrict__ k, const uint16_t *__restrict__ v, const float *__restrict__ state, int has_init,
    float *__restrict__ ws, unsigned *__restrict__ flags, unsigned epoch, int N, const SegTable &segs, int G, int seg, int u)
{
    constexpr int DV = 32 * NC, HP = NC / 2;      // HP: 64-column parts
    constexpr int NH = 4 / HP;                    // 32-token tiles of a step
    constexpr int PART = 32 * 64 * 2, TILE_K = 32 * DP * 2, STAGE = 4 * PART + NH * TILE_K, RING = 5;
    constexpr int IMAGE = image_bytes(NC), AT = hand_at(NC);
    static_assert(AT + RING * STAGE <= kLdsBytes && 11 * 4096 <= IMAGE && IMAGE <= kLdsBytes && AT + NC * 6 * 4096 <= kLdsBytes, "");
    const bool packed_state = (has_init & 2) != 0;
    has_init &= 1;
    const int tid = threadIdx.x, lane = tid & 63;
    const int w = __builtin_amdgcn_readfirstlane(tid >> 6), r4 = w & 3, grp = w >> 2;
    const int g = lane >> 5, n = lane & 31, m = lane & 15;
    const uint32_t lds_addr = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) unsigned char *)lds;

    const int tok_begin = segs.begin[seg], tok_end = segs.begin[seg + 1];   // (whole chunks: the sequence's last segment has no increment)
    const int steps = (tok_end - tok_begin + 32 * NH - 1) / (32 * NH);
    const uint16_t *ku = k + (size_t)u * N * DP, *vu = v + (size_t)u * N * DV;

    // Wave w moves 16 rows of part w / 2 (d_v 64: of tile w / 2; d_v 128: of tile w / 4, columns 64 (w / 2 % 2) ..) and, for w < NH, tile w of
    // K.  A tile past the end is the step's first once more.
    const uint32_t off_v = (uint32_t)((lane >> 3) * DV * 2 + 16 * ((lane & 7) ^ (4 * ((lane >> 4) & 1))));
    const int part_tile = HP == 1 ? w >> 1 : w >> 2, part_col = HP == 1 ? 0 : 64 * ((w >> 1) & 1);
    auto issue = [&](int step) {
        step = min(step, steps - 1);
        const int tok0 = tok_begin + 32 * NH * step;
        const uint32_t to = lds_addr + (uint32_t)(AT + step % RING * STAGE);
        const int tv = tok0 + 32 * part_tile < tok_end ? tok0 + 32 * part_tile : tok0;
        const uint16_t *vb = vu + (size_t)(tv + 16 * (w & 1)) * DV + part_col;
        const uint32_t vt = to + (uint32_t)((w >> 1) * PART + 2048 * (w & 1));
        dma16(vb, off_v, vt);
        dma16(vb + 8 * DV, off_v, vt + 1024);
        if (w < NH) {
            const int tk = tok0 + 32 * w < tok_end ? tok0 + 32 * w : tok0;
            dma16(ku + (size_t)tk * DP, 16 * lane, to + (uint32_t)(4 * PART + w * TILE_K));
        }
    };
    const bool imports = has_init && seg == 0;
    auto issue_first = [&]() {
#pragma unroll
        for (int i = 0; i < RING - 1; ++i) issue(i);
    };
    if (HP == 1 || !imports) issue_first();

    // 0/1 matrices as B operands
    const bf16x8 first_eye = one_at(g, m, 0x3F80u);                              // k_a
    const bf16x8 second_eye = one_at(g, (m + 2 * r4 + (n >> 4)) & 15, 0x3F80u);   // k_b of tile r
    const bf16x8 pair_eye = one_at(g, n >= 24 ? n - 24 : -1, 0x3F80u);           // k_b of tile 4's pairs (k_a: lane n holds a = n - 16)
    const float row_linear = n < 16 ? kSqrt2 : 0.f, row_one = n == 16 ? 1.f : 0.f;

    // This wave's column tiles are c0, c0 + 1; waves 2, 3, 4 and 5 have tile 4 of column tile c0 + r % 2 as well (a matrix pipe serves waves w
    // and w + 4), wave 1, at d_v 64 also 7, the moments.
    const int c0 = HP == 1 ? 0 : 2 * grp, e4 = r4 & 1;
    const bool has4 = (grp == 0) == (r4 >= 2), has_x = grp == 0 ? r4 == 1 : HP == 1 && r4 == 3;
    f32x16 S[2], E;   // tile r of the column tiles; tile 4, or the moments
    zero16(S[0]); zero16(S[1]); zero16(E);
    if (imports) {   // (the state buffer's image: as in the main pass)
        const float *Su = state + (size_t)u * (packed_state ? packed_state_stride(DP, DV) : state_stride(DP, DV));
        const float *zu = Su + (size_t)(packed_state ? packed_feature_dim(DP) : feature_dim(DP)) * DV;
        const bool starts = HP == 2 || grp == 0;   // of two groups the first one starts from it
        if (has_x && starts) {
#pragma unroll
            for (int r = 0; r < 16; ++r) E[r] = initial_moment(zu, 8 * (r >> 2) + 4 * g + (r & 3), n, packed_state);
        }
        float *image = reinterpret_cast<float *>(lds);
        import_state_image<NC>(image, Su, packed_state, tid);
        wg_sync();
        if (starts) {
            const float *at = image + c0 * 32 * NTILE * IMG_LD + 4 * g * IMG_LD + n;
#pragma unroll
            for (int r = 0; r < 16; ++r) {
                const int row = 8 * (r >> 2) + (r & 3);
#pragma unroll
                for (int c = 0; c < 2; ++c) S[c][r] = at[(c * 32 * NTILE + 32 * r4 + row) * IMG_LD];
                if (has4) E[r] = at[(e4 * 32 * NTILE + 128 + row) * IMG_LD];
            }
        }
        if (HP == 2) {
            wg_sync();   // the image has been read
            issue_first();
        }
    }

    const int tr_lane = ((m >> 2) + 4 * g) * 128 + ((32 * ((lane >> 4) & 1) + 8 * (m & 3)) ^ (64 * ((m >> 3) & 1)));
    auto load_v = [&](const unsigned char *part, int s, int c) {   // columns 32 c + n, tokens 16 s + 4 g + {0..3, 8..11}
        const unsigned char *p = part + (tr_lane ^ (64 * c)) + 16 * 128 * s;
        const s16x4 lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((__attribute__((address_space(3))) s16x4 *)p);
        const s16x4 hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((__attribute__((address_space(3))) s16x4 *)(p + 8 * 128));
        s16x8 o;
#pragma unroll
        for (int i = 0; i < 4; ++i) { o[i] = lo[i]; o[4 + i] = hi[i]; }
        return __builtin_bit_cast(bf16x8, o);
    };
    auto load_k = [&](const unsigned char *tile) {   // row n: elements 4 g .., 8 + 4 g ..
        const unsigned char *p = tile + 32 * n + 8 * g;
        const u32x2 a = *reinterpret_cast<const u32x2 *>(p), b = *reinterpret_cast<const u32x2 *>(p + 16);
        return as_bf16x8(u32x4{a[0], a[1], b[0], b[1]});
    };
    // KIND: 0 a tile, 1 a tile and the moments, 2 a tile and tile 4.  The factors of a tile of 32 rows are on their way while the products of the
    // tile before are built and multiplied.
    auto run = [&](auto kind) {
        constexpr int KIND = decltype(kind)::value;
        const unsigned char *const ring = lds + AT;
        f32x16 a[2], b[2], f[2];
        auto factors = [&](int step, int i) {
            const bf16x8 kr = load_k(ring + step % RING * STAGE + 4 * PART + (HP == 2 ? i : grp + 2 * i) * TILE_K);
            zero16(a[i]); zero16(b[i]);
            a[i] = mfma(kr, first_eye, a[i]);
            b[i] = mfma(kr, second_eye, b[i]);
            a[i] *= kRsqrt2;
            if (KIND == 2) {
#pragma unroll
                for (int r = 0; r < 16; ++r) f[i][r] = row_linear;
                f[i] = mfma(kr, pair_eye, f[i]);
            }
        };
        auto products = [&](int i, const bf16x8 (&vo)[2][2]) {
#pragma unroll
            for (int s = 0; s < 2; ++s) {
                float pr[8];
#pragma unroll
                for (int e = 0; e < 8; ++e) pr[e] = a[i][8 * s + e] * b[i][8 * s + e];
                const bf16x8 op = pack8(pr);
#pragma unroll
                for (int c = 0; c < 2; ++c) S[c] = mfma(op, vo[s][c], S[c]);
                if (KIND == 2) {   // linear rows, the constant, pairs
#pragma unroll
                    for (int e = 0; e < 8; ++e) pr[e] = fmaf(a[i][8 * s + e], f[i][8 * s + e], row_one);
                    E = mfma(pack8(pr), e4 ? vo[s][1] : vo[s][0], E);
                } else if (KIND == 1) {
#pragma unroll
                    for (int e = 0; e < 8; ++e) pr[e] = fmaf(a[i][8 * s + e], row_linear, row_one);
                    const bf16x8 x = pack8(pr);
                    E = mfma(x, x, E);
                }
            }
        };
        // All waves' pieces of a step are there after a barrier that each has passed with its own there; N: younger steps in flight.
        auto arrived = [&](auto younger) {
            constexpr int Y = decltype(younger)::value;
            if (w < NH) asm volatile("s_waitcnt vmcnt(%0)" : : "n"(3 * Y) : "memory");
            else asm volatile("s_waitcnt vmcnt(%0)" : : "n"(2 * Y) : "memory");
            wg_sync();
        };
        arrived(std::integral_constant<int, RING - 2>{});
        factors(0, 0);
        for (int t = 0; t < steps; ++t) {
            arrived(std::integral_constant<int, RING - 3>{});   // step t + 1; step t - 1 has been read
            issue(t + RING - 1);
            const unsigned char *stage = ring + t % RING * STAGE;
            // tiles 0, 1 of the step (d_v 128), or grp, grp + 2 (d_v 64; the segment may end before the second of them)
            const bool both = HP == 2 || tok_begin + 32 * NH * t + 64 < tok_end;
            bf16x8 vo[2][2][2];
#pragma unroll
            for (int i = 0; i < 2; ++i)
#pragma unroll
                for (int s = 0; s < 2; ++s)
#pragma unroll
                    for (int c = 0; c < 2; ++c) vo[i][s][c] = load_v(stage + (HP == 2 ? 2 * i + grp : grp + 2 * i) * PART, s, c);
            factors(t, 1);
            products(0, vo[0]);
            factors(t + 1 < steps ? t + 1 : t, 0);
            if (both) products(1, vo[1]);
        }
    };
    if (has4) run(std::integral_constant<int, 2>{});
    else if (has_x) run(std::integral_constant<int, 1>{});
    else run(std::integral_constant<int, 0>{});

    // ---- the entry: slot 6 c + T, and slot 5 (the moments) ----
    const bool publish = seg + 2 < G;   // later segments need it, too
    float *e = ws + (size_t)u * (G - 1) * entry_floats(NC) + (size_t)seg * entry_floats(NC) + (size_t)lane * 4;
    float *hand = reinterpret_cast<float *>(lds + AT) + 4 * lane;
    auto put = [&](int slot, const f32x16 &x) {
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            const f32x4 o = {x[4 * j], x[4 * j + 1], x[4 * j + 2], x[4 * j + 3]};
            *reinterpret_cast<f32x4 *>(hand + slot * kSlotFloats + j * 256) = o;
            if (publish) store16_coherent(e + (size_t)slot * kSlotFloats + (size_t)j * 256, o);
        }
    };
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    if (HP == 1) {   // the groups' sums: the first one finishes column tile 0, the other one column tile 1 and E
        float *x = reinterpret_cast<float *>(lds) + 4 * lane;   // (the image's place)
        auto give = [&](int i, const f32x16 &y) {
#pragma unroll
            for (int j = 0; j < 4; ++j) *reinterpret_cast<f32x4 *>(x + i * 1024 + j * 256) = f32x4{y[4 * j], y[4 * j + 1], y[4 * j + 2], y[4 * j + 3]};
        };
        auto take = [&](int i, f32x16 &y) {
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                const f32x4 t = *reinterpret_cast<const f32x4 *>(x + i * 1024 + j * 256);
#pragma unroll
                for (int q = 0; q < 4; ++q) y[4 * j + q] += t[q];
            }
        };
        give(grp == 0 ? 4 + r4 : r4, grp == 0 ? S[1] : S[0]);
        if (grp == 0 && has4) give(8 + e4, E);
        if (grp == 0 && has_x) give(10, E);
        wg_sync();
        if (grp == 0) {
            take(r4, S[0]);
            put(r4, S[0]);
        } else {
            take(4 + r4, S[1]);
            put(6 + r4, S[1]);
            if (has4) {
                take(8 + e4, E);
                put(6 * e4 + 4, E);
            }
            if (has_x) {
                take(10, E);
                put(6 * x_tile(NC) + 5, E);
            }
        }
    } else {
        wg_sync();   // (the last rows have been read)
        put(6 * c0 + r4, S[0]);
        put(6 * (c0 + 1) + r4, S[1]);
        if (has4) put(6 * (c0 + e4) + 4, E);
        if (has_x) put(6 * x_tile(NC) + 5, E);
    }
    if (publish) {   // the entry has reached memory (the stores are written through) before the flags are raised
        asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
        __syncthreads();
        if (tid >= 2 + seg && tid < G)
            __hip_atomic_store(flags + (size_t)u * G * G + (1 + seg) * G + tid, epoch, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
    } else {
        wg_sync();
    }
}

// Grid: segment by segment, so that a workgroup only waits for workgroups before it.  A launch of one segment is a kernel of its own, without the code of
// increments and entries: a short call runs its code once and waits for its instructions (16 units of 64 tokens: 6.5 and 7.8 us at the two widths with
// one kernel for all, 6.1 and 7.3).
// The workgroup of a segment g > 0 computes the increment of segment g - 1 itself, hands it to its main pass in LDS, and publishes it only if a later segment needs
// it.  (Before, increments were workgroups of their own and all main passes fetched entries: 128 units of 2048 tokens, d_v 64 36.7 -> 35.2 us, d_v 128
// 54.4 -> 49.1, 1024 tokens 33.5 -> 29.4; 64 units of 1024 20.8 -> 17.2, of 777, d_v 128, 25.7 -> 21.3: three and more segments of that many units were two
// rounds of the chip.)
template <int NC, bool SEG>
__global__ __launch_bounds__(64 * (NC + producers(NC)), 2) void prefill_mfma_kernel(
    const uint16_t *__restrict__ q, const uint16_t *__restrict__ k, const uint16_t *__restrict__ v,
    uint16_t *__restrict__ y, float *__restrict__ state, int has_init, float *__restrict__ ws,
    unsigned *__restrict__ flags, unsigned *__restrict__ status, int max_polls, unsigned epoch, int N,
    SegTable segs, int G, int U)
{
    __shared__ __align__(1024) unsigned char raw[kLdsBytes];
    __shared__ unsigned anew;
    Lds<NC> &lds = *reinterpret_cast<Lds<NC> *>(raw);
    if constexpr (!SEG) {
        prefill_body<NC, false>(lds, anew, q, k, v, y, state, has_init, ws, flags, status, max_polls, epoch, N, segs, 1, 0, blockIdx.x);
    } else {
        const int seg = blockIdx.x / U, u = blockIdx.x % U;
        if (seg > 0) increment_body<NC>(raw, k, v, state, has_init, ws, flags, epoch, N, segs, G, seg - 1, u);
        prefill_body<NC, true>(lds, anew, q, k, v, y, state, has_init, ws, flags, status, max_polls, epoch, N, segs, G, seg, u);
    }
}

// ---- host side ----------------------------------------------------------------------------------
namespace {

// Segments per sequence.  At most what fills the chip once (one workgroup per CU fits): beyond that a segment's workgroup waits for a CU as well (d_v 64, 2048
// tokens: 64 units 4 segments 25.5 us, 5 33.5; 128 units 2 35.2, 3 48.9).  With few units the chip is not the limit: G segments make a chain of
// chunks / G increment chunks, G - 2 entries to sum up and chunks / G chunks of the main pass, shortest for G ~ sqrt(2 chunks) (16 units, d_v 64: 8 chunks 1
// segment 15.2, 3 12.3, 4 11.9, 5 12.7; 13 chunks 1 21.8, 4 14.3, 5 13.7, 6 14.3; 32 chunks 5 21.5, 6 20.4, 8 19.1, 10 20.9; 64 chunks 6 29.6, 8 26.4, 10 25.4; d_v 128,
// 13 chunks 4 18.9, 5 17.5, 6 18.5; 32 chunks 6 26.4, 8 24.7, 10 26.9).  Below that a second segment does not pay for its increment (1 segment and 2, 16 and 128
// units: d_v 64, 4 chunks 9.9, 10.4 and 11.4, 12.0; 5 chunks 11.1, 10.5 and 12.7, 12.2; d_v 128, 5 chunks 13.9, 14.2 and 16.2, 16.6; 6 chunks 15.6, 15.2 and 17.8, 17.8,
// three of 6 chunks, 16 units: 10.9 and 13.9).  Four segments pay from 8 chunks on, at d_v 128 from 9 (us,
// three and four: d_v 64, 7 chunks, 16 units 11.1, 11.9, 51 12.2, 14.3, 64 12.1, 12.8, 8 chunks, 16 units 12.4, 11.8, 64 13.2, 12.9; d_v 128, 7 chunks 15.1, 15.3, 17.3,
// 20.6, 16.8, 17.3, 8 chunks 15.4, 15.4, 17.4, 20.6, 17.0, 17.1, 9 chunks, 16 units 16.7, 16.3, 64 18.5, 18.3).
// From a state (launch; the workspace has room for the number without one) the state is read twice and written by a third workgroup.  With a number of units that
// 8 divides these are on one XCD; otherwise the state travels between them, the longer the more units there are, and segments pay later.  (us from a state, one segment
// and several.  d_v 64: 42 units 6 chunks 14.5, 14.6, 7 15.9, 14.7; 60 units 6 14.8, 15.2, 7 16.1, 15.2; 85 units 6 15.1, 16.3, 8 17.8, 17.5, 9 19.1, 19.1; 102 units 9 19.4,
// 20.2, 10 20.8, 20.3; but 64 units 5 13.3, 13.0, 128 5 14.3, 14.2.  d_v 128: 12 units 6 17.8, 17.4; 28 units 7 19.8, 19.9, 8 21.3, 20.0; 29 units 7 20.4, 21.6; 44 units 8 22.1, 22.1; 45 units 8 22.7, 24.4; 51 units 8 21.7, 22.3, 9 23.4, 22.7; 85
// units 10 26.1, 26.4, 12 28.9, 27.9; 102 units 12 29.6, 29.6; but 64 units 6 19.0, 18.5, 96 6 19.8, 20.2, 8 22.6, 22.0, 128 7 22.4, 22.6, 8 23.1, 22.5.)
int pick_segments(int U, int N, int dv, bool from_state = false)
{
    const int chunks = (N + C - 1) / C;
    const bool wide = dv == 128;
    int least = !wide ? 5 : U > 85 ? 7 : 6;
    if (from_state && U % 8 != 0) least = wide ? 6 + (U + 3) / 16 : U > 85 ? 10 : 5 + U / 24;
    else if (from_state && wide && U > 85) least = 8;
    if (chunks < least) return 1;
    int G = 256 / U;
    int chain = chunks == 5 ? 2 : (int)(sqrtf(2.f * (float)chunks) + 0.5f);
    if (chunks < (wide ? 9 : 8) && chain > 3) chain = 3;
    if (G > chain) G = chain;
    if (G > kMaxSegments) G = kMaxSegments;
    return G < 1 ? 1 : G;
}

// Segment boundaries (multiples of the chunk length).  Returns the number of segments.
int make_segments(int N, int G, int dv, SegTable &t)
{
    const int T = (N + C - 1) / C;   // chunks
    if (G > T) G = T;
    if (G == 2) {
        // The first segment's main pass takes as long as its increment and the main pass of the second: a chunk of the increment is 0.46 of one of the main
        // pass (d_v 128: 0.6, where it is bound by memory), the second workgroup also fills its pipelines twice and writes the state (128 units, a chunk less, as
        // here and a chunk more: d_v 64, 1024 tokens 22.8, 21.9, 22.9 us, 2048 35.9, 35.2, 36.2, 4096 61.6, 63.3, 64.7; d_v 128 29.8, 29.4, 30.0,
        // 49.4, 49.1, 49.2, 99.5, 99.9, 97.8).
        const int first = dv == 64 ? (int)(0.65f * (float)T + 2.f) : (int)(0.72f * (float)T + 1.5f);
        t.begin[0] = 0;
        t.begin[1] = (first < T ? first : T - 1) * C;
        for (int g = 2; g <= kMaxSegments; ++g) t.begin[g] = T * C;
        return 2;
    }
    // More segments: the main pass of segment g waits for the increments of segments 0 .. g - 2 and sums as many entries, the last one also writes the final
    // state, so later segments get fewer chunks.  (The figures were set when the increments were workgroups of their own and not again since; segment 0, whose
    // workgroup has no increment to compute, gets no more for that.)
    int len[kMaxSegments];
    int sum = 0;
    for (int g = 0; g < G; ++g) {
        float off = 0.6f * (0.5f * (G - 1) - g);
        if (g == G - 1 && G > 1) off -= 0.5f;
        len[g] = T / G + (int)(off >= 0.f ? off + 0.5f : off - 0.5f);
        if (len[g] < 1) len[g] = 1;
        sum += len[g];
    }
    // hand the rounding remainder to (or take it from) the early segments, one chunk at a time
    for (int g = 0; sum != T; g = (g + 1) % G) {
        if (sum < T) { ++len[g]; ++sum; }
        else if (len[g] > 1) { --len[g]; --sum; }
    }
    int pos = 0;
    for (int g = 0; g < G; ++g) { t.begin[g] = pos * C; pos += len[g]; }
    for (int g = G; g <= kMaxSegments; ++g) t.begin[g] = pos * C;
    return G;
}

// Workspace: room for G entries per unit (G - 2 are used; what fits the static scratch is part of the interface), then G x G ready-flag words per unit (256-byte aligned).
size_t ws_entry_bytes(int U, int N, int dv)
{
    return (size_t)U * pick_segments(U, N, dv) * entry_floats(dv / 32) * sizeof(float);
}
size_t ws_flag_bytes(int U, int N, int dv)
{
    const size_t Gmax = (size_t)pick_segments(U, N, dv);
    const size_t flags = (size_t)U * Gmax * Gmax * sizeof(unsigned);
    return (flags + 255) / 256 * 256;
}

template <int NC>
hipError_t launch(const uint16_t *q, const uint16_t *k, const uint16_t *v, uint16_t *y, float *state, int flags_word,
                  void *workspace, unsigned *status, int U, int N, hipStream_t s)
{
    constexpr int dv = 32 * NC;
    SegTable segs;
    // a smaller G only uses a prefix of the workspace that was sized for pick_segments()
    const int Gmax = pick_segments(U, N, dv);
    const int G = make_segments(N, pick_segments(U, N, dv, (flags_word & 1) != 0), dv, segs);
    // what the kernels index must lie inside what the workspace was sized for
    if (G < 1 || G > Gmax || segs.begin[G] < N) return hipErrorInvalidValue;
    if ((long long)U * G >= (1ll << 31)) return hipErrorInvalidValue;
    float *ws = static_cast<float *>(workspace);
    unsigned *flags = reinterpret_cast<unsigned *>((char *)workspace + ws_entry_bytes(U, N, dv));
    // Every call raises its flags to a value no earlier call used: the flag words of a workspace
    // that has never been used hold whatever was in that memory.
    static std::atomic<unsigned> calls{0};
    const unsigned epoch = 0x5EED0000u + calls.fetch_add(1u) + 1u;
    const auto kernel = G > 1 ? prefill_mfma_kernel<NC, true> : prefill_mfma_kernel<NC, false>;
    hipLaunchKernelGGL(kernel, dim3((unsigned)(U * G)), dim3(64 * (NC + producers(NC))), 0, s, q, k, v,
                       y, state, flags_word, ws, flags, status, g_flag_poll_limit.load(), epoch, N, segs, G, U);
    return hipGetLastError();
}

}  // namespace

bool prefill_mfma_supported(int dp, int dv, int dtype)
{
    return dtype == BASED_BF16 && dp == DP && (dv == 64 || dv == 128);
}

size_t prefill_mfma_workspace_bytes(int U, int N, int dp, int dv)
{
    (void)dp;
    return ws_entry_bytes(U, N, dv) + ws_flag_bytes(U, N, dv);
}

void prefill_mfma_flags_region(int U, int N, int dp, int dv, size_t *offset, size_t *bytes)
{
    (void)dp;
    *offset = ws_entry_bytes(U, N, dv);
    *bytes = ws_flag_bytes(U, N, dv);
}

void prefill_mfma_set_poll_limit(int polls) { g_flag_poll_limit.store(polls < 0 ? kMaxFlagPolls : polls); }

hipError_t launch_prefill_mfma(const void *q, const void *k, const void *v, void *y, float *state,
                               int has_init, int packed_state, void *workspace, unsigned *status, int U, int N,
                               int dp, int dv, hipStream_t s)
{
    (void)dp;
    // the kernels' flag word (has_init arrives with bit 2 set for numerator-only outputs)
    const int flags_word = (has_init & 1) | (packed_state ? 2 : 0) | (has_init & 4);
    const uint16_t *q16 = (const uint16_t *)q, *k16 = (const uint16_t *)k, *v16 = (const uint16_t *)v;
    if (dv == 128)
        return launch<4>(q16, k16, v16, (uint16_t *)y, state, flags_word, workspace, status, U, N, s);
    return launch<2>(q16, k16, v16, (uint16_t *)y, state, flags_word, workspace, status, U, N, s);
}

}  // namespace based
