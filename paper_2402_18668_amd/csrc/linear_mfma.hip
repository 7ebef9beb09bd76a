// Bias-free linear projection y = x W^T on the gfx950 matrix cores (bf16 in, fp32 accumulate, bf16
// out): the q / k / v and output projections that surround the sequence mixers in a Based block
// (architecture of Sec. 3: projections of the d_model-wide input to H d' features for q and k and
// H d_v for v, and of the H d_v mixer output back to d_model; all without bias).
//
// x [M][K] and W [N][K] are both contiguous along K, so both MFMA operands are 16 contiguous bytes
// of a row per lane.  Products are computed transposed (rows of the matrix instruction = output features,
// columns = tokens), so that a lane holds runs of 4 consecutive features of one token.
//
// Two kernels, chosen by M (pick_variant):
//   linear_tile_kernel   a BM x BN tile of y per workgroup, x and W staged through LDS
//   linear_rows_kernel   a handful of tokens (decode): W streamed once from memory straight into registers
//
// Layouts.  The mixers read and write head-major tensors [B][H][N][d], the projections' natural output is
// token-major [B N][H d].  Rather than a transposing pass in between (one more read and write of q, k,
// v and of the mixer output through HBM), the kernels address head-major tensors directly:
//   SPLIT_OUT  the output features are three groups of heads (q, k, v: H d' + H d' + H d_v rows of W in
//              that order) and go to three head-major tensors; x is read once for all three;
//   HEADS_IN   the A operand is a head-major tensor (the mixer output): a K step of 64 lies inside one head.
#include "common.h"

#include <type_traits>
#include <utility>

namespace based {

namespace lin {

typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef __bf16 bf16x4 __attribute__((ext_vector_type(4)));
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));

constexpr int kXcds = 8;
constexpr int KQ = 64;         // K is a multiple of this
constexpr int NQ = 128;        // N is a multiple of this

__device__ __forceinline__ f32x4 mfma(u32x4 a, u32x4 b, f32x4 c)
{
    return __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, a), __builtin_bit_cast(bf16x8, b), c, 0,
                                                   0, 0);
}

// Head-major addressing: seq_len tokens per sequence, H heads; d[0..2] the head dims of the (up to) three
// output groups, y1 / y2 the second and third output tensor; d_in the head dim of a head-major input.
struct HeadLayout {
    int seq_len, H;
    int d[3];
    uint16_t *y1, *y2;
    int d_in;
};

// Where the 8 output features starting at f go in the head-major outputs: the tensor, its head dim, and the
// part of the element offset that does not depend on the token.  Offset of token t of sequence b:
// b * batch_stride + fixed + t * dh.  (Computed once per lane: the divisions are not cheap, and done per
// store they were most of the epilogue.)
struct FeatDst {
    uint16_t *dst;
    int dh;
    size_t fixed, batch_stride;
};
__device__ __forceinline__ FeatDst feat_dst(const HeadLayout &hl, uint16_t *y, int f)
{
    // group of the feature (boundaries are multiples of 8: a chunk lies inside one head)
    const int n0 = hl.H * hl.d[0], n1 = n0 + hl.H * hl.d[1];
    FeatDst r;
    r.dst = f < n0 ? y : (f < n1 ? hl.y1 : hl.y2);
    r.dh = f < n0 ? hl.d[0] : (f < n1 ? hl.d[1] : hl.d[2]);
    const int ff = f < n0 ? f : (f < n1 ? f - n0 : f - n1);
    r.fixed = (size_t)(ff / r.dh) * hl.seq_len * r.dh + ff % r.dh;
    r.batch_stride = (size_t)hl.H * hl.seq_len * r.dh;
    return r;
}
// (sequence, token) of a row, and of the rows after it
struct RowPos { int b, t; };
__device__ __forceinline__ RowPos row_pos(int row, int seq_len) { return {row / seq_len, row % seq_len}; }
__device__ __forceinline__ RowPos row_after(RowPos p, int delta, int seq_len)
{
    p.t += delta;
    while (p.t >= seq_len) { p.t -= seq_len; ++p.b; }
    return p;
}

// ---- tiles -------------------------------------------------------------------------------------------------
// WM x WN waves compute a BM x BN tile (tokens x features), each a (BM / WM) x (BN / WN) part of it in MFMA tiles of
// 16 x 16.
//
// Staging.  The rows go from memory to LDS directly (the 16-byte LDS DMA: no registers, no LDS write instructions), into
// a ring of ST stages of BK = 64 columns.  One instruction of a wave moves 1 KB: 64 lanes x 16 bytes land side by
// side in LDS, i.e. whole rows of BK elements without padding, so the bank spread comes from a permutation
// instead: 16-byte piece c of row r sits at place c ^ f(r), which the lanes produce for free by choosing what
// they fetch; the 8 rows that a group of lanes reads at a time then cover all banks.
//
// Pipeline.  One barrier per step, taken before the LAST 16-deep slab of a step: by then every operand of the step
// is in registers, so behind the barrier this step's stage is free for the DMA of step kt + ST, and
// the first operands of the next step are read under the matrix instructions of the last slab.  The DMA
// pieces are dealt out between the matrix instructions; the wait before the barrier counts them (s_waitcnt
// vmcnt), so ST - 1 stages stay in flight.  Steps past the end re-read the last one, which keeps the count
// constant.  (The DMA is inline asm: through the builtin the compiler makes every LDS read wait for all of it.)
//
// Groups.  KG > 1: groups of WM x WN waves, with stages of their own, take a KG-th of the steps each, and the first one adds up (all go through as
// many steps: a group whose share is one shorter starts one step early and clears its accumulators after that).  The stages of all groups are in flight at once, and a
// group's barriers and operand reads hide behind the others' products.
//
// The operand reads of the next slab and the DMA pieces sit one by one between the matrix instructions: in bursts they
// hold up the wave, and with it the matrix pipe, until the LDS and the memory pipeline have taken them.  16x16x32 matrix
// instructions, not 32x32x16: they move half the accumulator registers per product, and under this load the chip does not hold
// its clock (1.9 to 2.05 GHz by the cycle counters, 2.4 in the memory-bound kernels; q / k / v projection of the 1.3B-shaped layer,
// 32768 x 1792 x 2560, on one GPU: 271 against 252 us).  The same shape in steps: registers-staged 256 x 256 tiles of 32x32x16 284 us, DMA 276, reads and DMA
// between the matrix instructions 268, 16x16x32 252, the DMA of a stage out by 6/8 of a step 240 us = 1255 TFLOP/s.
constexpr int MT = 16;         // MFMA tile: 16 x 16, in
constexpr int SD = 32;         // slabs of 32 (the 16x16x32 instruction)
constexpr int BK = 64;         // columns of a stage
template <int BM_, int BN_, int WM_, int WN_, int ST_, int SPREAD_ = 8, int KG_ = 1> struct Tile {
    static constexpr int BM = BM_, BN = BN_, WM = WM_, WN = WN_, ST = ST_, SPREAD = SPREAD_;
    static constexpr int KG = KG_;                               // groups of NW waves that share out the steps
    static constexpr int NW = WM * WN, NT = 64 * NW * KG;
    static constexpr int TI = BM / WM / MT, TJ = BN / WN / MT;   // MFMA tiles of a wave: tokens, features
    static constexpr int CPR = BK / 8;                           // 16-byte pieces per staged row
    static constexpr int RPI = 64 / CPR;                         // rows one DMA instruction moves
    static constexpr int AP = BM / RPI / NW, BP = BN / RPI / NW, P = AP + BP;   // instructions of a wave per step
    static constexpr int KS = BK / SD;                           // slabs per step
    static constexpr int STAGE = (BM + BN) * BK * 2;             // bytes
    static constexpr int OUT_LD = BN / WN + 8;                   // bf16 elements per row of a wave's output staging
    static constexpr int OUT = NW * 32 * OUT_LD * 2;
    static constexpr int RING = ST * STAGE > OUT ? ST * STAGE : OUT, LDS = KG * RING;
    static_assert(BM % (RPI * NW) == 0 && BN % (RPI * NW) == 0 && KS % 2 == 0, "");
    static_assert(KG == 1 || 4 * BM * BN <= RING, "");
};

// f(0), f(1), .. f(N - 1) with constant arguments (the loops over accumulators must unroll, however long)
template <typename F, int... I> __device__ __forceinline__ void constexpr_for_seq(F &&f, std::integer_sequence<int, I...>)
{
    (f(std::integral_constant<int, I>{}), ...);
}
template <int N, typename F> __device__ __forceinline__ void constexpr_for(F &&f)
{
    constexpr_for_seq(f, std::make_integer_sequence<int, N>{});
}

// 16 bytes per lane from base (uniform) + off bytes (per lane) to LDS address `to` (uniform) + 16 lane
__device__ __forceinline__ void dma16(const void *base, uint32_t off, uint32_t to)
{
    asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, %2" : : "s"(to), "v"(off), "s"(base) : "memory", "m0");
}
// this wave's DMA is complete but for the N newest instructions, its LDS reads are complete; then the barrier
template <int N> __device__ __forceinline__ void dma_barrier()
{
    asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)\n\ts_barrier" : : "n"(N) : "memory");
}

// The tile whose first token is row0 and first feature col0.  K % 64 == 0, N % BN == 0 (checked by the launcher).
template <typename T, bool SPLIT_OUT, bool HEADS_IN>
__device__ __forceinline__ void tile_body(unsigned char *lds, const uint16_t *__restrict__ x, const uint16_t *__restrict__ W,
                                          uint16_t *__restrict__ y, int M, int K, int N, int row0, int col0, const HeadLayout &hl)
{
    constexpr int TI = T::TI, TJ = T::TJ, KS = T::KS, P = T::P, ST = T::ST, CPR = T::CPR;
    const int tid = threadIdx.x;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6), lane = tid & 63, g = lane / MT, n = lane % MT;
    const int w = wave % T::NW, group = wave / T::NW;
    const int wm = w / T::WN, wn = w % T::WN;

    // permutation of the 16-byte pieces of a row
    auto swz = [](int row) { return (row >> 1) & 7; };
    // DMA instruction p of this wave: rows (p NW + w) RPI + lane / CPR of the tile of x (p < AP) or W
    // (byte offsets from the tile's first row, whose address is uniform and moves along K)
    uint32_t src[P];
    const uint16_t *xbase, *wbase = W + (size_t)col0 * K;
    {
        static_assert(T::NW % 2 == 0, "the permutation of a wave's rows is the same in all its instructions");
        const int r = lane / CPR, c = 8 * ((lane % CPR) ^ swz(w * T::RPI + r));
        auto x_row = [&](int row) -> size_t {
            if (HEADS_IN)   // token t of sequence b, head 0: [b][h][t][d_in]
                return ((size_t)(row / hl.seq_len) * hl.H * hl.seq_len + row % hl.seq_len) * hl.d_in;
            return (size_t)row * K;
        };
        xbase = x + x_row(row0);
#pragma unroll
        for (int p = 0; p < T::AP; ++p)   // rows past M re-read the last one
            src[p] = (uint32_t)(2 * (x_row(min(row0 + (p * T::NW + w) * T::RPI + r, M - 1)) - x_row(row0) + c));
#pragma unroll
        for (int p = 0; p < T::BP; ++p) src[T::AP + p] = (uint32_t)(2 * ((size_t)((p * T::NW + w) * T::RPI + r) * K + c));
    }
    if (T::KG > 1) lds += group * T::RING;
    const uint32_t lds0 = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) unsigned char *)lds + (uint32_t)w * 1024;
    const int all_steps = K / BK, steps = (all_steps + T::KG - 1) / T::KG;   // of the tile, of a group
    int next = 0;   // the step the addresses stand at
    bool extra = false;   // the group's first step is the one before its share, and taken out again
    if (T::KG > 1 && group > 0) {
        next = (group * all_steps + T::KG - 1) / T::KG;
        extra = ((group + 1) * all_steps + T::KG - 1) / T::KG - next < steps;
        if (extra) --next;
        wbase += BK * next;
        const int head = HEADS_IN ? next * BK / hl.d_in : 0;
        xbase += HEADS_IN ? (size_t)head * hl.seq_len * hl.d_in + (next * BK - head * hl.d_in) : (size_t)(BK * next);
    }
    auto issue = [&](int p, int slot) {
        const int at = p < T::AP ? p * T::NW : T::BM / T::RPI + (p - T::AP) * T::NW;
        dma16(p < T::AP ? xbase : wbase, src[p], lds0 + (uint32_t)(slot * T::STAGE + at * 1024));
    };
    auto advance = [&]() {   // (the last step is re-read instead of a step past the end)
        if (next + 1 >= all_steps) return;
        ++next;
        wbase += BK;
        xbase += BK;   // head-major x: column k0 % d_in of head k0 / d_in, one head = seq_len rows on
        if (HEADS_IN && (next * BK) % hl.d_in == 0) xbase += (size_t)(hl.seq_len - 1) * hl.d_in;
    };

    // acc[j][i]: features 16 (TJ wn + j) .. (rows of the MFMA tile) x tokens 16 (TI wm + i) .. (columns)
    f32x4 acc[TJ][TI];
#pragma unroll
    for (int j = 0; j < TJ; ++j)
#pragma unroll
        for (int i = 0; i < TI; ++i) acc[j][i] = f32x4{0.f, 0.f, 0.f, 0.f};

    u32x4 fw[2][TJ], fx[2][TI];
    int off[KS];   // element offset of slab ks in this lane's row (rows 16 apart have the same permutation)
#pragma unroll
    for (int ks = 0; ks < KS; ++ks) off[ks] = n * BK + 8 * ((SD / 8 * ks + g) ^ swz(n));
    constexpr int NR = TI + TJ, NM = TI * TJ;   // operand reads and matrix instructions of a slab
    auto read_op = [&](int slot, int ks, int set, int r) {
        const uint16_t *a = reinterpret_cast<const uint16_t *>(lds + slot * T::STAGE) + off[ks];
        // (in the order the matrix instructions need them)
        if (r == 0 || r > TI) fw[set][r ? r - TI : 0] = *reinterpret_cast<const u32x4 *>(a + (T::BM + MT * (TJ * wn + (r ? r - TI : 0))) * BK);
        else fx[set][r - 1] = *reinterpret_cast<const u32x4 *>(a + MT * (TI * wm + r - 1) * BK);
    };

#pragma unroll
    for (int st = 0; st < ST; ++st) {
        if (st == ST - 1) break;
#pragma unroll
        for (int p = 0; p < P; ++p) issue(p, st);
        advance();
    }
    // the last stage's pieces: what the loop issues after a barrier for the step ST ahead, here for step ST - 1
    // Piece p of a stage goes out with matrix instruction p SPAN / P counted from the barrier that freed the stage, so that the
    // youngest has some time left until the barrier that waits for it.
    constexpr int SPAN = KS * NM * T::SPREAD / 8;
    constexpr int PK = (P * NM + SPAN - 1) / SPAN < P ? (P * NM + SPAN - 1) / SPAN : P;   // pieces of the first slab
#pragma unroll
    for (int p = 0; p < PK; ++p) issue(p, ST - 1);
    dma_barrier<(ST - 2) * P + PK>();
#pragma unroll
    for (int r = 0; r < NR; ++r) read_op(0, 0, 0, r);
    int slot = 0;
    for (int kt = 0; kt < steps; ++kt) {
        const int after = slot + 1 == ST ? 0 : slot + 1;       // slot of the next step
        const int fill = slot == 0 ? ST - 1 : slot - 1;        // slot being filled: step kt + ST - 1
        constexpr_for<KS>([&](auto kc) {
            constexpr int ks = decltype(kc)::value;
            if constexpr (ks + 1 == KS) {
                advance();
                dma_barrier<(ST - 2) * P>();
            }
            // the last slab starts the stage of step kt + ST, the others continue the one of step kt + ST - 1
            constexpr_for<NM>([&](auto mc) {
                constexpr int m = decltype(mc)::value;
                acc[m / TI][m % TI] = mfma(fw[ks & 1][m / TI], fx[ks & 1][m % TI], acc[m / TI][m % TI]);
                // between two matrix instructions: the share of the next slab's operand reads, and of the DMA
                constexpr_for<NR>([&](auto rc) {
                    constexpr int r = decltype(rc)::value;
                    if constexpr (r * NM / NR == m) read_op(ks + 1 < KS ? slot : after, (ks + 1) % KS, (ks + 1) & 1, r);
                });
                constexpr_for<P>([&](auto pc) {
                    constexpr int p = decltype(pc)::value;
                    if constexpr (p * SPAN / P == (ks + 1) % KS * NM + m) issue(p, ks + 1 < KS ? fill : slot);
                });
                __builtin_amdgcn_sched_barrier(0);
            });
        });
        slot = after;
        if (T::KG > 1 && kt == 0 && extra) {   // (uniform)
            constexpr_for<NM>([&](auto mc) { acc[decltype(mc)::value / TI][decltype(mc)::value % TI] = f32x4{0.f, 0.f, 0.f, 0.f}; });
        }
    }
    dma_barrier<0>();   // nothing lands in LDS any more
    if constexpr (T::KG > 1) {   // the other groups' sums, through their stages
        unsigned char *first = lds - group * T::RING;
        auto sums = [&](int of, int m) -> f32x4 & { return reinterpret_cast<f32x4 *>(first + of * T::RING)[(m * T::NW + w) * 64 + lane]; };
        if (group > 0) constexpr_for<NM>([&](auto mc) { sums(group, decltype(mc)::value) = acc[decltype(mc)::value / TI][decltype(mc)::value % TI]; });
        __syncthreads();
        if (group > 0) return;
        constexpr_for<T::KG - 1>([&](auto gc) {
            constexpr_for<NM>([&](auto mc) { acc[decltype(mc)::value / TI][decltype(mc)::value % TI] += sums(decltype(gc)::value + 1, decltype(mc)::value); });
        });
    }

    // epilogue: lane (g, n) of tile (j, i) holds token MT (TI wm + i) + n, features MT (TJ wn + j) + 4 g + e in register e.  32
    // tokens at a time through this wave's staging rows, then whole row segments.
    constexpr int OUT_LD = T::OUT_LD, CP = MT * TJ / 8;   // 16-byte pieces per row
    uint16_t *out = reinterpret_cast<uint16_t *>(lds) + (size_t)w * 32 * OUT_LD;
    const int oc = lane % CP, orow = lane / CP;
    const int f_lane = col0 + MT * TJ * wn + 8 * oc;   // first of this lane's 8 features
    const int r_lane = row0 + MT * TI * wm + orow;
    FeatDst fd{};
    RowPos rp0{};
    if (SPLIT_OUT) {
        fd = feat_dst(hl, y, f_lane);
        rp0 = row_pos(r_lane, hl.seq_len);
    }
    constexpr int IT = 32 / MT;   // MFMA tiles in 32 tokens
#pragma unroll
    for (int i32 = 0; i32 < TI / IT; ++i32) {
#pragma unroll
        for (int j = 0; j < TJ; ++j)
#pragma unroll
            for (int i = 0; i < IT; ++i)
                *reinterpret_cast<u32x2 *>(out + (size_t)(MT * i + n) * OUT_LD + MT * j + 4 * g) =
                    __builtin_bit_cast(u32x2, __builtin_convertvector(acc[j][i32 * IT + i], bf16x4));
        asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");   // the wave's own rows are complete in LDS
#pragma unroll
        for (int it = 0; it < CP / 2; ++it) {
            const int dr = it * (64 / CP);
            const u32x4 val = *reinterpret_cast<const u32x4 *>(out + (size_t)(dr + orow) * OUT_LD + 8 * oc);
            const int row = r_lane + 32 * i32 + dr;
            if (row < M) {
                if (SPLIT_OUT) {
                    const RowPos rp = row_after(rp0, 32 * i32 + dr, hl.seq_len);
                    *reinterpret_cast<u32x4 *>(fd.dst + (size_t)rp.b * fd.batch_stride + fd.fixed + (size_t)rp.t * fd.dh) = val;
                } else {
                    *reinterpret_cast<u32x4 *>(y + (size_t)row * N + f_lane) = val;
                }
            }
        }
        asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");   // read back before the next rows overwrite it
    }
}

// Blocks 0 .. : the first `whole` tiles of T; the blocks after them: the remaining tiles in halves of BM / 2 tokens (T2).
// Block -> tile: XCD b % 8 works through a contiguous eighth of the tiles, so that the tiles it has in hand share rows of x and W in
// its L2 (and a problem of one band of rows still uses all XCDs).  Features fastest, an XCD reads an eighth of x and all of W; rows fastest (rows_first;
// `fast` tiles), an eighth of W and all of x.
template <typename T, typename T2, bool SPLIT_OUT, bool HEADS_IN>
__global__ __launch_bounds__(T::NT, T::LDS > 80 * 1024 ? T::NT / 256 : T::NW / 2) void linear_tile_kernel(
    const uint16_t *__restrict__ x, const uint16_t *__restrict__ W, uint16_t *__restrict__ y, int M, int K, int N,
    int fast, int rows_fast, int whole, int halves, HeadLayout hl)
{
    __shared__ __align__(1024) unsigned char lds[T::LDS];
    const int per = (whole + kXcds - 1) / kXcds;
    struct RowCol { int row, col; };
    auto place = [&](int tile) {
        const int slow = __builtin_amdgcn_readfirstlane(tile / fast), rest = tile - slow * fast;
        return RowCol{(rows_fast ? rest : slow) * T::BM, (rows_fast ? slow : rest) * T::BN};
    };
    int b = blockIdx.x;
    if (b < per * kXcds) {
        const int tile = b % kXcds * per + b / kXcds;
        if (tile >= whole) return;   // uniform
        const RowCol at = place(tile);
        tile_body<T, SPLIT_OUT, HEADS_IN>(lds, x, W, y, M, K, N, at.row, at.col, hl);
    } else if constexpr (!std::is_same_v<T, T2>) {
        static_assert(T2::BM * 2 == T::BM && T2::BN == T::BN && T2::NT == T::NT && T2::LDS <= T::LDS, "");
        b -= per * kXcds;
        const int per2 = (halves + kXcds - 1) / kXcds, h = b % kXcds * per2 + b / kXcds;
        if (h >= halves) return;     // uniform
        const RowCol at = place(whole + h / 2);
        const int row0 = at.row + h % 2 * T2::BM;
        if (row0 >= M) return;       // uniform: the second half of a last band
        tile_body<T2, SPLIT_OUT, HEADS_IN>(lds, x, W, y, M, K, N, row0, at.col, hl);
    }
}

// ---- a handful of tokens -------------------------------------------------------------------------------------
// M of a few: bound by reading W once, by what a CU can take in of it and of x (which every workgroup reads whole), and by the latency of
// one trip to memory.  A workgroup takes F output features (a sixteenth of the matrix instruction's columns each, the rest idle: it is
// the CUs that count) and 16 TT tokens; its eight waves split K, each with the whole of its share of W (and x)
// requested up front, straight into operand registers (MFMA 16x16x32: lane = row n of W / token n, 8
// consecutive k); partial sums meet in LDS.  One workgroup of eight waves per CU puts the whole W in flight at once.  Where a thread's
// results go (divisions by the sequence length and the head dim) is worked out while the rows are on their way: 9 tokens, d_model
// 1792, H 16, d' 16, d_v 128: 5.2 and 5.7 us for the two projections with 16 features and that at the end, 5.0 and 5.1 with it here,
// 4.55 and 4.53 with 10 and 8 features.
constexpr int RW = 8;           // waves
template <int TT, bool SPLIT_OUT, bool HEADS_IN>
__global__ __launch_bounds__(64 * RW, 2) void linear_rows_kernel(const uint16_t *__restrict__ x,
                                                                 const uint16_t *__restrict__ W,
                                                                 uint16_t *__restrict__ y, int M, int K, int N, int F,
                                                                 HeadLayout hl)
{
    constexpr int G = TT == 4 ? 4 : 8;   // steps of 32 in flight per wave
    __shared__ __align__(16) float red[RW][16 * TT][20];   // (row stride 20: 16-byte writes of 16 rows spread over the banks)
    const int tid = threadIdx.x;
    const int w = __builtin_amdgcn_readfirstlane(tid >> 6), lane = tid & 63, g = lane >> 4, n = lane & 15;
    const int col0 = blockIdx.x * F, row0 = blockIdx.y * 16 * TT;

    const uint16_t *wp = W + (size_t)min(col0 + min(n, F - 1), N - 1) * K + 8 * g;   // (rows past the F-th re-read it)
    const uint16_t *xp[TT];
#pragma unroll
    for (int t = 0; t < TT; ++t) {   // rows past M re-read the last one
        const int row = min(row0 + 16 * t + n, M - 1);
        xp[t] = x + 8 * g + (HEADS_IN ? ((size_t)(row / hl.seq_len) * hl.H * hl.seq_len + row % hl.seq_len) * hl.d_in
                                      : (size_t)row * K);
    }
    f32x4 acc[TT];
#pragma unroll
    for (int t = 0; t < TT; ++t) acc[t] = f32x4{0.f, 0.f, 0.f, 0.f};
    const int steps = K / 32, s0 = steps * w / RW, s1 = steps * (w + 1) / RW;
    u32x4 a[G], b[G][TT];
    auto load = [&](int s) {
        int head = HEADS_IN ? 32 * s / hl.d_in : 0, in_head = 32 * s - head * hl.d_in;   // (d_in is a multiple of 32)
#pragma unroll
        for (int j = 0; j < G; ++j) {
            const int k0 = 32 * min(s + j, s1 - 1);
            const size_t xo = HEADS_IN ? (size_t)head * hl.seq_len * hl.d_in + in_head : (size_t)k0;
            a[j] = *reinterpret_cast<const u32x4 *>(wp + k0);
#pragma unroll
            for (int t = 0; t < TT; ++t) b[j][t] = *reinterpret_cast<const u32x4 *>(xp[t] + xo);
            if (HEADS_IN && s + j + 1 < s1) {
                in_head += 32;
                if (in_head >= hl.d_in) { in_head = 0; ++head; }
            }
        }
    };
    if (s0 < s1) load(s0);
    // where this thread's two features of one token go, worked out while the rows are on their way
    const int tok = tid >> 3, f2 = 2 * (tid & 7), f = col0 + f2, row = row0 + tok;
    const bool mine = tid < 128 * TT && row < M && f2 < F && f < N;
    uint16_t *dst = y;
    if (mine) {
        if (SPLIT_OUT) {
            const FeatDst fd = feat_dst(hl, y, f);
            const RowPos rp = row_pos(row, hl.seq_len);
            dst = fd.dst + (size_t)rp.b * fd.batch_stride + fd.fixed + (size_t)rp.t * fd.dh;
        } else {
            dst = y + (size_t)row * N + f;
        }
    }
    asm volatile("" : "+v"(dst));
    for (int s = s0; s < s1; s += G) {
        if (s > s0) load(s);
#pragma unroll
        for (int j = 0; j < G; ++j) {
            if (s + j < s1) {   // uniform
#pragma unroll
                for (int t = 0; t < TT; ++t)
                    acc[t] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, a[j]),
                                                                     __builtin_bit_cast(bf16x8, b[j][t]), acc[t], 0, 0, 0);
            }
        }
    }
    // lane (g, n): token n, features 4 g .. 4 g + 3
#pragma unroll
    for (int t = 0; t < TT; ++t) *reinterpret_cast<f32x4 *>(&red[w][16 * t + n][4 * g]) = acc[t];
    __syncthreads();
    if (!mine) return;
    float sum0 = 0.f, sum1 = 0.f;
#pragma unroll
    for (int v = 0; v < RW; ++v) { sum0 += red[v][tok][f2]; sum1 += red[v][tok][f2 + 1]; }
    *reinterpret_cast<uint32_t *>(dst) = (uint32_t)f32_to_bf16_bits(sum0) | ((uint32_t)f32_to_bf16_bits(sum1) << 16);
}

// ---- choice of the variant ---------------------------------------------------------------------------------
using T64 = Tile<64, 64, 2, 2, 4>;                 // 64 KB of LDS: two workgroups per CU
using T128N = Tile<128, 64, 2, 2, 3>;              // 72 KB: two
using T128 = Tile<128, 128, 2, 2, 2, 5>;       // 64 KB: two
using T256 = Tile<256, 256, 2, 2, 2, 6>;       // 128 KB: one
using T256H = Tile<128, 256, 2, 2, 2, 6>;
using T32S = Tile<32, 32, 1, 2, 4, 8, 4>;          // 128 KB: one
using T64S = Tile<64, 32, 2, 1, 3, 8, 4>;          // 144 KB: one
enum Variant { ROWS1, ROWS2, TILE32S, TILE64S, TILE64, TILE128N, TILE128, TILE256 };

inline long tiles_of(long M, long N, int bm, int bn) { return (M + bm - 1) / bm * (N / bn); }

// The ratios below are of launch times in three settings: the same operands again (they stay in the L2); other operands each time, in the last-level cache; and W
// from memory, as in a model whose weights that cache does not hold.
//
// Rows fastest over the XCDs: where W is enough larger than x, and the operands, not the output, are what a tile moves.  (Time of rows fastest by that of features
// fastest, 10 M < 7 N: 64 x 64 tiles, 16 steps of 64 columns and more, 0.94, 0.93, 0.98, up to 8 steps and 128 tiles 1.02, 1.02, 1.00; with 7 N <= 10 M < 10 N 0.99, 0.99, 0.98, beyond that up
// to 1.11, 1.09, 1.01.  128 x 64 tiles, up to 256 0.93, 0.95, 0.98, up to 512 0.88, 0.90, 1.04; over 1024 1.02 to 1.1.)
inline bool rows_first(long M, int K, long N)
{
    return 10 * M < 7 * N && K >= (tiles_of(M, N, 64, 64) > 128 ? 5 : 8) * BK && tiles_of(M, N, 128, 64) <= 1024;
}

// A handful of tokens: 16 or 32 per workgroup (above 32 tiles, which read W fewer times, are as fast or faster).
// Otherwise the tiling with the smallest expected time.  The figures are microseconds per 64-deep step, measured at
// K 768 .. 2048, 40 .. 5120 tiles: a launch of up to 256 tiles (one per CU) is bound by the latency of a step, after
// that each further tile per CU adds its share.  (The larger the tile the less it reads per product: at 32768 x 1792 x
// 2560 the four tilings take 630, 417, 308 and 240 us; at 512 x 1792 x 2560 they take 17, 12, 21 and 37.)
inline Variant pick_variant(int M, int K, int N)
{
    if (M <= 16) return ROWS1;
    if (M <= 18 || K >= (1 << 22)) return ROWS2;   // (tiles address their rows with 32-bit offsets)
    // Few tiles are bound by what a CU takes in of x and W and by the latency of a step: the smallest tiles that leave each CU at most one, the steps
    // shared out over four groups of waves, where there are enough of them to pay for the groups' start and sum.  (Time of
    // 32 x 32 by that before.  33 tokens and more, by 64 x 64, 10 M < 7 N: 9 steps 1.00, 1.00, 10 0.96, 0.97, 16 0.84, 0.86, 20 and more 0.75, 0.79, all with W from memory 0.76; otherwise 10
    // steps 0.94, 0.95 to 1.03, 0.89, 12 0.91, 0.92 to 1.00, 0.87, 26 0.73, 0.78 to 0.89, 0.72.  19 to 32, by ROWS2: 1
    // step 1.08, 1.10, 2 0.87, 0.88, 3 and more 0.74, 0.76, and with W from memory up to 17 steps 0.86, but from 18 on 1.05, there ROWS2 asks for more of W at once.
    // 64 x 32 by 64 x 64, 10 M < 7 N: 16 to 23 steps 0.97, 1.03, 0.93, 24 to 27 0.93, 1.00, 0.88, 28 and more 0.88, 0.96, 0.86; otherwise x is the larger operand and
    // read by twice as many tiles, 32 steps and more 0.88, 1.1, 0.86.  64 x 64 in two groups by one: 32 steps and more 0.95, 1.08, 1.01, fewer 0.97 to 1.02, 1.10, 1.04.  More
    // tiles than CUs take two rounds: 200 tokens, 1792 -> 2560, 8.3 us with 64 x 64, 17 with 32 x 32, 13 with 64 x 32.)
    const bool wide = 10ll * M < 7ll * N;
    if (K >= (M <= 32 ? 2 : wide ? 10 : 12) * BK && tiles_of(M, N, T32S::BM, T32S::BN) <= 256) return TILE32S;
    if (M <= 32) return ROWS2;
    if (wide && K >= 28 * BK && tiles_of(M, N, T64S::BM, T64S::BN) <= 224) return TILE64S;
    auto per_cu = [](long tiles) { return (float)((tiles + 255) / 256); };
    Variant best = TILE64;
    float t = 0.05f + 0.21f * per_cu(tiles_of(M, N, T64::BM, T64::BN));
    auto offer = [&](Variant v, float tv) {
        if (tv < t) { t = tv; best = v; }
    };
    offer(TILE128N, 0.02f + 0.31f * per_cu(tiles_of(M, N, T128N::BM, T128N::BN)));
    const long n128 = tiles_of(M, N, T128::BM, T128::BN);
    offer(TILE128, n128 <= 256 ? 0.7f : 0.9f * (float)((n128 + 511) / 512));   // two per CU run side by side
    if (N % T256::BN == 0) {
        const long n256 = tiles_of(M, N, T256::BM, T256::BN), rem = n256 % 256;
        offer(TILE256, 1.5f * (float)(n256 / 256) + (rem == 0 ? 0.f : rem <= 128 ? 1.f : 1.5f));   // (see launch_tile)
    }
    return best;
}

template <typename T, typename T2, bool SPLIT_OUT, bool HEADS_IN>
void launch_tile(const uint16_t *x, const uint16_t *W, uint16_t *y, int M, int K, int N, const HeadLayout &hl, hipStream_t s)
{
    const long tiles = tiles_of(M, N, T::BM, T::BN);
    // a last round of the chip that would be at most half full is dealt out in half tiles
    const long rem = tiles % 256, halves = !std::is_same_v<T, T2> && rem <= 128 ? 2 * rem : 0, whole = tiles - halves / 2;
    const bool rows_fast = rows_first(M, K, N);
    const long grid = (whole + kXcds - 1) / kXcds * kXcds + (halves + kXcds - 1) / kXcds * kXcds;
    hipLaunchKernelGGL((linear_tile_kernel<T, T2, SPLIT_OUT, HEADS_IN>), dim3((unsigned)grid), dim3(T::NT), 0, s, x, W, y, M, K,
                       N, rows_fast ? (M + T::BM - 1) / T::BM : N / T::BN, (int)rows_fast, (int)whole, (int)halves, hl);
}
template <int TT, bool SPLIT_OUT, bool HEADS_IN>
void launch_rows(const uint16_t *x, const uint16_t *W, uint16_t *y, int M, int K, int N, const HeadLayout &hl, hipStream_t s)
{
    // Features per workgroup: the smallest even number that leaves at most one workgroup per CU, 4 to 16.  (q / k / v and output projection of 9
    // tokens, d_model 1792, 2560 and 1792 features, us: 16 5.0 and 5.1, 12 4.7 and 4.8, 10 4.55 and 4.64, 8 6.5 and 4.53, 6 6.2 and 6.3; 3
    // tokens, d_model 512, 1024 features: 16 3.95, 8 3.4, 4 3.2.)
    const int per = (N + 255) / 256, even = (per + 1) / 2 * 2, F = even < 4 ? 4 : even > 16 ? 16 : even;
    hipLaunchKernelGGL((linear_rows_kernel<TT, SPLIT_OUT, HEADS_IN>), dim3((unsigned)((N + F - 1) / F), (unsigned)((M + 16 * TT - 1) / (16 * TT))),
                       dim3(64 * RW), 0, s, x, W, y, M, K, N, F, hl);
}
template <bool SPLIT_OUT, bool HEADS_IN>
hipError_t launch_variant(Variant v, const uint16_t *x, const uint16_t *W, uint16_t *y, int M, int K, int N,
                          const HeadLayout &hl, hipStream_t s)
{
    switch (v) {
    case ROWS1: launch_rows<1, SPLIT_OUT, HEADS_IN>(x, W, y, M, K, N, hl, s); break;
    case ROWS2: launch_rows<2, SPLIT_OUT, HEADS_IN>(x, W, y, M, K, N, hl, s); break;
    case TILE64: launch_tile<T64, T64, SPLIT_OUT, HEADS_IN>(x, W, y, M, K, N, hl, s); break;
    case TILE32S: launch_tile<T32S, T32S, SPLIT_OUT, HEADS_IN>(x, W, y, M, K, N, hl, s); break;
    case TILE64S: launch_tile<T64S, T64S, SPLIT_OUT, HEADS_IN>(x, W, y, M, K, N, hl, s); break;
    case TILE128N: launch_tile<T128N, T128N, SPLIT_OUT, HEADS_IN>(x, W, y, M, K, N, hl, s); break;
    case TILE128: launch_tile<T128, T128, SPLIT_OUT, HEADS_IN>(x, W, y, M, K, N, hl, s); break;
    case TILE256: launch_tile<T256, T256H, SPLIT_OUT, HEADS_IN>(x, W, y, M, K, N, hl, s); break;
    }
    return hipGetLastError();
}
template <bool SPLIT_OUT, bool HEADS_IN>
hipError_t launch_any(const uint16_t *x, const uint16_t *W, uint16_t *y, int M, int K, int N, const HeadLayout &hl,
                      hipStream_t s)
{
    return launch_variant<SPLIT_OUT, HEADS_IN>(pick_variant(M, K, N), x, W, y, M, K, N, hl, s);
}

}  // namespace lin

bool linear_supported(int M, int K, int N, int dtype)
{
    return dtype == BASED_BF16 && M >= 1 && K >= lin::KQ && K % lin::KQ == 0 && N >= lin::NQ && N % lin::NQ == 0;
}

hipError_t launch_linear(const void *x, const void *W, void *y, int M, int K, int N, hipStream_t s)
{
    return lin::launch_any<false, false>((const uint16_t *)x, (const uint16_t *)W, (uint16_t *)y, M, K, N,
                                         lin::HeadLayout{}, s);
}

bool project_qkv_supported(int K, int H, int d_feat, int d_v, int dtype)
{
    return dtype == BASED_BF16 && K >= lin::KQ && K % lin::KQ == 0 && H >= 1 && d_feat >= 8 && d_feat % 8 == 0 &&
           d_v >= 8 && d_v % 8 == 0 && (H * (2 * d_feat + d_v)) % lin::NQ == 0;
}

hipError_t launch_project_qkv(const void *x, const void *W, void *q, void *k, void *v, int B, int seq_len, int K,
                              int H, int d_feat, int d_v, hipStream_t s)
{
    const int M = B * seq_len, N = H * (2 * d_feat + d_v);
    lin::HeadLayout hl{seq_len, H, {d_feat, d_feat, d_v}, (uint16_t *)k, (uint16_t *)v, 0};
    return lin::launch_any<true, false>((const uint16_t *)x, (const uint16_t *)W, (uint16_t *)q, M, K, N, hl, s);
}

bool project_out_supported(int H, int d_v, int N, int dtype)
{
    return dtype == BASED_BF16 && H >= 1 && d_v >= lin::KQ && d_v % lin::KQ == 0 && N >= lin::NQ && N % lin::NQ == 0;
}

hipError_t launch_project_out(const void *y_heads, const void *W, void *out, int B, int seq_len, int H, int d_v,
                              int N, hipStream_t s)
{
    const int M = B * seq_len, K = H * d_v;
    lin::HeadLayout hl{seq_len, H, {0, 0, 0}, nullptr, nullptr, d_v};
    const uint16_t *x16 = (const uint16_t *)y_heads;
    uint16_t *o16 = (uint16_t *)out;
    const size_t seq_elems = (size_t)K * seq_len;
    if (B == 1 || seq_elems < (1u << 30))
        return lin::launch_any<false, true>(x16, (const uint16_t *)W, o16, M, K, N, hl, s);
    // a tile addresses its rows with 32-bit byte offsets, which must not have to reach from one such sequence into the next
    for (int b = 0; b < B; ++b) {
        const hipError_t e = lin::launch_any<false, true>(x16 + b * seq_elems, (const uint16_t *)W, o16 + (size_t)b * seq_len * N, seq_len, K, N, hl, s);
        if (e != hipSuccess) return e;
    }
    return hipSuccess;
}

}  // namespace based
