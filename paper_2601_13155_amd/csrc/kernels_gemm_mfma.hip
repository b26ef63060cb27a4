// bf16 matrix-core GEMM for gfx950:  C[M,N] = A[M,K] * B[N,K]^T, fp32 accumulation.
//
// Serves the dense contractions of the SPTS layer: K / Q / V / O projections, the gathered SwiGLU
// FFN and the low-rank proxy.  Both operands are K-contiguous, so MFMA fragments are plain 16-byte
// LDS reads with no transposition.
//
//  * 256x256 output tile per workgroup, 8 wavefronts (4x2), each owning 64x128 = 4x8 MFMA
//    16x16x32 blocks: 128 fp32 accumulators per lane, 32 MFMAs per 12 fragment reads, two wavefronts
//    per SIMD so that one wavefront's LDS reads, waits and barriers hide behind the other's MFMAs.
//    The same tile on 32x32x16 instructions has the same LDS traffic and rate on paper.  In a layer (8B shape, kernel
//    times on one GPU, 32x32x16 in row order -> 16x16x32 back and forth): gate/up of 13107 rows 2399 -> 2304 us (1336 TFLOP/s), of
//    3277 rows 627 -> 595; down 1131 -> 1125 and 325 -> 316; O 361 -> 350 and 109 -> 112; Q+V 470 -> 466 and 128 -> 127.  Products
//    that power does not bound lose instead (proxy z of 32768 rows, which reads 0.94 GB, 247 -> 262; proxy input of 20011 rows, 158 tiles,
//    110 -> 112); whole layers gain 2-5 %.
//  * K is consumed in slabs of 32.  Operands travel global memory -> LDS directly (global_load_lds_dwordx4: no VGPR
//    staging, no ds_write instructions) into a ring of stages (struct Ring): the loads of the next slabs are in flight while the
//    current one is multiplied.  The wavefront counts its own outstanding loads with
//    s_waitcnt vmcnt(n) and a workgroup barrier publishes a landed slab and frees the
//    stages consumed before it.
//  * The address of a load is a wavefront-uniform base in SGPRs, advanced along K by scalar adds, plus
//    a 32-bit per-lane offset fixed for the whole tile, and the steady state is unrolled over the ring
//    so that LDS stage offsets are immediates: the loop holds no vector address arithmetic (vector
//    instructions barely overlap with MFMAs on this chip: interleaved 1:1 they take 0.75 of the sum).
//  * A direct-to-LDS load puts lane i's 16 bytes at base + 16*i, so the XOR swizzle that makes the
//    16-lane b128 fragment reads bank-conflict free is applied on the global side: lane i fetches
//    the chunk that belongs at position i.
//  * A slab of 32 is two steps, one per half of the wavefront's columns.  Fragment reads of the next step are issued
//    between the MFMAs of the current one (sched_group_barrier pins the interleaving); the barrier sits a few MFMAs
//    into the last step so that the matrix pipe stays fed while wavefronts meet.
//  * Whole cache lines.  A load instruction that takes 64 bytes of each of 16 rows of a row-major operand requests every 128-byte line
//    twice (with the load of the next slab), and the kernel is bound by L2 requests.  Two ways round it:
//    (a) slab-major operands, [K/32][rows][32] (64 bytes per row and slab, neighbouring rows adjacent): the same 16 rows are 1 KB of
//    whole lines; only the addresses differ (row pitch 64 bytes, slab pitch rows * 64 bytes), the LDS image and the order of the
//    products do not.  B: weight copies (b_slab); A: activations that another kernel of this library wrote that way (a_slab; the SiLU
//    and store epilogues and the split-K finish write such a C on request, c_slab).
//    (b) 64 of K at a time: a load takes whole lines of 8 rows.  That costs LDS (32 KB a stage), and with 2 stages of both operands the loads
//    of the next stage arrive late.  So only the operands that are row-major are wide: A in 3 stages and a slab-major B in 4 stages of
//    32 (LAY_WIDE_A), or A in 3 and B in 2 (LAY_WIDE_AB) - A, which few workgroups share, comes from far away and gets the depth.
//    Measured alone (us, 32-wide slabs or 2 stages of 64 -> now): gate/up of 13107 gathered rows, slab-major weights 2294 -> 2140 (1440 TFLOP/s;
//    slab-major A 2167), of 3276 rows 577 -> 540; K projection of 32768 rows 229 -> 210; the proxy's input of 32768 rows 118 -> 103, of 20011 rows
//    100 -> 86; with row-major weights gate/up of 13107 rows 2504 -> 2290, down of 8192 rows 803 -> 718, K projection 252 -> 224.
//  * Rows of A may be gathered through an index list (the active-token gather of Eq. (skip) is
//    folded into the A loads: a row is 2*K contiguous bytes, so nothing is lost in coalescing),
//    rows of C may be scattered through one (the residual update X[T] += ...).
//  * The MFMA is issued as D^T = B * A^T so that a lane ends up with 4 consecutive output columns
//    of one row: lane-local rotary / SiLU-mul pairing, in-lane row sums, 8-byte packed pieces.
//  * The finished bf16 tile is staged through LDS (the operand ring is free by then) and leaves in
//    whole rows, 16 bytes per lane: stores straight from the fragment layout reach memory as 16-byte
//    pieces of 32 different rows per instruction, which cost a short-K GEMM a quarter of its time.
//  * Workgroup ids are remapped so that each of the 8 XCDs (own L2 each) walks a contiguous range
//    of tiles in groups of 4 row panels: concurrently running tiles share A and B panels in L2.
//  * One workgroup fits a CU, so tiles run in rounds of 256.  When the last round is partly filled
//    its tiles are split over K (tail split-K): several workgroups each take a share of K, write
//    fp32 partial tiles, and a small second kernel sums them and applies the epilogue.  A GEMM with
//    fewer than 256 tiles is the special case without whole rounds.
//  * The plain-store epilogue can take its B rows from two matrices (columns [0, N/2) from B0,
//    [N/2, N) from B1): the two down-projections of the proxy run as one launch.
//
// Epilogues: plain store (+ optional transposed copy for V), rotary embedding (pairs (j, j+d/2) sit
// in the same lane because an N block pair is d/2 apart), SiLU(gate)*up with gate and up columns
// interleaved per wavefront (row-major, slab-major or channel-major), residual add into scattered rows, per-row partial sums of squares.
#include "spts_internal.h"

namespace spts {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float f32x4 __attribute__((ext_vector_type(4)));

constexpr int BM = 256, BN = 256;

// LDS image of an operand tile, BK of K wide.  A tile row holds BK bf16 = CPR 16-byte chunks; chunk c of row `row` is stored at
// chunk position c ^ ((row / RP) % CPR) (RP = rows per 256 bytes), so the 16 lanes of a b128
// fragment read (16 consecutive rows, same chunk) cover all 64 LDS banks exactly once.
template <int BK> struct Image {
    static constexpr int ROW_BYTES = BK * 2;
    static constexpr int CPR = BK / 8;
    static constexpr int RP = 256 / ROW_BYTES;
    static constexpr int TILE_BYTES = 256 * ROW_BYTES;
    static constexpr int ROWS_PER_LOAD = 64 / CPR;   // tile rows moved by one direct-to-LDS load
    __device__ static inline int swz(int row) { return (row / RP) % CPR; }
    __device__ static inline int off(int row, int c) { return row * ROW_BYTES + ((c ^ swz(row)) << 4); }
};

// How the operands travel.  The loop's unit is a slab of 32 of K; a WIDE operand is moved 64 of K at a time, i.e. whole cache lines of a
// row-major matrix, and one of its stages serves two slabs.
enum Layout : int {
    LAY_SLABS = 0,   // both 32 wide, 4 stages each (3 with a second A operand): slab-major operands, K not a multiple of 64
    LAY_WIDE_A = 1,  // row-major A 64 wide in 3 stages, B (slab-major as a rule) 32 wide in 4: 96 + 64 KB
    LAY_WIDE_AB = 2, // both row-major and 64 wide, A in 3 stages and B in 2: 96 + 64 KB.  B, which many workgroups read, comes from L2
};
template <int LAY, bool DUAL_A> struct Ring {
    static constexpr bool AW = LAY != LAY_SLABS, BW = LAY == LAY_WIDE_AB;
    static constexpr int NSA = AW ? 3 : DUAL_A ? 3 : 4, NSB = BW ? 2 : DUAL_A ? 3 : 4;   // stages
    using IA = Image<AW ? 64 : 32>;
    using IB = Image<BW ? 64 : 32>;
    static constexpr int B0 = NSA * IA::TILE_BYTES, A1 = B0 + NSB * IB::TILE_BYTES;      // where B's and the second A's stages begin
    static constexpr int BYTES = A1 + (DUAL_A ? NSA * IA::TILE_BYTES : 0);
    static constexpr int UNROLL = AW ? 12 : 4;                                           // slabs after which every stage number recurs
};

__device__ inline uint32_t pack_bf16x2(float a, float b) { return cvt_pk_bf16(a, b); }
// SiLU with the hardware exponential and reciprocal (about 1 ulp each in fp32; the result is rounded to
// bf16): an IEEE division would cost ten more instructions per element, which shows in the short-K
// proxy GEMM whose epilogue is a quarter of the tile time
__device__ inline float silu_f(float g) {
    return g * __builtin_amdgcn_rcpf(1.0f + __builtin_amdgcn_exp2f(-1.4426950408889634f * g));
}

// tile number -> (row tile, column tile): grouped raster, GM row tiles per group, rows fastest inside
// a group, so that workgroups running together share A and B tiles in L2
__device__ __forceinline__ void tile_of(int id, int nM, int nN, int& tm, int& tn) {
    constexpr int GM = 4;
    const int group = id / (GM * nN);
    const int first_m = group * GM;
    const int gsz = (nM - first_m) < GM ? (nM - first_m) : GM;
    const int in_g = id % (GM * nN);
    tm = first_m + in_g % gsz;
    tn = in_g / gsz;
}

// NW wavefronts per workgroup: 4 (2x2 wavefronts of 128x128, one per SIMD) or 8 (4x2 wavefronts of
// 64x128, two per SIMD: a wavefront's memory instructions, waits and barriers hide behind the other's
// MFMAs at the price of 50 % more LDS fragment traffic).
template <int EPI, int LAY, bool DUAL_A, int NW>
__global__ void __launch_bounds__(NW * 64) gemm_mfma_kernel(GemmArgs a, int nM, int nN, int nfull, int nunits) {
    using R = Ring<LAY, DUAL_A>;
    using IA = typename R::IA;
    using IB = typename R::IB;
    static_assert(!DUAL_A || LAY == LAY_SLABS, "a second A operand travels in slabs of 32");
    constexpr bool AW = R::AW, BW = R::BW;
    constexpr int NSA = R::NSA, NSB = R::NSB;
    constexpr int MI = 32 / NW;                   // 16-row blocks per wavefront (8 or 4)
    constexpr int WROWS = 16 * MI;                // output rows per wavefront
    constexpr int LROWS = 256 / NW;               // operand tile rows each wavefront loads
    constexpr bool DUAL = (EPI == EPI_SILU_MUL || EPI == EPI_SILU_MUL_T);
    constexpr bool SEG = (EPI == EPI_ROPE_STORE);   // two products side by side: rotary columns, then stored columns
    constexpr bool CAN_SPLIT = (EPI == EPI_STORE || EPI == EPI_RESIDUAL || EPI == EPI_ROPE || SEG);
    constexpr int LPA = LROWS / IA::ROWS_PER_LOAD, LPB = LROWS / IB::ROWS_PER_LOAD;   // loads per wavefront per operand tile
    constexpr int PER = LROWS / 16 * (DUAL_A ? 3 : 2);   // direct-to-LDS loads per wavefront per slab (on average, of a wide operand)
    constexpr int STEPS = 2;                             // multiplication steps per slab: 32 of K times half of the wavefront's columns
    extern __shared__ __attribute__((aligned(16))) char smem[];

    // ---- work unit.  Workgroup b runs on XCD b % 8 as that XCD's (b / 8)-th workgroup.  Every XCD
    //      takes a contiguous range of whole tiles first, then a contiguous range of split units
    //      (a split unit = one K share of one of the tiles behind the first nfull), so that all
    //      XCDs run out of whole tiles at the same time.
    const int xcd = (int)(blockIdx.x % 8), pos = (int)(blockIdx.x / 8);
    const int pf = (nfull + 7) / 8;
    int id, split = 0, ksplit = 1;
    if (pos < pf) {
        id = xcd * pf + pos;
        if (id >= nfull) return;
    } else {
        if (!CAN_SPLIT) return;
        const int u = xcd * ((nunits + 7) / 8) + (pos - pf);
        if (u >= nunits) return;
        ksplit = a.ksplit;
        id = nfull + u / ksplit;
        split = u % ksplit;
    }
    const bool partial = CAN_SPLIT && ksplit > 1;
    int tm, tn;
    tile_of(id, nM, nN, tm, tn);

    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int wm = wave >> 1, wn = wave & 1;
    const int l16 = lane & 15, lq = lane >> 4;
    const int64_t row0 = (int64_t)tm * BM;
    constexpr int OUT_COLS = DUAL ? 128 : 256;   // output columns covered by one tile
    const int col0 = tn * OUT_COLS;

    // ---- direct-to-LDS assignment: wavefront w moves tile rows [LROWS * w, LROWS * (w + 1)) of every operand, 16
    //      (32 wide) or 8 (64 wide) rows = 1 KB per load; lane -> (row, LDS chunk position), and fetches
    //      the global chunk that the swizzle maps to that LDS position.
    // A load's address is a wavefront-uniform base (SGPR pair, advanced along K with scalar adds) plus a
    // 32-bit per-lane byte offset that never changes: no vector instructions for addresses in the loop.
    // Bases: A rows from row0 on (or the whole gather source when rows come through an index list, whose
    // byte size must then fit 32 bits); the B rows this wavefront moves.
    // Slab-major operands (32-wide slabs): a row of a slab is 64 bytes and consecutive rows are adjacent, so the row
    // pitch is 64 bytes and one slab further on is rows * 64 bytes.
    const bool a_slab = !AW && a.a_slab, b_slab = !BW && a.b_slab;
    const int64_t a_pitch = a_slab ? 64 : a.lda * 2, b_pitch = b_slab ? 64 : a.ldb * 2;      // bytes between rows
    const bool second = SEG && col0 >= a.n_split;   // this tile belongs to the second product (B1 -> C2)
    const int64_t a_kstep = a_slab ? a.M * 64 : IA::ROW_BYTES;                                       // bytes per tile along K
    const int64_t b_kstep = b_slab ? (second ? a.b_rows1 : a.b_rows) * 64 : IB::ROW_BYTES;
    uint32_t oa[LPA], ob[LPB];
    const char* abase = (const char*)a.A + (a.a_idx ? (int64_t)0 : row0 * a_pitch);
    const char* a1base = DUAL_A ? (const char*)a.A1 + (a.a_idx ? (int64_t)0 : row0 * a_pitch) : abase;
    const char* bbase;
    {
        const int rw = wave * LROWS;   // first B tile row of this wavefront
        if (DUAL) bbase = rw < 128 ? (const char*)a.B0 + (int64_t)(col0 + rw) * b_pitch
                                   : (const char*)a.B1 + (int64_t)(col0 + rw - 128) * b_pitch;
        else if (SEG) bbase = second ? (const char*)a.B1 + (int64_t)(col0 - a.n_split + rw) * b_pitch
                                     : (const char*)a.B0 + (int64_t)(col0 + rw) * b_pitch;
        else if (a.B1 && col0 >= a.N / 2) bbase = (const char*)a.B1 + (int64_t)(col0 - a.N / 2 + rw) * b_pitch;
        else bbase = (const char*)a.B0 + (int64_t)(col0 + rw) * b_pitch;
    }
#pragma unroll
    for (int q = 0; q < LPA; ++q) {
        const int r = wave * LROWS + q * IA::ROWS_PER_LOAD + lane / IA::CPR;
        const int c = (lane % IA::CPR) ^ IA::swz(r);
        int64_t grow = row0 + r;
        if (grow >= a.M) grow = a.M - 1;  // clamp: duplicates of the last row are never stored
        const int64_t srow = a.a_idx ? (int64_t)a.a_idx[grow] : grow - row0;
        oa[q] = (uint32_t)(srow * a_pitch + c * 16);
    }
#pragma unroll
    for (int q = 0; q < LPB; ++q) {
        const int rl = q * IB::ROWS_PER_LOAD + lane / IB::CPR;   // row inside the wavefront's share
        const int c = (lane % IB::CPR) ^ IB::swz(wave * LROWS + rl);
        ob[q] = (uint32_t)((int64_t)rl * b_pitch + c * 16);
    }
    const uint32_t lds0 = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) char*)smem;
    const uint32_t lds_a = lds0 + wave * (LROWS * IA::ROW_BYTES);           // this wavefront's rows inside an operand tile
    const uint32_t lds_b = lds0 + R::B0 + wave * (LROWS * IB::ROW_BYTES);
    // load q of operand tile t_ (counted from this workgroup's share of K): the tile goes to stage t_ % stages
#define SPTS_DMA_A(t_, q) dma16s(oa[q], abase + (a_t0 + (t_)) * a_kstep, lds_a + ((t_) % NSA) * IA::TILE_BYTES + (q) * 1024);
#define SPTS_DMA_B(t_, q) dma16s(ob[q], bbase + (b_t0 + (t_)) * b_kstep, lds_b + ((t_) % NSB) * IB::TILE_BYTES + (q) * 1024);
#define SPTS_DMA_A1(t_, q) dma16s(oa[q], a1base + (a_t0 + (t_)) * a_kstep, lds_a + R::A1 + ((t_) % NSA) * IA::TILE_BYTES + (q) * 1024);
    // Load number u_ of the PER or fewer that slab kt_ puts in flight.  LAY_SLABS: the slab NS - 1 further on, operands in turn.
    // LAY_WIDE_A: half of the A tile two pairs of slabs on, and B's slab three on.  LAY_WIDE_AB: the even slab of a pair fetches B's
    // next tile, the odd one A's next but one.  ISSUE: 1 = all, 2 = B only (A has no tile left).
#define SPTS_ISSUE(kt_, ISSUE, u_)                                                                           \
    {                                                                                                        \
        if (LAY == LAY_SLABS) {                                                                              \
            constexpr int OPS = DUAL_A ? 3 : 2;                                                              \
            if ((u_) < PER) {                                                                                \
                const int q_ = (u_) < PER ? (u_) / OPS : 0;                                                  \
                if ((u_) % OPS == 0) { SPTS_DMA_A((kt_) + NSA - 1, q_) }                                     \
                else if ((u_) % OPS == 1) { SPTS_DMA_B((kt_) + NSA - 1, q_) }                                \
                else { SPTS_DMA_A1((kt_) + NSA - 1, q_) }                                                    \
            }                                                                                                \
        } else if (LAY == LAY_WIDE_A) {                                                                      \
            if ((u_) < LPB) { SPTS_DMA_B((kt_) + 3, ((u_) < LPB ? (u_) : 0)) }                               \
            else if ((ISSUE) == 1 && (u_) < LPB + LPA / 2) { SPTS_DMA_A(((kt_) >> 1) + 2, (((kt_) & 1) * (LPA / 2) + ((u_) < LPB + LPA / 2 ? (u_) - LPB : 0))) } \
        } else {                                                                                             \
            if (((kt_) & 1) == 0) { if ((u_) < LPB) { SPTS_DMA_B(((kt_) >> 1) + 1, ((u_) < LPB ? (u_) : 0)) } } \
            else if ((ISSUE) == 1 && (u_) < LPA) { SPTS_DMA_A(((kt_) >> 1) + 2, ((u_) < LPA ? (u_) : 0)) }   \
        }                                                                                                    \
    }

    f32x4 acc[MI][8];
#pragma unroll
    for (int i = 0; i < MI; ++i)
#pragma unroll
        for (int j = 0; j < 8; ++j)
#pragma unroll
            for (int r = 0; r < 4; ++r) acc[i][j][r] = 0.f;

    // B tile row of this wavefront's N block j (16 columns)
    auto brow = [&](int j) { return DUAL ? (j >> 2) * 128 + wn * 64 + (j & 3) * 16 : wn * 128 + j * 16; };

    // A fragment is 16 rows of 32 K elements.  Step st of a slab multiplies its A fragments by the B fragments of columns
    // 64 * st .. + 63 of the wavefront's.
    bf16x8 af[2][MI], af1[DUAL_A ? MI : 1], bfr[2][4];
    // The fragments of slab kt_ sit in the 32-wide piece kt_ % 2 of a wide operand's stage.
#define SPTS_LOAD_A(buf, kt_)                                                                                \
    {                                                                                                        \
        const char* sA_ = smem + (AW ? ((kt_) >> 1) % NSA : (kt_) % NSA) * IA::TILE_BYTES;                   \
        _Pragma("unroll") for (int i = 0; i < MI; ++i)                                                       \
            af[buf][i] = *reinterpret_cast<const bf16x8*>(sA_ + IA::off(wm * WROWS + i * 16 + l16, (AW ? ((kt_) & 1) * 4 : 0) + lq)); \
    }
#define SPTS_LOAD_A1(kt_)                                                                                    \
    {                                                                                                        \
        const char* sA1_ = smem + R::A1 + ((kt_) % NSA) * IA::TILE_BYTES;                                    \
        _Pragma("unroll") for (int i = 0; i < (DUAL_A ? MI : 0); ++i)                                        \
            af1[i] = *reinterpret_cast<const bf16x8*>(sA1_ + IA::off(wm * WROWS + i * 16 + l16, lq));        \
    }
#define SPTS_LOAD_B(half, kt_)                                                                               \
    {                                                                                                        \
        const char* sB_ = smem + R::B0 + (BW ? ((kt_) >> 1) % NSB : (kt_) % NSB) * IB::TILE_BYTES;           \
        _Pragma("unroll") for (int j = 0; j < 4; ++j)                                                        \
            bfr[half][j] = *reinterpret_cast<const bf16x8*>(sB_ + IB::off(brow((half) * 4 + j) + l16, (BW ? ((kt_) & 1) * 4 : 0) + lq)); \
    }
    // MFMA m of a step: block row m / 4, block columns back and forth, so that each instruction shares an operand with the one before
#define SPTS_MJ(m) (((m) / 4) & 1 ? 3 - (m) % 4 : (m) % 4)
#define SPTS_MFMA(abuf, half, m)                                                                             \
    {                                                                                                        \
        if (DUAL_A && (half) == 1)                                                                           \
            acc[(m) / 4][(half) * 4 + SPTS_MJ(m)] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(bfr[half][SPTS_MJ(m)], af1[DUAL_A ? (m) / 4 : 0], acc[(m) / 4][(half) * 4 + SPTS_MJ(m)], 0, 0, 0); \
        else                                                                                                 \
            acc[(m) / 4][(half) * 4 + SPTS_MJ(m)] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(bfr[half][SPTS_MJ(m)], af[abuf][(m) / 4], acc[(m) / 4][(half) * 4 + SPTS_MJ(m)], 0, 0, 0); \
    }
    constexpr int NM = 4 * MI;                            // MFMAs per step
    constexpr int HS = NM / 2;                            // MFMA slots per half step
    constexpr int NR_ODD = DUAL_A ? MI + 4 : 4;           // fragment reads for the step of the second columns

    // K tiles of this workgroup: all of them, or the split's share (the first `units % ksplit` splits take one more); a unit is a slab,
    // or a pair of slabs where an operand is wide
    const int units = a.K / (AW ? 64 : 32);
    const int my_units = units / ksplit + (split < units % ksplit ? 1 : 0);
    const int unit0 = split * (units / ksplit) + (split < units % ksplit ? split : units % ksplit);
    const int nk = AW ? 2 * my_units : my_units;             // slabs
    const int64_t a_t0 = unit0, b_t0 = AW && !BW ? 2 * (int64_t)unit0 : unit0;   // first tile of A, of B
    // ---- prologue: what the ring holds ahead of slab 0, slab 0's operands first; they must have landed
    if (LAY == LAY_SLABS) {
        const int npre = nk < NSA - 1 ? nk : NSA - 1;
        for (int t = 0; t < npre; ++t) {
            _Pragma("unroll") for (int q = 0; q < LPA; ++q) {
                SPTS_DMA_A(t, q)
                SPTS_DMA_B(t, q)
                if (DUAL_A) SPTS_DMA_A1(t, q)
            }
        }
        if (npre == NSA - 1) { SPTS_WAIT_VMCNT((NSA - 2) * PER); } else { SPTS_WAIT_VMCNT(0); }
    } else {
        _Pragma("unroll") for (int q = 0; q < LPA; ++q) SPTS_DMA_A(0, q)
        _Pragma("unroll") for (int q = 0; q < LPB; ++q) SPTS_DMA_B(0, q)
        if (!BW) { _Pragma("unroll") for (int q = 0; q < LPB; ++q) SPTS_DMA_B(1, q) }
        if (nk > 2) {
            _Pragma("unroll") for (int q = 0; q < LPA; ++q) SPTS_DMA_A(1, q)
            if (!BW) { _Pragma("unroll") for (int q = 0; q < LPB; ++q) SPTS_DMA_B(2, q) }
            SPTS_WAIT_VMCNT(LPA + (BW ? 0 : 2 * LPB));
        } else { SPTS_WAIT_VMCNT(0); }
    }
    __syncthreads();
    SPTS_LOAD_A(0, 0)
    SPTS_LOAD_B(0, 0)

    // One slab of 32 = two steps of 16 MFMAs per wavefront.  Every memory instruction sits in the
    // shadow of an MFMA (an MFMA occupies the matrix pipe for 8 cycles while the wavefront may
    // issue other work):
    //   first step: the first half's MFMAs are interleaved with the fragment reads of the second step, the second half's with the
    //               direct-to-LDS loads (ISSUE);
    //   last step:  a quarter of the MFMAs, then (SYNC) wait for this wavefront's share of the next slab and meet the
    //               workgroup (the next slab is published, the stages read last by this one are free from here on),
    //               then the other MFMAs, interleaved with the first fragment reads of the next slab.
    // The loads of the two slabs behind the one being published may still be in flight (WAITN).  The even slab of a pair of wide
    // operands publishes and frees nothing (SYNC false).
    // ISSUE / SYNC / NEXT / PAR (buffer of the slab's A fragments) / COPY (hand the next slab its A fragments in buffer 0) are
    // literal constants at every expansion.
#define SPTS_SLAB(kt_, ISSUE, SYNC, NEXT, WAITN, PAR, COPY)                                                  \
    {                                                                                                        \
        constexpr int ab_ = (PAR);                                                                           \
        SPTS_LOAD_B(1, kt_)                                                                                  \
        SPTS_LOAD_A1(kt_)                                                                                    \
        _Pragma("unroll") for (int m_ = 0; m_ < HS; ++m_) SPTS_MFMA(ab_, 0, m_)                              \
        _Pragma("unroll") for (int g_ = 0; g_ < HS; ++g_) {                                                  \
            __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);                                               \
            __builtin_amdgcn_sched_group_barrier(0x100, (NR_ODD + HS - 1) / HS, 0);                          \
        }                                                                                                    \
        __builtin_amdgcn_sched_barrier(0);                                                                   \
        _Pragma("unroll") for (int m_ = HS; m_ < NM; ++m_) {                                                 \
            SPTS_MFMA(ab_, 0, m_)                                                                            \
            if (ISSUE) {                                                                                     \
                __builtin_amdgcn_sched_barrier(0);                                                           \
                SPTS_ISSUE(kt_, ISSUE, m_ - HS)                                                              \
                __builtin_amdgcn_sched_barrier(0);                                                           \
            }                                                                                                \
        }                                                                                                    \
        _Pragma("unroll") for (int m_ = 0; m_ < NM / 4; ++m_) SPTS_MFMA(ab_, 1, m_)                          \
        if (SYNC) {                                                                                          \
            if (NEXT) { SPTS_WAIT_VMCNT(WAITN); }                                                            \
            __syncthreads();                                                                                 \
        }                                                                                                    \
        if (NEXT) { SPTS_LOAD_A(ab_ ^ 1, (kt_) + 1) SPTS_LOAD_B(0, (kt_) + 1) }                              \
        _Pragma("unroll") for (int m_ = NM / 4; m_ < NM; ++m_) SPTS_MFMA(ab_, 1, m_)                         \
        if (NEXT) {                                                                                          \
            _Pragma("unroll") for (int g_ = 0; g_ < NM - NM / 4; ++g_) {                                     \
                __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);                                           \
                __builtin_amdgcn_sched_group_barrier(0x100, 1, 0);                                           \
            }                                                                                                \
        }                                                                                                    \
        __builtin_amdgcn_sched_barrier(0);                                                                   \
        if (NEXT && (COPY)) {                                                                                \
            _Pragma("unroll") for (int i = 0; i < MI; ++i) af[0][i] = af[1][i];                              \
        }                                                                                                    \
    }

    // Steady state, first in groups of UNROLL slabs, where the ring stage of every slab is a
    // compile-time constant and the LDS addresses of the fragment reads need no arithmetic in the loop.
    int kt = 0;
    if (LAY == LAY_SLABS) {
        // after the loads of slab kt + NSA - 1 are issued the slabs behind kt + 1 in flight are kt + 2 .. kt + NSA - 1
        if (NSA == 4) {
            int kb = 0;
            for (; kb * 4 + 6 < nk; ++kb) {
                _Pragma("unroll") for (int u = 0; u < 4; ++u) {
                    if (u & 1) SPTS_SLAB(kb * 4 + u, 1, true, true, (NSA - 2) * PER, 1, false)
                    else SPTS_SLAB(kb * 4 + u, 1, true, true, (NSA - 2) * PER, 0, false)
                }
            }
            kt = kb * 4;
        }
        for (; kt + NSA - 1 < nk; ++kt) SPTS_SLAB(kt, 1, true, true, (NSA - 2) * PER, 0, true)
        // drain: nothing left to issue; wait for everything that is still in flight
        for (; kt + 1 < nk; ++kt) SPTS_SLAB(kt, 0, true, true, 0, 0, true)
        SPTS_SLAB(kt, 0, true, false, 0, 0, false)
    } else {
        // a pair of slabs whose A tile two pairs on exists; LAY_WIDE_A: at the end of a slab the loads of it and of the one before may
        // be in flight, LAY_WIDE_AB: at the end of a pair those of its odd slab
        constexpr int W = BW ? LPA : 2 * PER;
        int kb = 0;
        for (; kb * R::UNROLL + R::UNROLL + 4 <= nk; ++kb) {
            _Pragma("unroll") for (int u = 0; u < R::UNROLL; u += 2) {
                SPTS_SLAB(kb * R::UNROLL + u, 1, !BW, true, W, 0, false)
                SPTS_SLAB(kb * R::UNROLL + u + 1, 1, true, true, W, 1, false)
            }
        }
        for (kt = kb * R::UNROLL; kt + 4 < nk; kt += 2) {
            SPTS_SLAB(kt, 1, !BW, true, W, 0, false)
            SPTS_SLAB(kt + 1, 1, true, true, W, 1, false)
        }
        // the last two pairs: A is all in flight or landed, B's last slab (last tile) is still to be fetched
        if (nk > 2) {
            SPTS_SLAB(kt, 2, !BW, true, PER + LPB, 0, false)
            SPTS_SLAB(kt + 1, 0, true, true, BW ? 0 : LPB, 1, false)
            kt += 2;
        }
        SPTS_SLAB(kt, 0, !BW, true, 0, 0, false)
        SPTS_SLAB(kt + 1, 0, true, false, 0, 1, false)
    }

    // ---- epilogue.  acc[i][j][r]: row = row0 + wm*WROWS + i*16 + l16, column (inside the wavefront's share) =
    //      16*j + 4*lq + r  -> 4 consecutive columns per block.
    bf16_t* Cb = (bf16_t*)a.C;
    if (partial) {
        // raw fp32 accumulators in fragment order: every store instruction of a wavefront writes 1 KB
        float* P = a.part32 + ((int64_t)(id - nfull) * ksplit + split) * (BM * 256);
#pragma unroll
        for (int i = 0; i < MI; ++i)
#pragma unroll
            for (int j = 0; j < 8; ++j) *reinterpret_cast<f32x4*>(P + (((wave * MI + i) * 8 + j) * 64 + lane) * 4) = acc[i][j];
        return;
    }
    if (EPI == EPI_SUMSQ) {
#pragma unroll
        for (int i = 0; i < MI; ++i) {
            float s = 0.f;
#pragma unroll
            for (int j = 0; j < 8; ++j)
#pragma unroll
                for (int r = 0; r < 4; ++r) s += acc[i][j][r] * acc[i][j][r];
            s += __shfl_xor(s, 16);
            s += __shfl_xor(s, 32);
            int64_t grow = row0 + wm * WROWS + i * 16 + l16;
            if (lq == 0 && grow < a.M) a.part[grow * a.part_ld + tn * 2 + wn] = s;
        }
        return;
    }
    // The finished values are packed to bf16 and staged through LDS (the operand ring is free now) so that
    // the tile leaves in whole rows: a lane owns 4 consecutive columns of 16 different rows per N block,
    // and stores straight from the fragment layout would reach memory as 16-byte pieces of 32 rows per
    // instruction.  Staged row tr keeps 16-byte chunk c at chunk position c ^ (tr % NCH): the 32 lanes of a
    // fragment write (32 rows, same chunk) and the row-wise reads are both spread over all banks.
    constexpr int NCH = OUT_COLS / 8;            // 16-byte chunks per staged row
    constexpr int ROWB = OUT_COLS * 2;           // bytes per staged row
    const int colshift = second ? a.n_split : 0; // the second product's outputs count their columns from n_split
    if (second) Cb = (bf16_t*)a.C2;
    const int64_t ldo = second ? a.ldc2 : a.ldc;
    auto stage = [&](int tr, int tc, uint2 o) {
        *reinterpret_cast<uint2*>(smem + tr * ROWB + ((((tc >> 3) ^ tr) & (NCH - 1)) << 4) + ((tc & 4) << 1)) = o;
    };
#pragma unroll
    for (int i = 0; i < MI; ++i) {
        const int tr = wm * WROWS + i * 16 + l16;
        const int64_t grow = row0 + tr;
        const bool rok = grow < a.M;
        const int64_t growc = rok ? grow : a.M - 1;
        const int64_t crow = a.c_idx ? (int64_t)a.c_idx[growc] : growc;
        if (EPI == EPI_STORE || (SEG && second)) {
#pragma unroll
            for (int j = 0; j < 8; ++j) {
                const int cb = col0 - colshift + wn * 128 + j * 16 + 4 * lq;   // column of this product's output
                uint2 o;
                o.x = pack_bf16x2(acc[i][j][0], acc[i][j][1]);
                o.y = pack_bf16x2(acc[i][j][2], acc[i][j][3]);
                stage(tr, cb - (col0 - colshift), o);
                if (a.Ct && grow < a.ldct) {
                    bf16_t* ct = (bf16_t*)a.Ct;
                    const uint16_t e[4] = {(uint16_t)(o.x & 0xffff), (uint16_t)(o.x >> 16), (uint16_t)(o.y & 0xffff), (uint16_t)(o.y >> 16)};
#pragma unroll
                    for (int t = 0; t < 4; ++t) ct[(int64_t)(cb + t) * a.ldct + vt_key_slot(grow)].v = e[t];
                }
            }
        } else if (EPI == EPI_RESIDUAL) {
            // the old values are read in the fragment layout (rows past M read the last row; they are not
            // stored): one rounding of old + acc, as without the staging
#pragma unroll
            for (int j = 0; j < 8; ++j) {
                const int cb = col0 + wn * 128 + j * 16 + 4 * lq;
                const uint2 old = *reinterpret_cast<const uint2*>(Cb + crow * a.ldc + cb);
                float x0 = __uint_as_float(old.x << 16), x1 = __uint_as_float(old.x & 0xffff0000u);
                float x2 = __uint_as_float(old.y << 16), x3 = __uint_as_float(old.y & 0xffff0000u);
                uint2 o;
                o.x = pack_bf16x2(x0 + acc[i][j][0], x1 + acc[i][j][1]);
                o.y = pack_bf16x2(x2 + acc[i][j][2], x3 + acc[i][j][3]);
                stage(tr, cb - col0, o);
            }
        } else if (EPI == EPI_SILU_MUL_T) {
            // channel-major: staged channel c keeps the 16-byte chunk (8 rows) r at chunk position r ^ (c % 32), which spreads the
            // 2-byte writes of a lane's four channels and the whole-channel reads over the banks
#pragma unroll
            for (int j = 0; j < 4; ++j)
#pragma unroll
                for (int r = 0; r < 4; ++r) {
                    const int c = wn * 64 + j * 16 + 4 * lq + r;
                    *reinterpret_cast<bf16_t*>(smem + c * 512 + ((((tr >> 3) ^ c) & 31) << 4) + ((tr & 7) << 1)) =
                        f32_to_bf16(silu_f(acc[i][j][r]) * acc[i][j + 4][r]);
                }
        } else if (EPI == EPI_SILU_MUL) {
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                float h[4];
#pragma unroll
                for (int t = 0; t < 4; ++t) h[t] = silu_f(acc[i][j][t]) * acc[i][j + 4][t];
                uint2 o; o.x = pack_bf16x2(h[0], h[1]); o.y = pack_bf16x2(h[2], h[3]);
                stage(tr, wn * 64 + j * 16 + 4 * lq, o);
            }
        } else if (EPI == EPI_ROPE || SEG) {
            const int64_t trow = a.rope_idx ? (int64_t)a.rope_idx[growc] : growc;
            const int half = a.head_dim >> 1;
            const float2* tab = a.rope + trow * half;
            const float rs = a.rope_scale != 0.f ? a.rope_scale : 1.f;
            // blocks j1 and j2 are d/2 columns apart; jj: the quad's first column inside the half head
            auto rotate = [&](int j1, int j2, int jj) {
                float lo[4], hi[4];
#pragma unroll
                for (int t = 0; t < 4; ++t) {
                    float2 cs = tab[jj + t];
                    float x1 = acc[i][j1][t], x2 = acc[i][j2][t];
                    lo[t] = (x1 * cs.x - x2 * cs.y) * rs;
                    hi[t] = (x2 * cs.x + x1 * cs.y) * rs;
                }
                uint2 o1, o2;
                o1.x = pack_bf16x2(lo[0], lo[1]); o1.y = pack_bf16x2(lo[2], lo[3]);
                o2.x = pack_bf16x2(hi[0], hi[1]); o2.y = pack_bf16x2(hi[2], hi[3]);
                stage(tr, wn * 128 + j1 * 16 + 4 * lq, o1);
                stage(tr, wn * 128 + j2 * 16 + 4 * lq, o2);
            };
            if (half == 64) {   // wavefront = one head of 128 columns
#pragma unroll
                for (int j = 0; j < 4; ++j) rotate(j, j + 4, j * 16 + 4 * lq);
            } else {            // d = 64: two heads per wavefront
#pragma unroll
                for (int j = 0; j < 4; ++j) rotate((j >> 1) * 4 + (j & 1), (j >> 1) * 4 + (j & 1) + 2, (j & 1) * 16 + 4 * lq);
            }
        }
    }
    // ---- the staged tile leaves row by row: NCH consecutive lanes write one row's OUT_COLS columns as
    //      16-byte pieces (whole 128-byte lines), rows through the scatter list when there is one
    __syncthreads();
    if (EPI == EPI_SILU_MUL_T) {
        // a channel's 256 rows are 512 contiguous bytes (rows past M are stored too: ldc covers whole tiles)
#pragma unroll 4
        for (int e = tid; e < 128 * 32; e += NW * 64) {
            const int c = e >> 5, ch = e & 31;
            *reinterpret_cast<u32x4*>(Cb + (int64_t)(col0 + c) * a.ldc + row0 + ch * 8) =
                *reinterpret_cast<const u32x4*>(smem + c * 512 + (((ch ^ c) & 31) << 4));
        }
        return;
    }
    if ((EPI == EPI_SILU_MUL || EPI == EPI_STORE) && a.c_slab) {
        // slab-major output: slab sl of the tile is 256 rows x 64 bytes, contiguous over the rows; 4 lanes per row
        constexpr int RPS = NW * 64 / 4;         // rows per pass
        const int oc4 = tid & 3, r_in = tid >> 2;
#pragma unroll
        for (int sl = 0; sl < OUT_COLS / 32; ++sl)
#pragma unroll
            for (int p = 0; p < 256 / RPS; ++p) {
                const int tr = p * RPS + r_in;
                const int64_t grow = row0 + tr;
                if (grow < a.M) {
                    const u32x4 v = *reinterpret_cast<const u32x4*>(smem + tr * ROWB + ((((sl * 4 + oc4) ^ tr) & (NCH - 1)) << 4));
                    *reinterpret_cast<u32x4*>(Cb + (((int64_t)(col0 >> 5) + sl) * a.M + grow) * 32 + oc4 * 8) = v;
                }
            }
        return;
    }
    constexpr int RPP = NW * 64 / NCH;           // rows per pass of the workgroup
    const int oc = tid % NCH, orow = tid / NCH;
#pragma unroll 4
    for (int p = 0; p < 256 / RPP; ++p) {
        const int tr = p * RPP + orow;
        const int64_t grow = row0 + tr;
        if (grow < a.M) {
            const int64_t crow = a.c_idx ? (int64_t)a.c_idx[grow] : grow;
            const u32x4 v = *reinterpret_cast<const u32x4*>(smem + tr * ROWB + (((oc ^ tr) & (NCH - 1)) << 4));
            *reinterpret_cast<u32x4*>(Cb + crow * ldo + (col0 - colshift) + oc * 8) = v;
        }
    }
}

int gemm_sumsq_blocks(int32_t N, bool mfma) { return mfma ? (N + 127) / 128 : (N + 63) / 64; }

static inline bool al16(const void* p) { return (reinterpret_cast<uintptr_t>(p) & 15u) == 0; }

bool gemm_mfma_supported(const GemmArgs& a) {
    if (a.c_is_f32) return false;
    const bool dual = a.epi == EPI_SILU_MUL || a.epi == EPI_SILU_MUL_T;
    const int ncols = dual ? 128 : 256;
    if (a.epi == EPI_SILU_MUL_T && (a.A1 || a.c_idx || a.Ct || a.c_slab || a.ldc < (a.M + BM - 1) / BM * BM)) return false;
    if (a.M <= 0 || a.N <= 0 || a.N % ncols != 0) return false;
    if (a.K < 32 || a.K % 32 != 0) return false;
    if (a.lda % 8 != 0 || a.ldb % 8 != 0) return false;
    // slab-major operands: served by the 32-wide-slab instantiations; A not gathered
    const bool seg = a.epi == EPI_ROPE_STORE;
    if ((a.a_slab || a.b_slab) && !dual && a.epi != EPI_RESIDUAL && a.epi != EPI_STORE && a.epi != EPI_ROPE && !seg) return false;
    if (seg) {
        if (a.n_split <= 0 || a.n_split >= a.N || a.n_split % 256 != 0 || a.c_idx || a.c_slab) return false;
        if (!a.B1 || !al16(a.B1) || !a.C2 || !al16(a.C2) || a.ldc2 % 8 != 0) return false;
        if (a.b_slab && (a.b_rows < a.n_split || a.b_rows1 < a.N - a.n_split)) return false;
    }
    if (a.a_slab && a.a_idx) return false;
    if (a.b_slab && !seg && a.b_rows < (a.epi == EPI_STORE && a.B1 ? a.N / 2 : a.N)) return false;   // rows of each B matrix
    if (a.c_slab && ((a.epi != EPI_SILU_MUL && a.epi != EPI_STORE) || a.c_idx || a.Ct)) return false;
    if (!al16(a.A) || !al16(a.B0) || (a.A1 && !al16(a.A1)) || (dual && !al16(a.B1))) return false;
    if (a.epi != EPI_SUMSQ) {
        if (a.ldc % 8 != 0 || !al16(a.C)) return false;
    }
    if ((a.epi == EPI_ROPE || seg) && a.head_dim != 128 && a.head_dim != 64) return false;
    if (a.Ct && a.epi != EPI_STORE && !seg) return false;
    if (a.epi == EPI_STORE && a.B1 && (a.N % 512 != 0 || !al16(a.B1))) return false;
    if (a.ksplit > 1) {
        if (!a.part32 || !al16(a.part32) || (a.epi != EPI_STORE && a.epi != EPI_RESIDUAL && a.epi != EPI_ROPE && !seg)) return false;
        if (a.K / 64 < a.ksplit || a.nfull < 0 || a.nfull > (a.M + BM - 1) / BM * (a.N / 256)) return false;
    }
    if (a.M > (int64_t)1 << 30) return false;
    // 32-bit byte offsets from the load bases: the gather source as a whole, 256 rows of A or B otherwise
    if (a.a_idx && (a.a_rows <= 0 || a.a_rows * a.lda * 2 >= ((int64_t)1 << 32))) return false;
    if (256 * a.lda * 2 >= ((int64_t)1 << 32) || 256 * a.ldb * 2 >= ((int64_t)1 << 32)) return false;
    return true;
}

template <int EPI, int LAY, bool DUAL_A, int NW>
static hipError_t launch_t(const GemmArgs& a, hipStream_t s) {
    const int ncols = EPI == EPI_SILU_MUL || EPI == EPI_SILU_MUL_T ? 128 : 256;
    const int nM = (int)((a.M + BM - 1) / BM), nN = a.N / ncols;
    const int tiles = nM * nN;
    const bool split = a.ksplit > 1;
    const int nfull = split ? a.nfull : tiles;
    const int nunits = split ? (tiles - nfull) * a.ksplit : 0;
    const int grid = 8 * ((nfull + 7) / 8 + (nunits + 7) / 8);
    const size_t lds = Ring<LAY, DUAL_A>::BYTES;
    {
        hipError_t e = ensure_dynamic_lds(reinterpret_cast<const void*>(&gemm_mfma_kernel<EPI, LAY, DUAL_A, NW>), (int)lds);
        if (e != hipSuccess) return e;
    }
    gemm_mfma_kernel<EPI, LAY, DUAL_A, NW><<<dim3(grid), dim3(NW * 64), lds, s>>>(a, nM, nN, nfull, nunits);
    return hipGetLastError();
}

template <int EPI, int NW>
static hipError_t launch_layout(const GemmArgs& a, hipStream_t s) {
    constexpr bool silu = EPI == EPI_SILU_MUL || EPI == EPI_SILU_MUL_T;
    if (a.a_slab || a.K % 64 != 0) return launch_t<EPI, LAY_SLABS, false, NW>(a, s);
    // row-major weights of the SiLU products: 32 wide as well, i.e. in halves of lines but three slabs ahead (gate/up of 13107 rows
    // 2440 -> 2333 us, of 3276 rows 615 -> 591); the other products are faster in whole lines (down of 8192 rows 736 against 762)
    if constexpr (silu) return launch_t<EPI, LAY_WIDE_A, false, NW>(a, s);
    else {
        if constexpr (EPI != EPI_SUMSQ) {   // which is refused with a slab-major B
            if (a.b_slab) return launch_t<EPI, LAY_WIDE_A, false, NW>(a, s);
        }
        return launch_t<EPI, LAY_WIDE_AB, false, NW>(a, s);
    }
}

// ---- tail split-K second pass: one thread per FIN_U accumulator-fragment quads (4 consecutive columns of FIN_U rows 16 apart) of a
//      split tile; sums the splits in split order and applies the epilogue exactly as the single-pass kernel does.  In a rotary
//      product (not in one that also stores) a thread owns the quad and its partner d/2 columns on, and only the first halves of
//      the heads have threads.  Bound: the memory-side cache, which the partial tiles were
//      just written to; with one quad per thread, half of a rotary product's wavefronts had nothing to do and a thread waited for
//      one load at a time: K projection of 8192 rows (256 shares) 26 -> 18 us, of 20011 rows 21 -> 15, stored products the same.
constexpr int FIN_U = 2;
template <int NW>
__global__ void __launch_bounds__(256) splitk_finish_kernel(GemmArgs a, int nM, int nN, int nfull) {
    constexpr int MI = 32 / NW, WROWS = 16 * MI, MG = MI / FIN_U;
    const int64_t g = (int64_t)blockIdx.x * 256 + threadIdx.x;
    const bool halves = a.epi == EPI_ROPE;         // 4 of the 8 column blocks have threads
    const int jb = halves ? 2 : 3;
    const int per_tile = 16384 / FIN_U >> (halves ? 1 : 0);
    const int rt = (int)(g / per_tile);            // split tile
    const int v = (int)(g % per_tile);
    const int lane = v & 63, jx = (v >> 6) & ((1 << jb) - 1), wi = v >> (6 + jb);
    const int wave = wi / MG, i0 = wi % MG * FIN_U;
    const int j = halves && a.head_dim == 64 ? (jx >> 1) * 4 + (jx & 1) : jx;
    const int wm = wave >> 1, wn = wave & 1, l16 = lane & 15, lq = lane >> 4;
    int tm, tn;
    tile_of(nfull + rt, nM, nN, tm, tn);
    const int col0 = tn * 256;
    const float* P = a.part32 + (int64_t)rt * a.ksplit * (BM * 256);
    auto quads = [&](int jj, f32x4 (&s)[FIN_U]) {
        const float* p = P + (((wave * MI + i0) * 8 + jj) * 64 + lane) * 4;
#pragma unroll
        for (int u = 0; u < FIN_U; ++u) s[u] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll 2
        for (int sp = 0; sp < a.ksplit; ++sp)
#pragma unroll
            for (int u = 0; u < FIN_U; ++u) s[u] += *reinterpret_cast<const f32x4*>(p + (int64_t)sp * (BM * 256) + u * 8 * 64 * 4);
    };
    bf16_t* Cb = (bf16_t*)a.C;
    // two products in one launch: a tile is either a rotary tile of the first or a stored tile of the second
    int epi = a.epi, colshift = 0;
    int64_t ldo = a.ldc;
    if (epi == EPI_ROPE_STORE) {
        if (col0 >= a.n_split) { epi = EPI_STORE; colshift = a.n_split; Cb = (bf16_t*)a.C2; ldo = a.ldc2; }
        else epi = EPI_ROPE;
    }
    const int half = a.head_dim >> 1;
    int j2 = j, jj = 0;   // rotary: block of the quad's partner; column inside the half head
    if (epi == EPI_ROPE) {
        if (half == 64) { if (j >= 4) return; j2 = j + 4; jj = j * 16 + 4 * lq; }
        else { if (j & 2) return; j2 = j + 2; jj = (j & 1) * 16 + 4 * lq; }
    }
    f32x4 s1[FIN_U], s2[FIN_U];
    quads(j, s1);
    if (epi == EPI_ROPE) quads(j2, s2);
    const int col = col0 - colshift + wn * 128 + (epi == EPI_ROPE ? (half == 64 ? 0 : (j >> 2) * 64) + jj : j * 16 + 4 * lq);
#pragma unroll
    for (int u = 0; u < FIN_U; ++u) {
        const f32x4 s = s1[u];
        const int64_t grow = (int64_t)tm * BM + wm * WROWS + (i0 + u) * 16 + l16;
        const bool rok = grow < a.M;
        const int64_t growc = rok ? grow : a.M - 1;
        const int64_t crow = a.c_idx ? (int64_t)a.c_idx[growc] : growc;
        if (epi == EPI_STORE) {
            u32x2 o = {pack_bf16x2(s.x, s.y), pack_bf16x2(s.z, s.w)};
            if (rok) {
                if (a.c_slab) *reinterpret_cast<u32x2*>(Cb + ((int64_t)(col >> 5) * a.M + grow) * 32 + (col & 31)) = o;   // slab-major C
                else *reinterpret_cast<u32x2*>(Cb + crow * ldo + col) = o;
            }
            if (a.Ct && grow < a.ldct) {
                bf16_t* ct = (bf16_t*)a.Ct;
                const uint16_t e[4] = {(uint16_t)(o.x & 0xffff), (uint16_t)(o.x >> 16), (uint16_t)(o.y & 0xffff), (uint16_t)(o.y >> 16)};
#pragma unroll
                for (int t = 0; t < 4; ++t) ct[(int64_t)(col + t) * a.ldct + vt_key_slot(grow)].v = e[t];
            }
        } else if (epi == EPI_RESIDUAL) {
            if (!rok) continue;
            u32x2* p = reinterpret_cast<u32x2*>(Cb + crow * a.ldc + col);
            const u32x2 old = *p;
            u32x2 o;
            o.x = pack_bf16x2(__uint_as_float(old.x << 16) + s.x, __uint_as_float(old.x & 0xffff0000u) + s.y);
            o.y = pack_bf16x2(__uint_as_float(old.y << 16) + s.z, __uint_as_float(old.y & 0xffff0000u) + s.w);
            *p = o;
        } else {   // EPI_ROPE
            if (!rok) continue;
            const int64_t trow = a.rope_idx ? (int64_t)a.rope_idx[grow] : grow;
            const float2* tab = a.rope + trow * half + jj;
            const float rs = a.rope_scale != 0.f ? a.rope_scale : 1.f;
            float lo[4], hi[4];
#pragma unroll
            for (int t = 0; t < 4; ++t) {
                const float2 cs = tab[t];
                lo[t] = (s[t] * cs.x - s2[u][t] * cs.y) * rs;
                hi[t] = (s2[u][t] * cs.x + s[t] * cs.y) * rs;
            }
            u32x2 o1 = {pack_bf16x2(lo[0], lo[1]), pack_bf16x2(lo[2], lo[3])};
            u32x2 o2 = {pack_bf16x2(hi[0], hi[1]), pack_bf16x2(hi[2], hi[3])};
            *reinterpret_cast<u32x2*>(Cb + crow * a.ldc + col) = o1;
            *reinterpret_cast<u32x2*>(Cb + crow * a.ldc + col + half) = o2;
        }
    }
}

// Cost model behind the split plan (one workgroup per CU, 256 CUs): a whole tile takes
// t_tile = 2*256*256*K flops at 4.2 TFLOP/s a CU (a chip of them reaches 1.3 times that now; the splits are as good as measured, see
// the time models of kernels_gemm_small.hip); the tail of `rem` tiles costs one t_tile
// unsplit, or ceil(rem*ks/256)/ks of it plus the partial-tile traffic (rem*ks tiles of 256 KB, written
// and read back) plus one more launch when split ks ways.
int gemm_pick_split(int64_t M, int32_t N, int32_t K, int epi, int32_t* nfull) {
    *nfull = 0;
    if (epi != EPI_STORE && epi != EPI_RESIDUAL && epi != EPI_ROPE && epi != EPI_ROPE_STORE) return 1;
    if (N % 256 != 0 || M <= 0) return 1;
    const int64_t tiles = ((M + BM - 1) / BM) * (N / 256);
    const int rem = (int)(tiles % 256);
    if (rem == 0) return 1;
    const double t_tile = 2.0 * 256 * 256 * K / 4.2e12;
    double best = t_tile;
    int best_ks = 1;
    for (int ks = 2; ks <= 8; ++ks) {
        if (K / ks < 512) break;
        const int rounds = (rem * ks + 255) / 256;
        const double t = t_tile * rounds / ks + (double)rem * ks * 262144.0 * 2.0 / 4.0e12 + 6e-6;
        if (t < best * 0.97) { best = t; best_ks = ks; }
    }
    *nfull = (int32_t)(tiles - rem);
    return best_ks;
}

// wavefronts per workgroup: the order of a split tile's shares follows it, in the launches and in both second passes
constexpr int GEMM_NW = 8;

static hipError_t launch_products(const GemmArgs& a, hipStream_t s) {
    constexpr int NW = GEMM_NW;
    hipError_t e;
    switch (a.epi) {
        case EPI_STORE: e = launch_layout<EPI_STORE, NW>(a, s); break;
        case EPI_RESIDUAL: e = launch_layout<EPI_RESIDUAL, NW>(a, s); break;
        case EPI_SUMSQ: e = launch_layout<EPI_SUMSQ, NW>(a, s); break;
        case EPI_ROPE: e = launch_layout<EPI_ROPE, NW>(a, s); break;
        case EPI_ROPE_STORE: e = launch_layout<EPI_ROPE_STORE, NW>(a, s); break;
        case EPI_SILU_MUL: e = a.A1 ? launch_t<EPI_SILU_MUL, LAY_SLABS, true, NW>(a, s) : launch_layout<EPI_SILU_MUL, NW>(a, s); break;
        case EPI_SILU_MUL_T: e = launch_layout<EPI_SILU_MUL_T, NW>(a, s); break;
        default: return hipErrorInvalidValue;
    }
    return e;
}

hipError_t launch_gemm_mfma(const GemmArgs& a, hipStream_t s) {
    constexpr int NW = GEMM_NW;
    const hipError_t e = launch_products(a, s);
    if (e != hipSuccess || a.ksplit <= 1) return e;
    const int nM = (int)((a.M + BM - 1) / BM), nN = a.N / 256;
    const int64_t threads = (int64_t)(nM * nN - a.nfull) * (16384 / FIN_U >> (a.epi == EPI_ROPE ? 1 : 0));
    if (threads <= 0) return hipSuccess;
    splitk_finish_kernel<NW><<<dim3((unsigned)(threads / 256)), dim3(256), 0, s>>>(a, nM, nN, a.nfull);
    return hipGetLastError();
}

// Second pass of a split product of 256 columns whose rows are wanted only for their norms (the proxy's z): c[n] = ||z[n, :]||, with z rounded to
// bf16 as the stored one would be, s[n] = c[n] * s_mha[n].  A workgroup takes 16 rows, which are 16 chunks of 1 KB in every share
// (fragment order: a chunk is 16 rows x 16 columns); wavefront w sums the shares of chunks 4 w .. 4 w + 3, squares, and the 16 row sums meet in
// LDS.  z is neither written nor read: 8192 rows in 8 shares 18.7 -> 13.4 us, 32768 in 2 22 -> 12, 11159 in 2 17 -> 10.3.
struct NormTiles { int tm, nM, nN; };   // tm: rows of a tile (64 / 128 / 192 x 128 of the short products, 256 x 256)
__global__ void __launch_bounds__(256) norm_finish_kernel(const float* __restrict__ part, NormTiles t, int ksplit, const float* __restrict__ s_mha,
                                                          float* __restrict__ c_ffn, float* __restrict__ s_ffn, int64_t M) {
    __shared__ float red[4][16];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, l16 = lane & 15;
    const int per_tile = t.tm / 16, tm = blockIdx.x / per_tile, gi = blockIdx.x - tm * per_tile;
    const int64_t row = (int64_t)tm * t.tm + gi * 16 + l16;
    const int64_t tiles = (int64_t)t.nM * t.nN, stride = t.tm == 256 ? 65536 : tiles * t.tm * 128;
    float sq = 0.f;
#pragma unroll
    for (int u = 0; u < 4; ++u) {
        const int c = wave * 4 + u;
        const float* p;
        if (t.tm == 256) {   // wavefront (gi / MI, c / 8) of the product, its block row gi % MI
            constexpr int MI = 32 / GEMM_NW;
            p = part + (int64_t)tm * ksplit * 65536 + ((gi / MI * 2 + (c >> 3)) * MI + gi % MI) * 2048 + (c & 7) * 256;
        }
        else {
            const int half = t.tm / 32, wm = gi / half, in = gi - wm * half;        // row groups of a wavefront
            const int group = tm / 8 * 8, gsz = t.nM - group < 8 ? t.nM - group : 8;
            const int64_t id = (int64_t)group * t.nN + (c >> 3) * gsz + (tm - group);   // as small_tile_of numbers the tiles
            p = part + id * t.tm * 128 + (((((wm * 2 + ((c >> 2) & 1)) * (t.tm / 64) + (in >> 1)) * 2 + ((c >> 1) & 1)) * 4 + (in & 1) * 2 + (c & 1)) * 64) * 4;
        }
        f32x4 z = {0.f, 0.f, 0.f, 0.f};
#pragma unroll 4
        for (int sp = 0; sp < ksplit; ++sp) z += *reinterpret_cast<const f32x4*>(p + sp * stride + lane * 4);
        const uint32_t lo = pack_bf16x2(z[0], z[1]), hi = pack_bf16x2(z[2], z[3]);
        const float v[4] = {__uint_as_float(lo << 16), __uint_as_float(lo & 0xffff0000u), __uint_as_float(hi << 16), __uint_as_float(hi & 0xffff0000u)};
#pragma unroll
        for (int e = 0; e < 4; ++e) sq += v[e] * v[e];
    }
    sq += __shfl_xor(sq, 16);
    sq += __shfl_xor(sq, 32);
    if (lane < 16) red[wave][l16] = sq;
    __syncthreads();
    if (threadIdx.x < 16 && row < M) {
        const float c = sqrtf(red[0][l16] + red[1][l16] + red[2][l16] + red[3][l16]);
        if (c_ffn) c_ffn[row] = c;
        if (s_ffn) s_ffn[row] = s_mha ? c * s_mha[row] : c;
    }
}

bool gemm_norm_supported(const GemmArgs& a, int wide_ksplit, int wide_nfull, const GemmSmallPlan* small) {
    if (a.epi != EPI_STORE || a.N != 256 || a.B1 || a.Ct || !gemm_mfma_supported(a)) return false;
    return small ? small->ksplit > 1 : wide_ksplit > 1 && wide_nfull == 0;
}
hipError_t launch_gemm_norm(const GemmArgs& a, const GemmSmallPlan* small, const float* s_mha, float* c_ffn, float* s_ffn, hipStream_t s) {
    const NormTiles t = small ? NormTiles{small->tm, (int)((a.M + small->tm - 1) / small->tm), 2} : NormTiles{256, (int)((a.M + BM - 1) / BM), 1};
    const hipError_t e = small ? launch_gemm_small_shares(a, *small, s) : launch_products(a, s);
    if (e != hipSuccess) return e;
    norm_finish_kernel<<<dim3((unsigned)(t.nM * (t.tm / 16))), dim3(256), 0, s>>>(a.part32, t, small ? small->ksplit : a.ksplit, s_mha, c_ffn, s_ffn, a.M);
    return hipGetLastError();
}

}  // namespace spts
