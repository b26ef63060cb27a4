// bf16 matrix-core GEMM for products that leave the 256x256 tiles of kernels_gemm_mfma.hip short of work: few rows (a short
// prompt, the probe queries, one request's active rows) or few columns (K projection, proxy factors).
//
//  * TM x 128 output tile (TM = 64, 128 or 192), 4 wavefronts (2x2) of TM/2 x 64 = (TM/32) x 4 MFMA 16x16x32 blocks.  32 / 64 / 96
//    accumulators per lane and a ring of 48 / 64 / 80 KB let two or three workgroups share a CU, which hides one's barriers,
//    fragment reads and epilogue behind the other's MFMAs; per flop it moves twice the operand bytes of the 256x256 tile, so it
//    pays only where that one leaves CUs idle or multiplies padding (the rule: gemm_small_pick).
//  * K in slabs of 32, travelling global memory -> LDS directly into a ring of 4 stages.  A slab's fragments are read between the matrix
//    instructions of the slab before (with a workgroup or two per CU nothing else hides the reads), so its stage is free again before
//    it is multiplied and 3 slabs (36 / 48 / 60 KB per workgroup) stay in flight, which is what keeps HBM busy when the product is
//    bound by reading its weights once.  Against reading the fragments right before they are used: products at the plan that is best
//    for them 0-14 % faster (800 rows of O 47.1 -> 40.7 us, 333 of down 58.6 -> 52.9, 133 of gate/up 65.0 -> 60.2, K projection of 1638 rows
//    30.5 -> 26.7).  Rings of 8 to 12 stages where a CU has one workgroup anyway: no faster, and the longer code costs short
//    products 1-2 us (16 slabs: 8.4 -> 10.3).
//    Slab-major operands as in kernels_gemm_mfma.hip (whole lines per load instruction), same swizzle, same LDS image.
//  * Split-K: `ksplit` workgroups share a tile, each leaves its raw fp32 accumulators (fragment order: every store is 1 KB),
//    small_finish_kernel sums them in split order and applies the epilogue.
//  * 32-wide column blocks of a wavefront: wavefront column wn, block j covers tile columns j * 64 + wn * 32 (or wn * 64 + j * 32 for
//    rotary heads of 64), so that block 0 and block 1 are the two members of a rotary pair, or gate and up of a channel: the
//    dual epilogues combine registers of one lane, also in the finish kernel.  The epilogue is chosen at run time; its finished
//    quads pass through 32 bytes of scratch memory per lane, once per product.
//
// Measured (us from launch to launch, weights from HBM, 256-wide tiles with their split -> here; slab-major weights, then row-major):
// 64 rows x 4096 x 4096 26.7 -> 17.0 and 30.0 -> 19.4 (4 shares of K), 133 rows of gate/up 67.2 -> 58.3 and 93.0 -> 79.9, of down
// 46.2 -> 38.1 and 60.4 -> 46.1 (the weights' HBM time: 39 and 20), proxy z of 512 rows 37.2 -> 16.8 and 39.6 -> 17.0.
#include "spts_internal.h"

namespace spts {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float f32x4 __attribute__((ext_vector_type(4)));

constexpr int SBN = 128;        // tile columns (weight rows)
constexpr int SBK = 32;         // K slab
constexpr int SROW = SBK * 2;   // bytes of a tile row in a slab
template <int TM> constexpr int small_stage_bytes() { return (TM + SBN) * SROW; }
constexpr int64_t ONCE_BYTES = 4 << 20;   // weights of a product from which on one row tile loads them as data that is read once
// ring stages: 48 / 64 / 80 KB (even, since the two fragment sets alternate)
constexpr int SMALL_STAGES = 4;

__device__ inline int small_off(int row, int c) { return row * SROW + ((c ^ ((row >> 2) & 3)) << 4); }
__device__ inline float small_silu(float g) { return g * __builtin_amdgcn_rcpf(1.0f + __builtin_amdgcn_exp2f(-1.4426950408889634f * g)); }

// what the epilogue of one 4-column quad (or pair of quads) needs to know about its tile
struct SmallTile { int col0; bool second; bool rope; int jstride, wstride; };

__device__ __forceinline__ SmallTile small_tile(const GemmArgs& a, int tn) {
    SmallTile t;
    t.col0 = tn * (a.epi == EPI_SILU_MUL ? SBN / 2 : SBN);
    t.second = a.epi == EPI_ROPE_STORE && t.col0 >= a.n_split;
    t.rope = a.epi == EPI_ROPE || (a.epi == EPI_ROPE_STORE && !t.second);
    const bool d64 = t.rope && a.head_dim == 64;
    t.jstride = d64 ? 32 : 64;
    t.wstride = d64 ? 64 : 32;
    return t;
}

// id -> (row tile, column tile): up to GM row tiles of a column tile are neighbours (they read the same weight panel), column
// tiles follow each other inside the group
__device__ __forceinline__ void small_tile_of(int id, int nM, int nN, int& tm, int& tn) {
    constexpr int GM = 8;
    const int group = id / (GM * nN), first = group * GM;
    const int gsz = nM - first < GM ? nM - first : GM;
    const int in_g = id - group * GM * nN;
    tm = first + in_g % gsz;
    tn = in_g / gsz;
}

// the two finished quads (block j = 0, 1; columns cq .. cq + 3 of the block) of output row grow -> bf16 pairs; returns how many quads
// there are (dual epilogues: SiLU leaves one)
__device__ __forceinline__ void small_epilogue(const GemmArgs& a, const SmallTile& t, int wn, int cq, int64_t growc, int64_t crow,
                                               f32x4 v0, f32x4 v1, u32x2& o0, u32x2& o1) {
    if (a.epi == EPI_SILU_MUL) {
        float h[4];
#pragma unroll
        for (int e = 0; e < 4; ++e) h[e] = small_silu(v0[e]) * v1[e];
        o0 = u32x2{cvt_pk_bf16(h[0], h[1]), cvt_pk_bf16(h[2], h[3])};
        return;
    }
    if (t.rope) {
        const int64_t trow = a.rope_idx ? (int64_t)a.rope_idx[growc] : growc;
        const int jj = (a.head_dim == 128 ? wn * 32 : 0) + cq;
        const float2* tab = a.rope + trow * (a.head_dim >> 1) + jj;
        const float rs = a.rope_scale != 0.f ? a.rope_scale : 1.f;
        float lo[4], hi[4];
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            const float2 cs = tab[e];
            lo[e] = (v0[e] * cs.x - v1[e] * cs.y) * rs;
            hi[e] = (v1[e] * cs.x + v0[e] * cs.y) * rs;
        }
        o0 = u32x2{cvt_pk_bf16(lo[0], lo[1]), cvt_pk_bf16(lo[2], lo[3])};
        o1 = u32x2{cvt_pk_bf16(hi[0], hi[1]), cvt_pk_bf16(hi[2], hi[3])};
        return;
    }
    if (a.epi == EPI_RESIDUAL) {   // one rounding of old + sum
        const bf16_t* c = (const bf16_t*)a.C + crow * a.ldc + t.col0 + wn * t.wstride + cq;
        const u32x2 p0 = *reinterpret_cast<const u32x2*>(c), p1 = *reinterpret_cast<const u32x2*>(c + t.jstride);
        v0 += f32x4{__uint_as_float(p0[0] << 16), __uint_as_float(p0[0] & 0xffff0000u), __uint_as_float(p0[1] << 16), __uint_as_float(p0[1] & 0xffff0000u)};
        v1 += f32x4{__uint_as_float(p1[0] << 16), __uint_as_float(p1[0] & 0xffff0000u), __uint_as_float(p1[1] << 16), __uint_as_float(p1[1] & 0xffff0000u)};
    }
    o0 = u32x2{cvt_pk_bf16(v0[0], v0[1]), cvt_pk_bf16(v0[2], v0[3])};
    o1 = u32x2{cvt_pk_bf16(v1[0], v1[1]), cvt_pk_bf16(v1[2], v1[3])};
}

// transposed copy of a stored quad (values of the attention): Ct[col + e, vt_key_slot(row)]
__device__ __forceinline__ void small_store_ct(const GemmArgs& a, int col, int64_t grow, u32x2 o) {
    bf16_t* ct = (bf16_t*)a.Ct;
    const uint16_t e[4] = {(uint16_t)(o[0] & 0xffff), (uint16_t)(o[0] >> 16), (uint16_t)(o[1] & 0xffff), (uint16_t)(o[1] >> 16)};
#pragma unroll
    for (int t = 0; t < 4; ++t) ct[(int64_t)(col + t) * a.ldct + vt_key_slot(grow)].v = e[t];
}

// workgroup `block` of a product.  PAIRS (row-major A): two slabs of A travel together, so that a load takes whole 128-byte lines of 8 rows and not
// halves of 16, which come twice.  The same LDS: two slots of a pair each, then the four stages of B.
template <int TM, bool PAIRS>
__device__ __forceinline__ void small_product(const GemmArgs& a, int nM, int nN, int ksplit, int block) {
    constexpr int MI = TM / 64;                 // 32-row blocks per wavefront
    constexpr int NST = SMALL_STAGES, STAGE = small_stage_bytes<TM>(), A_BYTES = TM * SROW;
    constexpr int LA = TM / 64, LB = 2, PER = LA + LB;   // direct-to-LDS loads per wavefront and slab: 16 rows each (row-major A: 2 LA of 8 rows per two slabs)
    constexpr int PAIR = TM * 2 * SROW, B_RING = 2 * PAIR, LQ = PAIRS ? 2 * LA : LA;
    extern __shared__ __attribute__((aligned(16))) char smem[];

    // XCD b % 8 takes a contiguous range of the units (split outermost): neighbouring units share operand panels in its L2
    const int tiles = nM * nN, units = tiles * ksplit;
    const int per_xcd = (units + 7) / 8;
    const int unit = block % 8 * per_xcd + block / 8;
    if (block / 8 >= per_xcd || unit >= units) return;
    const int split = unit / tiles, id = unit - split * tiles;
    int tm, tn;
    small_tile_of(id, nM, nN, tm, tn);
    const SmallTile st = small_tile(a, tn);

    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int wm = wave >> 1, wn = wave & 1, l16 = lane & 15, lq = lane >> 4;
    const int64_t row0 = (int64_t)tm * TM;

    // ---- load addresses: a wavefront-uniform base advanced along K plus a fixed 32-bit lane offset
    const bool second = st.second;
    const int64_t a_pitch = a.a_slab ? 64 : a.lda * 2, b_pitch = a.b_slab ? 64 : a.ldb * 2;
    const int64_t a_kstep = a.a_slab ? a.M * 64 : SROW, b_kstep = a.b_slab ? (second ? a.b_rows1 : a.b_rows) * 64 : SROW;
    const int lr = lane >> 2;                   // row of the load's 16
    uint32_t oa[LQ], ob[LB];
    const char* abase = (const char*)a.A + (a.a_idx ? (int64_t)0 : row0 * a_pitch);
    // This wavefront's 32 weight rows: which matrix, and from which row of it (one address for all epilogues, by selects)
    const int rw = wave * 32;
    const bool silu_b = a.epi == EPI_SILU_MUL;
    const bool upper = a.epi == EPI_STORE && a.B1 != nullptr && st.col0 >= a.N / 2;   // stacked B: columns [N/2, N) from B1
    const bool from_b1 = silu_b ? rw >= 64 : (second || upper);
    const int brow0 = (silu_b ? (rw & 63) : rw) + st.col0 - (second ? a.n_split : 0) - (upper ? a.N / 2 : 0);
    const char* bbase = (const char*)(from_b1 ? a.B1 : a.B0) + (int64_t)brow0 * b_pitch;
#pragma unroll
    for (int q = 0; q < LQ; ++q) {
        const int r = PAIRS ? wave * (TM / 4) + q * 8 + (lane >> 3) : wave * (TM / 4) + q * 16 + lr;
        int64_t grow = row0 + r;
        if (grow >= a.M) grow = a.M - 1;        // duplicates of the last row are never stored
        const int64_t srow = a.a_idx ? (int64_t)a.a_idx[grow] : grow - row0;
        oa[q] = (uint32_t)(srow * a_pitch + (PAIRS ? ((lane & 7) ^ (lane >> 3)) << 4 : ((lane & 3) ^ ((r >> 2) & 3)) << 4));
    }
    const uint32_t second_half = ((lane & 7) ^ (lane >> 3)) >= 4 ? SROW : 0;   // this lane's piece of a pair of slabs lies in the second one
#pragma unroll
    for (int q = 0; q < LB; ++q) {
        const int r = wave * 32 + q * 16 + lr;
        ob[q] = (uint32_t)((int64_t)(q * 16 + lr) * b_pitch + (((lane & 3) ^ ((r >> 2) & 3)) << 4));
    }
    const uint32_t lds0 = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) char*)smem;
    const uint32_t lds_a = lds0 + wave * (TM / 4) * (PAIRS ? 2 * SROW : SROW), lds_b = lds0 + (PAIRS ? B_RING : A_BYTES) + wave * 32 * SROW;
    const int nk_all = a.K / SBK;
    const int nk = nk_all / ksplit + (split < nk_all % ksplit ? 1 : 0);
    const int kbeg = split * (nk_all / ksplit) + (split < nk_all % ksplit ? split : nk_all % ksplit);
    // With one row tile no other workgroup reads these weights: they are loaded as such and leave the caches to the rows, which all do
    // (133 rows, in a layer: gate/up 67.5 -> 64.6 us, down 34 -> 29, O 14.6 -> 14; 333 rows, all products 338 -> 314).  Not products
    // below ONCE_BYTES, whose weights the caches keep from call to call at no cost to the rest (us a layer
    // of 130 rows, with these loads / without / from ONCE_BYTES on: hidden size 512, 16 layers 139.0 / 136.0 / 136.2; 1024, 24 layers
    // 152.0 / 156.4 / 151.2, 4 layers 151.0 / 144.7 / 148.3; 2048, 8 layers 171.9 / 178.2 / 172.1, 1 layer 172.1 / 164.8 / 171.5).
    const bool once = nM == 1 && (int64_t)a.N * a.K * (a.epi == EPI_SILU_MUL ? 4 : 2) >= ONCE_BYTES;
    auto issue_b = [&](int kt, uint32_t at) {
        const int64_t ks = kbeg + kt;
#pragma unroll
        for (int q = 0; q < LB; ++q) {
            if (once) dma16s_nt(ob[q], bbase + ks * b_kstep, lds_b + at + q * 1024);
            else dma16s(ob[q], bbase + ks * b_kstep, lds_b + at + q * 1024);
        }
    };
    auto issue = [&](int kt, int stage) {
        const int64_t ks = kbeg + kt;
        issue_b(kt, stage * STAGE);
#pragma unroll
        for (int q = 0; q < LA; ++q) dma16s(oa[q], abase + ks * a_kstep, lds_a + stage * STAGE + q * 1024);
    };

    f32x4 acc[MI][2][4];   // 32x32 block (i, j): quarter q = rows 16 * (q / 2), columns 16 * (q % 2)
#pragma unroll
    for (int i = 0; i < MI; ++i)
#pragma unroll
        for (int j = 0; j < 2; ++j)
#pragma unroll
            for (int q = 0; q < 4; ++q) acc[i][j][q] = f32x4{0.f, 0.f, 0.f, 0.f};

    bf16x8 fa[2][2 * MI], fb[2][4];
    auto multiply = [&](int buf) {
#pragma unroll
        for (int i = 0; i < 2 * MI; ++i)
#pragma unroll
            for (int j = 0; j < 4; ++j)
                acc[i >> 1][j >> 1][(i & 1) * 2 + (j & 1)] =
                    __builtin_amdgcn_mfma_f32_16x16x32_bf16(fb[buf][j], fa[buf][i], acc[i >> 1][j >> 1][(i & 1) * 2 + (j & 1)], 0, 0, 0);
    };
    // fragment reads between the matrix instructions
    auto interleave = [&]() {
#pragma unroll
        for (int g = 0; g < 4 + 2 * MI; ++g) {
            __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
            __builtin_amdgcn_sched_group_barrier(0x100, 1, 0);
        }
        __builtin_amdgcn_sched_barrier(0);
    };
    if constexpr (PAIRS) {
        const int npairs = (nk + 1) >> 1;
        auto issue_a = [&](int p, uint32_t at) {
            const uint32_t back = 2 * p + 1 < nk ? 0 : second_half;   // a pair whose second slab is not there: the first one twice
#pragma unroll
            for (int q = 0; q < LQ; ++q) dma16s(oa[q] - back, abase + (int64_t)(kbeg + 2 * p) * SROW, lds_a + at + q * 1024);
        };
        // slot / stage of the next pair and slab to load and of the slab whose fragments are next, in bytes
        uint32_t a_in = 0, b_in = 0, a_out = 0, b_out = 0;
        auto next_b = [](uint32_t& at) { at = (at + SBN * SROW) & (SMALL_STAGES * SBN * SROW - 1); };
        for (int t = 0; t < NST && t < nk + 1; ++t) {   // pair p is loaded before B's slab 2 p + 1 (t = nk: the pair of an odd last slab)
            if ((t & 1) && t / 2 < npairs) issue_a(t / 2, t / 2 * PAIR);
            if (t < nk) issue_b(t, t * SBN * SROW);
        }
        int pair = 2;   // the next pair to load: its slot is free after its predecessor's second slab
        const uint32_t fa0 = (wm * (TM / 2) + l16) * 2 * SROW + ((lq ^ (l16 & 7)) << 4);
        const uint32_t fb0 = B_RING + (uint32_t)small_off(wn * st.wstride + l16, lq);
        const uint32_t fbj = st.jstride * SROW;
        auto fragments = [&](int buf, int odd) {   // of slab `odd` of the pair at a_out, and of b_out
            const char* sb = smem + fb0 + b_out;
            const char* sa = smem + a_out + (odd ? fa0 ^ 64u : fa0);
#pragma unroll
            for (int j = 0; j < 4; ++j) fb[buf][j] = *reinterpret_cast<const bf16x8*>(sb + (j >> 1) * fbj + (j & 1) * 16 * SROW);
#pragma unroll
            for (int i = 0; i < 2 * MI; ++i) fa[buf][i] = *reinterpret_cast<const bf16x8*>(sa + i * 16 * 2 * SROW);
            next_b(b_out);
            if (odd) a_out ^= PAIR;
        };
        if (nk >= NST) { SPTS_WAIT_VMCNT(3 * LB + LQ); } else { SPTS_WAIT_VMCNT(0); }
        __syncthreads();
        fragments(0, 0);
        // Slab kt from one fragment set while the other takes kt + 1.  Loads that may be outstanding before that, as they were issued after those of kt + 1: B of
        // kt + 2 and kt + 3 and, with kt even, the pair of kt + 2.
        int kt = 0;
        auto step = [&](int odd, bool end) {
            if (!end && !odd) { SPTS_WAIT_VMCNT(2 * LB + LQ); }
            else if (!end || kt + 3 < nk) { SPTS_WAIT_VMCNT(2 * LB); }
            else if (kt + 2 < nk) { SPTS_WAIT_VMCNT(LB); }
            else { SPTS_WAIT_VMCNT(0); }
            __syncthreads();
            if (odd && pair < npairs) { issue_a(pair++, a_in); a_in ^= PAIR; }
            if (kt + NST < nk) { issue_b(kt + NST, b_in); next_b(b_in); }
            fragments(odd ^ 1, odd ^ 1);
            multiply(odd);
            interleave();
            ++kt;
        };
        while (kt + 4 < nk) {   // in here every load that the counts allow for has been issued
            step(0, false);
            step(1, false);
        }
        while (kt + 1 < nk) {
            step(0, true);
            if (kt + 1 < nk) step(1, true);
        }
        if (nk & 1) multiply(0);
        else multiply(1);
    } else {
    // All stages in flight; a slab's fragments are read while the slab before is multiplied, so its stage is free again when its
    // multiplication begins.
    const int npre = nk < NST ? nk : NST;
    for (int t = 0; t < npre; ++t) issue(t, t);
    auto fragments = [&](int buf, int stage) {
        const char* sa = smem + stage * STAGE;
        const char* sb = sa + A_BYTES;
#pragma unroll
        for (int j = 0; j < 4; ++j)
            fb[buf][j] = *reinterpret_cast<const bf16x8*>(sb + small_off((j >> 1) * st.jstride + wn * st.wstride + (j & 1) * 16 + l16, lq));
#pragma unroll
        for (int i = 0; i < 2 * MI; ++i) fa[buf][i] = *reinterpret_cast<const bf16x8*>(sa + small_off(wm * (TM / 2) + i * 16 + l16, lq));
    };
    if (npre == NST) { SPTS_WAIT_VMCNT((NST - 1) * PER); } else { SPTS_WAIT_VMCNT(0); }
    __syncthreads();
    fragments(0, 0);
    // Slab kt from one fragment set while the other takes slab kt + 1: this wavefront's loads of that have landed when only the `left`
    // slabs' behind it are outstanding; the barrier publishes everyone's and says that slab kt's stage has been read.
    int kt = 0;
    for (; kt + 2 * NST - 1 < nk; kt += NST) {   // ring stages are constants here
#pragma unroll
        for (int u = 0; u < NST; ++u) {
            SPTS_WAIT_VMCNT((NST - 2) * PER);
            __syncthreads();
            issue(kt + u + NST, u);
            fragments(~u & 1, (u + 1) % NST);
            multiply(u & 1);
            interleave();
        }
    }
    for (; kt + 1 < nk; ++kt) {
        const int left = nk - 2 - kt;
        if (left >= NST - 2) { SPTS_WAIT_VMCNT((NST - 2) * PER); }
        else if (left == 1) { SPTS_WAIT_VMCNT(PER); }
        else { SPTS_WAIT_VMCNT(0); }
        __syncthreads();
        if (kt + NST < nk) issue(kt + NST, kt % NST);
        fragments(1, (kt + 1) % NST);
        multiply(0);
        interleave();
#pragma unroll
        for (int i = 0; i < 2 * MI; ++i) fa[0][i] = fa[1][i];
#pragma unroll
        for (int j = 0; j < 4; ++j) fb[0][j] = fb[1][j];
    }
    multiply(0);
    }

    // ---- lane: output row l16 of its quarter block, columns 4 * lq + e
    if (ksplit > 1) {
        float* P = a.part32 + ((int64_t)split * tiles + id) * (TM * SBN);
#pragma unroll
        for (int i = 0; i < MI; ++i)
#pragma unroll
            for (int j = 0; j < 2; ++j)
#pragma unroll
                for (int q = 0; q < 4; ++q) *reinterpret_cast<f32x4*>(P + ((((wave * MI + i) * 2 + j) * 4 + q) * 64 + lane) * 4) = acc[i][j][q];
        return;
    }
    // staged through LDS (the ring is free once every wavefront is past its last fragment read) so that the tile leaves in
    // whole rows; 16-byte chunk c of row r at c ^ (r % chunks)
    __syncthreads();
    const bool silu = silu_b;
    const int nch = silu ? 8 : 16;               // chunks per staged row
#pragma unroll
    for (int i = 0; i < 2 * MI; ++i) {
        const int tr = wm * (TM / 2) + i * 16 + l16;
        const int64_t grow = row0 + tr;
        const int64_t growc = grow < a.M ? grow : a.M - 1;
        const int64_t crow = a.c_idx ? (int64_t)a.c_idx[growc] : growc;
#pragma unroll
        for (int h = 0; h < 2; ++h) {
            const int q = (i & 1) * 2 + h, cq = h * 16 + 4 * lq;
            u32x2 o[2];
            small_epilogue(a, st, wn, cq, growc, crow, acc[i >> 1][0][q], acc[i >> 1][1][q], o[0], o[1]);
#pragma unroll
            for (int j = 0; j < 2; ++j) {
                if (silu && j == 1) continue;
                const int tc = j * st.jstride + wn * st.wstride + cq;
                *reinterpret_cast<u32x2*>(smem + tr * (nch * 16) + ((((tc >> 3) ^ tr) & (nch - 1)) << 4) + ((tc & 4) << 1)) = o[j];
                if (a.Ct && !st.rope && grow < a.ldct) small_store_ct(a, st.col0 - (second ? a.n_split : 0) + tc, grow, o[j]);
            }
        }
    }
    __syncthreads();
    bf16_t* Cb = (bf16_t*)(second ? a.C2 : a.C);
    const int colb = st.col0 - (second ? a.n_split : 0);
    const int64_t ldo = second ? a.ldc2 : a.ldc;
    const int total = TM * nch;
    for (int e = tid; e < total; e += 256) {
        int tr, oc;
        if (a.c_slab) { oc = (e & 3) + 4 * (e / (TM * 4)); tr = (e >> 2) % TM; }   // slab by slab: 4 lanes per row, rows adjacent
        else { tr = e / nch; oc = e % nch; }
        const int64_t grow = row0 + tr;
        if (grow >= a.M) continue;
        const u32x4 v = *reinterpret_cast<const u32x4*>(smem + tr * (nch * 16) + (((oc ^ tr) & (nch - 1)) << 4));
        if (a.c_slab) {
            *reinterpret_cast<u32x4*>(Cb + (((int64_t)(colb >> 5) + (oc >> 2)) * a.M + grow) * 32 + (oc & 3) * 8) = v;
        } else {
            const int64_t crow = a.c_idx ? (int64_t)a.c_idx[grow] : grow;
            *reinterpret_cast<u32x4*>(Cb + crow * ldo + colb + oc * 8) = v;
        }
    }
}

// Pairs are for products that move more than they wait: shares of at least 96 slabs, tiles of 64 or 192 rows.  Gate/up of 64 / 133 / 333 / 700 rows
// of the 8B shape (128 slabs, slab-major weights) 44.4 -> 41.5, 60.2 -> 54.8, 108.9 -> 90.9, 190.2 -> 171.1 us.  14336 columns, weights from HBM, 64 / 180 / 550 rows: 96 slabs
// 33.4 -> 31.6, 57.0 -> 46.0, 123.8 -> 109.8; 104 36.1 -> 33.9, 61.9 -> 49.3, 136 -> 118; 112 39.1 -> 36.3, 67.3 -> 52.6, 146 -> 125 (Qwen layer of 384 rows 327 -> 295).  With all of
// a layer's weights in the memory-side cache 96 slabs can lose: 3072 wide, 8192 columns, 333 rows 43.6 -> 46.9.  A shorter share's first loads and last slabs
// cost what the lines save (4096 x 4096, 133 rows, 32 slabs 20.0 -> 21.3; 700 rows, 64 slabs 39.8 -> 40.8), and so it is with tiles of 128
// rows, where a slot has two iterations for its loads but half the work (gate/up of 133 rows 65.7 -> 69.6, 700 of 4096 x 4096 40.4 -> 44.2).
template <int TM> __host__ __device__ constexpr bool small_pairs(const GemmArgs& a, int ksplit) {
    return TM != 128 && !a.a_slab && a.K / SBK / ksplit >= 96;
}

template <int TM, bool PAIRS>
__global__ void __launch_bounds__(256, TM == 64 ? 3 : 2) gemm_small_kernel(GemmArgs a, int nM, int nN, int ksplit) {
    small_product<TM, PAIRS>(a, nM, nN, ksplit, blockIdx.x);
}

// Independent products of one tile height in one launch: product i has the blocks from first[i] on (multiples of 8: a block's XCD stays what
// it is in a launch of its own), and those from finish[i] on of the second pass.
struct SmallGroup { GemmArgs a[GEMM_GROUP_MAX]; int nM[GEMM_GROUP_MAX], nN[GEMM_GROUP_MAX], ksplit[GEMM_GROUP_MAX], first[GEMM_GROUP_MAX], finish[GEMM_GROUP_MAX]; };

template <int TM>
__global__ void __launch_bounds__(256, TM == 64 ? 3 : 2) gemm_small_group_kernel(SmallGroup g) {
    int i = 0;
#pragma unroll
    for (int q = 1; q < GEMM_GROUP_MAX; ++q) i += (int)blockIdx.x >= g.first[q] ? 1 : 0;
    if constexpr (TM != 128) {
        if (small_pairs<TM>(g.a[i], g.ksplit[i])) {
            small_product<TM, true>(g.a[i], g.nM[i], g.nN[i], g.ksplit[i], blockIdx.x - g.first[i]);
            return;
        }
    }
    small_product<TM, false>(g.a[i], g.nM[i], g.nN[i], g.ksplit[i], blockIdx.x - g.first[i]);
}

// Second pass of a split product: one thread per fragment quad pair (j = 0, 1), splits summed in order.
template <int TM>
__device__ __forceinline__ void small_finish(const GemmArgs& a, int nM, int nN, int ksplit, int block) {
    constexpr int MI = TM / 64, QPT = TM * SBN / 8;      // quad pairs per tile
    const int64_t g = (int64_t)block * 256 + threadIdx.x;
    const int id = (int)(g / QPT), v = (int)(g % QPT);
    const int lane = v & 63, q = (v >> 6) & 3, wi = v >> 8;
    const int wave = wi / MI, i = wi % MI;
    const int wm = wave >> 1, wn = wave & 1, l16 = lane & 15, lq = lane >> 4;
    const int tiles = nM * nN;
    int tm, tn;
    small_tile_of(id, nM, nN, tm, tn);
    const SmallTile st = small_tile(a, tn);
    const int64_t grow = (int64_t)tm * TM + wm * (TM / 2) + i * 32 + (q >> 1) * 16 + l16;
    const int cq = (q & 1) * 16 + 4 * lq;
    const bool rok = grow < a.M;
    if (!rok && !(a.Ct && !st.rope && grow < a.ldct)) return;
    const float* P = a.part32 + (int64_t)id * (TM * SBN) + (((wave * MI + i) * 2 * 4 + q) * 64 + lane) * 4;
    f32x4 s0 = {0.f, 0.f, 0.f, 0.f}, s1 = s0;
#pragma unroll 4
    for (int sp = 0; sp < ksplit; ++sp) {
        const float* p = P + (int64_t)sp * tiles * (TM * SBN);
        s0 += *reinterpret_cast<const f32x4*>(p);
        s1 += *reinterpret_cast<const f32x4*>(p + 4 * 64 * 4);
    }
    const int64_t growc = rok ? grow : a.M - 1;
    const int64_t crow = a.c_idx ? (int64_t)a.c_idx[growc] : growc;
    u32x2 o[2];
    small_epilogue(a, st, wn, cq, growc, crow, s0, s1, o[0], o[1]);
    bf16_t* Cb = (bf16_t*)(st.second ? a.C2 : a.C);
    const int64_t ldo = st.second ? a.ldc2 : a.ldc;
#pragma unroll
    for (int j = 0; j < 2; ++j) {
        if (a.epi == EPI_SILU_MUL && j == 1) continue;
        const int col = st.col0 - (st.second ? a.n_split : 0) + j * st.jstride + wn * st.wstride + cq;
        if (rok) {
            if (a.c_slab) *reinterpret_cast<u32x2*>(Cb + ((int64_t)(col >> 5) * a.M + grow) * 32 + (col & 31)) = o[j];
            else *reinterpret_cast<u32x2*>(Cb + crow * ldo + col) = o[j];
        }
        if (a.Ct && !st.rope && grow < a.ldct) small_store_ct(a, col, grow, o[j]);
    }
}

template <int TM>
__global__ void __launch_bounds__(256) small_finish_kernel(GemmArgs a, int nM, int nN, int ksplit) { small_finish<TM>(a, nM, nN, ksplit, blockIdx.x); }

template <int TM>
__global__ void __launch_bounds__(256) small_finish_group_kernel(SmallGroup g) {
    int i = 0;
#pragma unroll
    for (int q = 1; q < GEMM_GROUP_MAX; ++q) i += (int)blockIdx.x >= g.finish[q] ? 1 : 0;
    small_finish<TM>(g.a[i], g.nM[i], g.nN[i], g.ksplit[i], blockIdx.x - g.finish[i]);
}

bool gemm_small_supported(const GemmArgs& a) {
    if (a.epi != EPI_STORE && a.epi != EPI_SILU_MUL && a.epi != EPI_RESIDUAL && a.epi != EPI_ROPE && a.epi != EPI_ROPE_STORE) return false;
    if (a.A1 || a.ksplit > 1) return false;
    // everything the 256-wide kernel checks (alignment, 32-bit offsets, slab rows), which is for multiples of 256 (128) columns
    return gemm_mfma_supported(a);
}

// Time models (us) behind the choice between the two kernels and among this one's tiles and splits, fitted to 170 measured
// (product, rows) pairs x 24 (tile, split) pairs: rows 1 .. 16000 of the 8B shape's projections, FFN and proxy products, with kernels
// that read their fragments later and row-major operands in half lines.  The constants were not fitted again since; what counts is the
// choice, and that was measured with the present kernels (long shares of row-major rows in pairs of slabs), weights from HBM, 7 products x 18 row counts: against the
// best of everything tried it costs 0.5 % on the mean and 21 % at most (down of 100 rows, 8 shares for 6: 40.9 us, 33.9) with slab-major weights, 0.4 %
// and 11 % (proxy z of 800 rows) with row-major ones.
//  * this kernel: a K slab takes the load latency (0.18 / 0.31 / 0.38 us at TM = 64 / 128 / 192) or, with more workgroups, the
//    47 KB/us that a CU's slab loads reach together (rows past M repeat a line and cost a third); a split adds the finish launch
//    and its fp32 tiles written and read at 4 TB/s.
//  * 256-wide tiles: 0.41 us per slab + up to 0.36 us as the chip fills, a round of 256 tiles after the other, a partly filled
//    last round split over K as gemm_pick_split plans.
//  * The fitted products have K >= 4096, so the times per slab carry the epilogues.  Products of fewer than EPI_SLABS slabs (K < 2048) do
//    not, and get the rest: a start, and the epilogue per 128 rows of every workgroup that a CU runs, or per round of 256-wide
//    tiles.  Without it short products with many tiles came here too often: of 1095 measured with K < 2048, 66 took more than 2 % longer
//    than on the 256-wide tiles (up to 50 %; proxy z of 20011 rows on 512 channels 16.6 -> 18.4 us), with it none (0.73 of the
//    256-wide time on the mean, 0.74 without).
constexpr double EPI_SLABS = 64.0;
struct EpilogueTimes { double store, rope, resid, silu; };
static double short_share(const GemmArgs& a) { return a.K / SBK < EPI_SLABS ? 1.0 - a.K / SBK / EPI_SLABS : 0.0; }
static double epilogue_time(const EpilogueTimes& e, int epi) {
    return epi == EPI_SILU_MUL ? e.silu : epi == EPI_RESIDUAL ? e.resid : epi == EPI_STORE ? e.store : e.rope;
}
static double small_time(const GemmArgs& a, int tm, int ks) {
    const double lat = tm == 64 ? 0.18 : tm == 128 ? 0.31 : 0.38;
    const int64_t nM = (a.M + tm - 1) / tm, nN = a.N / (a.epi == EPI_SILU_MUL ? SBN / 2 : SBN), units = nM * nN * ks;
    const double fill = (double)units / 256.0, per_cu = fill <= 1.0 ? 1.0 : 0.5 * (fill + (double)((units + 255) / 256));
    const double rows = tm * (0.35 + 0.65 * (double)a.M / (double)(nM * tm));
    const double slab_kb = (rows + SBN) * SROW / 1024.0;
    const double per_slab = lat > per_cu * slab_kb / 47.0 ? lat : per_cu * slab_kb / 47.0;
    const double t = 2.6 + per_slab * (double)((a.K / SBK + ks - 1) / ks);
    if (ks > 1) return t + 2.5 + (double)units * tm * SBN * 8.0 / 4.0e6;
    return t + short_share(a) * (2.5 + per_cu * tm / 128.0 * epilogue_time(EpilogueTimes{5.0, 7.5, 5.5, 3.0}, a.epi));
}
static double wide_time(const GemmArgs& a, int ks, int nfull) {
    const int64_t tiles = (a.M + 255) / 256 * (a.N / (a.epi == EPI_SILU_MUL ? 128 : 256));
    const double slabs = a.K / SBK;
    auto per_slab = [](double busy) { return 0.41 + 0.36 * busy / 256.0; };
    const int64_t whole = ks > 1 ? nfull : tiles;
    const double epi = short_share(a) * epilogue_time(EpilogueTimes{9.0, 20.0, 15.0, 6.0}, a.epi);
    double t = 4.6 + (double)(whole / 256) * (slabs * per_slab(256) + epi);
    if (const int64_t rem = whole % 256) t += slabs * per_slab(whole > 256 && rem < 160 ? 160 : (double)rem) + epi * (0.3 + 0.7 * (double)rem / 256.0);
    if (ks > 1) {
        const int64_t units = (tiles - nfull) * ks;
        t += (double)((units + 255) / 256) * (double)((int)(slabs + ks - 1) / ks) * per_slab(units < 256 ? (double)units : 256.0) + 5.1 +
             (double)units * 262144.0 * 2.0 / 4.0e6;
    }
    return t;
}

bool gemm_small_pick(const GemmArgs& a, int wide_ksplit, int wide_nfull, size_t part_bytes, GemmSmallPlan* plan) {
    if (!gemm_small_supported(a)) return false;
    // 7 % in hand: where the two are that close the wider tile moves fewer bytes
    double best = 0.93 * wide_time(a, wide_ksplit, wide_nfull);
    bool found = false;
    for (const int tm : {64, 128, 192})
        for (const int ks : {1, 2, 3, 4, 6, 8, 12, 16}) {
            const GemmSmallPlan p{tm, ks};
            // Shares of at least 1024, at the price of 1-3 us a product (64 x 4096 x 4096: 18.1 us in 4 shares, 15.5 in 8).  A
            // product with K < 1024 is then never split (gemm_pick_split's shares are 512 at least) and is summed the same way
            // whatever its row count and whichever kernel takes it: a batched call and the calls one by one have the same sums (the
            // kernels' rotary epilogues still round a few values in a million differently).  From K = 1024 on the row count decides
            // the shares.
            if (ks > 1 && (a.K / ks < 1024 || gemm_small_part_bytes(a, p) > part_bytes)) break;
            const double t = small_time(a, tm, ks);
            if (t < best) { best = t; *plan = p; found = true; }
        }
    return found;
}

size_t gemm_small_part_bytes(const GemmArgs& a, const GemmSmallPlan& p) {
    const int64_t nN = a.N / (a.epi == EPI_SILU_MUL ? SBN / 2 : SBN);
    return p.ksplit > 1 ? (size_t)((a.M + p.tm - 1) / p.tm * nN) * p.ksplit * p.tm * SBN * sizeof(float) : 0;
}

template <int TM>
static hipError_t launch_small_t(const GemmArgs& a, int ksplit, bool finish, hipStream_t s) {
    const int nM = (int)((a.M + TM - 1) / TM), nN = a.N / (a.epi == EPI_SILU_MUL ? SBN / 2 : SBN);
    const int64_t units = (int64_t)nM * nN * ksplit;
    if (units > ((int64_t)1 << 30)) return hipErrorInvalidValue;
    constexpr int lds = SMALL_STAGES * small_stage_bytes<TM>();
    static_assert(lds >= TM * SBN * 2, "the finished tile is staged in the ring");
    const dim3 grid((unsigned)((units + 7) / 8 * 8));
    hipError_t e;
    if constexpr (TM != 128) {
        if (small_pairs<TM>(a, ksplit)) {
            if ((e = ensure_dynamic_lds(reinterpret_cast<const void*>(&gemm_small_kernel<TM, true>), lds)) != hipSuccess) return e;
            gemm_small_kernel<TM, true><<<grid, dim3(256), lds, s>>>(a, nM, nN, ksplit);
        }
    }
    if (!small_pairs<TM>(a, ksplit)) {
        if ((e = ensure_dynamic_lds(reinterpret_cast<const void*>(&gemm_small_kernel<TM, false>), lds)) != hipSuccess) return e;
        gemm_small_kernel<TM, false><<<grid, dim3(256), lds, s>>>(a, nM, nN, ksplit);
    }
    if ((e = hipGetLastError()) != hipSuccess || ksplit <= 1 || !finish) return e;
    const int64_t pairs = (int64_t)nM * nN * (TM * SBN / 8);
    small_finish_kernel<TM><<<dim3((unsigned)(pairs / 256)), dim3(256), 0, s>>>(a, nM, nN, ksplit);
    return hipGetLastError();
}

static hipError_t launch_small(const GemmArgs& a, const GemmSmallPlan& p, bool finish, hipStream_t s) {
    if (p.ksplit < 1 || p.ksplit > a.K / SBK || (p.ksplit > 1 && !a.part32)) return hipErrorInvalidValue;
    return p.tm == 192 ? launch_small_t<192>(a, p.ksplit, finish, s) : p.tm == 128 ? launch_small_t<128>(a, p.ksplit, finish, s) : launch_small_t<64>(a, p.ksplit, finish, s);
}
hipError_t launch_gemm_small(const GemmArgs& a, const GemmSmallPlan& p, hipStream_t s) { return launch_small(a, p, true, s); }
hipError_t launch_gemm_small_shares(const GemmArgs& a, const GemmSmallPlan& p, hipStream_t s) { return launch_small(a, p, false, s); }

template <int TM>
static hipError_t launch_small_group_t(const GemmArgs* a, const GemmSmallPlan* p, int n, hipStream_t s) {
    SmallGroup g{};
    int64_t blocks = 0, finish = 0;
    for (int i = 0; i < GEMM_GROUP_MAX; ++i) {
        g.first[i] = g.finish[i] = 0x7fffffff;
        if (i >= n) continue;
        g.a[i] = a[i];
        g.nM[i] = (int)((a[i].M + TM - 1) / TM);
        g.nN[i] = a[i].N / (a[i].epi == EPI_SILU_MUL ? SBN / 2 : SBN);
        g.ksplit[i] = p[i].ksplit;
        g.first[i] = (int)blocks;
        blocks += ((int64_t)g.nM[i] * g.nN[i] * p[i].ksplit + 7) / 8 * 8;
        g.finish[i] = (int)finish;
        if (p[i].ksplit > 1) finish += (int64_t)g.nM[i] * g.nN[i] * (TM * SBN / 8 / 256);
        if (blocks > 1 << 30 || finish > 1 << 30) return hipErrorInvalidValue;
    }
    constexpr int lds = SMALL_STAGES * small_stage_bytes<TM>();
    hipError_t e = ensure_dynamic_lds(reinterpret_cast<const void*>(&gemm_small_group_kernel<TM>), lds);
    if (e != hipSuccess) return e;
    gemm_small_group_kernel<TM><<<dim3((unsigned)blocks), dim3(256), lds, s>>>(g);
    if ((e = hipGetLastError()) != hipSuccess || finish == 0) return e;
    small_finish_group_kernel<TM><<<dim3((unsigned)finish), dim3(256), 0, s>>>(g);
    return hipGetLastError();
}

hipError_t launch_gemm_small_group(const GemmArgs* a, const GemmSmallPlan* p, int n, hipStream_t s) {
    if (n < 1 || n > GEMM_GROUP_MAX) return hipErrorInvalidValue;
    for (int i = 0; i < n; ++i)
        if (p[i].tm != p[0].tm || p[i].ksplit < 1 || p[i].ksplit > a[i].K / SBK || (p[i].ksplit > 1 && !a[i].part32)) return hipErrorInvalidValue;
    return p[0].tm == 192 ? launch_small_group_t<192>(a, p, n, s) : p[0].tm == 128 ? launch_small_group_t<128>(a, p, n, s) : launch_small_group_t<64>(a, p, n, s);
}

}  // namespace spts
