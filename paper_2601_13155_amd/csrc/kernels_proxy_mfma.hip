// Hidden layer of the low-rank proxy FFN on the matrix cores (Eq. (proxy_ffn)):
//   h[n, c] = silu( t_g[n, :] . Vg[c, :] ) * ( t_u[n, :] . Vu[c, :] ),   t_g = x Ug, t_u = x Uu  (K = r = 256)
// for all N candidates and all Dlow channels.  As a GEMM this is the least favourable shape of the layer: K is only 256,
// so a 256 x 128 output tile has 8 slabs between its prologue and an epilogue whose SiLU arithmetic (two
// quarter-rate transcendentals per element) takes about as much vector time as the 8 slabs take matrix time, one after
// the other.  This kernel turns the loops around:
//  * A wavefront owns 32 rows and keeps their t_g / t_u fragments in registers for its whole life (B operand of
//    h^T = V t^T, 16x16x32: 2 row blocks x 8 k-steps x 2 x 4 registers = 128); a workgroup = 8 wavefronts = 256 rows.
//  * The workgroup streams its share of the channels in tiles of 32 (Vg and Vu rows, 32 KB per tile for r = 256) through a
//    4-stage direct-to-LDS ring shared by the 8 wavefronts (tiles are published in pairs: one barrier per two tiles); per
//    tile a wavefront issues 64 MFMAs (two per LDS fragment).
//  * Two accumulator sets alternate: while the matrix pipe works on tile c, the vector ALU takes SiLU(gate) * up of tile
//    c - 1, packs it to bf16 and stores it -- written as 16 steps of four MFMAs, each
//    followed by a share of one element's arithmetic, fenced for the scheduler, so the two kinds of work are offered to the SIMD
//    side by side (32768 rows x 14336 channels: 443 us with 32x32x16 and an element per two MFMAs, 438 with the element behind
//    all four, 432 dealt out).
//  * LDS row 16 * cb + 4 * q + t of a weight tile holds channel 8 * q + 4 * cb + t: the accumulators of the two channel blocks
//    cb then give a lane 8 consecutive channels of its row, and the 16-byte pieces of a wavefront's 16 rows x 64 bytes are 1 KB of
//    whole lines per store instruction.
//  * Output: h slab-major [Dlow/32][N][32], the layout the following projection GEMM reads as whole lines.
//  * Grid: (row tiles of 256) x (channel shares); the share count is chosen so that the workgroups fill whole rounds of the
//    256 CUs.  Workgroups of one XCD take neighbouring ids, i.e. mostly the same channel share: its weights stay in that L2.
// Same products in the same k order as the GEMM path and the same SiLU: results are bit-identical to it.
#include "spts_internal.h"

namespace spts {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float f32x4 __attribute__((ext_vector_type(4)));

constexpr int PH_NSTG = 4;          // ring stages (tiles of 32 channels)
constexpr int PH_WAVES = 8;

__device__ inline float ph_silu(float g) {
    return g * __builtin_amdgcn_rcpf(1.0f + __builtin_amdgcn_exp2f(-1.4426950408889634f * g));
}

template <int KS>   // k-steps of 32: r = 32 * KS
__global__ void __launch_bounds__(PH_WAVES * 64) proxy_hidden_kernel(ProxyHiddenArgs a, int RT, int SC) {
    constexpr int NSL = KS;                       // 32-wide K slabs
    constexpr int MAT_BYTES = NSL * 2048;         // one matrix's tile: [NSL][32 channels][64 bytes]
    constexpr int STAGE = 2 * MAT_BYTES;          // Vg tile + Vu tile
    constexpr int LOADS = 2 * NSL * 2;            // 1 KB loads per tile
    constexpr int LPW = LOADS / PH_WAVES;         // per wavefront
    static_assert(KS == 8, "r = 256");             // 2 * KS steps per tile, one element of the previous tile in each
    extern __shared__ __attribute__((aligned(16))) char smem[];   // the ring: PH_NSTG stages of (Vg tile, Vu tile)

    // ---- work unit: (row tile, channel share); ids of one XCD are consecutive
    const int total = RT * SC;
    const int per = (total + 7) / 8;
    const int id = (int)(blockIdx.x % 8) * per + (int)(blockIdx.x / 8);
    if (id >= total) return;
    const int sc = id / RT, rt = id % RT;
    const int TT = a.Dlow / 32;
    const int tile_begin = (int)((int64_t)sc * TT / SC), tile_end = (int)((int64_t)(sc + 1) * TT / SC);
    const int ntiles = tile_end - tile_begin;
    if (ntiles <= 0) return;

    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int l16 = lane & 15, lq = lane >> 4;
    const int64_t row0w = (int64_t)rt * 256 + wave * 32;

    // ---- direct-to-LDS loads of a weight tile: load q = (matrix X, slab s, 16-row half hf); lane -> (LDS row, chunk position)
    const uint32_t lds0 = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) char*)smem;
    uint32_t goff[2];
#pragma unroll
    for (int hf = 0; hf < 2; ++hf) {
        const int m = hf * 16 + (lane >> 2);                 // LDS row of the tile
        const int ch = ((m & 12) << 1) | ((m >> 4) << 2) | (m & 3);   // channel (inside the tile) that belongs there
        const int c = (lane & 3) ^ ((m >> 2) & 3);           // global chunk for this LDS chunk position
        goff[hf] = (uint32_t)(ch * 64 + c * 16);
    }
    const char* Wg = (const char*)a.Vg_s;
    const char* Wu = (const char*)a.Vu_s;
#define SPTS_PH_DMA(tl_)                                                                                      \
    {                                                                                                         \
        const int tile_ = tile_begin + (tl_);                                                                 \
        const uint32_t st_ = lds0 + (uint32_t)(((tl_) % PH_NSTG) * STAGE);                                    \
        _Pragma("unroll") for (int u_ = 0; u_ < LPW; ++u_) {                                                  \
            const int q_ = wave * LPW + u_;                                                                   \
            const int X_ = q_ / (2 * NSL), s_ = (q_ % (2 * NSL)) >> 1, hf_ = q_ & 1;                          \
            const char* src_ = (X_ ? Wu : Wg) + ((int64_t)s_ * a.Dlow + (int64_t)tile_ * 32) * 64;            \
            dma16s(goff[hf_], src_, st_ + (uint32_t)(X_ * MAT_BYTES + s_ * 2048 + hf_ * 1024));               \
        }                                                                                                     \
    }

    // ---- prologue: the first four tiles in flight, then this wavefront's rows of t into registers
    {
        const int npre = ntiles < PH_NSTG ? ntiles : PH_NSTG;
        for (int t = 0; t < npre; ++t) SPTS_PH_DMA(t)
    }
    bf16x8 tg[2][KS], tu[2][KS];
#pragma unroll
    for (int rb = 0; rb < 2; ++rb) {
        int64_t row = row0w + rb * 16 + l16;
        if (row >= a.N) row = a.N - 1;
        const char* pg = (const char*)a.tg + row * a.t_row_pitch + lq * 16;
        const char* pu = (const char*)a.tu + row * a.t_row_pitch + lq * 16;
#pragma unroll
        for (int ks = 0; ks < KS; ++ks) {
            tg[rb][ks] = *reinterpret_cast<const bf16x8*>(pg + ks * a.t_slab_pitch);
            tu[rb][ks] = *reinterpret_cast<const bf16x8*>(pu + ks * a.t_slab_pitch);
        }
    }
    // fragment read offset inside a slab of a matrix tile (channel block 1 is 1 KB on)
    const uint32_t foff = (uint32_t)(l16 * 64 + ((lq ^ ((l16 >> 2) & 3)) << 4));
    char* hp = (char*)a.hp;
    const int64_t out_off = (row0w + l16) * 64 + lq * 16;   // the lane's 16 bytes inside a slab of the output, row block 0
    const bool row_ok[2] = {row0w + l16 < a.N, row0w + 16 + l16 < a.N};

    const f32x4 zero4 = {0.f, 0.f, 0.f, 0.f};
    f32x4 Ga[2][2], Ua[2][2], Gb[2][2], Ub[2][2];   // [channel block][row block]
#pragma unroll
    for (int c = 0; c < 2; ++c)
#pragma unroll
        for (int r = 0; r < 2; ++r) Ga[c][r] = Ua[c][r] = Gb[c][r] = Ub[c][r] = zero4;

    // One tile: 8*KS MFMAs into (GC, UC) from the ring stage of tile tl_, interleaved with the arithmetic of the previous
    // tile's accumulators (GP, UP), whose packed result is stored at the end (one 16-byte piece per lane and row block).
    // Step i: K piece i / 2, channel block i % 2.
    constexpr int FD = 3;   // fragment reads run FD steps ahead
#define SPTS_PH_FRAG(X_, i_) (*reinterpret_cast<const bf16x8*>(sT_ + (X_) * MAT_BYTES + ((i_) >> 1) * 2048 + ((i_) & 1) * 1024 + foff))
#define SPTS_PH_MFMA(ACC_, f_, t_, rb_, i_)                                                                    \
    ACC_[(i_) & 1][rb_] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(f_[(i_) % (FD + 1)], t_[rb_][(i_) >> 1], (i_) < 2 ? zero4 : ACC_[(i_) & 1][rb_], 0, 0, 0);
#define SPTS_PH_STORE(tile_, h_)                                                                              \
    {                                                                                                         \
        _Pragma("unroll") for (int rb_ = 0; rb_ < 2; ++rb_) {                                                 \
            u32x4 x_;                                                                                         \
            _Pragma("unroll") for (int j_ = 0; j_ < 4; ++j_) x_[j_] = cvt_pk_bf16(h_[rb_ * 8 + 2 * j_], h_[rb_ * 8 + 2 * j_ + 1]); \
            if (row_ok[rb_]) *reinterpret_cast<u32x4*>(hp + (int64_t)(tile_) * a.N * 64 + out_off + rb_ * 1024) = x_; \
        }                                                                                                     \
    }
#define SPTS_PH_TILE(tl_, GC, UC, GP, UP)                                                                      \
    {                                                                                                         \
        const char* sT_ = smem + ((tl_) % PH_NSTG) * STAGE;                                                   \
        const bool prev_ = (tl_) > 0;                                                                         \
        bf16x8 fg_[FD + 1], fu_[FD + 1];                                                                      \
        _Pragma("unroll") for (int i_ = 0; i_ < FD; ++i_) { fg_[i_] = SPTS_PH_FRAG(0, i_); fu_[i_] = SPTS_PH_FRAG(1, i_); } \
        float h_[16];   /* [row block][channel of the lane's 8] */                                            \
        _Pragma("unroll") for (int i_ = 0; i_ < 2 * KS; ++i_) {                                               \
            if (i_ + FD < 2 * KS) { fg_[(i_ + FD) % (FD + 1)] = SPTS_PH_FRAG(0, i_ + FD); fu_[(i_ + FD) % (FD + 1)] = SPTS_PH_FRAG(1, i_ + FD); } \
            /* the element's arithmetic is dealt out between the four MFMAs: each share runs in the shadow of one */ \
            const float g_ = GP[(i_ >> 2) & 1][i_ >> 3][i_ & 3], u_ = UP[(i_ >> 2) & 1][i_ >> 3][i_ & 3];     \
            SPTS_PH_MFMA(GC, fg_, tg, 0, i_)                                                                  \
            const float x_ = __builtin_amdgcn_exp2f(-1.4426950408889634f * g_);                               \
            __builtin_amdgcn_sched_barrier(0);                                                                \
            SPTS_PH_MFMA(UC, fu_, tu, 0, i_)                                                                  \
            const float y_ = __builtin_amdgcn_rcpf(1.0f + x_);                                                \
            __builtin_amdgcn_sched_barrier(0);                                                                \
            SPTS_PH_MFMA(GC, fg_, tg, 1, i_)                                                                  \
            h_[i_] = g_ * y_ * u_;                                                                            \
            __builtin_amdgcn_sched_barrier(0);                                                                \
            SPTS_PH_MFMA(UC, fu_, tu, 1, i_)                                                                  \
            __builtin_amdgcn_sched_barrier(0);                                                                \
        }                                                                                                     \
        if (prev_) SPTS_PH_STORE(tile_begin + (tl_) - 1, h_)                                                  \
    }

    // Everything in flight lands here (the t fragments included): the compiler does not see the direct-to-LDS loads, so
    // a wait it would place later for its own loads must find none outstanding.
    SPTS_WAIT_VMCNT(0);
    __syncthreads();
    // Tiles are taken in pairs: one wait + one workgroup barrier publishes tiles tl and tl + 1 (their loads were issued
    // right after the previous barrier) and frees the two stages the previous pair was read from, which the loads of
    // tiles tl + 2 and tl + 3 then refill.  The only operations a wavefront issued after those loads are the previous pair's
    // four output stores (two per tile), so "all but the newest 4" covers the loads -- provided the stores were really
    // issued: a wavefront whose rows reach past N may skip some (no active lane), so it waits for everything instead.
    const bool full_wave = row0w + 32 <= a.N;
    for (int tl = 0; tl < ntiles; tl += 2) {
        if (tl > 0) {
            if (full_wave) { SPTS_WAIT_VMCNT(4); } else { SPTS_WAIT_VMCNT(0); }
            __syncthreads();
            if (tl + 2 < ntiles) SPTS_PH_DMA(tl + 2)
            if (tl + 3 < ntiles) SPTS_PH_DMA(tl + 3)
        }
        SPTS_PH_TILE(tl, Ga, Ua, Gb, Ub)
        if (tl + 1 < ntiles) SPTS_PH_TILE(tl + 1, Gb, Ub, Ga, Ua)
    }
    // the last tile's accumulators: a slot without MFMAs
    {
        const bool odd = (ntiles & 1) != 0;   // last tile index is even -> it used (Ga, Ua)
        float h[16];
#pragma unroll
        for (int e = 0; e < 16; ++e) {
            const int c = (e >> 2) & 1, r = e >> 3, t = e & 3;
            h[e] = odd ? ph_silu(Ga[c][r][t]) * Ua[c][r][t] : ph_silu(Gb[c][r][t]) * Ub[c][r][t];
        }
        SPTS_PH_STORE(tile_end - 1, h)
    }
}

bool proxy_hidden_supported(const ProxyHiddenArgs& a) {
    if (a.r != 256) return false;   // the rank every configuration uses; other ranks take the GEMM path
    if (a.N <= 0 || a.N >= ((int64_t)1 << 31) || a.Dlow <= 0 || a.Dlow % 32 != 0) return false;
    if (!a.Vg_s || !a.Vu_s || !a.tg || !a.tu || !a.hp) return false;
    auto al = [](const void* p) { return (reinterpret_cast<uintptr_t>(p) & 15u) == 0; };
    if (!al(a.Vg_s) || !al(a.Vu_s) || !al(a.tg) || !al(a.tu) || !al(a.hp)) return false;
    if (a.t_row_pitch % 16 != 0 || a.t_slab_pitch % 16 != 0) return false;
    return true;
}

// channel shares per row tile: the smallest count (each share at least 4 tiles of 32 channels) whose workgroups fill
// whole rounds of the 256 CUs to within 3 % of the best (at least 8 tiles, which left 333 rows 112 workgroups: 19.7 -> 16.8 us)
static int pick_shares(int RT, int TT) {
    int best = 1;
    double best_eff = 0.0;
    for (int sc = 1; sc <= 128 && TT / sc >= 4; ++sc) {
        const int64_t wg = (int64_t)RT * sc;
        const int64_t rounds = (wg + 255) / 256;
        const double eff = (double)wg / (double)(rounds * 256);
        if (eff > best_eff * 1.03) { best_eff = eff; best = sc; }
    }
    return best;
}

hipError_t launch_proxy_hidden(const ProxyHiddenArgs& a, hipStream_t s) {
    const int RT = (int)((a.N + 255) / 256), TT = a.Dlow / 32;
    const int SC = pick_shares(RT, TT);
    const int total = RT * SC;
    const int grid = (total + 7) / 8 * 8;
    const int ks = a.r / 32;
    const size_t lds = (size_t)PH_NSTG * 2 * ks * 2048;
    if (a.r != 256) return hipErrorInvalidValue;
    hipError_t e = ensure_dynamic_lds(reinterpret_cast<const void*>(&proxy_hidden_kernel<8>), (int)lds);
    if (e != hipSuccess) return e;
    proxy_hidden_kernel<8><<<dim3(grid), dim3(PH_WAVES * 64), lds, s>>>(a, RT, SC);
    return hipGetLastError();
}

}  // namespace spts
