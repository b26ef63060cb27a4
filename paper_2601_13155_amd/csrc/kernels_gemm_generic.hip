// C = A * B^T (A [M,K] rows optionally gathered, B [N,K]) with fp32 accumulation and the SPTS epilogues for whatever the
// 256-wide matrix-core kernel does not take: fp32, and bf16 with dimensions that are not tile multiples.
//
//  * gemm_tile32_kernel (rows of whole 16-byte chunks): 32x32 output tile per workgroup, its four or eight wavefronts split K and
//    meet in LDS.  fp32 runs on the fp32 matrix instruction (v_mfma_f32_32x32x2_f32: fp32 products and sums, 157 TFLOP/s,
//    twice what the vector ALU has without packed instructions), bf16 on the 32x32x16 one.  What bounds it: latency.  The
//    products of the fp32 configuration (M <= 512, K <= 688) are 1-200 MFLOP; with small tiles there are enough workgroups for
//    the chip, with K over the wavefronts a wavefront's whole share of both operands (two or three groups of 128 bytes per
//    row) is in flight at once, and nothing waits for a barrier before the final sum.  Operand fragments come straight from
//    global memory: a lane takes 16 consecutive bytes of its row, which is four (fp32) products' operands or one (bf16)
//    product's; which k an instruction multiplies is free as long as both operands agree.  256 x 256 x 256 fp32: 34 us (64x64
//    tiles, 16-wide K steps through LDS, two barriers each) -> 7 us; 256 x 256 x 688 with the residual: 101 -> 10 us; the whole
//    fp32 layer of 512 tokens with the probe and attention of kernels_attn_generic.hip 1590 -> 172 us, its error against 64
//    bits 2.9e-7 -> 1.6e-7 (four or eight partial sums instead of one chain).
//  * gemm_generic_kernel: element-wise loads, any K and any leading dimension.
#include "spts_internal.h"

namespace spts {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float f32x16 __attribute__((ext_vector_type(16)));
typedef float f32x4 __attribute__((ext_vector_type(4)));

// ONE: one product.  SILU: a second product (A1 / B1).  ROPE: columns c and c + d/2 of a head (B rows d/2 apart).  WIDE:
// columns c and c + 32 (the row sums of squares keep their 64-column blocks).
enum Tile32Mode : int { T32_ONE, T32_SILU, T32_ROPE, T32_WIDE };

__device__ inline f32x16 tile32_mfma(u32x4 b, u32x4 a, f32x16 c, float) {
#pragma unroll
    for (int j = 0; j < 4; ++j) c = __builtin_amdgcn_mfma_f32_32x32x2f32(__uint_as_float(b[j]), __uint_as_float(a[j]), c, 0, 0, 0);
    return c;
}
__device__ inline f32x16 tile32_mfma(u32x4 b, u32x4 a, f32x16 c, bf16_t) {
    return __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, b), __builtin_bit_cast(bf16x8, a), c, 0, 0, 0);
}

// Partial sums of an element: one per wavefront, four; eight for a plain fp32 product of K > 256 (partial c: every eighth group of 32 from the c-th on),
// which are added in order.  Who computes them is the launch's choice: eight wavefronts one each, or four two each.  The rule
// for the number knows nothing of the launch or the row count: a product has the same sums alone, in a group and for any rows beside its own.
template <typename T> __host__ __device__ constexpr int tile32_partials(int mode, int K) { return sizeof(T) == 4 && mode == T32_ONE && K > 256 ? 8 : 4; }

// Eight wavefronts while every tile has a CU for itself: with their second set of loads they take 122 registers against 72 and twice the LDS.  K = 512,
// N = 512, M = 512 / 768 / 1500 / 6000 (256, 384, 752, 3008 tiles) with eight 7.6 / 13.2 / 18.3 / 62 us, with four 7.8 / 10.8 / 14.4 / 52; K = 688, N = 256, M = 256 /
// 1024 / 1500 / 6000 8.7 / 9.2 / 16.7 / 46, with four 9.7 / 10.0 / 16.1 / 43.5.  (Two products to a tile, SiLU and rotary, have registers for one workgroup of eight
// per CU: gate/up of 750 rows 16.4 -> 23.4 us.)  And for long sums of very many rows to few columns: K = 1376, N = 128 / 256, 24000 rows 170 / 333, with four 185 / 351; K = 2752,
// N = 64, 24000 rows 180 / 219, N = 256, 6000 rows 173 / 233; not at K = 1024 (N = 256, 6000 / 24000 rows 65 / 239, with four 59 / 234) or fewer tiles (K = 1376,
// N = 128, 6000 rows, 752 of them, 47 / 42.5).
// (A group: the first of the two, over all its tiles.)
constexpr int64_t TILE32_EIGHT_TILES = 256;
static bool tile32_eight_waves(int64_t tiles, int N, int K) { return tiles <= TILE32_EIGHT_TILES || (tiles > 4 * TILE32_EIGHT_TILES && N <= 256 && K > 1024); }

// tile (bx, by) of a product
template <typename T, int MODE, int W, int CH = 1>   // CH: partial sums per wavefront
__device__ __forceinline__ void tile32_product(const GemmArgs& a, int bx, int by, float (*red)[W][32][36]) {
    constexpr int EPC = 16 / (int)sizeof(T);   // elements per 16-byte chunk
    constexpr int KS = 2 * EPC;                // k per step: one chunk for each half of the wavefront
    constexpr int U = 4;                       // steps per group: 128 consecutive bytes of a row
    constexpr int NP = MODE == T32_ONE ? 1 : 2;
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int l32 = lane & 31, lh = lane >> 5;
    const int64_t row0 = (int64_t)by * 32;
    const int col0 = bx * (MODE == T32_WIDE ? 64 : 32);
    const int ncols = MODE == T32_ROPE ? a.N / 2 : a.N;   // rotary: a column stands for its pair
    const int half = MODE == T32_ROPE ? a.head_dim >> 1 : 1;

    int64_t arow = row0 + l32 < a.M ? row0 + l32 : a.M - 1;   // rows and columns past the end repeat the last one (never stored)
    if (a.a_idx) arow = a.a_idx[arow];
    const T* pa = (const T*)a.A + arow * a.lda + lh * EPC;
    const T* pa1 = MODE == T32_SILU && a.A1 ? (const T*)a.A1 + arow * a.lda + lh * EPC : pa;
    const int c = col0 + l32 < ncols ? col0 + l32 : ncols - 1;
    int64_t brow = c, brow1 = c;
    if (MODE == T32_ROPE) { brow = (int64_t)(c / half) * a.head_dim + c % half; brow1 = brow + half; }
    if (MODE == T32_WIDE) brow1 = col0 + 32 + l32 < ncols ? col0 + 32 + l32 : ncols - 1;
    const T* pb = (const T*)a.B0 + brow * a.ldb + lh * EPC;
    const T* pb1 = (const T*)(MODE == T32_SILU ? a.B1 : a.B0) + brow1 * a.ldb + lh * EPC;

    static_assert(CH == 1 || (CH == 2 && W == 4 && NP == 1), "eight partial sums");
    constexpr int NA = NP * CH;
    f32x16 acc[NA];   // of either product, or either partial sum
#pragma unroll
    for (int p = 0; p < NA; ++p)
#pragma unroll
        for (int r = 0; r < 16; ++r) acc[p][r] = 0.f;
    // K % EPC == 0: a chunk is inside or outside as a whole.  Loads past K read the last chunk instead and count as zeros: a load
    // under a lane mask is a branch of its own, and the group's loads would then wait for one another.
    auto load = [&](const T* p, int k0) -> u32x4 {
        const bool in = k0 + lh * EPC < a.K;
        u32x4 v = *reinterpret_cast<const u32x4*>(p + (in ? k0 : a.K - EPC - lh * EPC));
#pragma unroll
        for (int e = 0; e < 4; ++e) v[e] = in ? v[e] : 0u;
        return v;
    };
    constexpr int SETS = W == 8 ? 2 : 1;   // plain fp32 products: a group's loads are in flight while the group before is multiplied
    u32x4 fa[SETS][U], fb[SETS][U], fa1[U], fb1[U];
    auto load_group = [&](int set, int k0) {
#pragma unroll
        for (int u = 0; u < U; ++u) {
            fa[set][u] = load(pa, k0 + u * KS);
            fb[set][u] = load(pb, k0 + u * KS);
            if (NP == 2) fb1[u] = load(pb1, k0 + u * KS);
            if (MODE == T32_SILU) fa1[u] = load(pa1, k0 + u * KS);
        }
    };
    auto multiply_group = [&](int set, int to = 0) {
#pragma unroll
        for (int u = 0; u < U; ++u) {
            acc[to] = tile32_mfma(fb[set][u], fa[set][u], acc[to], T{});
            if (NP == 2) acc[NP - 1] = tile32_mfma(fb1[u], MODE == T32_SILU ? fa1[u] : fa[set][u], acc[NP - 1], T{});
        }
    };
    constexpr int STEP = W * U * KS;
    if (CH == 2) {
        for (int k0 = wave * (U * KS); k0 < a.K; k0 += 2 * STEP) {
            load_group(0, k0);
            multiply_group(0);
            if (k0 + STEP < a.K) { load_group(0, k0 + STEP); multiply_group(0, NA - 1); }
        }
    } else if (SETS == 1) {
        for (int k0 = wave * (U * KS); k0 < a.K; k0 += STEP) { load_group(0, k0); multiply_group(0); }
    } else {
        int k0 = wave * (U * KS);
        if (k0 < a.K) load_group(0, k0);
        for (; k0 < a.K; k0 += 2 * STEP) {
            if (k0 + STEP < a.K) load_group(SETS - 1, k0 + STEP);
            multiply_group(0);
            if (k0 + STEP >= a.K) break;
            if (k0 + 2 * STEP < a.K) load_group(0, k0 + 2 * STEP);
            multiply_group(SETS - 1);
        }
    }
    // lane: output row l32, columns 8 * (r / 4) + 4 * lh + r % 4
    const int r = tid >> 3, c4 = (tid & 7) * 4;
    f32x4 v[2];
#pragma unroll
    for (int ch = 0; ch < CH; ++ch) {
        if (ch > 0) __syncthreads();
#pragma unroll
        for (int p = 0; p < NP; ++p)
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                const f32x16& s = acc[p + ch];
                *reinterpret_cast<f32x4*>(&red[p][wave][l32][8 * q + 4 * lh]) = f32x4{s[4 * q], s[4 * q + 1], s[4 * q + 2], s[4 * q + 3]};
            }
        __syncthreads();
        if (tid >= 256) return;   // (of eight wavefronts, which have one partial sum each)
#pragma unroll
        for (int p = 0; p < NP; ++p)
#pragma unroll
            for (int w = 0; w < W; ++w) {   // fixed order
                const f32x4 s = *reinterpret_cast<const f32x4*>(&red[p][w][r][c4]);
                v[p] = ch == 0 && w == 0 ? s : v[p] + s;
            }
    }
    const int64_t grow = row0 + r;
    if (MODE == T32_WIDE) {   // EPI_SUMSQ
        float ss = 0.f;
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            if (col0 + c4 + e < a.N) ss += v[0][e] * v[0][e];
            if (col0 + 32 + c4 + e < a.N) ss += v[NP - 1][e] * v[NP - 1][e];
        }
        ss += __shfl_xor(ss, 1); ss += __shfl_xor(ss, 2); ss += __shfl_xor(ss, 4);
        if ((tid & 7) == 0 && grow < a.M) a.part[grow * a.part_ld + bx] = ss;
        return;
    }
    if (grow >= a.M) return;
    const int64_t crow = a.c_idx ? (int64_t)a.c_idx[grow] : grow;
    T* C = (T*)a.C + crow * a.ldc;
#pragma unroll
    for (int e = 0; e < 4; ++e) {
        const int col = col0 + c4 + e;
        if (col >= ncols) continue;
        if (MODE == T32_ROPE) {
            const int head = col / half, j = col % half;
            const float2 cs = a.rope[(a.rope_idx ? (int64_t)a.rope_idx[grow] : grow) * half + j];
            const float rs = a.rope_scale != 0.f ? a.rope_scale : 1.f, x1 = v[0][e], x2 = v[NP - 1][e];
            C[(int64_t)head * a.head_dim + j] = from_f32<T>((x1 * cs.x - x2 * cs.y) * rs);
            C[(int64_t)head * a.head_dim + j + half] = from_f32<T>((x2 * cs.x + x1 * cs.y) * rs);
        } else if (MODE == T32_SILU) {
            const float g = v[0][e];
            const T o = from_f32<T>(g / (1.0f + expf(-g)) * v[NP - 1][e]);
            C[col] = o;
            if (a.Ct) ((T*)a.Ct)[(int64_t)col * a.ldct + vt_key_slot(grow)] = o;
        } else if (a.epi == EPI_RESIDUAL) {
            C[col] = from_f32<T>(to_f32(C[col]) + v[0][e]);
        } else if (a.c_is_f32) {
            ((float*)a.C)[crow * a.ldc + col] = v[0][e];
        } else {
            const T o = from_f32<T>(v[0][e]);
            C[col] = o;
            if (a.Ct) ((T*)a.Ct)[(int64_t)col * a.ldct + vt_key_slot(grow)] = o;
        }
    }
}

template <typename T, int MODE, int W, int CH = 1>
__global__ void __launch_bounds__(64 * W) gemm_tile32_kernel(GemmArgs a) {
    __shared__ __attribute__((aligned(16))) float red[MODE == T32_ONE ? 1 : 2][W][32][36];
    tile32_product<T, MODE, W, CH>(a, blockIdx.x, blockIdx.y, red);
}

// independent products, rotary or plain, in one launch: product i has the blocks from first[i] on, nx[i] of them to a row of tiles
struct Tile32Group { GemmArgs a[GEMM_GROUP_MAX]; int first[GEMM_GROUP_MAX], nx[GEMM_GROUP_MAX]; };
// EIGHT: there are products of eight partial sums among them
template <typename T, int WG, bool EIGHT>
__global__ void __launch_bounds__(64 * WG) gemm_tile32_group_kernel(Tile32Group g) {
    __shared__ __attribute__((aligned(16))) float red[2 * 4 * 32 * 36];
    static_assert(sizeof(red) >= sizeof(float) * WG * 32 * 36, "one product of WG wavefronts or two of four");
    int i = 0;
#pragma unroll
    for (int q = 1; q < GEMM_GROUP_MAX; ++q) i += (int)blockIdx.x >= g.first[q] ? 1 : 0;
    const int b = blockIdx.x - g.first[i], by = b / g.nx[i], bx = b - by * g.nx[i];
    const bool rope = g.a[i].epi == EPI_ROPE, eight = EIGHT && tile32_partials<T>(rope ? T32_ROPE : T32_ONE, g.a[i].K) == 8;
    if (WG == 8 && eight) {
        tile32_product<T, T32_ONE, WG>(g.a[i], bx, by, reinterpret_cast<float (*)[WG][32][36]>(red));
        return;
    }
    if (threadIdx.x >= 256) return;
    auto* red4 = reinterpret_cast<float (*)[4][32][36]>(red);
    if constexpr (WG == 4 && EIGHT)
        if (eight) {
            tile32_product<T, T32_ONE, 4, 2>(g.a[i], bx, by, red4);
            return;
        }
    if (rope) tile32_product<T, T32_ROPE, 4>(g.a[i], bx, by, red4);
    else tile32_product<T, T32_ONE, 4>(g.a[i], bx, by, red4);
}

constexpr int GT = 64;   // tile edge
constexpr int GK = 16;   // k step

template <typename T, bool DUAL>
__global__ void __launch_bounds__(256) gemm_generic_kernel(GemmArgs a) {
    __shared__ float As[GK][GT + 1];
    __shared__ float Bs[GK][GT + 1];
    __shared__ float Bs1[DUAL ? GK : 1][GT + 1];
    __shared__ float As1[DUAL ? GK : 1][GT + 1];
    __shared__ float red[GT][17];

    const T* A = (const T*)a.A;
    const T* A1 = a.A1 ? (const T*)a.A1 : A;
    const T* B0 = (const T*)a.B0;
    const T* B1 = (const T*)a.B1;
    const int tx = threadIdx.x & 15, ty = threadIdx.x >> 4;
    const int64_t row0 = (int64_t)blockIdx.y * GT;
    const int col0 = blockIdx.x * GT;

    float acc[4][4] = {}, acc1[4][4] = {};

    // loader mapping: thread loads element (r = tid / 16 + 16 * i, kk = tid % 16)
    const int lk = threadIdx.x & 15, lr = threadIdx.x >> 4;
    for (int k0 = 0; k0 < a.K; k0 += GK) {
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            int r = lr + 16 * i;
            int64_t grow = row0 + r;
            int kk = k0 + lk;
            float va = 0.f, va1 = 0.f, vb = 0.f, vb1 = 0.f;
            if (grow < a.M && kk < a.K) {
                int64_t srow = a.a_idx ? (int64_t)a.a_idx[grow] : grow;
                va = to_f32(A[srow * a.lda + kk]);
                if (DUAL) va1 = to_f32(A1[srow * a.lda + kk]);
            }
            int gcol = col0 + r;
            if (gcol < a.N && kk < a.K) {
                vb = to_f32(B0[(int64_t)gcol * a.ldb + kk]);
                if (DUAL) vb1 = to_f32(B1[(int64_t)gcol * a.ldb + kk]);
            }
            As[lk][r] = va;
            Bs[lk][r] = vb;
            if (DUAL) { Bs1[lk][r] = vb1; As1[lk][r] = va1; }
        }
        __syncthreads();
#pragma unroll
        for (int kk = 0; kk < GK; ++kk) {
            float av[4], av1[4], bv[4], bv1[4];
#pragma unroll
            for (int i = 0; i < 4; ++i) { av[i] = As[kk][ty * 4 + i]; bv[i] = Bs[kk][tx * 4 + i]; if (DUAL) { bv1[i] = Bs1[kk][tx * 4 + i]; av1[i] = As1[kk][ty * 4 + i]; } }
#pragma unroll
            for (int i = 0; i < 4; ++i)
#pragma unroll
                for (int j = 0; j < 4; ++j) {
                    acc[i][j] = fmaf(av[i], bv[j], acc[i][j]);
                    if (DUAL) acc1[i][j] = fmaf(av1[i], bv1[j], acc1[i][j]);
                }
        }
        __syncthreads();
    }

    if (a.epi == EPI_SUMSQ) {
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            float ssq = 0.f;
#pragma unroll
            for (int j = 0; j < 4; ++j) { int gcol = col0 + tx * 4 + j; if (gcol < a.N) ssq += acc[i][j] * acc[i][j]; }
            red[ty * 4 + i][tx] = ssq;
        }
        __syncthreads();
        if (threadIdx.x < GT) {
            int64_t grow = row0 + threadIdx.x;
            if (grow < a.M) {
                float t = 0.f;
                for (int j = 0; j < 16; ++j) t += red[threadIdx.x][j];
                a.part[grow * a.part_ld + blockIdx.x] = t;
            }
        }
        return;
    }

#pragma unroll
    for (int i = 0; i < 4; ++i) {
        int64_t grow = row0 + ty * 4 + i;
        if (grow >= a.M) continue;
        int64_t crow = a.c_idx ? (int64_t)a.c_idx[grow] : grow;
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            int gcol = col0 + tx * 4 + j;
            if (gcol >= a.N) continue;
            float v = acc[i][j];
            if (DUAL) { float g = v; v = g / (1.0f + expf(-g)) * acc1[i][j]; }
            if (a.epi == EPI_RESIDUAL) {
                T* c = (T*)a.C + crow * a.ldc + gcol;
                *c = from_f32<T>(to_f32(*c) + v);
            } else if (a.c_is_f32) {
                ((float*)a.C)[crow * a.ldc + gcol] = v;
            } else {
                T o = from_f32<T>(v);
                ((T*)a.C)[crow * a.ldc + gcol] = o;
                if (a.Ct) ((T*)a.Ct)[(int64_t)gcol * a.ldct + vt_key_slot(grow)] = o;
            }
        }
    }
}

// Rows of whole 16-byte chunks at 16-byte addresses; every epilogue but the merged rotary + store and the channel-major one, no stacked B.
bool gemm_tile32_supported(const GemmArgs& a, bool bf16) {
    const int epc = bf16 ? 8 : 4;
    auto al = [](const void* p) { return (reinterpret_cast<uintptr_t>(p) & 15u) == 0; };
    if (a.M <= 0 || a.N <= 0 || a.K <= 0 || a.K % epc != 0 || a.lda % epc != 0 || a.ldb % epc != 0) return false;
    if ((a.M + 31) / 32 > 65535) return false;   // grid y
    if (!al(a.A) || !al(a.B0) || (a.A1 && !al(a.A1)) || (a.B1 && !al(a.B1))) return false;
    if (a.a_slab || a.b_slab || a.c_slab || a.epi == EPI_ROPE_STORE || a.epi == EPI_SILU_MUL_T || (a.epi == EPI_STORE && a.B1)) return false;
    if (a.epi == EPI_ROPE && (a.head_dim <= 0 || a.head_dim % 2 != 0 || a.N % a.head_dim != 0 || a.c_is_f32 || a.Ct)) return false;
    if (a.c_is_f32 && a.epi != EPI_STORE) return false;
    return true;
}

// wavefronts of a product in a launch of its own
int gemm_tile32_waves(const GemmArgs& a, bool bf16) {
    if (bf16 || (a.epi != EPI_STORE && a.epi != EPI_RESIDUAL) || tile32_partials<float>(T32_ONE, a.K) != 8) return 4;
    return tile32_eight_waves((a.M + 31) / 32 * ((a.N + 31) / 32), a.N, a.K) ? 8 : 4;
}

template <typename T>
static void launch_tile32_t(const GemmArgs& a, hipStream_t s) {
    const unsigned ny = (unsigned)((a.M + 31) / 32), nx = (unsigned)((a.N + 31) / 32);
    const dim3 b4(256);
    switch (a.epi) {
        case EPI_SILU_MUL: gemm_tile32_kernel<T, T32_SILU, 4><<<dim3(nx, ny), b4, 0, s>>>(a); break;
        case EPI_ROPE: gemm_tile32_kernel<T, T32_ROPE, 4><<<dim3((unsigned)((a.N / 2 + 31) / 32), ny), b4, 0, s>>>(a); break;
        case EPI_SUMSQ: gemm_tile32_kernel<T, T32_WIDE, 4><<<dim3((unsigned)((a.N + 63) / 64), ny), b4, 0, s>>>(a); break;
        default:
            if constexpr (sizeof(T) == 4)
                if (tile32_partials<T>(T32_ONE, a.K) == 8) {
                    if (gemm_tile32_waves(a, false) == 8) gemm_tile32_kernel<T, T32_ONE, 8><<<dim3(nx, ny), dim3(512), 0, s>>>(a);
                    else gemm_tile32_kernel<T, T32_ONE, 4, 2><<<dim3(nx, ny), b4, 0, s>>>(a);
                    break;
                }
            gemm_tile32_kernel<T, T32_ONE, 4><<<dim3(nx, ny), b4, 0, s>>>(a);
            break;
    }
}

hipError_t launch_gemm_generic(const GemmArgs& a, bool bf16, hipStream_t s) {
    if (a.M == 0 || a.N == 0) return hipSuccess;
    if (gemm_tile32_supported(a, bf16)) {
        if (bf16) launch_tile32_t<bf16_t>(a, s); else launch_tile32_t<float>(a, s);
        return hipGetLastError();
    }
    if (a.epi == EPI_ROPE || a.epi == EPI_ROPE_STORE || a.epi == EPI_SILU_MUL_T) return hipErrorInvalidValue;
    dim3 grid((unsigned)((a.N + GT - 1) / GT), (unsigned)((a.M + GT - 1) / GT)), block(256);
    bool dual = a.epi == EPI_SILU_MUL;
    if (bf16) {
        if (dual) gemm_generic_kernel<bf16_t, true><<<grid, block, 0, s>>>(a);
        else gemm_generic_kernel<bf16_t, false><<<grid, block, 0, s>>>(a);
    } else {
        if (dual) gemm_generic_kernel<float, true><<<grid, block, 0, s>>>(a);
        else gemm_generic_kernel<float, false><<<grid, block, 0, s>>>(a);
    }
    return hipGetLastError();
}

static int tile32_columns(const GemmArgs& a) { return ((a.epi == EPI_ROPE ? a.N / 2 : a.N) + 31) / 32; }   // tiles of a plain or rotary product

bool gemm_tile32_group_supported(const GemmArgs* a, int n, bool bf16) {
    if (n < 1 || n > GEMM_GROUP_MAX) return false;
    int64_t blocks = 0;
    for (int i = 0; i < n; ++i) {
        if (!gemm_tile32_supported(a[i], bf16) || (a[i].epi != EPI_ROPE && a[i].epi != EPI_STORE && a[i].epi != EPI_RESIDUAL)) return false;
        blocks += (int64_t)tile32_columns(a[i]) * ((a[i].M + 31) / 32);
    }
    return blocks <= 1 << 23;   // one grid dimension of 256 threads each
}

hipError_t launch_gemm_tile32_group(const GemmArgs* a, int n, bool bf16, hipStream_t s) {
    if (!gemm_tile32_group_supported(a, n, bf16)) return hipErrorInvalidValue;
    Tile32Group g{};
    int64_t blocks = 0;
    for (int i = 0; i < GEMM_GROUP_MAX; ++i) {
        g.first[i] = 0x7fffffff;
        g.nx[i] = 1;
        if (i >= n) continue;
        g.a[i] = a[i];
        g.first[i] = (int)blocks;
        g.nx[i] = tile32_columns(a[i]);
        blocks += (int64_t)g.nx[i] * ((a[i].M + 31) / 32);
    }
    bool eight = false;
    for (int i = 0; i < n; ++i) eight |= !bf16 && tile32_partials<float>(a[i].epi == EPI_ROPE ? T32_ROPE : T32_ONE, a[i].K) == 8;
    const dim3 grid((unsigned)blocks);
    if (bf16) gemm_tile32_group_kernel<bf16_t, 4, false><<<grid, dim3(256), 0, s>>>(g);
    else if (!eight) gemm_tile32_group_kernel<float, 4, false><<<grid, dim3(256), 0, s>>>(g);
    else if (blocks <= TILE32_EIGHT_TILES) gemm_tile32_group_kernel<float, 8, true><<<grid, dim3(512), 0, s>>>(g);
    else gemm_tile32_group_kernel<float, 4, true><<<grid, dim3(256), 0, s>>>(g);
    return hipGetLastError();
}

}  // namespace spts
