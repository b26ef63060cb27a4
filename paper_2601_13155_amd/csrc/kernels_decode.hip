// Decode phase over the per-layer KV caches left by the token-skipped prefill (Alg. 1 with
// Is_prefill_phase() false: both branches dense for the one new token; Sec. 3.2 last paragraph and
// the appendix on KV-cache flexibility say what a cache holds: the active pairs of the prefill plus
// every decoded token's pair).
//
// One token means every contraction is a matrix-vector product whose cost is reading the weights
// once, so the whole step is HBM-bound (8B-shaped model: 13.9 GB of bf16 weights per token):
//   * gemv_kernel: y = W x with W [R, K] row-major.  A workgroup of 4 wavefronts owns 2 rows (4 where it
//     normalises x itself, for Q/K/V and for the head) and splits K across its 256 lanes in
//     16-byte chunks, with several independent 16-byte weight loads per lane in flight before the first use; bf16
//     pairs are multiplied with v_dot2c_f32_bf16 (fp32 accumulate, no conversion instructions).
//     Lanes reduce by shuffles, wavefronts through LDS.  Up to three matrices that share x run as
//     one launch (Q, K, V).  Epilogues: store, SiLU(gate)*up, residual add, fp32 store (logits).
//   * decode_attn_kernel: flash-decoding.  Grid = (key splits, KV heads); 64/LPK keys per wavefront
//     step (LPK lanes hold one key row as 16-byte pieces), every lane group keeps its own running
//     (max, sum, weighted values) for all query heads of the KV head, a lane the maximum and sum of one head; groups, wavefronts and splits
//     are merged with the usual (max, sum) algebra in a fixed order (deterministic).
//   * small kernels: rotary embedding of q / k for the new position + cache append, merge of the
//     splits, argmax with ties to the lowest token id, table row gather.
#include "spts_internal.h"
#include "spts_lanes.h"

namespace spts {

// ------------------------------------------------------------------------------------------- GEMV
// 16-byte chunk of T -> chunk of T holding from_f32(x[e] * inv * gamma[e]) (RMSNorm's last step)
__device__ inline u32x4 norm_chunk(u32x4 xv, u32x4 gv, float inv, bf16_t) {
    u32x4 o;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        const float x0 = __uint_as_float(xv[i] << 16), x1 = __uint_as_float(xv[i] & 0xffff0000u);
        const float g0 = __uint_as_float(gv[i] << 16), g1 = __uint_as_float(gv[i] & 0xffff0000u);
        o[i] = (uint32_t)f32_to_bf16(x0 * inv * g0).v | ((uint32_t)f32_to_bf16(x1 * inv * g1).v << 16);
    }
    return o;
}
__device__ inline u32x4 norm_chunk(u32x4 xv, u32x4 gv, float inv, float) {
    u32x4 o;
#pragma unroll
    for (int i = 0; i < 4; ++i) o[i] = __float_as_uint(__uint_as_float(xv[i]) * inv * __uint_as_float(gv[i]));
    return o;
}
__device__ inline float chunk_sumsq(u32x4 v, bf16_t) {
    float s = 0.f;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        const float a = __uint_as_float(v[i] << 16), b = __uint_as_float(v[i] & 0xffff0000u);
        s += a * a; s += b * b;
    }
    return s;
}
__device__ inline float chunk_sumsq(u32x4 v, float) {
    float s = 0.f;
#pragma unroll
    for (int i = 0; i < 4; ++i) { const float a = __uint_as_float(v[i]); s += a * a; }
    return s;
}

// the sum over the wavefront's lanes, in every lane: six DPP steps (a shuffle through the LDS crossbar takes about a hundred cycles)
__device__ __forceinline__ float wave_total(float v) {
    auto bits = [](float f) { return __builtin_bit_cast(int, f); };
    v += __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, bits(v), 0x111, 0xF, 0xF, false));   // row_shr 1
    v += __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, bits(v), 0x112, 0xF, 0xF, false));   // row_shr 2
    v += __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, bits(v), 0x114, 0xF, 0xF, false));   // row_shr 4
    v += __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, bits(v), 0x118, 0xF, 0xF, false));   // row_shr 8
    v += __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, bits(v), 0x142, 0xA, 0xF, false));   // row_bcast 15
    v += __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, bits(v), 0x143, 0xC, 0xF, false));   // row_bcast 31
    return __builtin_bit_cast(float, __builtin_amdgcn_readlane(bits(v), 63));
}

// NORM: x is normalised on the way in (NCH chunks of it and of every row per lane, all in registers).  ROWS: dot products per workgroup.
template <typename T, int MODE, bool NORM, int ROWS, int NCH>
__global__ void __launch_bounds__(256) gemv_kernel(GemvArgs a) {
    constexpr int EPC = 16 / (int)sizeof(T);          // elements per 16-byte chunk
    static_assert(MODE != GEMV_QKV_ROPE || ROWS == 4, "two rotary pairs");
    __shared__ float sred[4][ROWS];
    __shared__ float snorm[4];
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;

    // rows of this workgroup: ROWS consecutive rows of one matrix, or (SiLU) ROWS / 2 gate rows and the same up rows.
    // Without a norm two rows per workgroup measured best where the epilogue allows it (O-proj 8.0 -> 7.5 us, down 19.7 -> 19.3 us,
    // gate/up 36.9 -> 35.3 us against four; one row and eight rows are slower); Q/K/V keep the four rows of two
    // rotary pairs
    const T* wrow[ROWS];
    int64_t out_row;      // first output element of this workgroup
    int which = 0;        // matrix the rows belong to
    if (MODE == GEMV_SILU) {
        out_row = (int64_t)blockIdx.x * (ROWS / 2);
#pragma unroll
        for (int r = 0; r < ROWS; ++r)
            wrow[r] = (const T*)(r < ROWS / 2 ? a.W[0] : a.W[1]) + (out_row + (r % (ROWS / 2))) * a.K;
    } else if (MODE == GEMV_QKV_ROPE) {
        // Q and K blocks own the rows (j, j+1, j+d/2, j+d/2+1) of one head, so that both members of the
        // two rotary pairs are reduced by the same workgroup; V blocks own 4 consecutive rows
        int64_t blk = blockIdx.x;
        if (blk >= a.R[0] / 4) { blk -= a.R[0] / 4; which = 1; if (blk >= a.R[1] / 4) { blk -= a.R[1] / 4; which = 2; } }
        if (which < 2) {
            const int qd = a.head_dim / 4;                       // blocks per head
            out_row = (blk / qd) * a.head_dim + 2 * (blk % qd);  // j of the first pair
#pragma unroll
            for (int r = 0; r < ROWS; ++r)
                wrow[r] = (const T*)a.W[which] + (out_row + (r & 1) + (r >> 1) * (a.head_dim / 2)) * a.K;
        } else {
            out_row = blk * ROWS;
#pragma unroll
            for (int r = 0; r < ROWS; ++r) wrow[r] = (const T*)a.W[2] + (out_row + r) * a.K;
        }
    } else {
        int64_t row = (int64_t)blockIdx.x * ROWS;
        if (row >= a.R[0]) { row -= a.R[0]; which = 1; if (row >= a.R[1]) { row -= a.R[1]; which = 2; } }
        out_row = row;
#pragma unroll
        for (int r = 0; r < ROWS; ++r) wrow[r] = (const T*)a.W[which] + (row + r) * a.K;
    }

    const int nchunks = a.K / EPC;
    const T* x = (const T*)a.x;
    float acc[ROWS];
    for (int r = 0; r < ROWS; ++r) acc[r] = 0.f;
    if (NORM) {
        // the weight loads do not depend on the norm: issue them first, then normalise x while they fly
        u32x4 wv[NCH][ROWS], xc[NCH], gc[NCH];
#pragma unroll
        for (int i = 0; i < NCH; ++i) {
            const int c = tid + 256 * i;
            if (c < nchunks) {
                xc[i] = *reinterpret_cast<const u32x4*>(x + (int64_t)c * EPC);
                gc[i] = *reinterpret_cast<const u32x4*>((const T*)a.gamma + (int64_t)c * EPC);
#pragma unroll
                for (int r = 0; r < ROWS; ++r) wv[i][r] = __builtin_nontemporal_load(reinterpret_cast<const u32x4*>(wrow[r] + (int64_t)c * EPC));
            }
        }
        float ss = 0.f;
#pragma unroll
        for (int i = 0; i < NCH; ++i)
            if (tid + 256 * i < nchunks) ss += chunk_sumsq(xc[i], T{});
        ss = wave_total(ss);
        if (lane == 0) snorm[wave] = ss;
        __syncthreads();
        const float inv = 1.0f / sqrtf((snorm[0] + snorm[1] + snorm[2] + snorm[3]) / (float)a.K + a.eps);
#pragma unroll
        for (int i = 0; i < NCH; ++i) {
            const int c = tid + 256 * i;
            if (c < nchunks) {
                const u32x4 xn = norm_chunk(xc[i], gc[i], inv, T{});
#pragma unroll
                for (int r = 0; r < ROWS; ++r) acc[r] = dot16(wv[i][r], xn, acc[r], T{});
            }
        }
    } else {
#pragma unroll 4
        for (int c = tid; c < nchunks; c += 256) {
            const u32x4 xv = *reinterpret_cast<const u32x4*>(x + (int64_t)c * EPC);
            u32x4 wv[ROWS];
#pragma unroll
            for (int r = 0; r < ROWS; ++r) wv[r] = __builtin_nontemporal_load(reinterpret_cast<const u32x4*>(wrow[r] + (int64_t)c * EPC));
#pragma unroll
            for (int r = 0; r < ROWS; ++r) acc[r] = dot16(wv[r], xv, acc[r], T{});
        }
    }
#pragma unroll
    for (int r = 0; r < ROWS; ++r) {
        acc[r] = wave_total(acc[r]);
        if (lane == 0) sred[wave][r] = acc[r];
    }
    __syncthreads();
    if (tid >= ROWS) return;
    const float v = sred[0][tid] + sred[1][tid] + sred[2][tid] + sred[3][tid];
    if (MODE == GEMV_SILU) {
        if (tid < ROWS / 2) {
            const float g = v;
            const float u = sred[0][tid + ROWS / 2] + sred[1][tid + ROWS / 2] + sred[2][tid + ROWS / 2] + sred[3][tid + ROWS / 2];
            const float h = g / (1.0f + __expf(-g)) * u;
            ((T*)a.y[0])[out_row + tid] = from_f32<T>(h);
        }
    } else if (MODE == GEMV_QKV_ROPE) {
        if (blockIdx.x == 0 && tid == 0 && a.pos_out) *a.pos_out = a.pos_val;
        if (which == 2) {
            ((T*)a.y[2])[out_row + tid] = from_f32<T>(v);
        } else {
            // tid: 0, 1 = first members (j, j+1), 2, 3 = their partners at +d/2
            const int half = a.head_dim / 2;
            const int j = (int)(out_row % a.head_dim) + (tid & 1);
            const float2 cs = a.rope[j];
            const float other = sred[0][tid ^ 2] + sred[1][tid ^ 2] + sred[2][tid ^ 2] + sred[3][tid ^ 2];
            const float res = tid < 2 ? v * cs.x - other * cs.y : v * cs.x + other * cs.y;
            ((T*)a.y[which])[out_row + (tid & 1) + (tid >> 1) * half] = from_f32<T>(res);
        }
    } else if (MODE == GEMV_RESID) {
        T* y = (T*)a.y[which] + out_row + tid;
        *y = from_f32<T>(to_f32(*y) + v);
    } else {   // GEMV_F32
        ((float*)a.y[which])[out_row + tid] = v;
    }
}

bool gemv_supported(const GemvArgs& a, bool bf16) {
    const int epc = bf16 ? 8 : 4;
    if (a.K <= 0 || a.K % epc != 0) return false;
    for (int i = 0; i < 3; ++i) {
        if (a.R[i] < 0 || a.R[i] % 4 != 0) return false;
        if (a.R[i] > 0 && (!a.W[i] || (reinterpret_cast<uintptr_t>(a.W[i]) & 15u))) return false;
    }
    if (!a.x || (reinterpret_cast<uintptr_t>(a.x) & 15u)) return false;
    if (a.gamma && ((reinterpret_cast<uintptr_t>(a.gamma) & 15u) || a.K / epc > 1024)) return false;
    return true;
}

// With the norm inside, a workgroup of gate/up rows takes two of each, so that normalising x (a barrier and a round trip to the L2) comes once per
// 32 KB of weights that are in flight meanwhile: 1 / 2 / 4 row pairs 338.9 / 331.8 / 333.3 us for two layers of the 8B shape, 13107 cached pairs, and a head of 128256 rows,
// Qwen shape 335.4 / 329.6 / 330.3, hidden size 2048, 8 layers 352 / 349 / 351, fp32, 4 layers 236 / 232 / 234.  The head with four rows 336.1 and 330.2 (8B, Qwen), with eight
// 341.9 and 330.6.  Half as many registers where a lane holds two chunks (Q/K/V: 1536 workgroups, six per CU, at once instead of in two rounds).
// Against a launch for each norm (the head of 32000 rows, 500 cached pairs): hidden size 1024, 16 layers 479 -> 414; 2048, 8 layers 344 -> 299; 4096, 2 layers 226 -> 210; with
// four chunks to a lane 5120 / 6144 / 8192, 2 layers 275 -> 256, 350 -> 327, 628 -> 612; fp32 1024, 8 layers 283 -> 249, 3072 / 4096, 2 layers 238 -> 224, 347 -> 331.
template <typename T>
static hipError_t launch_gemv_t(const GemvArgs& a, hipStream_t s) {
    const int64_t rows = (int64_t)a.R[0] + a.R[1] + a.R[2];
    if (rows == 0) return hipSuccess;
    const dim3 b(256);
    const bool n = a.gamma != nullptr;
    const bool two = a.K / (16 / (int)sizeof(T)) <= 512;   // chunks of x per lane, with the norm: 2, or 4
    auto grid = [&](int per) { return dim3((unsigned)(rows / per)); };
    switch (a.mode) {
        case GEMV_SILU:
            if (!n) gemv_kernel<T, GEMV_SILU, false, 2, 1><<<grid(1), b, 0, s>>>(a);
            else if (two) gemv_kernel<T, GEMV_SILU, true, 4, 2><<<grid(2), b, 0, s>>>(a);
            else gemv_kernel<T, GEMV_SILU, true, 4, 4><<<grid(2), b, 0, s>>>(a);
            break;
        case GEMV_RESID: if (n) return hipErrorInvalidValue; gemv_kernel<T, GEMV_RESID, false, 2, 1><<<grid(2), b, 0, s>>>(a); break;
        case GEMV_F32:
            if (!n) gemv_kernel<T, GEMV_F32, false, 4, 1><<<grid(4), b, 0, s>>>(a);
            else if (two) gemv_kernel<T, GEMV_F32, true, 4, 2><<<grid(4), b, 0, s>>>(a);
            else gemv_kernel<T, GEMV_F32, true, 4, 4><<<grid(4), b, 0, s>>>(a);
            break;
        case GEMV_QKV_ROPE:
            if (!a.rope || a.head_dim % 4 != 0 || a.R[0] % a.head_dim != 0 || a.R[1] % a.head_dim != 0) return hipErrorInvalidValue;
            if (!n) gemv_kernel<T, GEMV_QKV_ROPE, false, 4, 1><<<grid(4), b, 0, s>>>(a);
            else if (two) gemv_kernel<T, GEMV_QKV_ROPE, true, 4, 2><<<grid(4), b, 0, s>>>(a);
            else gemv_kernel<T, GEMV_QKV_ROPE, true, 4, 4><<<grid(4), b, 0, s>>>(a);
            break;
        default: return hipErrorInvalidValue;
    }
    return hipGetLastError();
}

hipError_t launch_gemv(const GemvArgs& a, bool bf16, hipStream_t s) {
    return bf16 ? launch_gemv_t<bf16_t>(a, s) : launch_gemv_t<float>(a, s);
}

// ------------------------------------------------------------------- GEMV over a few input vectors
// Y[b, r] = W[r, :] . X[b, :] for b < NB (a decode step over NB sequences): the weights are still read
// once, every weight chunk meets the NB input chunks in registers.  X [NB, K] and Y[i] [NB, R[i]] are
// row-major and contiguous.
// A wavefront owns RW rows on its own (RW/2 gate rows and the same up rows for the SiLU variant) and
// splits K over its 64 lanes; a workgroup is four such wavefronts on consecutive rows (they read the
// same input chunks at about the same time).  The RW*NB accumulators of a lane are reduced over the
// wavefront with a halving butterfly: at every step a lane hands half of its accumulators to its
// partner and adds the partner's other half, so 64 sums cost 63 exchanges instead of 64*6; lane
// (i << (6 - log2(RW*NB))) ends up with the total of accumulator i.
template <typename T, int MODE, int NB, int RW>
__global__ void __launch_bounds__(256) gemv_nb_kernel(GemvArgs a) {
    constexpr int EPC = 16 / (int)sizeof(T);
    constexpr int HR = RW / 2;
    constexpr int NA = RW * NB;                     // accumulators per lane (a power of two <= 64)
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const T* wrow[RW];
    int64_t out_row;
    int which = 0;
    if (MODE == GEMV_SILU) {
        out_row = ((int64_t)blockIdx.x * 4 + wave) * HR;
#pragma unroll
        for (int r = 0; r < RW; ++r) wrow[r] = (const T*)(r < HR ? a.W[0] : a.W[1]) + (out_row + r % HR) * a.K;
    } else {
        int64_t row = ((int64_t)blockIdx.x * 4 + wave) * RW;
        if (row >= a.R[0]) { row -= a.R[0]; which = 1; if (row >= a.R[1]) { row -= a.R[1]; which = 2; } }
        out_row = row;
#pragma unroll
        for (int r = 0; r < RW; ++r) wrow[r] = (const T*)a.W[which] + (row + r) * a.K;
    }
    const int nchunks = a.K / EPC;
    const T* x = (const T*)a.x;
    float acc[NA];
#pragma unroll
    for (int i = 0; i < NA; ++i) acc[i] = 0.f;
#pragma unroll 2
    for (int c = lane; c < nchunks; c += 64) {
        u32x4 wv[RW], xv[NB];
#pragma unroll
        for (int r = 0; r < RW; ++r) wv[r] = __builtin_nontemporal_load(reinterpret_cast<const u32x4*>(wrow[r] + (int64_t)c * EPC));
#pragma unroll
        for (int b = 0; b < NB; ++b) xv[b] = *reinterpret_cast<const u32x4*>(x + ((int64_t)b * a.K + (int64_t)c * EPC));
#pragma unroll
        for (int r = 0; r < RW; ++r)
#pragma unroll
            for (int b = 0; b < NB; ++b) acc[r * NB + b] = dot16(wv[r], xv[b], acc[r * NB + b], T{});
    }
    // halving butterfly over the 64 lanes
    int n = NA;
#pragma unroll
    for (int off = 32; off >= 1; off >>= 1) {
        if (n > 1) {
            const int half = n / 2;
            const bool up = (lane & off) != 0;
#pragma unroll
            for (int i = 0; i < NA / 2; ++i) {
                if (i < half) {
                    const float lo = acc[i], hi = acc[i + half];
                    acc[i] = (up ? hi : lo) + __shfl_xor(up ? lo : hi, off);
                }
            }
            n = half;
        } else {
            acc[0] += __shfl_xor(acc[0], off);
        }
    }
    constexpr int SH = NA == 64 ? 0 : NA == 32 ? 1 : NA == 16 ? 2 : NA == 8 ? 3 : NA == 4 ? 4 : NA == 2 ? 5 : 6;
    const float v = acc[0];
    const int idx = lane >> SH;                     // accumulator this lane holds the total of
    const int r = idx / NB, b = idx % NB;
    float u = 0.f;
    if (MODE == GEMV_SILU) u = __shfl(v, ((idx + HR * NB) % NA) << SH);   // the up row's total (read by the gate row's lane)
    if ((lane & ((1 << SH) - 1)) != 0) return;
    if (MODE == GEMV_SILU) {
        if (r < HR) ((T*)a.y[0])[(int64_t)b * a.R[0] + out_row + r] = from_f32<T>(v / (1.0f + __expf(-v)) * u);
    } else if (MODE == GEMV_RESID) {
        T* y = (T*)a.y[which] + (int64_t)b * a.R[which] + out_row + r;
        *y = from_f32<T>(to_f32(*y) + v);
    } else {   // GEMV_F32
        ((float*)a.y[which])[(int64_t)b * a.R[which] + out_row + r] = v;
    }
}

template <typename T, int NB, int RW>
static hipError_t launch_gemv_nb_tr(const GemvArgs& a, hipStream_t s) {
    const int64_t rows = (int64_t)a.R[0] + a.R[1] + a.R[2];
    const dim3 b(256);
    const dim3 g((unsigned)(a.mode == GEMV_SILU ? a.R[0] / (4 * (RW / 2)) : rows / (4 * RW)));
    switch (a.mode) {
        case GEMV_SILU: gemv_nb_kernel<T, GEMV_SILU, NB, RW><<<g, b, 0, s>>>(a); break;
        case GEMV_RESID: gemv_nb_kernel<T, GEMV_RESID, NB, RW><<<g, b, 0, s>>>(a); break;
        case GEMV_F32: gemv_nb_kernel<T, GEMV_F32, NB, RW><<<g, b, 0, s>>>(a); break;
        default: return hipErrorInvalidValue;
    }
    return hipGetLastError();
}

// rows per wavefront: 4 when every matrix has a multiple of 16 rows (8 outputs for the SiLU variant), else 2 (multiples
// of 8 / 4); row counts that divide neither are refused (the callers' shapes are multiples of 16)
template <typename T, int NB>
static hipError_t launch_gemv_nb_t(const GemvArgs& a, hipStream_t s) {
    const int64_t rows = (int64_t)a.R[0] + a.R[1] + a.R[2];
    if (rows == 0) return hipSuccess;
    auto divides = [&](int unit) { return a.R[0] % unit == 0 && a.R[1] % unit == 0 && a.R[2] % unit == 0; };
    const bool silu = a.mode == GEMV_SILU;
    if (divides(silu ? 8 : 16)) return launch_gemv_nb_tr<T, NB, 4>(a, s);
    if (divides(silu ? 4 : 8)) return launch_gemv_nb_tr<T, NB, 2>(a, s);
    return hipErrorInvalidValue;
}

// ------------------------------------------------------------------- the same on the matrix cores (bf16)
// Y[b, r] = W[r, :] . X[b, :] for up to 16 input vectors with v_mfma_f32_16x16x32_bf16: a weight row is an MFMA
// operand row (row = lane % 16, 8 consecutive k of group lane / 16) and an input vector is an operand column (lanes
// >= nb feed zeros).  No dot instructions, no lane reductions: the vector ALU only moves the 4 results per lane.
//
// The operand layout gives a row only 4 lanes, i.e. 64 bytes per load instruction, and weight streams read as
// half cache lines by two different instructions run at ~60 % of the rate of whole-line reads (measured: 4.1 against
// 6.4 TB/s on the 14336 x 4096 gate/up pair).  So the weights (and the input vectors, same shape: 16 rows with row
// stride K) go through LDS with direct-to-LDS loads whose lanes are laid out for memory, not for the matrix core:
// one instruction = 8 rows x one whole 128-byte line, two instructions = a 16-row strip x 64 k.  Fragments are then
// 16-byte LDS reads; the 16-byte chunk c of row r sits at slot c ^ (r >> 1) (the permutation is applied to the
// global addresses, since the hardware places lane l's 16 bytes at 16 * l), which spreads the 16 rows a fragment
// read touches over all banks.
//
// A workgroup of 4 wavefronts owns a strip of 16 rows (a gate strip and the same up strip for the SiLU variant)
// and splits K four ways (8 wavefronts with deeper or shallower rings measured the same or slower); every wavefront runs its own ring of DEPTH stages of 64 k (no workgroup barrier in the
// loop: a wavefront reads only what it loaded itself, after its own vmcnt wait).  The partial 16x16 tiles meet
// in LDS.  Needs K % 256 == 0 and row counts that are multiples of 16.
// The weights are read once and are loaded as such (nt): kept in the caches they push out the input vectors, which every strip reads.
// 8 vectors: table of 128256 x 4096 178 -> 155 us (6.8 TB/s), gate/up 41 -> 36.5, down 22.2 -> 20.5; a step of two layers and the head 467 -> 432.
// Models that the 256 MB memory-side cache holds from step to step pay for it, the others gain, and a call sees one product only.  Steps of 8
// vectors, 32000 words, cached -> nt: hidden size 512, 16 layers 598 -> 604 us; 1024, 2 / 8 / 24 layers 95.6 -> 99.4 / 338.7 -> 331.1 /
// 1005 -> 954; 2048, 1 / 2 / 8 layers 75.4 -> 81.5 / 139.1 -> 131.6 / 462.6 -> 440.  By the product's bytes instead (cached below 4, 16 or 32 MB) the
// cached products' weights push out the rest: 1024 x 24 layers 954 (4 MB), 1030 (16), 1030 (32); 2048 x 8 layers 448 (4), 442 (16), 465 (32).
// (8 instead of 16 rows of input vectors in a stage, which makes room for three workgroups per CU or six stages: no faster.)
typedef __bf16 mfma_bf16x8 __attribute__((ext_vector_type(8)));
typedef float mfma_f32x4 __attribute__((ext_vector_type(4)));

constexpr int GEMV_MFMA_WAVES = 4;

constexpr int GEMV_NORM_K = 4096;   // longest norm inside a product: the ring and gamma are 80 KB, two workgroups per CU
// GEMV_QKV_ROPE of several sequences: where the new pairs go, and the rotation's exponent per channel pair
struct GemvRopeBatch { DecodeBatch db; double neg2_over_d_log2base; };
struct GemvNoRope {};
template <int MODE> struct GemvRopeOf { typedef GemvNoRope type; };
template <> struct GemvRopeOf<GEMV_QKV_ROPE> { typedef GemvRopeBatch type; };

// NORM: x is normalised on the way in.  The product that wrote x (GEMV_RESID with ssq) has left the sum of squares of each strip of 16 rows; every workgroup
// adds them up while its ring fills, gamma stands in LDS, and fragments are normalised and rounded as rmsnorm_kernel does it.  (From x itself, which is
// then read twice per strip, gate/up of eight vectors took 45.6 us instead of 41.5: no less than the norm's launch.)
// GEMV_QKV_ROPE: a strip of Q or K has the rows j .. j + 7 and j + d/2 .. j + d/2 + 7 of one head, both members of eight rotary pairs, and the epilogue
// rotates them and writes keys and values into the caches, which was a launch of its own.
// Both are the work of four more wavefronts: one that waits for loads of its own waits for its whole ring.
template <int MODE, bool NORM> constexpr int gemv_mfma_threads() { return GEMV_MFMA_WAVES * (NORM || MODE == GEMV_QKV_ROPE ? 128 : 64); }
template <int MODE, int XI, bool NORM>
__global__ void __launch_bounds__((gemv_mfma_threads<MODE, NORM>()), 2) gemv_mfma_kernel(GemvArgs a, int nb, typename GemvRopeOf<MODE>::type rb) {
    constexpr int NW = GEMV_MFMA_WAVES;
    constexpr bool HELP = NORM || MODE == GEMV_QKV_ROPE;
    constexpr int NS = MODE == GEMV_SILU ? 2 : 1;          // weight strips per workgroup (gate, up)
    constexpr int DEPTH = NS == 2 ? 3 : 4;                 // ring stages per wavefront (64 / 72 KB: two workgroups per CU)
    constexpr int NI = NS * 2 + XI;                        // direct-to-LDS loads per stage
    constexpr uint32_t STRIP_B = 2048, STAGE_B = (NS + 1) * STRIP_B, WAVE_B = DEPTH * STAGE_B;
    static_assert((DEPTH - 1) * NI <= 63, "vmcnt field");
    static_assert(NW * 64 >= 256 && (size_t)NW * WAVE_B >= (size_t)NW * NS * 16 * 17 * 4, "the partial tiles reuse the ring");
    extern __shared__ __attribute__((aligned(16))) char gsm[];
    const int lane = threadIdx.x & 63, wave_ = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), wave = wave_ & (NW - 1);
    const bool helper = HELP && wave_ >= NW;
    const int l16 = lane & 15, kg = lane >> 4;
    int64_t row0 = (int64_t)blockIdx.x * 16;
    int which = 0;
    int64_t upper = 8;                                      // strip row 8 + i is `upper` rows after row i
    const int nstage = a.K / (NW * 64);
    const int64_t kw = (int64_t)wave * nstage * 64;         // first k of this wavefront's contiguous share
    const char* wb[NS];
    if (MODE == GEMV_SILU) {
        wb[0] = (const char*)((const bf16_t*)a.W[0] + row0 * a.K + kw);
        wb[NS - 1] = (const char*)((const bf16_t*)a.W[1] + row0 * a.K + kw);
    } else {
        if (row0 >= a.R[0]) { row0 -= a.R[0]; which = 1; if (row0 >= a.R[1]) { row0 -= a.R[1]; which = 2; } }
        if (MODE == GEMV_QKV_ROPE && which < 2) {
            const int64_t head = row0 / a.head_dim;
            row0 = head * a.head_dim + (row0 - head * a.head_dim) / 2;
            upper = a.head_dim / 2;
        }
        wb[0] = (const char*)((const bf16_t*)a.W[which] + row0 * a.K + kw);
    }
    const char* xb = (const char*)((const bf16_t*)a.x + kw);
    // load lanes: instruction j covers strip rows 8j .. 8j+7, lane -> (row 8j + lane / 8, slot lane % 8)
    uint32_t voff_w[2], voff_x[2];
#pragma unroll
    for (int j = 0; j < 2; ++j) {
        const int r = 8 * j + (lane >> 3), chunk = (lane & 7) ^ (r >> 1);
        const int xr = r < nb ? r : nb - 1;                 // rows beyond the batch: any valid row (their lanes feed zeros)
        voff_w[j] = (uint32_t)(((j * upper + (r & 7)) * a.K + chunk * 8) * 2);
        voff_x[j] = (uint32_t)(((int64_t)xr * a.K + chunk * 8) * 2);
    }
    const uint32_t ring = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) char*)gsm + (uint32_t)wave * WAVE_B;
    auto issue = [&](int st) {                              // stage st -> ring slot st % DEPTH
        const uint32_t slot = ring + (uint32_t)(st % DEPTH) * STAGE_B;
        const int64_t koff = (int64_t)st * 128;
#pragma unroll
        for (int s = 0; s < NS; ++s)
#pragma unroll
            for (int j = 0; j < 2; ++j) dma16s_nt(voff_w[j], wb[s] + koff, slot + s * STRIP_B + j * 1024);
#pragma unroll
        for (int j = 0; j < XI; ++j) dma16s(voff_x[j], xb + koff, slot + NS * STRIP_B + j * 1024);
    };
    const int npre = nstage < DEPTH ? nstage : DEPTH;
    if (!helper)
        for (int st = 0; st < npre; ++st) issue(st);
    // the helpers: 1 / rms of the vectors, gamma; for the epilogue, which is theirs (strip row t / 16, vector t % 16 of their t = 0 .. 255), rotation and cache row
    const int t = (int)threadIdx.x - (HELP ? NW * 64 : 0);
    float cs = 1.f, sn = 0.f, inv = 0.f;
    bf16_t* out = nullptr;
    const bf16_t* const gam = reinterpret_cast<const bf16_t*>(gsm + NW * WAVE_B);   // [K], with NORM
    if constexpr (NORM) {
        float* const sums = reinterpret_cast<float*>(gsm + NW * WAVE_B);   // [NW][16], in gamma's place until everyone has them
        constexpr int GC = GEMV_NORM_K / 8 / (NW * 64);
        u32x4 g[GC];
        if (helper) {
#pragma unroll
            for (int i = 0; i < GC; ++i) g[i] = reinterpret_cast<const u32x4*>(a.gamma)[min(t + i * NW * 64, a.K / 8 - 1)];
            float ss = 0.f;
#pragma unroll 8
            for (int i = t; i < a.K; i += NW * 64) ss += a.ssq[i];   // [K / 16][16]: lane's vector t % 16
            ss += __shfl_xor(ss, 16);
            ss += __shfl_xor(ss, 32);
            if (lane < 16) sums[wave * 16 + lane] = ss;
        }
        __syncthreads();
        float ss = 0.f;
#pragma unroll
        for (int w = 0; w < NW; ++w) ss += sums[w * 16 + l16];
        inv = 1.0f / sqrtf(ss / (float)a.K + a.eps);
        __syncthreads();
        if (helper) {
#pragma unroll
            for (int i = 0; i < GC; ++i)
                if (t + i * NW * 64 < a.K / 8) reinterpret_cast<u32x4*>(gsm + NW * WAVE_B)[t + i * NW * 64] = g[i];
        }
        __syncthreads();
    }
    if constexpr (MODE == GEMV_QKV_ROPE) {
        if (helper) {
            const int er = t >> 4, eb = (t & 15) < nb ? t & 15 : nb - 1;
            if (which < 2) {
                const int j = (int)(row0 % a.head_dim) + (er & 7);
                double dc, ds;
                sincos((double)rb.db.pos[eb] * exp2((double)j * rb.neg2_over_d_log2base), &ds, &dc);
                cs = (float)dc; sn = (float)ds;
            }
            out = which == 0 ? (bf16_t*)a.y[0] + (int64_t)eb * a.R[0] : (bf16_t*)(which == 1 ? rb.db.cache_k[eb] : rb.db.cache_v[eb]) + rb.db.count[eb] * a.R[which];
            if (blockIdx.x == 0 && t < nb) rb.db.cache_pos[t][rb.db.count[t]] = rb.db.pos[t];
        }
    }
    // fragment reads: lane (row l16, k group kg), half h of the stage -> chunk 4h + kg of its row
    const char* myring = gsm + (size_t)wave * WAVE_B;
    uint32_t foff[2];
#pragma unroll
    for (int h = 0; h < 2; ++h) foff[h] = (uint32_t)(l16 * 128 + (((4 * h + kg) ^ (l16 >> 1)) * 16));
    const bool tok = l16 < nb;
    mfma_f32x4 acc[NS];
#pragma unroll
    for (int s = 0; s < NS; ++s) acc[s] = mfma_f32x4{0.f, 0.f, 0.f, 0.f};
    for (int st = 0; st < (helper ? 0 : nstage); ++st) {
        // stages issued so far: min(nstage, st + DEPTH); all but the DEPTH - 1 youngest must have landed
        if (st + DEPTH <= nstage) SPTS_WAIT_VMCNT((DEPTH - 1) * NI); else SPTS_WAIT_VMCNT(0);
        asm volatile("" ::: "memory");
        const char* slot = myring + (size_t)(st % DEPTH) * STAGE_B;
        u32x4 wv[NS][2], xv[2], gv[2];
#pragma unroll
        for (int h = 0; h < 2; ++h) {
#pragma unroll
            for (int s = 0; s < NS; ++s) wv[s][h] = *reinterpret_cast<const u32x4*>(slot + s * STRIP_B + foff[h]);
            xv[h] = *reinterpret_cast<const u32x4*>(slot + NS * STRIP_B + foff[h]);
            if (NORM) gv[h] = *reinterpret_cast<const u32x4*>(gam + kw + st * 64 + (4 * h + kg) * 8);
            if (!NORM && !tok) xv[h] = u32x4{0u, 0u, 0u, 0u};
        }
        // the slot is refilled only after its fragments have arrived in registers
        asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
        if (st + DEPTH < nstage) issue(st + DEPTH);
        if (NORM) {
#pragma unroll
            for (int h = 0; h < 2; ++h)
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    const float x0 = __uint_as_float(xv[h][i] << 16), x1 = __uint_as_float(xv[h][i] & 0xffff0000u);
                    const float g0 = __uint_as_float(gv[h][i] << 16), g1 = __uint_as_float(gv[h][i] & 0xffff0000u);
                    xv[h][i] = tok ? cvt_pk_bf16(x0 * inv * g0, x1 * inv * g1) : 0u;
                }
        }
#pragma unroll
        for (int h = 0; h < 2; ++h)
#pragma unroll
            for (int s = 0; s < NS; ++s)
                acc[s] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(mfma_bf16x8, wv[s][h]),
                                                                 __builtin_bit_cast(mfma_bf16x8, xv[h]), acc[s], 0, 0, 0);
    }
    // every wavefront is done with its ring (nothing in flight: the last stage waited for vmcnt 0); the partial
    // tiles take its place.  Lane (token l16, row group kg) holds rows 4*kg .. 4*kg+3 of its tile.
    __syncthreads();
    float (*sred)[NS][16][17] = reinterpret_cast<float (*)[NS][16][17]>(gsm);
    if (!helper) {
#pragma unroll
        for (int s = 0; s < NS; ++s)
#pragma unroll
            for (int r = 0; r < 4; ++r) sred[wave][s][4 * kg + r][l16] = acc[s][r];
    }
    __syncthreads();
    if (t < 0) return;
    const int r = t >> 4, b = t & 15;
    if (MODE == GEMV_RESID && a.ssq) {   // + the strip's sum of squares of each vector, as stored
        float v = 0.f, y = 0.f;
#pragma unroll
        for (int w = 0; w < NW; ++w) v += sred[w][0][r][b];
        if (b < nb) {
            bf16_t* p = (bf16_t*)a.y[which] + (int64_t)b * a.R[which] + row0 + r;
            const bf16_t s = f32_to_bf16(bf16_to_f32(*p) + v);
            *p = s;
            y = bf16_to_f32(s);
        }
        float ss = y * y;
        ss += __shfl_xor(ss, 16);
        ss += __shfl_xor(ss, 32);
        __syncthreads();
        float* const sums = reinterpret_cast<float*>(gsm);
        if (lane < 16) sums[wave * 16 + lane] = ss;
        __syncthreads();
        if (t < 16) a.ssq[blockIdx.x * 16 + t] = sums[t] + sums[16 + t] + sums[32 + t] + sums[48 + t];
        return;
    }
    if (b >= nb) return;
    float v = 0.f, u = 0.f;
#pragma unroll
    for (int w = 0; w < NW; ++w) { v += sred[w][0][r][b]; if (NS == 2) u += sred[w][NS - 1][r][b]; }
    if constexpr (MODE == GEMV_QKV_ROPE) {
        if (which < 2) {
            float other = 0.f;
#pragma unroll
            for (int w = 0; w < NW; ++w) other += sred[w][0][r ^ 8][b];
            v = r < 8 ? v * cs - other * sn : v * cs + other * sn;
        }
        out[row0 + (r >> 3) * upper + (r & 7)] = f32_to_bf16(v);
    } else if (MODE == GEMV_SILU) {
        ((bf16_t*)a.y[0])[(int64_t)b * a.R[0] + row0 + r] = f32_to_bf16(v / (1.0f + __expf(-v)) * u);
    } else if (MODE == GEMV_RESID) {
        bf16_t* y = (bf16_t*)a.y[which] + (int64_t)b * a.R[which] + row0 + r;
        *y = f32_to_bf16(bf16_to_f32(*y) + v);
    } else {   // GEMV_F32
        ((float*)a.y[which])[(int64_t)b * a.R[which] + row0 + r] = v;
    }
}

static int gemv_mfma_lds(const GemvArgs& a) {   // the ring, and gamma behind it
    const int ns = a.mode == GEMV_SILU ? 2 : 1, depth = ns == 2 ? 3 : 4;
    return GEMV_MFMA_WAVES * depth * (ns + 1) * 2048 + (a.gamma ? a.K * 2 : 0);
}

bool gemv_mfma_supported(const GemvArgs& a, int nb) {
    if (nb < 1 || nb > 16 || a.K <= 0 || a.K % 256 != 0) return false;
    if (a.mode != GEMV_SILU && a.mode != GEMV_RESID && a.mode != GEMV_F32 && a.mode != GEMV_QKV_ROPE) return false;
    if (a.gamma && (a.mode != GEMV_SILU || !a.ssq || a.K > GEMV_NORM_K)) return false;
    if (a.mode == GEMV_QKV_ROPE && (a.head_dim <= 0 || a.head_dim % 16 != 0 || a.R[0] % a.head_dim != 0 || a.R[1] % a.head_dim != 0)) return false;
    for (int i = 0; i < 3; ++i)
        if (a.R[i] < 0 || a.R[i] % 16 != 0) return false;
    // per-lane byte offsets are 32-bit: 16 rows of K elements, or half a head's
    const int64_t rows = a.mode == GEMV_QKV_ROPE && a.head_dim > 16 ? a.head_dim : 16;
    if (rows * a.K * 2 >= ((int64_t)1 << 32)) return false;
    return true;
}

template <int MODE, int XI, bool NORM>
static hipError_t launch_gemv_mfma_t(const GemvArgs& a, int nb, const typename GemvRopeOf<MODE>::type& rb, unsigned grid, hipStream_t s) {
    const hipError_t e = ensure_dynamic_lds(reinterpret_cast<const void*>(&gemv_mfma_kernel<MODE, XI, NORM>), NORM ? 80 * 1024 : gemv_mfma_lds(a));   // (NORM: the longest gamma)
    if (e != hipSuccess) return e;
    gemv_mfma_kernel<MODE, XI, NORM><<<dim3(grid), dim3(gemv_mfma_threads<MODE, NORM>()), gemv_mfma_lds(a), s>>>(a, nb, rb);
    return hipGetLastError();
}

template <int MODE, bool NORM>
static hipError_t launch_gemv_mfma_m(const GemvArgs& a, int nb, const typename GemvRopeOf<MODE>::type& rb, hipStream_t s) {
    const int64_t rows = MODE == GEMV_SILU ? (int64_t)a.R[0] : (int64_t)a.R[0] + a.R[1] + a.R[2];
    if (rows == 0) return hipSuccess;
    const unsigned grid = (unsigned)(rows / 16);
    return nb > 8 ? launch_gemv_mfma_t<MODE, 2, NORM>(a, nb, rb, grid, s) : launch_gemv_mfma_t<MODE, 1, NORM>(a, nb, rb, grid, s);
}

hipError_t launch_gemv_mfma(const GemvArgs& a, int nb, hipStream_t s) {
    if (!gemv_mfma_supported(a, nb)) return hipErrorInvalidValue;
    const GemvNoRope none{};
    switch (a.mode) {
        case GEMV_SILU: return a.gamma ? launch_gemv_mfma_m<GEMV_SILU, true>(a, nb, none, s) : launch_gemv_mfma_m<GEMV_SILU, false>(a, nb, none, s);
        case GEMV_RESID: return launch_gemv_mfma_m<GEMV_RESID, false>(a, nb, none, s);
        case GEMV_F32: return launch_gemv_mfma_m<GEMV_F32, false>(a, nb, none, s);
        default: return hipErrorInvalidValue;
    }
}

hipError_t launch_gemv_qkv_batched(const GemvArgs& a, const DecodeBatch& db, float base, hipStream_t s) {
    if (a.mode != GEMV_QKV_ROPE || db.n < 1 || db.n > DECODE_MAX_BATCH || !gemv_mfma_supported(a, db.n)) return hipErrorInvalidValue;
    const GemvRopeBatch rb{db, -2.0 / (double)a.head_dim * log2((double)base)};
    return launch_gemv_mfma_m<GEMV_QKV_ROPE, false>(a, db.n, rb, s);
}

// nb input vectors (1 <= nb <= 16).  bf16 with tile-friendly shapes runs on the matrix cores; otherwise the
// dot-product kernel, instantiated for 2, 4 and 8 vectors: other counts run as a sum of those (rows of X and Y are
// contiguous, so a group of vectors is the same call on shifted pointers)
hipError_t launch_gemv_nb(const GemvArgs& a, int nb, bool bf16, hipStream_t s) {
    if (nb < 1 || nb > DECODE_MAX_BATCH || a.mode == GEMV_QKV_ROPE) return hipErrorInvalidValue;
    if (bf16 && nb > 1 && gemv_mfma_supported(a, nb)) return launch_gemv_mfma(a, nb, s);
    if (a.gamma) return hipErrorInvalidValue;
    const size_t eb = bf16 ? 2 : 4;
    int done = 0;
    while (done < nb) {
        const int left = nb - done;
        const int take = left >= 8 ? 8 : left >= 4 ? 4 : left >= 2 ? 2 : 1;
        GemvArgs g = a;
        g.x = (const char*)a.x + (size_t)done * a.K * eb;
        for (int i = 0; i < 3; ++i)
            if (a.y[i]) g.y[i] = (char*)a.y[i] + (size_t)done * a.R[i] * (a.mode == GEMV_F32 ? 4 : eb);
        hipError_t e;
        if (take == 1) e = launch_gemv(g, bf16, s);
        else if (bf16) e = take == 8 ? launch_gemv_nb_t<bf16_t, 8>(g, s) : take == 4 ? launch_gemv_nb_t<bf16_t, 4>(g, s) : launch_gemv_nb_t<bf16_t, 2>(g, s);
        else e = take == 8 ? launch_gemv_nb_t<float, 8>(g, s) : take == 4 ? launch_gemv_nb_t<float, 4>(g, s) : launch_gemv_nb_t<float, 2>(g, s);
        if (e != hipSuccess) return e;
        done += take;
    }
    return hipSuccess;
}

// ------------------------------------------------------------------- rotary table of one position
__global__ void decode_rope_row_kernel(int pos, int half, double neg2_over_d_log2base, float2* __restrict__ table) {
    const int j = blockIdx.x * blockDim.x + threadIdx.x;
    if (j >= half) return;
    double sn, cs;
    sincos((double)pos * exp2((double)j * neg2_over_d_log2base), &sn, &cs);
    table[j] = make_float2((float)cs, (float)sn);
}

hipError_t launch_decode_rope_row(int pos, int d, float base, float2* table, hipStream_t s) {
    const int half = d / 2;
    decode_rope_row_kernel<<<dim3((unsigned)((half + 63) / 64)), dim3(64), 0, s>>>(pos, half, -2.0 / (double)d * log2((double)base),
                                                                                 table);
    return hipGetLastError();
}

// ------------------------------------------------------------------- rotary + cache append
// Rotary embedding and cache append for a batch of sequences (blockIdx.y = sequence), from the fp32 sums of the projections: q32 [B, H, d],
// k32 / v32 [B, Hkv, d] -> q [B, H, d] and the new cache rows, rounded to T once, after the rotation (as the
// single-sequence GEMV's epilogue does); every sequence has its own cache, row and position (by-value descriptor: at
// most DECODE_MAX_BATCH sequences)
template <typename T>
__global__ void decode_rope_append_batched_kernel(const float* __restrict__ q32, const float* __restrict__ k32,
                                                  const float* __restrict__ v32, T* __restrict__ q, int H, int Hkv, int d,
                                                  double neg2_over_d_log2base, DecodeBatch db) {
    const int half = d / 2;
    const int b = blockIdx.y;
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    const int pos = db.pos[b];
    const int64_t row = db.count[b];
    if (i == 0) db.cache_pos[b][row] = pos;
    if (i >= (H + Hkv) * half) return;
    const int head = i / half, j = i % half;
    double sn, cs;
    sincos((double)pos * exp2((double)j * neg2_over_d_log2base), &sn, &cs);
    const float c = (float)cs, s = (float)sn;
    if (head < H) {
        const int64_t o = ((int64_t)b * H + head) * d + j;
        const float x0 = q32[o], x1 = q32[o + half];
        q[o] = from_f32<T>(x0 * c - x1 * s);
        q[o + half] = from_f32<T>(x1 * c + x0 * s);
    } else {
        const int g = head - H;
        const int64_t i0 = ((int64_t)b * Hkv + g) * d + j;
        const float x0 = k32[i0], x1 = k32[i0 + half];
        T* o = (T*)db.cache_k[b] + (row * Hkv + g) * (int64_t)d + j;
        o[0] = from_f32<T>(x0 * c - x1 * s);
        o[half] = from_f32<T>(x1 * c + x0 * s);
        T* ov = (T*)db.cache_v[b] + (row * Hkv + g) * (int64_t)d + j;
        ov[0] = from_f32<T>(v32[i0]);
        ov[half] = from_f32<T>(v32[i0 + half]);
    }
}

hipError_t launch_decode_rope_append_batched(const float* q32, const float* k32, const float* v32, void* q, int H, int Hkv, int d,
                                             float base, const DecodeBatch& db, bool bf16, hipStream_t s) {
    if (db.n < 1 || db.n > DECODE_MAX_BATCH) return hipErrorInvalidValue;
    const int n = (H + Hkv) * (d / 2);
    const double kk = -2.0 / (double)d * log2((double)base);
    const dim3 g((unsigned)((n + 255) / 256), (unsigned)db.n), b(256);
    if (bf16)
        decode_rope_append_batched_kernel<bf16_t><<<g, b, 0, s>>>(q32, k32, v32, (bf16_t*)q, H, Hkv, d, kk, db);
    else
        decode_rope_append_batched_kernel<float><<<g, b, 0, s>>>(q32, k32, v32, (float*)q, H, Hkv, d, kk, db);
    return hipGetLastError();
}

// ------------------------------------------------------------------------- decode attention
// partial layout: part[((g * nsplit + split) * GRP_MAX + hg) * (d + 2)] = (max, sum, weighted values[d])
constexpr int GRP_MAX = 8;

// ---- the lanes of a key (LPK of them, each with a piece of the row) and the query heads: every lane owns one of GL heads, number lane % GL
template <int CTRL> __device__ __forceinline__ float dpp(float v) {
    return __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, v), CTRL, 0xF, 0xF, true));
}
constexpr int DPP_XOR1 = 0xB1, DPP_XOR2 = 0x4E, DPP_HALF_MIRROR = 0x141, DPP_ROR4 = 0x124, DPP_ROR8 = 0x128;   // (quad permutes, lane 7 - i of 8, rotations of 16)

// p[h]: this lane's part of head h's sum -> the whole sum of the lane's own head.  As many heads as there are left are halved with the lanes, one
// partner keeping either half, so that all heads together take GL - 1 additions and a few more, not GL log2(LPK).
template <int LPK, int GL>
__device__ __forceinline__ float sum_own_head(float (&p)[GL], int lane) {
    if (GL == 8) {
#pragma unroll
        for (int h = 0; h < GL / 2; ++h) {
            const float keep = lane & 4 ? p[GL / 2 + h] : p[h], send = lane & 4 ? p[h] : p[GL / 2 + h];
            p[h] = keep + dpp<DPP_HALF_MIRROR>(send);
        }
    } else if (LPK == 8) {
#pragma unroll
        for (int h = 0; h < GL; ++h) p[h] += dpp<DPP_HALF_MIRROR>(p[h]);
    }
    if (GL >= 4) {
        constexpr int H2 = GL >= 4 ? 2 : 0;
#pragma unroll
        for (int h = 0; h < H2; ++h) {
            const float keep = lane & 2 ? p[H2 + h] : p[h], send = lane & 2 ? p[h] : p[H2 + h];
            p[h] = keep + dpp<DPP_XOR2>(send);
        }
    }
    if (GL >= 2) {
        constexpr int H1 = GL >= 2 ? 1 : 0;
        const float keep = lane & 1 ? p[H1] : p[0], send = lane & 1 ? p[0] : p[H1];
        p[0] = keep + dpp<DPP_XOR1>(send);
    }
    float v = p[0];
    if (GL == 1 && LPK >= 2) v += dpp<DPP_XOR1>(v);
    if (GL <= 2 && LPK >= 4) v += dpp<DPP_XOR2>(v);
    if (LPK >= 16) {
        v += dpp<DPP_ROR8>(v);
        if (GL < 8) v += dpp<DPP_ROR4>(v);
    }
    if (LPK >= 32) v += __shfl_xor(v, 16);
    return v;
}

// v: a value of the lane's own head -> every head's, in every lane of the key
template <int GL>
__device__ __forceinline__ void all_heads(float v, int lane, float (&out)[GL]) {
    if (GL == 1) out[0] = v;
    if (GL == 2) { out[0] = dpp<0xA0>(v); out[GL / 2] = dpp<0xF5>(v); }   // quad_perm [0,0,2,2], [1,1,3,3]
    if (GL >= 4) {
        const float q[4] = {dpp<0x00>(v), dpp<0x55>(v), dpp<0xAA>(v), dpp<0xFF>(v)};
#pragma unroll
        for (int h = 0; h < 4; ++h) {
            const float other = GL == 8 ? dpp<DPP_HALF_MIRROR>(q[h]) : 0.f;
            out[h & (GL - 1)] = GL == 8 && (lane & 4) ? other : q[h];
            if (GL == 8) out[(4 + h) & (GL - 1)] = lane & 4 ? q[h] : other;
        }
    }
}

// G: query heads per KV head the register arrays are sized for (>= H / Hkv)
// What bounds it besides the caches' bytes is instructions: per key and head a reduction over the key's lanes, a maximum, an exponential and the test for a
// new maximum.  The lanes of a key hold the same sums, so each does that for one head only.
// U: keys that a lane takes at a time (see decode_attn_pairs).
template <typename T, int D, int G, int U>
__device__ __forceinline__ void decode_attn_body(const T* __restrict__ q, const T* __restrict__ K, const T* __restrict__ V,
                                                 int64_t M, int H, int Hkv, float scale_log2e, float* __restrict__ part) {
    constexpr int EPC = 16 / (int)sizeof(T);
    constexpr int LPK = D / EPC;          // lanes that hold one key row
    constexpr int KPW = 64 / LPK;         // keys per wavefront step
    constexpr int GL = G < LPK ? G : LPK, R = G / GL;   // heads that share the lanes, heads per lane
    __shared__ float sm[4][G][2];
    __shared__ float sacc[4][G][D];

    const int split = blockIdx.x, nsplit = gridDim.x, g = blockIdx.y;
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int sub = lane % LPK, kslot = lane / LPK;
    const int grp = H / Hkv;
    const int64_t per = (M + nsplit - 1) / nsplit;
    const int64_t m_begin = (int64_t)split * per;
    const int64_t m_end = m_begin + per < M ? m_begin + per : M;

    // this lane's piece of every query head of the group
    u32x4 qv[G];
#pragma unroll
    for (int hg = 0; hg < G; ++hg) {
        const int h = g * grp + (hg < grp ? hg : 0);
        qv[hg] = *reinterpret_cast<const u32x4*>(q + (int64_t)h * D + sub * EPC);
    }
    float mrun[R], lrun[R], acc[G][EPC];
#pragma unroll
    for (int r = 0; r < R; ++r) { mrun[r] = -INFINITY; lrun[r] = 0.f; }
#pragma unroll
    for (int hg = 0; hg < G; ++hg)
#pragma unroll
        for (int e = 0; e < EPC; ++e) acc[hg][e] = 0.f;

    // keys of this lane: m_begin + wave*KPW + kslot + it * 4*KPW, U of them at a time; the next U are loaded before the
    // current ones are used
    const T* Kg = K + m_begin * Hkv * D + (int64_t)g * D + sub * EPC;
    const T* Vg = V + m_begin * Hkv * D + (int64_t)g * D + sub * EPC;
    const int64_t rstride = (int64_t)Hkv * D;
    const int n = m_begin < m_end ? (int)(m_end - m_begin) : 0;
    u32x4 kn[U], vn[U];
    auto load = [&](int i0) {
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int64_t at = min(i0 + u * 4 * KPW, n - 1) * rstride;
            kn[u] = *reinterpret_cast<const u32x4*>(Kg + at);
            vn[u] = *reinterpret_cast<const u32x4*>(Vg + at);
        }
    };
    if (n > 0) load(wave * KPW + kslot);
    for (int i0 = wave * KPW; i0 < n; i0 += U * 4 * KPW) {
        const int i = i0 + kslot;
        u32x4 kv[U], vv[U];
#pragma unroll
        for (int u = 0; u < U; ++u) { kv[u] = kn[u]; vv[u] = vn[u]; }
        load(i + U * 4 * KPW);
        float s[U][R];
#pragma unroll
        for (int u = 0; u < U; ++u)
#pragma unroll
            for (int r = 0; r < R; ++r) {
                float p[GL];
#pragma unroll
                for (int h = 0; h < GL; ++h) p[h] = r * GL + h < grp ? dot16(kv[u], qv[r * GL + h], 0.f, T{}) : 0.f;
                const float t = sum_own_head<LPK, GL>(p, lane);
                s[u][r] = i + u * 4 * KPW < n ? t * scale_log2e : -INFINITY;
            }
#pragma unroll
        for (int r = 0; r < R; ++r) {
            float mn = mrun[r];
#pragma unroll
            for (int u = 0; u < U; ++u) mn = fmaxf(mn, s[u][r]);
            const float mu = mn == -INFINITY ? 0.f : mn;
            // the running maximum rarely moves after the first keys: rescale only when it did for some lane
            if (__ballot(mn != mrun[r]) != 0) {
                const float alpha = __builtin_amdgcn_exp2f(mrun[r] - mu);
                lrun[r] *= alpha;
                mrun[r] = mn;
                float ah[GL];
                all_heads<GL>(alpha, lane, ah);
#pragma unroll
                for (int h = 0; h < GL; ++h)
#pragma unroll
                    for (int e = 0; e < EPC; ++e) acc[r * GL + h][e] *= ah[h];
            }
#pragma unroll
            for (int u = 0; u < U; ++u) {
                const float p = __builtin_amdgcn_exp2f(s[u][r] - mu);
                lrun[r] += p;
                float ph[GL];
                all_heads<GL>(p, lane, ph);
#pragma unroll
                for (int h = 0; h < GL; ++h)
                    if (r * GL + h < grp) {
#pragma unroll
                        for (int e = 0; e < EPC; ++e) acc[r * GL + h][e] = __builtin_fmaf(ph[h], chunk_elem(vv[u], e, T{}), acc[r * GL + h][e]);
                    }
            }
        }
    }
    // merge the KPW lane groups of the wavefront (lanes with equal `sub`)
#pragma unroll
    for (int r = 0; r < R; ++r) {
#pragma unroll
        for (int off = LPK; off < 64; off <<= 1) {
            const float mo = __shfl_xor(mrun[r], off), lo = __shfl_xor(lrun[r], off);
            const float mn = fmaxf(mrun[r], mo);
            const float mu = mn == -INFINITY ? 0.f : mn;
            const float a0 = __builtin_amdgcn_exp2f(mrun[r] - mu), a1 = __builtin_amdgcn_exp2f(mo - mu);
            lrun[r] = lrun[r] * a0 + lo * a1;
            mrun[r] = mn;
            float h0[GL], h1[GL];
            all_heads<GL>(a0, lane, h0);
            all_heads<GL>(a1, lane, h1);
#pragma unroll
            for (int h = 0; h < GL; ++h)
                if (r * GL + h < grp) {
#pragma unroll
                    for (int e = 0; e < EPC; ++e) acc[r * GL + h][e] = acc[r * GL + h][e] * h0[h] + __shfl_xor(acc[r * GL + h][e], off) * h1[h];
                }
        }
        if (lane < GL) { sm[wave][r * GL + lane][0] = mrun[r]; sm[wave][r * GL + lane][1] = lrun[r]; }
    }
    if (kslot == 0) {
#pragma unroll
        for (int hg = 0; hg < G; ++hg)
            if (hg < grp) {
#pragma unroll
                for (int e = 0; e < EPC; ++e) sacc[wave][hg][sub * EPC + e] = acc[hg][e];
            }
    }
    __syncthreads();
    // merge the 4 wavefronts: thread t < grp * D handles (hg, element)
    for (int t = tid; t < grp * D; t += 256) {
        const int hg = t / D, e = t % D;
        float mn = -INFINITY;
#pragma unroll
        for (int w = 0; w < 4; ++w) mn = fmaxf(mn, sm[w][hg][0]);
        const float mu = mn == -INFINITY ? 0.f : mn;
        float l = 0.f, o = 0.f;
#pragma unroll
        for (int w = 0; w < 4; ++w) {
            const float aw = __builtin_amdgcn_exp2f(sm[w][hg][0] - mu);
            l += sm[w][hg][1] * aw;
            o += sacc[w][hg][e] * aw;
        }
        float* dst = part + (((int64_t)g * nsplit + split) * GRP_MAX + hg) * (D + 2);
        if (e == 0) { dst[0] = mn; dst[1] = l; }
        dst[2 + e] = o;
    }
}

template <typename T, int D, int G, int U>
__global__ void __launch_bounds__(256) decode_attn_kernel(const T* __restrict__ q, const T* __restrict__ K,
                                                          const T* __restrict__ V, int64_t M, int H, int Hkv, float scale_log2e,
                                                          float* __restrict__ part) {
    decode_attn_body<T, D, G, U>(q, K, V, M, H, Hkv, scale_log2e, part);
}
// blockIdx.z = sequence: its query [H, D], its cache (count[b] + 1 pairs: the new pair is already appended) and its
// share of the partial buffer
template <typename T, int D, int G, int U>
__global__ void __launch_bounds__(256) decode_attn_batched_kernel(const T* __restrict__ q, DecodeBatch db, int H, int Hkv,
                                                                  float scale_log2e, float* __restrict__ part, int64_t part_stride) {
    const int b = blockIdx.z;
    decode_attn_body<T, D, G, U>(q + (int64_t)b * H * D, (const T*)db.cache_k[b], (const T*)db.cache_v[b], db.count[b] + 1, H, Hkv,
                              scale_log2e, part + (int64_t)b * part_stride);
}

// out[h, e] = sum over splits of the weighted values / sum of sums.  One workgroup of 1024 threads per
// query head: thread s < 256 takes split s for the (max, sum) part; the weighted values are summed by
// 1024 / D thread groups that each walk a strided subset of the splits with independent loads.
template <typename T>
__global__ void __launch_bounds__(1024) decode_attn_merge_kernel(const float* __restrict__ part, int nsplit, int H, int Hkv, int D,
                                                                 T* __restrict__ out, int64_t part_stride) {
    __shared__ float sa[256];
    __shared__ float sw[16], sl[16];
    __shared__ float so[1024];
    const int h = blockIdx.x, tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int grp = H / Hkv, g = h / grp, hg = h % grp;
    part += (int64_t)blockIdx.y * part_stride;      // blockIdx.y = sequence of a batched step
    out += (int64_t)blockIdx.y * H * D;
    const float* base = part + ((int64_t)g * nsplit * GRP_MAX + hg) * (D + 2);
    const int64_t stride = (int64_t)GRP_MAX * (D + 2);
    const float m = tid < nsplit ? base[tid * stride] : -INFINITY;       // nsplit <= 256: wavefronts 0-3
    const float l = tid < nsplit ? base[tid * stride + 1] : 0.f;
    float mx = m;
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) mx = fmaxf(mx, __shfl_xor(mx, off));
    if (lane == 0) sw[wave] = mx;
    __syncthreads();
    mx = fmaxf(fmaxf(sw[0], sw[1]), fmaxf(sw[2], sw[3]));
    const float mu = mx == -INFINITY ? 0.f : mx;
    const float a = __builtin_amdgcn_exp2f(m - mu);     // 0 for absent or empty splits
    if (tid < 256) sa[tid] = a;
    const float ls = wave_sum(l * a);
    if (lane == 0) sl[wave] = ls;
    __syncthreads();
    const float L = sl[0] + sl[1] + sl[2] + sl[3];
    const int ngroups = 1024 / D, grp_id = tid / D, e = tid % D;
    float o = 0.f;
    if (grp_id < ngroups) {
#pragma unroll 8
        for (int s = grp_id; s < nsplit; s += ngroups) o += base[s * stride + 2 + e] * sa[s];
    }
    so[tid] = o;
    __syncthreads();
    if (tid < D) {
        float t = 0.f;
        for (int k = 0; k < ngroups; ++k) t += so[k * D + tid];
        out[(int64_t)h * D + tid] = from_f32<T>(L > 0.f ? t / L : 0.f);
    }
}

// number of key splits per sequence: two workgroups per CU over the whole launch (measured best on 4.6K-13K cached
// pairs, one sequence: 32 / 64 / 128 / 256 splits of 8 KV heads take 14.6 / 11.7 / 12.8 / 14.3 us; 8 sequences of
// 8.3K pairs: 8 / 16 / 32 / 64 splits take 61 / 62 / 65 / 69 us, 4 splits 89 us), at least 64 keys each, and no
// more than the scratch buffer (scratch_floats, per sequence) holds
int decode_attn_splits(int64_t M, int Hkv, int d, size_t scratch_floats, int nseq) {
    int64_t s = 512 / ((int64_t)(Hkv > 0 ? Hkv : 1) * (nseq > 0 ? nseq : 1));
    if (s > (M + 63) / 64) s = (M + 63) / 64;
    const int64_t cap = (int64_t)(scratch_floats / ((size_t)Hkv * GRP_MAX * (d + 2)));
    if (s > cap) s = cap;
    if (s > 256) s = 256;
    if (s < 1) s = 1;
    return (int)s;
}
// Two keys at a time per lane, four loads in flight instead of two and one test for a new maximum, where a split has keys enough to fill the
// longer pipeline: attention of two layers with 750 keys to a split (8 sequences of 6001 .. 2851 pairs, 16 of 3000 .. 1313) 79.9 -> 68.5 us and 80.6 -> 69.6, with
// 375 (2 of 12000 and 8400) 46.1 -> 48.5, with 205 (one of 13107) 37.0 -> 39.4.  (One head per lane instead of all heads in every lane came to 80.3, 80.4, 51.2 and
// 41.0 -> the first figures.  Three keys: 69.8, 70.6, 50.7, 41.5.)
static bool decode_attn_pairs(int64_t M, int nsplit) { return (M + nsplit - 1) / nsplit >= 512; }
size_t decode_attn_min_scratch_floats(int Hkv, int d) { return (size_t)Hkv * GRP_MAX * (d + 2); }

bool decode_attn_supported(int H, int Hkv, int d, bool bf16) {
    (void)bf16;
    if (Hkv <= 0 || H % Hkv != 0 || H / Hkv > GRP_MAX) return false;
    return d == 16 || d == 32 || d == 64 || d == 128;
}

template <typename T>
static hipError_t launch_decode_attn_t(const T* q, const T* K, const T* V, int64_t M, int H, int Hkv, int d, float* part,
                                       size_t part_floats, T* out, hipStream_t s) {
    const int nsplit = decode_attn_splits(M, Hkv, d, part_floats, 1);
    const float scale_log2e = 1.4426950408889634f / sqrtf((float)d);
    const dim3 g((unsigned)nsplit, (unsigned)Hkv), b(256);
    const int grp = H / Hkv;
    const bool two = decode_attn_pairs(M, nsplit);
#define SPTS_DEC_ATTN_U(D_, G_)                                                                             \
    if (two) decode_attn_kernel<T, D_, G_, 2><<<g, b, 0, s>>>(q, K, V, M, H, Hkv, scale_log2e, part);       \
    else decode_attn_kernel<T, D_, G_, 1><<<g, b, 0, s>>>(q, K, V, M, H, Hkv, scale_log2e, part);
#define SPTS_DEC_ATTN(D_)                                                                                   \
    if (grp <= 1) { SPTS_DEC_ATTN_U(D_, 1) }                                                                \
    else if (grp <= 2) { SPTS_DEC_ATTN_U(D_, 2) }                                                           \
    else if (grp <= 4) { SPTS_DEC_ATTN_U(D_, 4) }                                                           \
    else { SPTS_DEC_ATTN_U(D_, GRP_MAX) }
    switch (d) {
        case 128: SPTS_DEC_ATTN(128) break;
        case 64: SPTS_DEC_ATTN(64) break;
        case 32: SPTS_DEC_ATTN(32) break;
        case 16: SPTS_DEC_ATTN(16) break;
        default: return hipErrorInvalidValue;
    }
#undef SPTS_DEC_ATTN
#undef SPTS_DEC_ATTN_U
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    decode_attn_merge_kernel<T><<<dim3((unsigned)H), dim3(1024), 0, s>>>(part, nsplit, H, Hkv, d, out, 0);
    return hipGetLastError();
}

hipError_t launch_decode_attn(const void* q, const void* K, const void* V, int64_t M, int H, int Hkv, int d, float* part,
                              size_t part_floats, void* out, bool bf16, hipStream_t s) {
    if (M <= 0 || part_floats < decode_attn_min_scratch_floats(Hkv, d)) return hipErrorInvalidValue;
    if (bf16)
        return launch_decode_attn_t<bf16_t>((const bf16_t*)q, (const bf16_t*)K, (const bf16_t*)V, M, H, Hkv, d, part, part_floats,
                                            (bf16_t*)out, s);
    return launch_decode_attn_t<float>((const float*)q, (const float*)K, (const float*)V, M, H, Hkv, d, part, part_floats, (float*)out, s);
}

// the same for a batch of sequences in one launch (grid z = sequence); every sequence takes the same number of
// splits, chosen for the longest cache; out [B, H, d]
template <typename T>
static hipError_t launch_decode_attn_batched_t(const T* q, const DecodeBatch& db, int H, int Hkv, int d, float* part,
                                               size_t part_floats, T* out, hipStream_t s) {
    int64_t mmax = 1;
    for (int b = 0; b < db.n; ++b) mmax = db.count[b] + 1 > mmax ? db.count[b] + 1 : mmax;
    const int nsplit = decode_attn_splits(mmax, Hkv, d, part_floats / (size_t)db.n, db.n);
    const int64_t stride = (int64_t)Hkv * nsplit * GRP_MAX * (d + 2);
    const float scale_log2e = 1.4426950408889634f / sqrtf((float)d);
    const dim3 g((unsigned)nsplit, (unsigned)Hkv, (unsigned)db.n), b(256);
    const int grp = H / Hkv;
    const bool two = decode_attn_pairs(mmax, nsplit);
#define SPTS_DEC_ATTN_BU(D_, G_)                                                                                          \
    if (two) decode_attn_batched_kernel<T, D_, G_, 2><<<g, b, 0, s>>>(q, db, H, Hkv, scale_log2e, part, stride);          \
    else decode_attn_batched_kernel<T, D_, G_, 1><<<g, b, 0, s>>>(q, db, H, Hkv, scale_log2e, part, stride);
#define SPTS_DEC_ATTN_B(D_)                                                                                               \
    if (grp <= 1) { SPTS_DEC_ATTN_BU(D_, 1) }                                                                             \
    else if (grp <= 2) { SPTS_DEC_ATTN_BU(D_, 2) }                                                                        \
    else if (grp <= 4) { SPTS_DEC_ATTN_BU(D_, 4) }                                                                        \
    else { SPTS_DEC_ATTN_BU(D_, GRP_MAX) }
    switch (d) {
        case 128: SPTS_DEC_ATTN_B(128) break;
        case 64: SPTS_DEC_ATTN_B(64) break;
        case 32: SPTS_DEC_ATTN_B(32) break;
        case 16: SPTS_DEC_ATTN_B(16) break;
        default: return hipErrorInvalidValue;
    }
#undef SPTS_DEC_ATTN_B
#undef SPTS_DEC_ATTN_BU
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    decode_attn_merge_kernel<T><<<dim3((unsigned)H, (unsigned)db.n), dim3(1024), 0, s>>>(part, nsplit, H, Hkv, d, out, stride);
    return hipGetLastError();
}

hipError_t launch_decode_attn_batched(const void* q, const DecodeBatch& db, int H, int Hkv, int d, float* part, size_t part_floats,
                                      void* out, bool bf16, hipStream_t s) {
    if (db.n < 1 || db.n > DECODE_MAX_BATCH || part_floats / (size_t)db.n < decode_attn_min_scratch_floats(Hkv, d)) return hipErrorInvalidValue;
    if (bf16) return launch_decode_attn_batched_t<bf16_t>((const bf16_t*)q, db, H, Hkv, d, part, part_floats, (bf16_t*)out, s);
    return launch_decode_attn_batched_t<float>((const float*)q, db, H, Hkv, d, part, part_floats, (float*)out, s);
}

// ------------------------------------------------------------------------------ greedy head
// token[b] = argmax of logits row b [V], ties to the lowest id; x_next[b] = table[token[b]].  Two launches for the whole
// batch: ARGMAX_PARTS workgroups per row leave the (value, id) of their share, then one workgroup per row picks among
// those and copies the table row.  Bound: launch latency (a row is 0.5 MB).  One workgroup per row is limited by the loads
// one CU keeps in flight: 60 us + 4.5 us for the row copy at V = 128256, row after row (520 of the 990 us of a two-layer
// step over 8 sequences); now about 10 us for 1 and for 8 sequences (that step: 962 -> 468 us, one sequence 405 -> 363).
struct ArgBest { float v; int i; };
__device__ inline ArgBest better(ArgBest a, ArgBest b) { return (b.v > a.v || (b.v == a.v && b.i < a.i)) ? b : a; }
__device__ inline ArgBest wave_best(ArgBest a) {
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) a = better(a, ArgBest{__shfl_xor(a.v, off), __shfl_xor(a.i, off)});
    return a;
}

__global__ void __launch_bounds__(256) argmax_part_kernel(const float* __restrict__ logits, int V, ArgBest* __restrict__ part) {
    __shared__ ArgBest sb[4];
    const float* row = logits + (int64_t)blockIdx.y * V;
    const int quads = V / 4, per = (quads + (int)gridDim.x - 1) / (int)gridDim.x;      // V % 4 == 0, rows 16-byte aligned
    const int q0 = (int)blockIdx.x * per, q1 = q0 + per < quads ? q0 + per : quads;
    ArgBest best{-INFINITY, 0x7fffffff};
#pragma unroll 4
    for (int q = q0 + (int)threadIdx.x; q < q1; q += 256) {
        const f32x4 v = *reinterpret_cast<const f32x4*>(row + (int64_t)q * 4);
#pragma unroll
        for (int e = 0; e < 4; ++e) best = better(best, ArgBest{v[e], q * 4 + e});
    }
    best = wave_best(best);
    if ((threadIdx.x & 63) == 0) sb[threadIdx.x >> 6] = best;
    __syncthreads();
    if (threadIdx.x == 0) part[blockIdx.y * ARGMAX_PARTS + blockIdx.x] = better(better(sb[0], sb[1]), better(sb[2], sb[3]));
}

template <typename T>
__global__ void __launch_bounds__(1024) argmax_pick_kernel(const ArgBest* __restrict__ part, int nparts, int32_t* __restrict__ token,
                                                           const T* __restrict__ table, int D, T* __restrict__ x_next) {
    __shared__ int stok;
    const int b = blockIdx.x;
    if (threadIdx.x < 64) {
        ArgBest best{-INFINITY, 0x7fffffff};
        if ((int)threadIdx.x < nparts) best = part[b * ARGMAX_PARTS + threadIdx.x];
        best = wave_best(best);
        if (threadIdx.x == 0) {
            stok = best.i == 0x7fffffff ? 0 : best.i;   // nothing compares above -inf (NaN logits): id 0
            token[b] = stok;
        }
    }
    if (!x_next) return;
    __syncthreads();
    const T* src = table + (int64_t)stok * D;
    for (int i = threadIdx.x; i < D; i += 1024) x_next[(int64_t)b * D + i] = src[i];
}

hipError_t launch_argmax_rows(const float* logits, int V, int nrows, int32_t* token, const void* table, int D, void* x_next, bool bf16,
                              void* scratch, hipStream_t s) {
    static_assert(sizeof(ArgBest) * ARGMAX_PARTS * DECODE_MAX_BATCH <= ARGMAX_SCRATCH_BYTES && ARGMAX_PARTS <= 64, "argmax scratch");
    if (nrows < 1 || nrows > DECODE_MAX_BATCH || V % 4 != 0) return hipErrorInvalidValue;
    ArgBest* part = (ArgBest*)scratch;
    int nparts = (V / 4 + 255) / 256;
    if (nparts > ARGMAX_PARTS) nparts = ARGMAX_PARTS;
    argmax_part_kernel<<<dim3((unsigned)nparts, (unsigned)nrows), dim3(256), 0, s>>>(logits, V, part);
    if (bf16) argmax_pick_kernel<bf16_t><<<dim3((unsigned)nrows), dim3(1024), 0, s>>>(part, nparts, token, (const bf16_t*)table, D, (bf16_t*)x_next);
    else argmax_pick_kernel<float><<<dim3((unsigned)nrows), dim3(1024), 0, s>>>(part, nparts, token, (const float*)table, D, (float*)x_next);
    return hipGetLastError();
}

}  // namespace spts
