// Causal GQA attention and PAP probe scoring with fp32 arithmetic, any even head dimension up to 256: the fp32 configuration
// and the head dimensions / types the bf16 matrix-core kernels do not take.
//
// All products run on the fp32 matrix instruction v_mfma_f32_32x32x2_f32 (fp32 products and sums; bf16 inputs are widened).
// What bounds these kernels at the fp32 configuration's sizes (256-2048 rows, d = 64) is the latency of dependent loads, so
// operand fragments come straight from global memory, a lane's whole row piece at once (element j of a lane's 4-element
// piece is the operand of product j: which k an instruction multiplies is free as long as both operands agree), and the
// wavefronts of a workgroup split the keys (attention, statistics) or the probe rows (scores) and meet in LDS, all at once (the
// attention's one after the other: 24.3 us for 256 queries over 512 keys, 53.0 for 750 over 1500; now 21.0 and 47.2).
// Measured at N = 512, 4 heads, d = 64: attention of 256 queries 50 -> 21 us against one wavefront per query row; probe of 32
// rows 1001 -> 22 us (two launches) against one lane per candidate that walked all P * H rows.  Dense fp32 layers of 6000 rows (D = 512,
// H d = 512, Dff = 512), 7-9 ms with those: d = 16 1.61 ms, 32 1.01, 64 0.95, 128 1.30, 256 1.52; the attention in them 1231, 634, 578, 925 and 1127 us.
#include "spts_internal.h"

namespace spts {

typedef float f32x16 __attribute__((ext_vector_type(16)));
typedef float f32x4 __attribute__((ext_vector_type(4)));

// Wavefronts per workgroup: eight up to d = 64, four beyond (up to 512 registers each).  At d = 64 the attention then keeps 3 registers in
// scratch memory and reloads them in the key loop; four wavefronts without spills are slower (attention of 256 queries over 512 keys
// 23.9 -> 26.6 us, dense layer of 6000 rows 1.21 -> 1.41 ms).  At d = 256 a lane's row pieces exceed 512 registers: 1.3 KB of scratch per lane
// in the attention, 0.45 KB in the two probe kernels (the attention's 134 KB of LDS cost nothing: registers allow one workgroup per CU).
template <int D> constexpr int f32_waves() { return D <= 64 ? 8 : 4; }
constexpr float LOG2E = 1.4426950408889634f;

// elements c .. c+3 of a row of d elements as fp32, zeros past its end; d4: d % 4 == 0 (the piece is then one aligned load).  Loads
// are unconditional from clamped places and the zeros selected afterwards: a load under a lane mask is a branch of its own, and a
// row's loads then wait for one another (attention of 256 queries over 512 keys: 35 us with masked loads).
__device__ inline f32x4 load4(const float* row, int c, int d, bool d4) {
    f32x4 v;
    if (d4) {
        v = *reinterpret_cast<const f32x4*>(row + (c < d ? c : d - 4));
    } else {
#pragma unroll
        for (int e = 0; e < 4; ++e) v[e] = row[c + e < d ? c + e : d - 1];
    }
#pragma unroll
    for (int e = 0; e < 4; ++e) v[e] = c + e < d ? v[e] : 0.f;
    return v;
}
__device__ inline f32x4 load4(const bf16_t* row, int c, int d, bool d4) {
    f32x4 v;
    if (d4) {
        const u32x2 w = *reinterpret_cast<const u32x2*>(row + (c < d ? c : d - 4));
        v = f32x4{__uint_as_float(w[0] << 16), __uint_as_float(w[0] & 0xffff0000u), __uint_as_float(w[1] << 16), __uint_as_float(w[1] & 0xffff0000u)};
    } else {
#pragma unroll
        for (int e = 0; e < 4; ++e) v[e] = bf16_to_f32(row[c + e < d ? c + e : d - 1]);
    }
#pragma unroll
    for (int e = 0; e < 4; ++e) v[e] = c + e < d ? v[e] : 0.f;
    return v;
}

// acc += a b^T over the 32-row operands whose row pieces (8 s + 4 lh ..) are in fa / fb
template <int NS>
__device__ inline f32x16 mma_rows(const f32x4 (&fa)[NS], const f32x4 (&fb)[NS]) {
    f32x16 s = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int t = 0; t < NS; ++t)
#pragma unroll
        for (int j = 0; j < 4; ++j) s = __builtin_amdgcn_mfma_f32_32x32x2f32(fa[t][j], fb[t][j], s, 0, 0, 0);
    return s;
}
// row (or key) inside a 32-block that accumulator register r of lane half lh holds
__device__ inline int acc_row(int r, int lh) { return 8 * (r >> 2) + 4 * lh + (r & 3); }

// ---------------------------------------------------------------- attention
// Workgroup = 32 queries of one head.  A wavefront takes every GW-th block of 32 keys: S^T = K Q^T (one query per lane column:
// the softmax is in-lane), online softmax, O^T += V^T P^T with the probabilities as they left the first product.  D: head
// dimension rounded up to 32 / 64 / 128 / 256.
template <typename T, int D>
__global__ void __launch_bounds__(64 * f32_waves<D>()) attention_f32_kernel(AttnArgs a) {
    constexpr int NS = D / 8, DB = D / 32, GW = f32_waves<D>();
    __shared__ float sm[GW][32], sl[GW][32];
    __shared__ __attribute__((aligned(16))) float so[GW][32][D + 4];
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int l32 = lane & 31, lh = lane >> 5;
    const int h = blockIdx.y, g = h / (a.H / a.Hkv), d = a.d;
    const int64_t q0 = (int64_t)(gridDim.x - 1 - blockIdx.x) * 32;   // longest causal ranges first
    const bool d4 = d % 4 == 0;
    const float scale = LOG2E / sqrtf((float)d) / (a.q_scale != 0.f ? a.q_scale : 1.0f);   // q may arrive pre-scaled
    const int64_t qi = q0 + l32 < a.Mq ? q0 + l32 : a.Mq - 1;
    const int qp = a.qpos[qi];
    const int qp_last = a.qpos[(q0 + 32 < a.Mq ? q0 + 32 : a.Mq) - 1];
    const T* K = (const T*)a.k + (int64_t)g * d;
    const T* V = (const T*)a.v + (int64_t)g * d;
    const int64_t rstride = (int64_t)a.Hkv * d;
    f32x4 qf[NS];
    {
        const T* qr = (const T*)a.q + (qi * a.H + h) * (int64_t)d;
#pragma unroll
        for (int t = 0; t < NS; ++t) qf[t] = load4(qr, 8 * t + 4 * lh, d, d4);
    }
    float m = -INFINITY, l = 0.f;
    f32x16 o[DB];
#pragma unroll
    for (int db = 0; db < DB; ++db)
#pragma unroll
        for (int r = 0; r < 16; ++r) o[db][r] = 0.f;

    // The block's loads go out beside the one that says whether it is visible at all, where they leave registers: beyond d = 64 that costs more
    // spills (d = 256) and a worse schedule than the wait (attention of 6000 rows, d = 16 / 64 / 128 / 256, waiting and not: 1282 -> 1230, 626 -> 580,
    // 924 -> 931, 1145 -> 2180 us).
    constexpr bool LOAD_FIRST = D <= 64;
    for (int64_t j0 = wave * 32; j0 < a.Mk; j0 += 32 * GW) {
        const int first = a.kpos[j0];
        if (!LOAD_FIRST && first > qp_last) break;   // ascending positions: nothing visible from here on
        const int64_t jk = j0 + l32 < a.Mk ? j0 + l32 : a.Mk - 1;
        f32x4 kf[NS];
#pragma unroll
        for (int t = 0; t < NS; ++t) kf[t] = load4(K + jk * rstride, 8 * t + 4 * lh, d, d4);
        int kp[16];
#pragma unroll
        for (int r = 0; r < 16; ++r) {
            const int64_t j = j0 + acc_row(r, lh);
            kp[r] = a.kpos[j < a.Mk ? j : a.Mk - 1];
        }
        if (LOAD_FIRST && first > qp_last) break;
        const f32x16 s = mma_rows<NS>(kf, qf);
        float p[16], mx = m;
#pragma unroll
        for (int r = 0; r < 16; ++r) {
            p[r] = j0 + acc_row(r, lh) < a.Mk && kp[r] <= qp ? s[r] * scale : -INFINITY;
            mx = fmaxf(mx, p[r]);
        }
        mx = fmaxf(mx, __shfl_xor(mx, 32));
        const float mu = mx == -INFINITY ? 0.f : mx;   // none of the query's keys seen yet
        const float alpha = __builtin_amdgcn_exp2f(m - mu);
        m = mx;
        l *= alpha;
#pragma unroll
        for (int r = 0; r < 16; ++r) { p[r] = __builtin_amdgcn_exp2f(p[r] - mu); l += p[r]; }
#pragma unroll
        for (int db = 0; db < DB; ++db) {
            const int c = db * 32 + l32;
            float vv[16];
#pragma unroll
            for (int r = 0; r < 16; ++r) {
                int64_t j = j0 + acc_row(r, lh);
                if (j >= a.Mk) j = a.Mk - 1;   // its probability is zero
                vv[r] = to_f32(V[j * rstride + (c < d ? c : d - 1)]);
            }
#pragma unroll
            for (int t = 0; t < 16; ++t) o[db][t] *= alpha;
#pragma unroll
            for (int r = 0; r < 16; ++r) o[db] = __builtin_amdgcn_mfma_f32_32x32x2f32(c < d ? vv[r] : 0.f, p[r], o[db], 0, 0, 0);
        }
    }
    l += __shfl_xor(l, 32);
    if (lh == 0) { sm[wave][l32] = m; sl[wave][l32] = l; }
    __syncthreads();
    float mg = -INFINITY, lg = 0.f;
#pragma unroll
    for (int w = 0; w < GW; ++w) mg = fmaxf(mg, sm[w][l32]);
    const float mu = mg == -INFINITY ? 0.f : mg;
#pragma unroll
    for (int w = 0; w < GW; ++w) lg += sl[w][l32] * __builtin_amdgcn_exp2f(sm[w][l32] - mu);
    const float f = __builtin_amdgcn_exp2f(m - mu) * (lg > 0.f ? 1.0f / lg : 0.f);
#pragma unroll
    for (int db = 0; db < DB; ++db)
#pragma unroll
        for (int q = 0; q < 4; ++q)
            *reinterpret_cast<f32x4*>(&so[wave][l32][db * 32 + 8 * q + 4 * lh]) = f32x4{o[db][4 * q] * f, o[db][4 * q + 1] * f, o[db][4 * q + 2] * f, o[db][4 * q + 3] * f};
    __syncthreads();
    for (int t = tid; t < 32 * d; t += 64 * GW) {
        const int r = t / d, c = t - r * d;
        float v = so[0][r][c];
#pragma unroll
        for (int w = 1; w < GW; ++w) v += so[w][r][c];   // fixed order
        if (q0 + r < a.Mq) ((T*)a.out)[((q0 + r) * a.H + h) * (int64_t)d + c] = from_f32<T>(v);
    }
}

template <typename T>
static void launch_attention_f32_t(const AttnArgs& a, hipStream_t s) {
    const dim3 grid((unsigned)((a.Mq + 31) / 32), (unsigned)a.H);
    if (a.d <= 32) attention_f32_kernel<T, 32><<<grid, dim3(64 * f32_waves<32>()), 0, s>>>(a);
    else if (a.d <= 64) attention_f32_kernel<T, 64><<<grid, dim3(64 * f32_waves<64>()), 0, s>>>(a);
    else if (a.d <= 128) attention_f32_kernel<T, 128><<<grid, dim3(64 * f32_waves<128>()), 0, s>>>(a);
    else attention_f32_kernel<T, 256><<<grid, dim3(64 * f32_waves<256>()), 0, s>>>(a);
}

hipError_t launch_attention_generic(const AttnArgs& a, bool bf16, hipStream_t s) {
    if (a.Mq == 0) return hipSuccess;
    if (a.d > 256) return hipErrorInvalidValue;
    if (bf16) launch_attention_f32_t<bf16_t>(a, s); else launch_attention_f32_t<float>(a, s);
    return hipGetLastError();
}

// ---------------------------------------------------------------- probe (Eq. (mha_importance))
// Probe row rr = p * grp + hg of kv head g <-> qp[p, g * grp + hg, :]; window row p sees candidates 0 .. N - P + p.
// Pass 1: a workgroup takes 32 probe rows of one kv head and all candidates (its wavefronts every GW-th block of 32), leaving
// the rows' maximum (log2 units) and 1 / sum of exponentials.
template <typename T, int D>
__global__ void __launch_bounds__(64 * f32_waves<D>()) probe_stats_f32_kernel(ProbeArgs a) {
    constexpr int NS = D / 8, GW = f32_waves<D>();
    __shared__ float sm[GW][32], sl[GW][32];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int l32 = lane & 31, lh = lane >> 5;
    const int grp = a.H / a.Hkv, g = blockIdx.y, R = a.P * grp, d = a.d;
    const int rr = blockIdx.x * 32 + l32, rc = rr < R ? rr : R - 1;
    const bool d4 = d % 4 == 0;
    const float scale = LOG2E / sqrtf((float)d) / (a.q_scale != 0.f ? a.q_scale : 1.0f);
    const int64_t last = a.N - a.P + rc / grp;   // last candidate the lane's row sees
    const int64_t rstride = (int64_t)a.Hkv * d;
    f32x4 qf[NS];
    {
        const T* qr = (const T*)a.qp + ((int64_t)(rc / grp) * a.H + g * grp + rc % grp) * d;
#pragma unroll
        for (int t = 0; t < NS; ++t) qf[t] = load4(qr, 8 * t + 4 * lh, d, d4);
    }
    float m = -INFINITY, l = 0.f;
    for (int64_t n0 = wave * 32; n0 < a.N; n0 += 32 * GW) {
        const int64_t nk = n0 + l32 < a.N ? n0 + l32 : a.N - 1;
        const T* kr = (const T*)a.k + nk * rstride + (int64_t)g * d;
        f32x4 kf[NS];
#pragma unroll
        for (int t = 0; t < NS; ++t) kf[t] = load4(kr, 8 * t + 4 * lh, d, d4);
        const f32x16 s = mma_rows<NS>(kf, qf);
        float v[16], mx = m;
#pragma unroll
        for (int r = 0; r < 16; ++r) { v[r] = n0 + acc_row(r, lh) <= last ? s[r] * scale : -INFINITY; mx = fmaxf(mx, v[r]); }
        mx = fmaxf(mx, __shfl_xor(mx, 32));
        const float mu = mx == -INFINITY ? 0.f : mx;
        l *= __builtin_amdgcn_exp2f(m - mu);
        m = mx;
#pragma unroll
        for (int r = 0; r < 16; ++r) l += __builtin_amdgcn_exp2f(v[r] - mu);
    }
    l += __shfl_xor(l, 32);
    if (lh == 0) { sm[wave][l32] = m; sl[wave][l32] = l; }
    __syncthreads();
    if (threadIdx.x < 32 && rr < R) {
        float mg = -INFINITY, lg = 0.f;
#pragma unroll
        for (int w = 0; w < GW; ++w) mg = fmaxf(mg, sm[w][l32]);
#pragma unroll
        for (int w = 0; w < GW; ++w) lg += sl[w][l32] * __builtin_amdgcn_exp2f(sm[w][l32] - mg);   // a row sees at least one candidate
        float* st = a.stats + ((int64_t)g * R + rr) * 2;
        st[0] = mg;
        st[1] = 1.0f / lg;
    }
}

// Pass 2: a workgroup takes 32 candidates, its wavefronts every GW-th (kv head, 32 probe rows): S = Q K^T (one candidate per lane
// column: the sum over rows is in-lane), fixed order of all sums.
template <typename T, int D>
__global__ void __launch_bounds__(64 * f32_waves<D>()) probe_scores_f32_kernel(ProbeArgs a) {
    constexpr int NS = D / 8, GW = f32_waves<D>();
    __shared__ float ss[GW][32];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int l32 = lane & 31, lh = lane >> 5;
    const int grp = a.H / a.Hkv, R = a.P * grp, nrb = (R + 31) / 32, d = a.d;
    const bool d4 = d % 4 == 0;
    const float scale = LOG2E / sqrtf((float)d) / (a.q_scale != 0.f ? a.q_scale : 1.0f);
    const int64_t n = (int64_t)blockIdx.x * 32 + l32, nc = n < a.N ? n : a.N - 1;
    float acc = 0.f;
    for (int item = wave; item < a.Hkv * nrb; item += GW) {
        const int g = item / nrb, r0 = (item % nrb) * 32;
        const int rc = r0 + l32 < R ? r0 + l32 : R - 1;
        const T* qr = (const T*)a.qp + ((int64_t)(rc / grp) * a.H + g * grp + rc % grp) * d;
        const T* kr = (const T*)a.k + (nc * a.Hkv + g) * (int64_t)d;
        f32x4 qf[NS], kf[NS];
#pragma unroll
        for (int t = 0; t < NS; ++t) { qf[t] = load4(qr, 8 * t + 4 * lh, d, d4); kf[t] = load4(kr, 8 * t + 4 * lh, d, d4); }
        float2 st[16];
#pragma unroll
        for (int r = 0; r < 16; ++r) {
            const int rr = r0 + acc_row(r, lh);
            st[r] = *reinterpret_cast<const float2*>(a.stats + ((int64_t)g * R + (rr < R ? rr : R - 1)) * 2);
        }
        const f32x16 s = mma_rows<NS>(qf, kf);
#pragma unroll
        for (int r = 0; r < 16; ++r) {
            const int rr = r0 + acc_row(r, lh);
            if (rr < R && n <= a.N - a.P + rr / grp) acc += __builtin_amdgcn_exp2f(s[r] * scale - st[r].x) * st[r].y;
        }
    }
    acc += __shfl_xor(acc, 32);
    if (lh == 0) ss[wave][l32] = acc;
    __syncthreads();
    if (threadIdx.x < 32 && n < a.N) {
        float t = 0.f;
#pragma unroll
        for (int w = 0; w < GW; ++w) t += ss[w][l32];
        a.S[n] = t / (float)(a.P * a.H);
    }
}

template <typename T, int D>
static void launch_probe_f32_t(const ProbeArgs& a, hipStream_t s) {
    const int R = a.P * (a.H / a.Hkv);
    probe_stats_f32_kernel<T, D><<<dim3((unsigned)((R + 31) / 32), (unsigned)a.Hkv), dim3(64 * f32_waves<D>()), 0, s>>>(a);
    probe_scores_f32_kernel<T, D><<<dim3((unsigned)((a.N + 31) / 32)), dim3(64 * f32_waves<D>()), 0, s>>>(a);
}
template <typename T>
static void launch_probe_f32_d(const ProbeArgs& a, hipStream_t s) {
    if (a.d <= 32) launch_probe_f32_t<T, 32>(a, s);
    else if (a.d <= 64) launch_probe_f32_t<T, 64>(a, s);
    else if (a.d <= 128) launch_probe_f32_t<T, 128>(a, s);
    else launch_probe_f32_t<T, 256>(a, s);
}

hipError_t launch_probe_generic(const ProbeArgs& a, bool bf16, hipStream_t s) {
    if (a.N == 0) return hipSuccess;
    if (a.d > 256) return hipErrorInvalidValue;
    if (bf16) launch_probe_f32_d<bf16_t>(a, s); else launch_probe_f32_d<float>(a, s);
    return hipGetLastError();
}

}  // namespace spts
