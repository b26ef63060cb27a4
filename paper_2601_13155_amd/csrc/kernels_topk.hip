// TopK(S, k): the k largest scores under (score descending, index ascending), written in ascending
// index order (Sec. 3.2 TopK; Eq. (ffn_selection); Eq. (stage_prune)).
//
// Design for gfx950: N <= 2^17..2^20 fp32 scores are 0.5-4 MB, i.e. L2-resident and latency-bound, so
// one workgroup of 1024 lanes (16 wavefronts) owns the whole problem and never leaves the CU:
//   1. MSB-first radix select on order-preserving 32-bit keys, 4 passes of 8 bits, with a 256-bin
//      LDS histogram per pass (integer LDS atomics: order-independent, hence deterministic) -> the
//      exact key T of the k-th largest element, the number of keys above it, and how many keys equal
//      to T are still needed (those are taken lowest index first: the tie rule).
//      Scores of one layer are probabilities of similar magnitude, so almost all keys share their
//      top bits and fall into one or two bins: lanes whose bin equals that of the wavefront's first
//      active lane are counted with one ballot and a single atomic instead of 64 serialised ones.
//   2. Ordered stream compaction without a per-chunk workgroup barrier: every wavefront owns one
//      contiguous slice; a first sweep counts its (greater, equal) elements with ballots, a 16-entry
//      LDS prefix gives each wavefront its output offsets, a second sweep ranks every element inside
//      the wavefront with ballot + mbcnt (lane prefix popcount) and writes
//      out[gt_before + min(eq_before, need_eq)].
// Up to 32768 scores the keys are read once and stay in registers (KPT per lane, wavefront w holding
// the contiguous slice [64*KPT*w, 64*KPT*(w+1))), and the threshold is found by halving the range of keys
// (topk_reg_kernel); longer inputs re-read the scores in every sweep.
// Shortcut for step 1 (long-row kernels): one pass builds an 8192-bin histogram
// of the top 13 key bits, the keys of the bin that holds the k-th largest go to LDS and the remaining
// 19 bits are resolved there; the four 8-bit passes over all keys remain as the route for rows whose
// threshold bin does not fit (heavily tied scores).  Both routes yield the same exact threshold.
#include "spts_internal.h"

#include <mutex>

namespace spts {

constexpr int TOPK_THREADS = 1024;
constexpr int TOPK_WAVES = TOPK_THREADS / 64;

__device__ inline uint32_t order_key(float f) {
    f = f + 0.0f;  // -0.0 -> +0.0
    uint32_t u = __float_as_uint(f);
    return (u & 0x80000000u) ? ~u : (u | 0x80000000u);
}

__device__ inline uint32_t load_key(const float* __restrict__ s, int64_t i, int64_t N, int protect_last) {
    uint32_t key = order_key(s[i]);
    if (protect_last && i == N - 1) key = 0xFFFFFFFFu;
    return key;
}

__device__ inline int lane_prefix_popc(uint64_t mask) {
    // number of set bits below this lane
    return __builtin_amdgcn_mbcnt_hi((uint32_t)(mask >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)mask, 0));
}

// hist[bin] += 1 for every active lane.  Lanes that share the bin of the first active lane are
// counted by that lane alone (one atomic for the whole group); the others add for themselves.
__device__ inline void hist_add(int* hist, bool active, int bin) {
    const uint64_t act = __ballot(active);
    if (act == 0) return;
    const int first = __builtin_ctzll(act);
    const int lead = __builtin_amdgcn_readlane(bin, first);
    const bool same = active && bin == lead;
    const uint64_t m = __ballot(same);
    const int lane = threadIdx.x & 63;
    if (lane == first) atomicAdd(&hist[lead], (int)__popcll(m));
    else if (active && !same) atomicAdd(&hist[bin], 1);
}

// wavefront 0: from the 256-bin histogram and the rank `need` still wanted, the bin that holds the
// need-th largest element of the current bucket; updates (prefix, need) in LDS.  I: int64_t, or int where ranks fit
template <typename I>
__device__ inline void pick_bin(const int* hist, int lane, int shift, uint32_t prefix, I need, uint32_t* sh_prefix, I* sh_need) {
    // bins in descending order: lane l owns bins 255-4l .. 252-4l
    int c0 = hist[255 - 4 * lane], c1 = hist[254 - 4 * lane], c2 = hist[253 - 4 * lane], c3 = hist[252 - 4 * lane];
    I tot = (I)c0 + c1 + c2 + c3;
    I incl = tot;
    for (int off = 1; off < 64; off <<= 1) {
        I o = __shfl_up(incl, off);
        if (lane >= off) incl += o;
    }
    I excl = incl - tot;  // elements in bins above this lane's bins
    if (excl < need && need <= incl) {
        I rem = need - excl;
        int bin;
        if (rem <= c0) { bin = 255 - 4 * lane; }
        else if (rem <= (I)c0 + c1) { bin = 254 - 4 * lane; rem -= c0; }
        else if (rem <= (I)c0 + c1 + c2) { bin = 253 - 4 * lane; rem -= (I)c0 + c1; }
        else { bin = 252 - 4 * lane; rem -= (I)c0 + c1 + c2; }
        *sh_prefix = prefix | ((uint32_t)bin << shift);
        *sh_need = rem;
    }
}

// ---- the threshold bin resolved in LDS (long-row kernels) -------------------
// A first histogram over the keys' top 13 bits (sign, exponent, four mantissa bits: a bin is 4.4 % wide in value) finds the
// bin of the k-th largest key; every wavefront then copies the low 19 bits of ITS keys of that bin into its own LDS
// region, and three radix passes over those few keys (8 + 8 + 3 bits) give the exact threshold, the number of keys equal
// to it that are still wanted, and each wavefront's (greater, equal) counts.  A wavefront whose share of the bin does not
// fit its region (heavily tied scores) makes the caller fall back to 8-bit passes over all keys.
constexpr int T13_BINS = 8192;
constexpr int T13_LOW = 19;
// Half of a CU's 160 KB with the small arrays below, so that two workgroups share a CU where the registers allow it (at 80 KB without
// the arrays they did not: 512 rows of 131072, k = 52428: 140 us, now 119).  The regions take the place of the histogram once the bin is
// known.
constexpr int T13_LDS_BYTES = 78 * 1024;
constexpr int T13_CW = T13_LDS_BYTES / (TOPK_WAVES * 4);                 // keys per wavefront region: 1248
struct TopkShared {
    int64_t need;
    int hist[256];
    int wave_gt[TOPK_WAVES], wave_eq[TOPK_WAVES], wave_tot[TOPK_WAVES], wave_in[TOPK_WAVES];
    uint32_t prefix, lo, hi;
    int bin, over, rank_lo, rank;
};
static_assert(T13_LDS_BYTES + sizeof(TopkShared) <= 80 * 1024, "two workgroups share a CU's LDS");
static_assert(T13_BINS * 4 <= T13_LDS_BYTES && TOPK_WAVES * 256 * 4 <= T13_LDS_BYTES, "the histograms fit");

// all 1024 lanes: from the 8192-bin histogram the bin that holds the k-th largest key (-> *sh_bin) and the rank wanted
// inside it (-> *sh_need); ends with a barrier
__device__ inline void t13_pick(const int* h13, int64_t k, int* wave_tot, int* sh_bin, int64_t* sh_need) {
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    constexpr int BPT = T13_BINS / TOPK_THREADS;   // bins per lane, descending
    int c[BPT], tot = 0;
#pragma unroll
    for (int q = 0; q < BPT; ++q) { c[q] = h13[T13_BINS - 1 - BPT * tid - q]; tot += c[q]; }
    int incl = tot;
    for (int off = 1; off < 64; off <<= 1) {
        const int o = __shfl_up(incl, off);
        if (lane >= off) incl += o;
    }
    if (lane == 63) wave_tot[wave] = incl;
    __syncthreads();
    int64_t excl = incl - tot;
    for (int w = 0; w < wave; ++w) excl += wave_tot[w];
    if (excl < k && k <= excl + tot) {
        int64_t rem = k - excl;
        int q = 0;
#pragma unroll
        for (int t = 0; t < BPT - 1; ++t)
            if (q == t && rem > c[t]) { rem -= c[t]; q = t + 1; }
        *sh_bin = T13_BINS - 1 - BPT * tid - q;
        *sh_need = rem;
    }
    __syncthreads();
}

// all 1024 lanes: cand[0 .. cnt) = low 19 bits of this wavefront's keys of the bin, `need` = rank wanted inside the bin.
// Returns the low 19 bits of the threshold; *need_eq = keys equal to it still wanted; *g / *e = this wavefront's
// candidates above / equal to it.
__device__ inline uint32_t t13_resolve(const uint32_t* cand, int cnt, int64_t need, int* hist, uint32_t* sh_prefix,
                                       int64_t* sh_need, int* need_eq, int* g, int* e) {
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    uint32_t prefix = 0;
    const int cnt64 = (cnt + 63) & ~63;
#pragma unroll
    for (int pass = 0; pass < 3; ++pass) {
        const int shift = pass == 0 ? 11 : pass == 1 ? 3 : 0;
        const uint32_t dmask = pass == 2 ? 0x7u : 0xFFu;
        const uint32_t hi_mask = pass == 0 ? 0u : pass == 1 ? 0x7F800u : 0x7FFF8u;
        if (tid < 256) hist[tid] = 0;
        __syncthreads();
        for (int j = lane; j < cnt64; j += 64) {
            const uint32_t c = j < cnt ? cand[j] : 0u;
            hist_add(hist, j < cnt && (c & hi_mask) == prefix, (int)((c >> shift) & dmask));
        }
        __syncthreads();
        if (wave == 0) pick_bin(hist, lane, shift, prefix, need, sh_prefix, sh_need);
        __syncthreads();
        prefix = *sh_prefix;
        need = *sh_need;
    }
    *need_eq = (int)need;
    int gg = 0, ee = 0;
    for (int j = lane; j < cnt64; j += 64) {
        const uint32_t c = j < cnt ? cand[j] : 0u;
        gg += (int)__popcll(__ballot(j < cnt && c > prefix));
        ee += (int)__popcll(__ballot(j < cnt && c == prefix));
    }
    *g = gg; *e = ee;
    return prefix;
}

// sums / minima / maxima over the wavefront's 64 lanes in six DPP steps, the result uniform.  (A lane-crossing shuffle goes through
// the LDS crossbar: about a hundred cycles a step.)
template <typename F>
__device__ __forceinline__ uint32_t wave_reduce_u32(uint32_t v, uint32_t identity, F f) {
    auto step = [&](auto dpp) { v = f(v, dpp()); };
    step([&] { return (uint32_t)__builtin_amdgcn_update_dpp((int)identity, (int)v, 0x111, 0xF, 0xF, false); });   // row_shr 1
    step([&] { return (uint32_t)__builtin_amdgcn_update_dpp((int)identity, (int)v, 0x112, 0xF, 0xF, false); });   // row_shr 2
    step([&] { return (uint32_t)__builtin_amdgcn_update_dpp((int)identity, (int)v, 0x114, 0xF, 0xF, false); });   // row_shr 4
    step([&] { return (uint32_t)__builtin_amdgcn_update_dpp((int)identity, (int)v, 0x118, 0xF, 0xF, false); });   // row_shr 8
    step([&] { return (uint32_t)__builtin_amdgcn_update_dpp((int)identity, (int)v, 0x142, 0xA, 0xF, false); });   // row_bcast 15
    step([&] { return (uint32_t)__builtin_amdgcn_update_dpp((int)identity, (int)v, 0x143, 0xC, 0xF, false); });   // row_bcast 31
    return (uint32_t)__builtin_amdgcn_readlane((int)v, 63);
}

// Register-resident variant: N <= 64 * KPT * W, one workgroup of W wavefronts per problem.  Lane keeps keys[j] = key of element
// lo + 64*j + lane, lo = 64*KPT*wave; slots at or beyond N hold key 0.  So does a score that is the NaN with every bit set: the search counts keys that
// reach a value above 0 only, and where the threshold itself is 0 an empty slot is the last of the equal keys, behind the k <= N selected.
// The threshold is searched for between the row's smallest and largest key: a round counts the keys that reach the middle (a
// compare per key, summed on the scalar unit -- of 12 and more keys every third on the vector unit, since the scalar one runs out --, one LDS
// atomic per wavefront, one barrier) and keeps one half, until that holds at most 64 keys or a single value.  Those keys go to LDS, and
// every wavefront decides the rest of the threshold for itself, bit by bit, one key per lane, without a barrier.  A round that leaves
// every key in has met few values: the range then shrinks to the outermost of them, so ties need no route of their own.
// Bound: latency (a launch that does nothing takes 4.3 us; a round 0.25 us at 8 keys per lane, 10 of them), from 16 keys per
// lane on also the compares and the output's ranks.  With a histogram of the keys' top 13 bits (LDS atomics that meet in few bins, 8192 bins
// cleared and scanned, three more passes for the other bits) in the place of the rounds a row of 700 scores took 8.9 us, now 4.5; 2048 9.1, now
// 5.2; 8192 10.6, now 9.1; 20001 24.7, now 14.4; 32768 27.1, now 20.1; 512 rows of them 17.9, 18.4, 21.6, 64.7, 70.9, now 5.5, 7.7, 15.3, 27.5, 49.4.
// Up to 512 scores: one wavefront that decided all 32 bits 5.9, now 4.4 (512 rows 6.5, now 4.9).  Three thresholds a round: 10.5 us at 8192.
// MAP: map.in[i] goes where i goes.  (An instantiation of its own: a test in the place where indices are written costs the others 0.7 us.)
template <int KPT, int W, bool MAP>
__global__ void __launch_bounds__(64 * W) __attribute__((amdgpu_waves_per_eu(8, 8))) topk_reg_kernel(const float* __restrict__ scores, int64_t N, int64_t k,
                                                            int protect_last, int32_t* __restrict__ idx_out, TopkSegments seg, TopkMap map) {
    constexpr int ROUNDS = 33;   // a round leaves at most half of a 32-bit range
    __shared__ int count[ROUNDS];
    __shared__ uint32_t cand[64], wave_min[W], wave_max[W];
    __shared__ int cands, wave_ge[W], wave_gt[W];

    int base = 0;   // what the written indices count from
    // one independent problem per workgroup: equal rows, or the segment the descriptors give it
    if (seg.offsets) {
        const int64_t b0 = seg.offsets[blockIdx.x];
        N = seg.offsets[blockIdx.x + 1] - b0;
        k = seg.k[blockIdx.x];
        if (seg.whole) base = (int)b0;
        scores += b0;
        idx_out += seg.out_offsets[blockIdx.x];
        if (k > N) k = N;
        if (k <= 0 || N <= 0) return;
    } else {
        scores += (int64_t)blockIdx.x * N;
        idx_out += (int64_t)blockIdx.x * k;
        if (MAP) map.out += (int64_t)blockIdx.x * k;
    }
    auto put = [&](int at, int i) {
        idx_out[(uint32_t)at] = base + i;
        if (MAP) map.out[(uint32_t)at] = map.in[i];
    };
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int n = (int)N, kk = (int)k, last = protect_last ? n - 1 : -1;   // the protected score is above all others: left out of the search
    const int lo = wave * (64 * KPT);

    auto umin = [](uint32_t a, uint32_t b) { return min(a, b); };
    auto umax = [](uint32_t a, uint32_t b) { return max(a, b); };
    auto uadd = [](uint32_t a, uint32_t b) { return a + b; };
    // sum of the first `m` wavefronts' entries
    auto sum_of = [&](const int* per_wave, int m) { return (int)wave_reduce_u32(lane < m ? (uint32_t)per_wave[lane & (W - 1)] : 0u, 0u, uadd); };
    uint32_t keys[KPT];
    if (tid < ROUNDS) count[tid] = 0;
    if (tid == 0) cands = 0;
    if (tid < 64) cand[tid] = 0;
    {
        float v[KPT];
        uint32_t mn = 0xFFFFFFFFu, mx = 0u;
        if (lo + 64 * KPT <= n && !(last >= lo && last < lo + 64 * KPT)) {   // every slot has a key that is searched
            const float* p = scores + lo + lane;
#pragma unroll
            for (int j = 0; j < KPT; ++j) v[j] = p[64 * j];
#pragma unroll
            for (int j = 0; j < KPT; ++j) {
                keys[j] = order_key(v[j]);
                mn = min(mn, keys[j]);
                mx = max(mx, keys[j]);
            }
        } else {
#pragma unroll
            for (int j = 0; j < KPT; ++j) {
                v[j] = 0.f;
                if (lo + 64 * j < n) v[j] = scores[min(lo + 64 * j + lane, n - 1)];
            }
#pragma unroll
            for (int j = 0; j < KPT; ++j) {
                const int i = lo + 64 * j + lane;
                const uint32_t key = order_key(v[j]);
                const bool in = i < n && i != last;
                keys[j] = in ? key : 0u;
                mn = min(mn, in ? key : 0xFFFFFFFFu);
                mx = max(mx, keys[j]);
            }
        }
        mn = wave_reduce_u32(mn, 0xFFFFFFFFu, umin);
        mx = wave_reduce_u32(mx, 0u, umax);
        if (lane == 0) { wave_min[wave] = mn; wave_max[wave] = mx; }
    }
    __syncthreads();
    const int want = protect_last ? kk - 1 : kk;   // rank of the threshold among the searched keys
    uint32_t T = 0xFFFFFFFFu;
    if (want > 0) {
        // the threshold lies in [lo_key, lo_key + width]: c_lo >= want keys reach the lower end, c_hi < want are above the upper one
        uint32_t lo_key = wave_reduce_u32(wave_min[lane & (W - 1)], 0xFFFFFFFFu, umin);
        uint32_t width = wave_reduce_u32(wave_max[lane & (W - 1)], 0u, umax) - lo_key;
        int c_lo = protect_last ? n - 1 : n, c_hi = 0, held = 0;
        for (int round = 0; c_lo - c_hi > 64 && width > 0; ++round) {
            const uint32_t off = (width >> 1) + 1, t = lo_key + off;   // > 0: no empty slot counts
            int c = 0, mine = 0;
#pragma unroll
            for (int j = 0; j < KPT; ++j) {
                if (KPT >= 12 && j % 3 == 2) mine += keys[j] >= t ? 1 : 0;
                else c += (int)__popcll(__ballot(keys[j] >= t));
            }
            if (KPT >= 12) c += (int)wave_reduce_u32((uint32_t)mine, 0u, uadd);
            if (lane == 0) atomicAdd(&count[round], c);
            __syncthreads();
            c = __builtin_amdgcn_readfirstlane(count[round]);
            if (c >= want) { lo_key = t; width -= off; c_lo = c; }
            else { width = off - 1; c_hi = c; }
            const int inside = c_lo - c_hi;
            if (inside == held && inside > 64) {
                // a round that left every key in: the part's keys are few values, and its ends move to the outermost of them
                uint32_t mn = 0xFFFFFFFFu, mx = 0u;
#pragma unroll
                for (int j = 0; j < KPT; ++j) {
                    const uint32_t d = keys[j] - lo_key;
                    mn = min(mn, d <= width ? d : 0xFFFFFFFFu);
                    mx = max(mx, d <= width ? d : 0u);
                }
                mn = wave_reduce_u32(mn, 0xFFFFFFFFu, umin);
                mx = wave_reduce_u32(mx, 0u, umax);
                if (lane == 0) { wave_min[wave] = mn; wave_max[wave] = mx; }
                __syncthreads();
                mn = wave_reduce_u32(wave_min[lane & (W - 1)], 0xFFFFFFFFu, umin);
                mx = wave_reduce_u32(wave_max[lane & (W - 1)], 0u, umax);
                lo_key += mn;
                width = mx - mn;
            }
            held = inside;
        }
        T = lo_key;
        if (width > 0) {
            const uint32_t first = lo_key, above = max(first, 1u), span = width - (above - first);   // (distance 0 from key 0 is in cand already)
#pragma unroll
            for (int j = 0; j < KPT; ++j)
                if (keys[j] - above <= span) cand[atomicAdd(&cands, 1) & 63] = keys[j] - first;
            __syncthreads();
            const uint32_t d = cand[lane];
            const int rank = want - c_hi;
            uint32_t t = 0;
            for (int bit = 31 - __builtin_clz(width); bit >= 0; --bit) {
                const uint32_t at = t | (1u << bit);
                if ((int)__popcll(__ballot(d >= at)) >= rank) t = at;
            }
            T = first + t;
        }
    }
    if (last >= lo && last < lo + 64 * KPT) {
#pragma unroll
        for (int j = 0; j < KPT; ++j)
            if (lo + 64 * j + lane == last) keys[j] = 0xFFFFFFFFu;
    }

    int ge = 0;
#pragma unroll
    for (int j = 0; j < KPT; ++j) ge += (int)__popcll(__ballot(keys[j] >= T));
    if (lane == 0) wave_ge[wave] = ge;
    __syncthreads();
    const int total = sum_of(wave_ge, W);
    int before = sum_of(wave_ge, wave);
    if (total == kk) {   // every key that reaches the threshold is selected
#pragma unroll
        for (int j = 0; j < KPT; ++j) {
            const bool sel = keys[j] >= T;
            const uint64_t m = __ballot(sel);
            const int at = __builtin_amdgcn_mbcnt_hi((uint32_t)(m >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)m, before));
            if (sel) put(at, lo + 64 * j + lane);
            before += (int)__popcll(m);
        }
        return;
    }
    // of the keys equal to the threshold only the first need_eq are taken
    int gt = 0, eq = 0;
#pragma unroll
    for (int j = 0; j < KPT; ++j) {
        gt += (int)__popcll(__ballot(keys[j] > T));
        eq += (int)__popcll(__ballot(keys[j] == T));
    }
    __syncthreads();
    if (lane == 0) { wave_gt[wave] = gt; wave_ge[wave] = eq; }
    __syncthreads();
    const int need_eq = kk - sum_of(wave_gt, W);
    int gt_before = sum_of(wave_gt, wave), eq_before = sum_of(wave_ge, wave);
#pragma unroll
    for (int j = 0; j < KPT; ++j) {
        const int i = lo + 64 * j + lane;
        const bool g_ = keys[j] > T, e_ = keys[j] == T;
        const uint64_t mgt = __ballot(g_), meq = __ballot(e_);
        const int my_gt = gt_before + lane_prefix_popc(mgt);
        const int my_eq = eq_before + lane_prefix_popc(meq);
        if (g_ || (e_ && my_eq < need_eq)) put(my_gt + (my_eq < need_eq ? my_eq : need_eq), i);
        gt_before += (int)__popcll(mgt);
        eq_before += (int)__popcll(meq);
    }
}

__global__ void __launch_bounds__(TOPK_THREADS) topk_kernel(const float* __restrict__ scores, int64_t N, int64_t k,
                                                            int protect_last, int32_t* __restrict__ idx_out, TopkSegments seg) {
    __shared__ int hist[256];
    __shared__ uint32_t sh_prefix;     // key bits decided so far
    __shared__ int64_t sh_need;        // how many elements are still to be taken inside the current bucket
    __shared__ int64_t wave_gt[TOPK_WAVES], wave_eq[TOPK_WAVES];

    int base = 0;   // what the written indices count from
    // one independent problem per workgroup: equal rows, or the segment the descriptors give it
    if (seg.offsets) {
        const int64_t b0 = seg.offsets[blockIdx.x];
        N = seg.offsets[blockIdx.x + 1] - b0;
        k = seg.k[blockIdx.x];
        if (seg.whole) base = (int)b0;
        scores += b0;
        idx_out += seg.out_offsets[blockIdx.x];
        if (k > N) k = N;
        if (k <= 0 || N <= 0) return;
    } else {
        scores += (int64_t)blockIdx.x * N;
        idx_out += (int64_t)blockIdx.x * k;
    }
    const int tid = threadIdx.x;
    const int lane = tid & 63, wave = tid >> 6;

    if (tid == 0) { sh_prefix = 0; sh_need = k; }
    uint32_t prefix = 0;
    int64_t need = k;

    // ---- 1. radix select
    for (int pass = 0; pass < 4; ++pass) {
        const int shift = 24 - 8 * pass;
        const uint32_t hi_mask = pass == 0 ? 0u : (0xFFFFFFFFu << (shift + 8));
        if (tid < 256) hist[tid] = 0;
        __syncthreads();
        // every lane runs the same number of rounds (hist_add uses wavefront-wide ballots)
        for (int64_t at0 = 0; at0 < N; at0 += TOPK_THREADS) {
            const int64_t i = at0 + tid;
            uint32_t key = i < N ? load_key(scores, i, N, protect_last) : 0u;
            hist_add(hist, i < N && (key & hi_mask) == prefix, (int)((key >> shift) & 0xFF));
        }
        __syncthreads();
        if (wave == 0) pick_bin(hist, lane, shift, prefix, need, &sh_prefix, &sh_need);
        __syncthreads();
        prefix = sh_prefix;
        need = sh_need;
    }
    const uint32_t T = prefix;     // key of the k-th largest element
    const int64_t need_eq = need;  // elements equal to T to take (lowest indices first), >= 1

    // ---- 2. ordered compaction, one contiguous slice per wavefront (slice length multiple of 64)
    int64_t per_wave = ((N + TOPK_WAVES - 1) / TOPK_WAVES + 63) / 64 * 64;
    int64_t lo = (int64_t)wave * per_wave;
    int64_t hi = lo + per_wave < N ? lo + per_wave : N;
    int64_t cgt = 0, ceq = 0;
    for (int64_t at0 = lo; at0 < hi; at0 += 64) {
        int64_t i = at0 + lane;
        bool gt = false, eq = false;
        if (i < hi) { uint32_t key = load_key(scores, i, N, protect_last); gt = key > T; eq = key == T; }
        cgt += __popcll(__ballot(gt));
        ceq += __popcll(__ballot(eq));
    }
    if (lane == 0) { wave_gt[wave] = cgt; wave_eq[wave] = ceq; }
    __syncthreads();
    int64_t gt_before = 0, eq_before = 0;
    for (int w = 0; w < wave; ++w) { gt_before += wave_gt[w]; eq_before += wave_eq[w]; }
    for (int64_t at0 = lo; at0 < hi; at0 += 64) {
        int64_t i = at0 + lane;
        bool gt = false, eq = false;
        if (i < hi) { uint32_t key = load_key(scores, i, N, protect_last); gt = key > T; eq = key == T; }
        uint64_t mgt = __ballot(gt), meq = __ballot(eq);
        int64_t my_gt = gt_before + lane_prefix_popc(mgt);
        int64_t my_eq = eq_before + lane_prefix_popc(meq);
        if (gt || (eq && my_eq < need_eq)) {
            int64_t o = my_gt + (my_eq < need_eq ? my_eq : need_eq);
            idx_out[o] = base + (int32_t)i;
        }
        gt_before += __popcll(mgt);
        eq_before += __popcll(meq);
    }
}

// Long rows of a batch (N > 32768, equal rows): one workgroup per row as above, but written for streaming.
// Every wavefront owns one contiguous slice in all sweeps and reads it as 16-byte loads, four per lane in flight (64 KB per
// workgroup).
// Three sweeps over the row in the usual case: (1) an 8192-bin histogram of the keys' top 13 bits (sign, exponent, four
// mantissa bits) finds the bin of the k-th largest key; (2) every wavefront copies the low 19 bits of its keys of that bin
// into its own LDS region and counts the keys of higher bins -- scores of one layer spread over several octaves, so the
// bin (4.4 % wide in value) holds a few percent of the row --, the remaining 19 bits are then resolved by three radix passes
// over LDS, which also leave each wavefront's (greater, equal) counts; (3) the ordered compaction.  If a wavefront's
// keys of the bin do not fit its region (heavily tied scores), the kernel falls back to four 8-bit passes over the row with
// histograms private to the wavefront, six sweeps in all; both routes end in the same exact (threshold, rank) pair.
// A length that is no multiple of 4 leaves rows at 4-byte addresses, which 16-byte loads take (512 rows of 131071: 112 us, of 131072
// 113; one row 46 and 46, where scores read one by one in six sweeps took 477 and 231), and a last piece of one to three scores, which is loaded from the row's end, moved into place and padded with the NaN
// whose key is 0: no score's key is smaller and none comes later, so a padded place is never among the k <= N selected.  (Minus infinity is
// not enough: NaNs with the sign bit set come below it.)
typedef float f32x4v __attribute__((ext_vector_type(4)));
typedef float f32x4u __attribute__((ext_vector_type(4), aligned(4)));
constexpr int LONG_U = 4;                       // 16-byte loads in flight per lane
constexpr int LONG_STEP = 64 * 4 * LONG_U;      // scores a wavefront takes per iteration

// the piece [i0, i0 + 4) of a row of n scores, key 0 in the places past it, from the four scores at min(i0, n - 4); for i0 >= n any of these
__device__ __forceinline__ f32x4v end_piece(f32x4v v, int i0, int n) {
    const int by = i0 - min(i0, n - 4);
    const float none = __uint_as_float(0xFFFFFFFFu);
    if (by & 1) v = f32x4v{v[1], v[2], v[3], none};
    if (by & 2) v = f32x4v{v[2], v[3], none, none};
    return v;
}

// HINT: a caller that has reason to believe that the k-th largest key begins with the 16 bits `top16` (>= 0) skips the sweeps and passes before
// those that resolve the other 16; the counts of the first of them tell when it does not, and all four follow.
template <bool HINT>
__device__ __forceinline__ void topk_long_rows(const float* __restrict__ scores, int64_t N, int64_t k, int protect_last, int32_t* __restrict__ idx_out, char* lsm, TopkShared& sh,
                                               int top16 = -1) {
    int* h13 = reinterpret_cast<int*>(lsm);                                                     // [T13_BINS]
    uint32_t (*cand)[T13_CW] = reinterpret_cast<uint32_t (*)[T13_CW]>(lsm);                     // [TOPK_WAVES][T13_CW], after the histogram
    int (*whist)[256] = reinterpret_cast<int (*)[256]>(lsm);                                    // 8-bit passes only, same bytes
    int* const hist = sh.hist;
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int n = (int)N;
    const int per_wave = ((n + TOPK_WAVES - 1) / TOPK_WAVES + LONG_STEP - 1) / LONG_STEP * LONG_STEP;
    const int lo = __builtin_amdgcn_readfirstlane(wave * per_wave);
    const int hi = lo + per_wave < n ? lo + per_wave : n;   // of a piece that starts below hi, places past it have key 0
    auto load_step = [&](int base, f32x4v (&v)[LONG_U]) {   // the pieces of one iteration
#pragma unroll
        for (int u = 0; u < LONG_U; ++u) v[u] = *reinterpret_cast<const f32x4u*>(scores + (uint32_t)min(base + u * 256 + lane * 4, n - 4));
        if (base + LONG_STEP > n) {
#pragma unroll
            for (int u = 0; u < LONG_U; ++u) v[u] = end_piece(v[u], base + u * 256 + lane * 4, n);
        }
    };
    const uint32_t last_key_at = protect_last ? (uint32_t)(n - 1) : 0xFFFFFFFFu;

    // one iteration of a sweep over the wavefront's slice: the keys of load u, element e (index i0 + e) go to BODY
#define SPTS_LONG_SWEEP(BODY)                                                                              \
    for (int base = lo; base < hi; base += LONG_STEP) {                                                    \
        f32x4v v[LONG_U];                                                                                  \
        load_step(base, v);                                                                                \
        _Pragma("unroll") for (int u = 0; u < LONG_U; ++u) {                                               \
            const int i0 = base + u * 256 + lane * 4;                                                      \
            const bool valid = i0 < hi;                                                                    \
            _Pragma("unroll") for (int e = 0; e < 4; ++e) {                                                \
                uint32_t key = order_key(v[u][e]);                                                         \
                if ((uint32_t)(i0 + e) == last_key_at) key = 0xFFFFFFFFu;                                  \
                BODY                                                                                       \
            }                                                                                              \
        }                                                                                                  \
    }

    uint32_t T = 0;
    int need_eq = 0;
    uint32_t b12 = 0;
    int64_t need = 0;
    int cnt = 0, cgt = 0;
    bool over = HINT && top16 >= 0;
    if (!over) {
        // ---- sweep 1: top 13 bits
        for (int i = tid; i < T13_BINS; i += TOPK_THREADS) h13[i] = 0;
        if (tid == 0) { sh.over = 0; sh.bin = 0; sh.need = k; }
        __syncthreads();
        SPTS_LONG_SWEEP({ hist_add(h13, valid, (int)(key >> T13_LOW)); })
        __syncthreads();
        t13_pick(h13, k, sh.wave_tot, &sh.bin, &sh.need);
        b12 = (uint32_t)__builtin_amdgcn_readfirstlane(sh.bin);
        need = __builtin_amdgcn_readfirstlane((int)sh.need);
        // ---- sweep 2: the wavefront's keys of that bin into its LDS region (low 19 bits), keys of higher bins counted
        SPTS_LONG_SWEEP({
            const uint32_t top = key >> T13_LOW;
            cgt += (int)__popcll(__ballot(valid && top > b12));
            const bool in = valid && top == b12;
            const uint64_t m = __ballot(in);
            const int at = cnt + lane_prefix_popc(m);
            if (in && at < T13_CW) cand[wave][at] = key & ((1u << T13_LOW) - 1u);
            cnt += (int)__popcll(m);
        })
        if (lane == 0 && cnt > T13_CW) sh.over = 1;
        __syncthreads();
        over = sh.over != 0;
    }
    if (!over) {
        int g, e;
        const uint32_t low = t13_resolve(cand[wave], cnt, need, hist, &sh.prefix, &sh.need, &need_eq, &g, &e);
        T = (b12 << T13_LOW) | low;
        if (lane == 0) { sh.wave_gt[wave] = cgt + g; sh.wave_eq[wave] = e; }
    } else {
        // ---- fallback: four 8-bit passes over the row
        __syncthreads();   // every wavefront has read sh.over before the regions are reused as histograms
        uint32_t prefix = HINT && top16 >= 0 ? (uint32_t)top16 << 16 : 0u;
        need = k;
        cgt = 0;   // last pass, and the first one after a hint: keys of this wavefront's slice whose decided bits exceed the prefix
        for (int pass = HINT && top16 >= 0 ? 2 : 0; pass < 4; ++pass) {
            if (HINT) cgt = 0;
            const bool hinted = HINT && top16 >= 0 && pass == 2;
            const int shift = 24 - 8 * pass;
            const uint32_t hi_mask = pass == 0 ? 0u : (0xFFFFFFFFu << (shift + 8));
            for (int i = lane; i < 256; i += 64) whist[wave][i] = 0;
            __syncthreads();
            SPTS_LONG_SWEEP({
                hist_add(whist[wave], valid && (key & hi_mask) == prefix, (int)((key >> shift) & 0xFF));
                if (pass == 3 || hinted) cgt += (int)__popcll(__ballot(valid && (key & hi_mask) > prefix));
            })
            if (hinted && lane == 0) sh.wave_gt[wave] = cgt;
            if (HINT && tid == 0) sh.need = 0;
            __syncthreads();
            if (tid < 256) {
                int t = 0;
#pragma unroll
                for (int w = 0; w < TOPK_WAVES; ++w) t += whist[w][tid];
                hist[tid] = t;
            }
            if (hinted) {
                int above = 0;
                for (int w = 0; w < TOPK_WAVES; ++w) above += sh.wave_gt[w];
                need -= __builtin_amdgcn_readfirstlane(above);
            }
            __syncthreads();
            if (wave == 0) pick_bin(hist, lane, shift, prefix, need, &sh.prefix, &sh.need);
            __syncthreads();
            prefix = (uint32_t)__builtin_amdgcn_readfirstlane(sh.prefix);
            need = __builtin_amdgcn_readfirstlane((int)sh.need);
            if (HINT && need == 0) {   // no bin holds that rank: not the key's first bits
                prefix = 0; need = k; top16 = -1; pass = -1;
            }
        }
        T = prefix;
        need_eq = (int)need;
        // this wavefront's keys above T / equal to T, from its own last-digit histogram
        const int digit = (int)(T & 0xFFu);
        int above = 0;
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            const int b = lane * 4 + q;
            above += b > digit ? whist[wave][b] : 0;
        }
#pragma unroll
        for (int off = 32; off > 0; off >>= 1) above += __shfl_xor(above, off);
        if (lane == 0) { sh.wave_gt[wave] = above + cgt; sh.wave_eq[wave] = whist[wave][digit]; }
    }
    __syncthreads();
    int gt_before = 0, eq_before = 0;
    for (int w = 0; w < wave; ++w) { gt_before += sh.wave_gt[w]; eq_before += sh.wave_eq[w]; }
    // ordered compaction of the slice: index order inside an iteration is (load u, lane, element e)
    for (int base = lo; base < hi; base += LONG_STEP) {
        f32x4v v[LONG_U];
        load_step(base, v);
#pragma unroll
        for (int u = 0; u < LONG_U; ++u) {
            const int i0 = base + u * 256 + lane * 4;
            const bool valid = i0 < hi;
            bool gt[4], eq[4];
            int lower_gt = 0, lower_eq = 0, tot_gt = 0, tot_eq = 0;   // selected keys of lower lanes / of the whole wavefront, this load
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                uint32_t key = order_key(v[u][e]);
                if ((uint32_t)(i0 + e) == last_key_at) key = 0xFFFFFFFFu;
                gt[e] = valid && key > T;
                eq[e] = valid && key == T;
                const uint64_t mg = __ballot(gt[e]), me = __ballot(eq[e]);
                lower_gt += lane_prefix_popc(mg); lower_eq += lane_prefix_popc(me);
                tot_gt += (int)__popcll(mg); tot_eq += (int)__popcll(me);
            }
            int my_gt = gt_before + lower_gt, my_eq = eq_before + lower_eq;
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                if (gt[e] || (eq[e] && my_eq < need_eq)) idx_out[my_gt + (my_eq < need_eq ? my_eq : need_eq)] = i0 + e;
                my_gt += gt[e] ? 1 : 0;
                my_eq += eq[e] ? 1 : 0;
            }
            gt_before += tot_gt;
            eq_before += tot_eq;
        }
    }
}

__global__ void __launch_bounds__(TOPK_THREADS) __attribute__((amdgpu_waves_per_eu(8, 8))) topk_long_kernel(const float* __restrict__ scores, int64_t N, int64_t k,
                                                                 int protect_last, int32_t* __restrict__ idx_out) {
    extern __shared__ __attribute__((aligned(16))) char lsm[];
    __shared__ TopkShared sh;
    topk_long_rows<false>(scores + (int64_t)blockIdx.x * N, N, k, protect_last, idx_out + (int64_t)blockIdx.x * k, lsm, sh);
}

// The same rows read from memory once (32768 < N <= LONG1_MAX_N).  A sample of 8192 scores spread over the row gives, through
// the 8192-bin histogram and 8 more bits of the keys in its bins, two keys that bracket the k-th largest with four standard
// deviations of the sample's quantile on either side (about 4 % of the row lies between them, whatever the scores' spread).  One
// sweep over the row then leaves, per score, a bit of the lane's own in LDS (above the bracket), and the keys inside the bracket, with
// their places, in the wavefront's LDS region; counts tell whether the bracket holds the threshold.  The exact threshold is
// resolved among those keys, the selected ones set their bits, and the index list is written from the bits.  A region keeps
// 21 bits of a key's distance from the bracket's lower end; where the bracket is wider, the keys that share the threshold's 21 bits
// (a handful) are read again for the rest.  Rows of which the sample says that a wavefront's share of the bracket does not fit its region
// (a few equal values, scores ordered by position) take the route of topk_long_rows at once, and so do the rare ones (1 in 10^4 of
// ordinary rows) that turn out not to fit or not to hold the threshold after the sweep; where the bracket's ends share 16 bits (equal
// values, as a rule), only the last 16 are left to resolve there: two passes and the output instead of seven sweeps.
// Bound: HBM for one read of the scores and the index list (68 us for 512 rows of 131072, k = 52428, at 5.5 TB/s) and about 25
// vector instructions per score and wavefront.  Measured there, three sweeps -> this kernel: 196 -> 116 us for scores within an
// octave, 191 -> 117 for scores over many (log-spread 1.5 to 3), 189 -> 116 for signed normal ones, 194 -> 148 for fifty values, 410 -> 192
// for equal ones; k = 5 % 182 -> 97, k = 95 % 225 -> 168.  16 rows 86 -> 48-51, of equal values 186 -> 96; one row of 33000 30 -> 24-27.
// Scores sorted by position pay the sample and the sweeps: 512 rows 349 -> 196 (their bin fits the regions now, and two workgroups share a CU), 16
// rows 160 -> 98, but one of 33000 36 -> 43 and 256 of 65536 66 -> 76.
constexpr int LONG1_MAX_N = 131072;                               // one bit per score: 16 KB; longer rows keep to the three sweeps
constexpr int LONG1_WORDS = LONG1_MAX_N / TOPK_WAVES / 64 / 32;  // 32-score words per lane
constexpr int LONG1_SAMPLES = 8192;
constexpr int LONG1_BITS = LONG1_WORDS * TOPK_THREADS * 4;       // bytes of those bits; the regions take what is left of the LDS
constexpr int LONG1_CW = (T13_LDS_BYTES - LONG1_BITS) / (TOPK_WAVES * 4);   // keys per wavefront region: 992, 12 % of the longest slice
struct topk_true { static constexpr bool value = true; };
struct topk_false { static constexpr bool value = false; };

// all 1024 lanes: the 13-bit bins of the sampled histogram that hold ranks r_hi <= r_lo (1 = largest) and the ranks inside them ->
// sh.hi / sh.rank and sh.lo / sh.rank_lo, samples in those bins and the seven around them -> sh.bin, sh.over; ends with a barrier
__device__ inline void sample_bins(const int* h13, int r_hi, int r_lo, TopkShared& sh) {
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    constexpr int BPT = T13_BINS / TOPK_THREADS;
    int c[BPT], tot = 0;
#pragma unroll
    for (int q = 0; q < BPT; ++q) { c[q] = h13[T13_BINS - 1 - BPT * tid - q]; tot += c[q]; }
    int incl = tot;
    for (int off = 1; off < 64; off <<= 1) {
        const int o = __shfl_up(incl, off);
        if (lane >= off) incl += o;
    }
    if (lane == 63) sh.wave_tot[wave] = incl;
    __syncthreads();
    int excl = incl - tot;
    for (int w = 0; w < wave; ++w) excl += sh.wave_tot[w];
#pragma unroll
    for (int end = 0; end < 2; ++end) {
        const int rank = end ? r_lo : r_hi;
        if (excl < rank && rank <= excl + tot) {
            int rem = rank - excl, q = 0;
#pragma unroll
            for (int t = 0; t < BPT - 1; ++t)
                if (q == t && rem > c[t]) { rem -= c[t]; q = t + 1; }
            *(end ? &sh.lo : &sh.hi) = (uint32_t)(T13_BINS - 1 - BPT * tid - q);
            *(end ? &sh.rank_lo : &sh.rank) = rem;
            *(end ? &sh.over : &sh.bin) = tot;
        }
    }
    __syncthreads();
}

__global__ void __launch_bounds__(TOPK_THREADS) __attribute__((amdgpu_waves_per_eu(8, 8))) topk_once_kernel(const float* __restrict__ scores, int64_t N, int64_t k,
                                                                 int protect_last, int32_t* __restrict__ idx_out) {
    extern __shared__ __attribute__((aligned(16))) char lsm[];
    int* h13 = reinterpret_cast<int*>(lsm);                                                   // [T13_BINS], the sample's
    uint32_t (*sel)[TOPK_THREADS] = reinterpret_cast<uint32_t (*)[TOPK_THREADS]>(lsm);        // [LONG1_WORDS][1024], after the sample
    uint32_t (*cand)[LONG1_CW] = reinterpret_cast<uint32_t (*)[LONG1_CW]>(lsm + LONG1_BITS);  // [TOPK_WAVES][LONG1_CW], after the sample
    __shared__ TopkShared sh;
    int* const hist = sh.hist;
    scores += (int64_t)blockIdx.x * N;
    idx_out += (int64_t)blockIdx.x * k;
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int n = (int)N;
    const int per_wave = ((n + TOPK_WAVES - 1) / TOPK_WAVES + LONG_STEP - 1) / LONG_STEP * LONG_STEP;   // a wavefront's slice
    // ---- bracket from the sample: two 16-byte pieces per lane, spread evenly
    int* const h8 = h13 + T13_BINS;   // two 256-bin histograms
    uint32_t smp[8];
    {
        const int quads = n / 4;
        f32x4v v[2];
#pragma unroll
        for (int p = 0; p < 2; ++p)
            v[p] = *reinterpret_cast<const f32x4u*>(scores + 4 * (int64_t)((int64_t)(2 * tid + p) * quads / (LONG1_SAMPLES / 4)));
        for (int i = tid; i < T13_BINS; i += TOPK_THREADS) h13[i] = 0;
        if (tid < 512) h8[tid] = 0;
        __syncthreads();
#pragma unroll
        for (int e = 0; e < 8; ++e) {
            smp[e] = order_key(v[e >> 2][e & 3]);
            hist_add(h13, true, (int)(smp[e] >> T13_LOW));
        }
    }
    __syncthreads();
    // (the budgets that come here leave at least 79 ranks of the sample above the bracket and below it)
    const float frac = (float)k / (float)n, r = frac * LONG1_SAMPLES, dev = 4.f * sqrtf(r * (1.f - frac)) + 4.f;
    sample_bins(h13, (int)(r - dev), (int)(r + dev) + 1, sh);
    {
        const uint32_t bh = sh.hi, bl = sh.lo;
        const bool many = sh.bin + sh.over > LONG1_SAMPLES / 2;   // else a few lanes of a wavefront, which need no grouping
#pragma unroll
        for (int e = 0; e < 8; ++e) {
            const bool eh = smp[e] >> T13_LOW == bh, el = smp[e] >> T13_LOW == bl;
            const int b8 = (int)(smp[e] >> 11 & 0xFFu);
            if (many) {
                hist_add(h8, eh, b8);
                hist_add(h8 + 256, el, b8);
            } else {
                if (eh) atomicAdd(&h8[b8], 1);
                if (el) atomicAdd(&h8[256 + b8], 1);
            }
        }
        __syncthreads();
        if (wave == 0) pick_bin(h8, lane, 11, bh << T13_LOW, sh.rank, &sh.hi, &sh.rank);
        if (wave == 1) pick_bin(h8 + 256, lane, 11, bl << T13_LOW, sh.rank_lo, &sh.lo, &sh.rank_lo);
        __syncthreads();
    }
    const uint32_t hi_key = __builtin_amdgcn_readfirstlane(sh.hi) | 0x7FFu, lo_key = __builtin_amdgcn_readfirstlane(sh.lo), width = hi_key - lo_key;
    const int shift = width >> 21 ? 11 - __builtin_clz(width) : 0;   // lower bits of a distance that do not fit in 21
    // A wavefront's samples lie in its own slice (or, where slices are rounded up, its neighbour's): the share of them that the
    // bracket holds, times the slice, has to fit a region (scores in no order of position fill a third of it).
    bool fits = true;
    {
        int in = 0, most = 0;
#pragma unroll
        for (int e = 0; e < 8; ++e) in += (int)__popcll(__ballot(smp[e] - lo_key <= width));
        if (lane == 0) sh.wave_eq[wave] = in;   // (next written two barriers on)
        __syncthreads();
#pragma unroll
        for (int w = 0; w < TOPK_WAVES; ++w) most = sh.wave_eq[w] > most ? sh.wave_eq[w] : most;
        fits = most * per_wave <= LONG1_CW * (LONG1_SAMPLES / TOPK_WAVES);
    }

    // ---- the one sweep: wavefront w owns a contiguous slice
    const int lo = wave * per_wave;
    const int hi = lo + per_wave < n ? lo + per_wave : n;   // of a piece that starts below hi, places past it have key 0
    const int last = protect_last ? n - 1 : -1;
    // Bit 31 - (4 u + e) of word w: element e of the slice's load 8 w + u lies above the bracket (later: is selected).  A key inside the bracket is kept as (key - lo_key) >> shift << 11 | (4 u + e) << 6 | lane;
    // its word follows from the region's fill at the word's end.
    const int words = (fits && hi > lo ? hi - lo + 2 * LONG_STEP - 1 : 0) / (2 * LONG_STEP);   // of this wavefront; none without a sweep
    int cnt = 0, cgt = 0, word_end[LONG1_WORDS];
#pragma unroll
    for (int w = 0; w < LONG1_WORDS; ++w) {
        if (w < words) {
            uint32_t gw = 0;
            // ALL: every score exists and none of them is the protected one
            auto half_word = [&](int half, auto all_tag) {
                constexpr bool ALL = decltype(all_tag)::value;
                const int base = lo + (w * 2 + half) * LONG_STEP;
                f32x4v v[LONG_U];
#pragma unroll
                for (int u = 0; u < LONG_U; ++u) {
                    const int i0 = base + u * 256 + lane * 4;
                    v[u] = *reinterpret_cast<const f32x4u*>(scores + (ALL ? (uint32_t)i0 : (uint32_t)min(i0, n - 4)));
                    if (!ALL && (n & 3) != 0) v[u] = end_piece(v[u], i0, n);
                }
#pragma unroll
                for (int u = 0; u < LONG_U; ++u) {
                    const int i0 = base + u * 256 + lane * 4;
#pragma unroll
                    for (int e = 0; e < 4; ++e) {
                        uint32_t key = order_key(v[u][e]);
                        if (!ALL && i0 + e == last) key = 0xFFFFFFFFu;
                        const uint32_t delta = key - lo_key;
                        const bool in = (ALL || i0 < hi) && delta <= width;
                        gw = (gw << 1) | ((ALL || i0 < hi) && key > hi_key ? 1u : 0u);
                        const uint64_t m = __ballot(in);
                        const int at = __builtin_amdgcn_mbcnt_hi((uint32_t)(m >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)m, cnt));
                        if (in && at < LONG1_CW) cand[wave][at] = (delta >> shift << 11) | (uint32_t)((half * 16 + u * 4 + e) << 6) | (uint32_t)lane;
                        cnt += (int)__popcll(m);
                    }
                }
            };
#pragma unroll
            for (int half = 0; half < 2; ++half) {
                const int base = lo + (w * 2 + half) * LONG_STEP;
                if (base + LONG_STEP <= hi && !(last >= base && last < base + LONG_STEP)) half_word(half, topk_true{});
                else half_word(half, topk_false{});
            }
            sel[w][tid] = gw;
            cgt += __popc(gw);
        }
        word_end[w] = cnt;
    }
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) cgt += __shfl_xor(cgt, off);
    if (lane == 0) { sh.wave_gt[wave] = cgt; sh.wave_in[wave] = cnt; }
    __syncthreads();
    int above = 0, inside = 0;
#pragma unroll
    for (int w = 0; w < TOPK_WAVES; ++w) { above += sh.wave_gt[w]; inside += sh.wave_in[w]; fits &= sh.wave_in[w] <= LONG1_CW; }
    if (!fits || (int64_t)above >= k || (int64_t)above + inside < k) {
        __syncthreads();
        topk_long_rows<true>(scores, N, k, protect_last, idx_out, lsm, sh, (hi_key ^ lo_key) >> 16 == 0 ? (int)(lo_key >> 16) : -1);
        return;
    }
    auto place = [&](uint32_t c, int j) {   // of region entry j = c, in index order inside the slice: word, load, lane, element
        int w = 0;
#pragma unroll
        for (int q = 0; q < LONG1_WORDS - 1; ++q) w += j >= word_end[q] ? 1 : 0;
        const uint32_t ue = (c >> 6) & 31u;
        return ((uint32_t)w << 11) | ((ue >> 2) << 8) | ((c & 63u) << 2) | (ue & 3u);
    };
    // ---- exact threshold among the keys of the bracket: 8 + 8 + 5 bits of their distance from its lower end
    uint32_t prefix = 0;
    int need = (int)(k - above);
    const int cnt64 = (cnt + 63) & ~63;
#pragma unroll
    for (int pass = 0; pass < 3; ++pass) {
        const int shift = pass == 0 ? 24 : pass == 1 ? 16 : 11;
        const uint32_t hi_mask = pass == 0 ? 0u : pass == 1 ? 0xFF000000u : 0xFFFF0000u;
        if (tid < 256) hist[tid] = 0;
        __syncthreads();
        for (int j = lane; j < cnt64; j += 64) {
            const uint32_t c = j < cnt ? cand[wave][j] : 0u;
            hist_add(hist, j < cnt && (c & hi_mask) == prefix, (int)((c >> shift) & (pass == 2 ? 0x1Fu : 0xFFu)));
        }
        __syncthreads();
        if (wave == 0) pick_bin(hist, lane, shift, prefix, need, &sh.prefix, &sh.rank);
        __syncthreads();
        prefix = sh.prefix;
        need = sh.rank;
    }
    uint32_t T = prefix >> 11;   // the threshold's distance from lo_key, as far as the regions keep it
    if (shift > 0) {
        // 8 + 3 more bits among the keys that share those 21, then every entry's distance becomes 2 / 1 / 0: above / equal / below
        auto low_bits = [&](uint32_t c, int j) {
            const int at = lo + (int)place(c, j);
            return ((at < n ? load_key(scores, at, N, protect_last) : 0u) - lo_key) & ((1u << shift) - 1u);
        };
        prefix = 0;
#pragma unroll
        for (int pass = 0; pass < 2; ++pass) {
            if (tid < 256) hist[tid] = 0;
            __syncthreads();
            for (int j = lane; j < cnt64; j += 64) {
                const uint32_t c = j < cnt ? cand[wave][j] : 0u;
                const bool in = j < cnt && c >> 11 == T;
                const uint32_t d = in ? low_bits(c, j) : 0u;
                hist_add(hist, in && (pass == 0 || (d & 0x7F8u) == prefix), (int)(pass == 0 ? d >> 3 : d & 7u));
            }
            __syncthreads();
            if (wave == 0) pick_bin(hist, lane, pass == 0 ? 3 : 0, prefix, need, &sh.prefix, &sh.rank);
            __syncthreads();
            prefix = sh.prefix;
            need = sh.rank;
        }
        for (int j = lane; j < cnt; j += 64) {
            const uint32_t c = cand[wave][j];
            uint32_t order = c >> 11 > T ? 2u : 0u;
            if (c >> 11 == T) {
                const uint32_t d = low_bits(c, j);
                order = d > prefix ? 2u : d == prefix ? 1u : 0u;
            }
            cand[wave][j] = (order << 11) | (c & 0x7FFu);
        }
        T = 1;
    }
    const int need_eq = need;
    int g = 0, ne = 0;
    for (int j = lane; j < cnt64; j += 64) {
        const uint32_t c = j < cnt ? cand[wave][j] >> 11 : 0u;
        g += (int)__popcll(__ballot(j < cnt && c > T));
        ne += (int)__popcll(__ballot(j < cnt && c == T));
    }
    if (lane == 0) sh.wave_eq[wave] = ne;
    __syncthreads();
    int eq_before = 0;
#pragma unroll
    for (int w = 0; w < TOPK_WAVES; ++w) eq_before += w < wave ? sh.wave_eq[w] : 0;
    // ---- the bracket's selected keys join the words.  Of the keys equal to the threshold the first `eq_taken` of this slice are taken; in
    //      the one wavefront where that is some but not all, they get words of their own (where the last histogram was) and are
    //      counted off in index order.
    const int eq_taken = need_eq - eq_before < 0 ? 0 : need_eq - eq_before < ne ? need_eq - eq_before : ne;
    const bool part = eq_taken > 0 && eq_taken < ne;
    uint32_t* const eqw = reinterpret_cast<uint32_t*>(hist);   // [LONG1_WORDS][64]
    static_assert(LONG1_WORDS * 64 <= 256, "the equal keys' words fit the histogram's place");
    if (part) {
#pragma unroll
        for (int w = 0; w < LONG1_WORDS; ++w) eqw[w * 64 + lane] = 0;
    }
    for (int j = lane; j < cnt; j += 64) {
        const uint32_t c = cand[wave][j], at = place(c, j), lane_at = (at >> 2) & 63u, bit = 1u << (31 - (((at >> 8) & 7u) * 4 + (at & 3u)));
        const bool eq = (c >> 11) == T;
        if (eq && part) atomicOr(&eqw[(at >> 11) * 64 + lane_at], bit);
        else if ((c >> 11) > T || (eq && eq_taken > 0)) atomicOr(&sel[at >> 11][wave * 64 + lane_at], bit);
    }
    if (lane == 0) sh.wave_in[wave] = cgt + g + eq_taken;   // selected scores of this slice
    __syncthreads();
    int out = 0;
    for (int w = 0; w < wave; ++w) out += sh.wave_in[w];
    if (part) {
        int seen = 0;
        for (int w = 0; w < words; ++w) {
            const uint32_t ew = eqw[w * 64 + lane];
            uint32_t take = 0;
#pragma unroll
            for (int q = 0; q < 8; ++q) {
                int mine = seen;   // equal keys before this lane's first of load q
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    const uint64_t m = __ballot((ew >> (31 - (q * 4 + e))) & 1u);
                    mine += lane_prefix_popc(m);
                    seen += (int)__popcll(m);
                }
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    const uint32_t bit = ew & (1u << (31 - (q * 4 + e)));
                    if (bit && mine < eq_taken) take |= bit;
                    mine += bit ? 1 : 0;
                }
            }
            sel[w][tid] |= take;
        }
    }

    // ---- ordered index list from the words; index order inside a load is (lane, element e)
    for (int w = 0; w < words; ++w) {
        const uint32_t sw = sel[w][tid];
#pragma unroll
        for (int q = 0; q < 8; ++q) {
            const int i0 = lo + (w * 8 + q) * 256 + lane * 4;
            int at = out;
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                const uint64_t m = __ballot((sw >> (31 - (q * 4 + e))) & 1u);
                at = __builtin_amdgcn_mbcnt_hi((uint32_t)(m >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)m, at));
                out += (int)__popcll(m);
            }
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                const bool s_ = (sw >> (31 - (q * 4 + e))) & 1u;
                if (s_) idx_out[at] = i0 + e;
                at += s_ ? 1 : 0;
            }
        }
    }
}

// ---------------------------------------------------------------------------------------------
// One problem spread over the chip (N up to TOPK_MULTI_MAX_N): the same radix select, but every 8-bit
// pass is its own launch of G workgroups, and no workgroup ever communicates with another one inside
// a launch: no atomics, no fences, no counters, nothing to clear between calls.  Workgroup g owns the
// contiguous slice [g * 1024 * KPT, (g + 1) * 1024 * KPT) (keys in registers for the duration of a
// launch), counts its share of the current digit into a private LDS histogram and stores those 256
// counters as row g of a table in the scratch.  The NEXT launch starts with every workgroup adding
// up the G rows for itself (G * 1 KB from L2, sixteen 16-byte loads in flight per lane) and picking
// the bin -- all workgroups reach the same (prefix, need) because the sums are integers -- before it
// counts the next digit into the other of two tables.  The fifth launch picks the last digit, turns
// the last table into its own output offsets (keys above the threshold and keys equal to it in the
// slices before its own) and writes its piece of the ascending index list.
struct TopkMultiScratch {
    int32_t rows[2][TOPK_MULTI_MAX_WG][256];   // histogram rows of the even / odd passes
    int32_t gt_hi[TOPK_MULTI_MAX_WG];          // last pass: keys of the slice whose decided 24 bits exceed the prefix
    uint32_t prefix[4]; int32_t need[4];       // state after pass p (written by workgroup 0 of launch p + 1)
};
static_assert(sizeof(TopkMultiScratch) <= TOPK_MULTI_SCRATCH_BYTES, "scratch size constant too small");

typedef int i32x4 __attribute__((ext_vector_type(4)));

// hist[0..256) = column sums of the G rows of `table`; all 1024 lanes take part, ends with a barrier
__device__ inline void topk_sum_rows(const int32_t (*table)[256], int G, int (*part)[256], int* hist) {
    const int tid = threadIdx.x;
    const int c4 = (tid & 63) * 4;
    i32x4 sum = {0, 0, 0, 0};
    for (int r = tid >> 6; r < G; r += 16) sum += *(const i32x4*)&table[r][c4];
    *(i32x4*)&part[tid >> 6][c4] = sum;
    __syncthreads();
    if (tid < 256) {
        int t = 0;
#pragma unroll
        for (int q = 0; q < 16; ++q) t += part[q][tid];
        hist[tid] = t;
    }
    __syncthreads();
}

template <int KPT>
__global__ void __launch_bounds__(TOPK_THREADS) topk_multi_hist_kernel(const float* __restrict__ scores, int N, int k,
                                                                       int protect_last, TopkMultiScratch* scr, int pass) {
    __shared__ int hist[256];
    __shared__ __attribute__((aligned(16))) int part[16][256];
    __shared__ uint32_t sh_prefix;
    __shared__ int64_t sh_need;
    __shared__ int wave_cnt[TOPK_WAVES];
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int g = blockIdx.x, G = gridDim.x;
    const int lo = g * (1024 * KPT) + wave * (64 * KPT);
    uint32_t keys[KPT];
#pragma unroll
    for (int j = 0; j < KPT; ++j) {
        const int i = lo + 64 * j + lane;
        keys[j] = i < N ? load_key(scores, i, N, protect_last) : 0u;
    }
    // state after the previous pass: the bin choice the previous launch's table implies
    uint32_t prefix = 0u;
    int64_t need = k;
    if (pass > 0) {
        if (pass > 1) { prefix = scr->prefix[pass - 2]; need = scr->need[pass - 2]; }
        if (tid == 0) { sh_prefix = prefix; sh_need = need; }
        topk_sum_rows(scr->rows[(pass - 1) & 1], G, part, hist);
        if (wave == 0) pick_bin(hist, lane, 24 - 8 * (pass - 1), prefix, need, &sh_prefix, &sh_need);
        __syncthreads();
        prefix = sh_prefix;
        need = sh_need;
        if (g == 0 && tid == 0) { scr->prefix[pass - 1] = prefix; scr->need[pass - 1] = (int32_t)need; }
    }
    const int shift = 24 - 8 * pass;
    const uint32_t hi_mask = pass == 0 ? 0u : (0xFFFFFFFFu << (shift + 8));
    __syncthreads();
    if (tid < 256) hist[tid] = 0;
    __syncthreads();
    int cgt = 0;
#pragma unroll
    for (int j = 0; j < KPT; ++j) {
        const bool valid = lo + 64 * j + lane < N;
        hist_add(hist, valid && (keys[j] & hi_mask) == prefix, (int)((keys[j] >> shift) & 0xFF));
        if (pass == 3) cgt += (int)__popcll(__ballot(valid && (keys[j] & hi_mask) > prefix));
    }
    if (lane == 0) wave_cnt[wave] = cgt;
    __syncthreads();
    if (tid < 256) scr->rows[pass & 1][g][tid] = hist[tid];
    if (tid == 0 && pass == 3) {
        int t = 0;
        for (int w = 0; w < TOPK_WAVES; ++w) t += wave_cnt[w];
        scr->gt_hi[g] = t;
    }
}

template <int KPT>
__global__ void __launch_bounds__(TOPK_THREADS) topk_multi_write_kernel(const float* __restrict__ scores, int N, int protect_last,
                                                                        const TopkMultiScratch* scr, int32_t* __restrict__ idx_out) {
    __shared__ int hist[256];
    __shared__ __attribute__((aligned(16))) int part[16][256];
    __shared__ uint32_t sh_prefix;
    __shared__ int64_t sh_need;
    __shared__ int wave_gt[TOPK_WAVES], wave_eq[TOPK_WAVES];
    __shared__ int red_gt[TOPK_WAVES], red_eq[TOPK_WAVES];
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int g = blockIdx.x, G = gridDim.x;
    const int lo = g * (1024 * KPT) + wave * (64 * KPT);
    uint32_t keys[KPT];
#pragma unroll
    for (int j = 0; j < KPT; ++j) {
        const int i = lo + 64 * j + lane;
        keys[j] = i < N ? load_key(scores, i, N, protect_last) : 0u;
    }
    // the last digit: threshold key T and the number of keys equal to T still to be taken
    const int32_t (*table)[256] = scr->rows[1];
    {
        const uint32_t prefix = scr->prefix[2];
        const int64_t need = scr->need[2];
        if (tid == 0) { sh_prefix = prefix; sh_need = need; }
        topk_sum_rows(table, G, part, hist);
        if (wave == 0) pick_bin(hist, lane, 0, prefix, need, &sh_prefix, &sh_need);
        __syncthreads();
    }
    const uint32_t T = sh_prefix;
    const int need_eq = (int)sh_need;
    const int digit = (int)(T & 0xFFu);
    // keys above T / equal to T in the slices before this one: eight lanes per row of the table, each 32 consecutive
    // bins (eight 16-byte loads), rows at or beyond g contribute nothing
    int row_gt = 0, row_eq = 0;
    {
        const int r = tid >> 3, sub = tid & 7;
        if (r < g) {
#pragma unroll
            for (int q = 0; q < 8; ++q) {
                const int b = sub * 32 + q * 4;
                const i32x4 v = *(const i32x4*)&table[r][b];
                row_gt += (b > digit ? v[0] : 0) + (b + 1 > digit ? v[1] : 0) + (b + 2 > digit ? v[2] : 0) + (b + 3 > digit ? v[3] : 0);
            }
            if (sub == 0) { row_gt += scr->gt_hi[r]; row_eq = table[r][digit]; }
        }
    }
    int cgt = 0, ceq = 0;
#pragma unroll
    for (int j = 0; j < KPT; ++j) {
        const bool valid = lo + 64 * j + lane < N;
        cgt += (int)__popcll(__ballot(valid && keys[j] > T));
        ceq += (int)__popcll(__ballot(valid && keys[j] == T));
    }
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) { row_gt += __shfl_xor(row_gt, off); row_eq += __shfl_xor(row_eq, off); }
    if (lane == 0) { wave_gt[wave] = cgt; wave_eq[wave] = ceq; red_gt[wave] = row_gt; red_eq[wave] = row_eq; }
    __syncthreads();
    int gt_before = 0, eq_before = 0;
    for (int w = 0; w < TOPK_WAVES; ++w) { gt_before += red_gt[w]; eq_before += red_eq[w]; }
    for (int w = 0; w < wave; ++w) { gt_before += wave_gt[w]; eq_before += wave_eq[w]; }
#pragma unroll
    for (int j = 0; j < KPT; ++j) {
        const int i = lo + 64 * j + lane;
        const bool valid = i < N;
        const bool gt = valid && keys[j] > T, eq = valid && keys[j] == T;
        const uint64_t mgt = __ballot(gt), meq = __ballot(eq);
        const int my_gt = gt_before + lane_prefix_popc(mgt);
        const int my_eq = eq_before + lane_prefix_popc(meq);
        if (gt || (eq && my_eq < need_eq)) idx_out[my_gt + (my_eq < need_eq ? my_eq : need_eq)] = i;
        gt_before += (int)__popcll(mgt);
        eq_before += (int)__popcll(meq);
    }
}

template <int KPT>
static hipError_t topk_multi_launch(const float* scores, int N, int k, int protect_last, int32_t* idx_out,
                                    TopkMultiScratch* scr, hipStream_t s) {
    const int G = (N + 1024 * KPT - 1) / (1024 * KPT);
    for (int pass = 0; pass < 4; ++pass)
        topk_multi_hist_kernel<KPT><<<dim3(G), dim3(TOPK_THREADS), 0, s>>>(scores, N, k, protect_last, scr, pass);
    topk_multi_write_kernel<KPT><<<dim3(G), dim3(TOPK_THREADS), 0, s>>>(scores, N, protect_last, scr, idx_out);
    return hipGetLastError();
}

// Scratch of the no-allocation entry point: one array per GPU, in the code object's own device memory.  Nothing in it
// has to start at zero: every word a call reads was written earlier in the same call.
static __device__ __align__(256) __attribute__((used)) unsigned char scratch[TOPK_MULTI_SCRATCH_BYTES];

hipError_t topk_static_scratch(void** out) {
    // In host code the array's name is only a handle for the runtime: the address a kernel can use comes from
    // hipGetSymbolAddress, once per device (every GPU holds its own copy at its own address).
    constexpr int MAX_DEV = 64;
    static std::mutex mtx;
    static void* dev_ptr[MAX_DEV] = {};
    int dev = 0;
    hipError_t e = hipGetDevice(&dev);
    if (e != hipSuccess) return e;
    if (dev < 0 || dev >= MAX_DEV) return hipErrorInvalidDevice;
    std::lock_guard<std::mutex> lock(mtx);
    if (!dev_ptr[dev]) {
        void* p = nullptr;
        e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
        if (e != hipSuccess) return e;
        if (!p) return hipErrorInvalidSymbol;
        dev_ptr[dev] = p;
    }
    *out = dev_ptr[dev];
    return hipSuccess;
}

hipError_t launch_topk_multi(const float* scores, int64_t N, int64_t k, int protect_last, int32_t* idx_out, void* scratch,
                             hipStream_t s) {
    if (k <= 0 || N <= 0) return hipSuccess;
    if (N > TOPK_MULTI_MAX_N || k > N || !scratch) return hipErrorInvalidValue;
    TopkMultiScratch* scr = (TopkMultiScratch*)scratch;
    // slices of 4096 keys (32 workgroups at N = 131072: every workgroup re-adds all rows of the table, so a small
    // grid keeps that cheap); longer rows take 8192 so that the grid stays within the table
    if (N <= (int64_t)TOPK_MULTI_MAX_WG * 4096) return topk_multi_launch<4>(scores, (int)N, (int)k, protect_last, idx_out, scr, s);
    return topk_multi_launch<8>(scores, (int)N, (int)k, protect_last, idx_out, scr, s);
}

// ---------------------------------------------------------------------------------------------
// Mean of the k largest |values| of every row of a [rows, T] matrix (Eq. (channel_importance): the
// importance of an FFN channel is the mean of the top-rho fraction of its saliencies over the
// calibration tokens; rows = channels).  Same radix select as above on the keys of |v| (exact
// k-th value and how many copies of it count), then a sum of everything above it in a fixed order
// (per lane, shuffle tree, wavefronts in order): deterministic.  One workgroup per row; the row is
// re-read in every sweep and stays in L2 meanwhile.
template <typename T>
__global__ void __launch_bounds__(TOPK_THREADS) topk_mean_kernel(const T* __restrict__ vals, int64_t ld, int64_t n, int64_t k,
                                                                 float* __restrict__ out) {
    __shared__ int hist[256];
    __shared__ uint32_t sh_prefix;
    __shared__ int64_t sh_need;
    __shared__ float wsum[TOPK_WAVES];
    const T* row = vals + (int64_t)blockIdx.x * ld;
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    if (tid == 0) { sh_prefix = 0; sh_need = k; }
    uint32_t prefix = 0;
    int64_t need = k;
    // bf16 values widen to keys whose low 16 bits are zero: two 8-bit passes decide the whole key
    constexpr int NPASS = sizeof(T) == 2 ? 2 : 4;
    for (int pass = 0; pass < NPASS; ++pass) {
        const int shift = 24 - 8 * pass;
        const uint32_t hi_mask = pass == 0 ? 0u : (0xFFFFFFFFu << (shift + 8));
        if (tid < 256) hist[tid] = 0;
        __syncthreads();
        for (int64_t base = 0; base < n; base += TOPK_THREADS) {
            const int64_t i = base + tid;
            const uint32_t key = i < n ? order_key(fabsf(to_f32(row[i]))) : 0u;
            hist_add(hist, i < n && (key & hi_mask) == prefix, (int)((key >> shift) & 0xFF));
        }
        __syncthreads();
        if (wave == 0) pick_bin(hist, lane, shift, prefix, need, &sh_prefix, &sh_need);
        __syncthreads();
        prefix = sh_prefix;
        need = sh_need;
    }
    const uint32_t Tk = prefix;       // key of the k-th largest |value|
    float s = 0.f, tval = 0.f;
    for (int64_t base = 0; base < n; base += TOPK_THREADS) {
        const int64_t i = base + tid;
        if (i < n) {
            const float v = fabsf(to_f32(row[i]));
            const uint32_t key = order_key(v);
            if (key > Tk) s += v;
            if (key == Tk) tval = v;
        }
    }
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) { s += __shfl_xor(s, off); tval = fmaxf(tval, __shfl_xor(tval, off)); }
    __shared__ float wt[TOPK_WAVES];
    if (lane == 0) { wsum[wave] = s; wt[wave] = tval; }
    __syncthreads();
    if (tid == 0) {
        float tot = 0.f, tv = 0.f;
        for (int w = 0; w < TOPK_WAVES; ++w) { tot += wsum[w]; tv = fmaxf(tv, wt[w]); }
        out[blockIdx.x] = (tot + (float)need * tv) / (float)k;
    }
}

// Rows of at most 64 * KPT values: one wavefront per row, the row read once into registers.  The key of the k-th largest |value| lies between a key that k keys
// reach and one that fewer do, and the two close in: first to either side of the same quantile of 256 of the keys, as far as its error and the usual slope of such
// a row suggest and then eight times as far each time, after that to their middle.  What is found does not depend on the guesses.  Up to 1024 values in bf16 the
// key's 15 bits are decided one by one instead.
// Counting is one compare per key whose lane mask is summed on the scalar unit, so there are no histograms, no LDS and no
// barrier.  The scalar unit is what that runs out of (two instructions a key against one), so every third key is counted on the
// vector unit instead (one more), lane by lane.  Bound: the counts, and one read of the row (20 us for 14336 rows of 4096).  Measured there: 283 us with
// the workgroup-per-row kernel above (two histogram passes over 1024-lane strides), 72 with a count for each of a key's 15 bits, 45 here (1000
// values to a row of 18944: 26).  14336 rows of 256 / 1000 / 2048 / 4096 products of two normal values, k a fifth: bf16 bit by bit 11.9 / 18.8 / 31.0 / 58, from
// the sample 15.2 / 18.9 / 26 / 42; fp32 31 / 35 / 55 / 108 and 17 / 24 / 36 / 63.  Rows that are one value repeated end later than those: 2048 in bf16 36.6, in fp32 50.
template <typename T, int KPT>
__global__ void __launch_bounds__(256) topk_mean_wave_kernel(const T* __restrict__ vals, int64_t ld, int64_t rows, int n, int k, int wide,
                                                             float* __restrict__ out) {
    constexpr int VN = 16 / (int)sizeof(T), BITS = sizeof(T) == 2 ? 15 : 31;
    static_assert(KPT % VN == 0, "whole 16-byte loads");
    const int64_t r = (int64_t)blockIdx.x * 4 + (threadIdx.x >> 6);
    if (r >= rows) return;
    const int lane = threadIdx.x & 63;
    const T* row = vals + r * ld;
    auto key_of = [](uint32_t raw) { return raw & (sizeof(T) == 2 ? 0x7fffu : 0x7fffffffu); };   // order of |v|; slots past n hold key 0
    uint32_t key[KPT];
    if (wide) {   // rows at 16-byte addresses
#pragma unroll
        for (int j = 0; j < KPT / VN; ++j) {
            const int i0 = (j * 64 + lane) * VN;
            u32x4 v = {0u, 0u, 0u, 0u};
            if (i0 + VN <= n) v = *reinterpret_cast<const u32x4*>(row + i0);
            else
                for (int e = 0; e < VN; ++e)
                    if (i0 + e < n) {
                        const uint32_t raw = sizeof(T) == 2 ? (uint32_t)reinterpret_cast<const uint16_t*>(row)[i0 + e] : reinterpret_cast<const uint32_t*>(row)[i0 + e];
                        if (sizeof(T) == 2) v[e >> 1] |= raw << (16 * (e & 1)); else v[e] = raw;
                    }
#pragma unroll
            for (int e = 0; e < VN; ++e) key[j * VN + e] = key_of(sizeof(T) == 2 ? v[e >> 1] >> (16 * (e & 1)) : v[e]);
        }
    } else {
#pragma unroll
        for (int j = 0; j < KPT; ++j) {
            const int i = j * 64 + lane;
            key[j] = i < n ? key_of(sizeof(T) == 2 ? (uint32_t)reinterpret_cast<const uint16_t*>(row)[i] : reinterpret_cast<const uint32_t*>(row)[i]) : 0u;
        }
    }
    auto reach = [&](uint32_t c) {   // keys that reach c
        int cnt = 0, mine = 0;
#pragma unroll
        for (int j = 0; j < KPT; ++j) {
            if (j % 3 == 2) mine += key[j] >= c ? 1 : 0;
            else cnt += (int)__popcll(__ballot(key[j] >= c));
        }
        return cnt + (int)wave_reduce_u32((uint32_t)mine, 0u, [](uint32_t a, uint32_t b) { return a + b; });
    };
    uint32_t t = 0;
    if constexpr (BITS == 15 && KPT <= 16) {   // bit by bit: a count costs no more than the sample's share of the other way
        for (int b = BITS - 1; b >= 0; --b) {
            const uint32_t c = t | (1u << b);
            if (reach(c) >= k) t = c;
        }
    } else {
        uint32_t guess = 0;
        const int rank = (int)(((int64_t)k * 4 + KPT - 1) / KPT);   // of 256 keys out of 64 KPT
        for (int b = BITS - 1; b > BITS - 16; --b) {
            const uint32_t c = guess | (1u << b);
            int cnt = 0;
#pragma unroll
            for (int q = 0; q < 4; ++q) cnt += (int)__popcll(__ballot(key[KPT / 4 * q] >= c));
            if (cnt >= rank) guess = c;
        }
        uint32_t end = 1u << BITS, c = guess > 0 ? guess : 1u, step = 0;   // k keys or more reach t, fewer end
        int at_t = 64 * KPT + 1;   // keys that reach t (0: all)
        bool up = false, closing = false;
        for (int left = 16; (BITS == 15 || left > 0) && end - t > 1 && at_t != k; --left) {
            const int cnt = reach(c);
            const bool enough = cnt >= k;
            if (enough) { t = c; at_t = cnt; } else end = c;
            if (step == 0) {   // twice as far as it is where keys thin out to a third within an octave
                const float octaves = fminf((float)(enough ? cnt - k : k - cnt) / (float)k, 64.f);
                step = (uint32_t)(octaves * (float)(2 << (BITS - 8))) + (2u << (BITS - 15));   // (0.7 / 1 / 1.4 octaves for that: 46 / 47 / 46 us, two 45)
                up = enough;
            } else closing = closing || up != enough;
            const uint32_t room = end - t;
            if (closing || step >= room) { c = t + room / 2; closing = true; }
            else { c = up ? t + step : end - step; step *= 8; }
        }
        // fp32, and not there yet: few values, or rare ones, and up to 30 bits between them.  The ends move to the outermost keys, and then to their
        // middle for some rounds.  (In bf16 there are 15 bits in all.)
        while (BITS == 31 && end - t > 1 && at_t != k) {
            uint32_t mn = 0xFFFFFFFFu, mx = 0u;
#pragma unroll
            for (int j = 0; j < KPT; ++j) {
                const uint32_t d = key[j] - t;
                const bool in = d < end - t;
                mn = min(mn, in ? d : 0xFFFFFFFFu);
                mx = max(mx, in ? d : 0u);
            }
            mn = wave_reduce_u32(mn, 0xFFFFFFFFu, [](uint32_t a, uint32_t b) { return min(a, b); });
            mx = wave_reduce_u32(mx, 0u, [](uint32_t a, uint32_t b) { return max(a, b); });
            end = t + mx + 1;
            t += mn;
            if (mn == mx) break;
            for (int left = 6; left > 0 && end - t > 1 && at_t != k; --left) {
                c = t + (end - t) / 2;
                const int cnt = reach(c);
                if (cnt >= k) { t = c; at_t = cnt; } else end = c;
            }
        }
        if (at_t == k && end - t > 1) {   // exactly k keys reach t: the smallest of them
            uint32_t mn = 0xFFFFFFFFu;
#pragma unroll
            for (int j = 0; j < KPT; ++j) mn = min(mn, key[j] >= t ? key[j] : 0xFFFFFFFFu);
            t = wave_reduce_u32(mn, 0xFFFFFFFFu, [](uint32_t a, uint32_t b) { return min(a, b); });
        }
    }
    auto value = [](uint32_t q) { return __uint_as_float(sizeof(T) == 2 ? q << 16 : q); };
    float s = 0.f;
    int above = 0;
#pragma unroll
    for (int j = 0; j < KPT; ++j) {
        above += (int)__popcll(__ballot(key[j] > t));
        s += key[j] > t ? value(key[j]) : 0.f;
    }
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) s += __shfl_xor(s, off);   // fixed order
    if (lane == 0) out[r] = (s + (float)(k - above) * value(t)) / (float)k;
}

template <typename T>
static bool launch_topk_mean_wave(const T* vals, int64_t ld, int64_t rows, int64_t n, int64_t k, float* out, hipStream_t s) {
    constexpr int MAXK = sizeof(T) == 2 ? 128 : 64;   // registers: two or more wavefronts per SIMD
    if (n > 64 * MAXK || rows > (int64_t)1 << 32) return false;
    const dim3 g((unsigned)((rows + 3) / 4)), b(256);
    const int wide = (ld * (int)sizeof(T)) % 16 == 0 && (reinterpret_cast<uintptr_t>(vals) & 15u) == 0;
    if (n <= 64 * 8) topk_mean_wave_kernel<T, 8><<<g, b, 0, s>>>(vals, ld, rows, (int)n, (int)k, wide, out);
    else if (n <= 64 * 16) topk_mean_wave_kernel<T, 16><<<g, b, 0, s>>>(vals, ld, rows, (int)n, (int)k, wide, out);
    else if (n <= 64 * 32) topk_mean_wave_kernel<T, 32><<<g, b, 0, s>>>(vals, ld, rows, (int)n, (int)k, wide, out);
    else if (n <= 64 * 64) topk_mean_wave_kernel<T, 64><<<g, b, 0, s>>>(vals, ld, rows, (int)n, (int)k, wide, out);
    else topk_mean_wave_kernel<T, MAXK><<<g, b, 0, s>>>(vals, ld, rows, (int)n, (int)k, wide, out);
    return true;
}

hipError_t launch_topk_mean(const void* vals, int64_t ld, int64_t rows, int64_t n, int64_t k, float* out, bool bf16,
                            hipStream_t s) {
    if (rows <= 0 || n <= 0 || k <= 0) return hipSuccess;
    if (bf16 ? launch_topk_mean_wave((const bf16_t*)vals, ld, rows, n, k, out, s) : launch_topk_mean_wave((const float*)vals, ld, rows, n, k, out, s))
        return hipGetLastError();
    const dim3 g((unsigned)rows), b(TOPK_THREADS);
    if (bf16) topk_mean_kernel<bf16_t><<<g, b, 0, s>>>((const bf16_t*)vals, ld, n, k, out);
    else topk_mean_kernel<float><<<g, b, 0, s>>>((const float*)vals, ld, n, k, out);
    return hipGetLastError();
}

hipError_t launch_topk(const float* scores, int64_t N, int64_t k, int protect_last, int32_t* idx_out, int batch,
                       hipStream_t s, TopkSegments seg, TopkMap map) {
    // with segments N is the longest segment (it picks the kernel variant) and k is ignored
    if ((k <= 0 && !seg.offsets) || N <= 0 || batch <= 0) return hipSuccess;
    if (map.out && (seg.offsets || N > TOPK_ONE_MAX_N)) return hipErrorInvalidValue;
    const dim3 g((unsigned)batch), b(TOPK_THREADS);
    if (N <= TOPK_REG_MAX_N) {
        // The smallest of these workgroups that holds the row: a round costs a compare per slot, empty or not, and 16 wavefronts wait
        // longer for one another than 8 (4000 scores: 6.6 us with 8 x 8 slots, 7.3 with 4 x 16; 6000: 8.2 with 6 x 16, 8.6 with 12 x 8).
#define SPTS_TOPK_REG(KPT, W)                                                                                              \
    do {                                                                                                                   \
        if (map.out) topk_reg_kernel<KPT, W, true><<<g, dim3(64 * W), 0, s>>>(scores, N, k, protect_last, idx_out, seg, map); \
        else topk_reg_kernel<KPT, W, false><<<g, dim3(64 * W), 0, s>>>(scores, N, k, protect_last, idx_out, seg, map);        \
    } while (0)
        if (N <= 512) SPTS_TOPK_REG(2, 4);
        else if (N <= 1024) SPTS_TOPK_REG(4, 4);
        else if (N <= 2048) SPTS_TOPK_REG(4, 8);
        else if (N <= 3072) SPTS_TOPK_REG(6, 8);
        else if (N <= 4096) SPTS_TOPK_REG(8, 8);
        else if (N <= 6144) SPTS_TOPK_REG(6, 16);
        else if (N <= 8192) SPTS_TOPK_REG(8, 16);
        else if (N <= 12288) SPTS_TOPK_REG(12, 16);
        else if (N <= 16384) SPTS_TOPK_REG(16, 16);
        else if (N <= 20480) SPTS_TOPK_REG(20, 16);
        else if (N <= 24576) topk_reg_kernel<24, 16, false><<<g, b, 0, s>>>(scores, N, k, protect_last, idx_out, seg, map);   // (no map)
        else topk_reg_kernel<32, 16, false><<<g, b, 0, s>>>(scores, N, k, protect_last, idx_out, seg, map);
#undef SPTS_TOPK_REG
    }
    else if (!seg.offsets && N < ((int64_t)1 << 30)) {
        // the bracket needs sample ranks on both of its sides: budgets between 1/64 and 63/64 of the row (k = 0.5 % of 512 x 131072: three
        // sweeps, 152 us)
        if (N <= LONG1_MAX_N && k * 64 >= N && (N - k) * 64 >= N) {
            hipError_t e = ensure_dynamic_lds(reinterpret_cast<const void*>(&topk_once_kernel), T13_LDS_BYTES);
            if (e != hipSuccess) return e;
            topk_once_kernel<<<g, b, T13_LDS_BYTES, s>>>(scores, N, k, protect_last, idx_out);
        } else {
            hipError_t e = ensure_dynamic_lds(reinterpret_cast<const void*>(&topk_long_kernel), T13_LDS_BYTES);
            if (e != hipSuccess) return e;
            topk_long_kernel<<<g, b, T13_LDS_BYTES, s>>>(scores, N, k, protect_last, idx_out);
        }
    }
    else topk_kernel<<<g, b, 0, s>>>(scores, N, k, protect_last, idx_out, seg);
    return hipGetLastError();
}

}  // namespace spts
