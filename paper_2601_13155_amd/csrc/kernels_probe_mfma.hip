// PAP probe scoring on the matrix cores (Eq. (mha_importance) with a probe window of P rows):
//   S[n] = 1/(P*H) * sum over probe rows (p, h) of softmax_n( qp[p,h].k[n,g(h)] / sqrt(d) )[n],
// probe row p being candidate N-P+p, which sees candidates 0..N-P+p.
//
// A softmax needs the full-row denominator before any probability can be averaged over rows, so
// K is streamed twice:
//   pass 1  per (kv head g, chunk of keys): (max, sum-exp) of every probe row of that
//           head group over the chunk  ->  stats_part[chunk][g][row]
//   combine per (g, row): global max M and 1/sum over the chunks; where those are few every workgroup of pass 2 does it for itself
//   pass 2  per (g, chunk): logits again, p = exp2(s - M) / L summed over the rows of the group
//           ->  part[g][n];   final: S[n] = sum_g part[g][n] / (P*H)   (fixed order: deterministic)
// The R = P*H/Hkv probe rows of one KV head form a dense [R x d] operand that stays in registers
// (32*RB rows per wavefront); K tiles of 64 keys go through LDS (swizzled, shared by the 4
// wavefronts).  The scores of a sequence are the same bits alone and inside any batch, although both the chunk length and who combines
// depend on the whole call: the statistics of 64-key tiles always meet in the same tree (pairs, groups of 256 keys, the
// groups over JOIN_LANES lanes).  Pass 1 computes S^T = K Q^T (one probe row per lane column: row max in-lane),
// pass 2 computes S = Q K^T (one key per lane column: the sum over rows is in-lane).
// Up to 512 rows per kv head are one workgroup's; more (7 query heads per kv head x 128 probe rows = 896, say) are dealt to
// row groups of 512 (grid z), each of which streams K for itself and leaves its own part[group][g][n].  (They used to take the
// fp32 kernels: a layer of 8192 tokens with 896 probe rows per kv head, 64.4 -> 2.03 ms.)
#include "spts_internal.h"

#include <type_traits>

namespace spts {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float f32x16 __attribute__((ext_vector_type(16)));

constexpr int PKV = 64;          // keys per tile
constexpr int CHUNK_MAX = 256;   // keys of the longest chunk: a group of tiles
// Chunks up to which pass 2 combines their statistics itself: every workgroup then reads 8 bytes per row and chunk once more, which is less
// than a launch of its own.  Pass 2 with the combine before it -> with it inside: 32 chunks 19.4 -> 16.9 us, 24 sequences of at most
// 6 chunks 23.3 -> 13.9; 64 chunks cost 33 (with two passes over the statistics).
constexpr int FOLD_CHUNKS = 32;

// Statistics of a probe row over some keys: the largest exponent, and the sum of 2^(exponent - m).  join() is the same roundings
// wherever two halves of a group meet, and joining nothing changes no bit.  Both passes with one tree for every chunk length, against
// running sums in the chunk and whatever order suited each of the two combines: 333 candidates 20.2 -> 20.3 us, 1000 21.3 -> 21.7,
// 8192 37.4 -> 38.1, 20000 71 -> 66, 32768 87.5 -> 84, 24 ragged sequences 35.0 -> 34.6.
struct RowStats { float m, l; };
__device__ constexpr RowStats NO_KEYS{-INFINITY, 0.f};
__device__ __forceinline__ RowStats join(RowStats a, RowStats b) {
    const bool up = a.m >= b.m;
    const float hi = fmaxf(a.m, b.m), lo = fminf(a.m, b.m);
    const float e = lo == -INFINITY ? 0.f : __builtin_amdgcn_exp2f(lo - hi);
    return RowStats{hi, fmaf(up ? b.l : a.l, e, up ? a.l : b.l)};
}

// a group from the PG chunks it was cut into
template <int PG>
__device__ __forceinline__ RowStats group_of(const RowStats* c) {
    if constexpr (PG == 1) return c[0];
    else if constexpr (PG == 2) return join(c[0], c[1]);
    else return join(join(c[0], c[1]), join(c[2], c[3]));
}
// The groups of a row meet in JOIN_LANES lanes: lane i joins groups i, i + JOIN_LANES, ... in turn, then the lanes meet in halves.
// Here by one thread, for a row of at most FOLD_CHUNKS chunks, PG to a group; sp: the row's first chunk, `step` floats to the next.
constexpr int JOIN_LANES = 8;
template <int PG>
__device__ __forceinline__ RowStats join_chunks(const float* sp, int64_t step, int nchunks) {
    RowStats acc[JOIN_LANES];
#pragma unroll
    for (int u = 0; u < JOIN_LANES; ++u) acc[u] = NO_KEYS;
#pragma unroll
    for (int c0 = 0; c0 < FOLD_CHUNKS; c0 += 8) {
        if (c0 >= nchunks) break;
        RowStats cs[8];
#pragma unroll
        for (int u = 0; u < 8; ++u) {
            const float2 v = *reinterpret_cast<const float2*>(sp + (c0 + u < nchunks ? c0 + u : nchunks - 1) * step);
            cs[u] = c0 + u < nchunks ? RowStats{v.x, v.y} : NO_KEYS;
        }
#pragma unroll
        for (int u = 0; u < 8; u += PG) {
            const RowStats g = group_of<PG>(cs + u);
            const int q = (c0 + u) / PG;
            acc[q % JOIN_LANES] = q < JOIN_LANES ? g : join(acc[q % JOIN_LANES], g);
        }
    }
#pragma unroll
    for (int off = JOIN_LANES / 2; off > 0; off >>= 1)
#pragma unroll
        for (int u = 0; u < off; ++u) acc[u] = join(acc[u], acc[u + off]);
    return acc[0];
}

// last b with pref[b] <= i (pref ascending, pref[0] = 0, i < pref[n])
__device__ inline int segment_of(const int64_t* pref, int n, int64_t i) {
    int lo = 0, hi = n;
    while (hi - lo > 1) {
        const int mid = (lo + hi) >> 1;
        if (pref[mid] <= i) lo = mid; else hi = mid;
    }
    return lo;
}

template <int D> struct ProbeLds {
    static constexpr int CPRK = D / 8;
    static constexpr int RPK = 256 / (2 * D);
    static constexpr int K_BYTES = PKV * D * 2;
    __device__ static inline int koff(int row, int c) { return row * (2 * D) + ((c ^ ((row / RPK) % CPRK)) << 4); }
};

// Offset that turns a logit's exponent into the probability's, log2(1 / L) - M; -inf for a row that weighs nothing
__device__ inline float probe_offset(float M, float inv_l) { return inv_l > 0.f ? __builtin_amdgcn_logf(inv_l) - M : -INFINITY; }

// stats_part: [nchunks][Hkv][Rp][2]; stats: [Hkv][Rp][2] (M, 1/L), or null where pass 2 combines stats_part itself; part: [Hkv][Np]
// NWV wavefronts per workgroup, 32 * RB probe rows each.  Two wavefronts per SIMD are asked of the register allocator
// where the rows fit (RB <= 2; left alone it used 270-280 registers and ran one).
template <int D, int RB, int PASS, int NWV>
__global__ void __launch_bounds__(64 * NWV) __attribute__((amdgpu_waves_per_eu(RB <= 2 ? 2 : 1, 8))) probe_mfma_kernel(ProbeArgs a, int Rp, int64_t Np, float qmul, int chunk_keys, int nchunks,
                                                         float* __restrict__ stats_part, const float* __restrict__ stats, ProbeSegments seg) {
    using L = ProbeLds<D>;
    constexpr int KS = D / 16;
    __shared__ __attribute__((aligned(16))) char sK[2][L::K_BYTES];
    constexpr int NT = 64 * NWV;
    __shared__ float sRed[NWV][PKV];
    __shared__ float sOff[PASS == 2 ? 32 * RB * NWV : 1];

    // one sequence, or the sequence of a batch that this chunk belongs to
    int chunk = blockIdx.x;
    const int g = blockIdx.y;
    int64_t seq_row0 = 0;
    const bf16_t* Q = (const bf16_t*)a.qp;
    if (seg.n > 0) {
        const int b = segment_of(seg.chunk, seg.n, blockIdx.x);
        chunk = (int)(blockIdx.x - seg.chunk[b]);
        seq_row0 = seg.off[b];
        a.N = seg.off[b + 1] - seq_row0;
        Q += (int64_t)b * a.P * a.H * D;
        if (PASS == 2) {
            if (stats) stats += (int64_t)b * a.Hkv * Rp * 2;
            nchunks = __builtin_amdgcn_readfirstlane((int)(seg.chunk[b + 1] - seg.chunk[b]));
            stats_part += seg.chunk[b] * a.Hkv * Rp * 2;
        }
    }
    const int row_base = (int)blockIdx.z * (32 * RB * NWV);   // first probe row of this row group
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int l32 = lane & 31, lh = lane >> 5;
    const int grp = a.H / a.Hkv;
    const int R = a.P * grp;
    const int64_t key_begin = (int64_t)chunk * chunk_keys;
    const int64_t key_end = key_begin + chunk_keys < a.N ? key_begin + chunk_keys : a.N;
    const int n_tiles = (int)((key_end - key_begin + PKV - 1) / PKV);

    // ---- probe-row fragments: row rr = p * grp + hg  <->  qp[p, g*grp + hg, :]
    bf16x8 qf[RB][KS];
    int vis_last[RB];   // last candidate index visible to the lane's row in block rb (pass 1 layout)
#pragma unroll
    for (int rb = 0; rb < RB; ++rb) {
        int rr = row_base + wave * 32 * RB + rb * 32 + l32;
        int rc = rr < R ? rr : R - 1;
        int p = rc / grp, hg = rc % grp;
        vis_last[rb] = rr < R ? (int)(a.N - a.P + p) : -1;
        const bf16_t* qr = Q + ((int64_t)p * a.H + g * grp + hg) * D + 8 * lh;
#pragma unroll
        for (int ks = 0; ks < KS; ++ks) qf[rb][ks] = *reinterpret_cast<const bf16x8*>(qr + 16 * ks);
        // qp normally arrives carrying log2(e)/sqrt(d) (qmul == 1): the logits leave the matrix core as exponents of 2;
        // otherwise the rest of the factor is folded in here (a second bf16 rounding)
        if (qmul != 1.0f) {
#pragma unroll
            for (int ks = 0; ks < KS; ++ks) {
                u32x4 raw = __builtin_bit_cast(u32x4, qf[rb][ks]);
#pragma unroll
                for (int j = 0; j < 4; ++j)
                    raw[j] = cvt_pk_bf16(__uint_as_float(raw[j] << 16) * qmul, __uint_as_float(raw[j] & 0xffff0000u) * qmul);
                qf[rb][ks] = __builtin_bit_cast(bf16x8, raw);
            }
        }
    }
    // pass 2: the lane's 16 rows per block keep their exponent offset log2(1/L) - M in registers, laid out as the C operand
    // that starts a block's product: the MFMA then delivers log2 of the probability itself (padded rows and empty rows:
    // offset -inf, probability 0)
    f32x16 coff[PASS == 2 ? RB : 1];
    // ... and, for the tiles that reach into the probe window, (window row p of the register's probe row) + 1, two per
    // register: candidate N - P + j is hidden from the row when j >= p + 1 (0 for padded rows, whose offset is -inf anyway)
    uint32_t pvis[PASS == 2 ? RB : 1][8];
    if (PASS == 2) {
        for (int i = tid; i < 32 * RB * NWV; i += NT) {
            const int rr = row_base + i;
            if (stats) {
                const float2 st = *reinterpret_cast<const float2*>(stats + ((int64_t)g * Rp + rr) * 2);
                sOff[i] = probe_offset(st.x, st.y);
            } else {
                const float* sp = stats_part + ((int64_t)g * Rp + rr) * 2;
                const int64_t step = (int64_t)a.Hkv * Rp * 2;
                const RowStats all = chunk_keys == CHUNK_MAX ? join_chunks<1>(sp, step, nchunks)
                                     : chunk_keys == CHUNK_MAX / 2 ? join_chunks<2>(sp, step, nchunks) : join_chunks<4>(sp, step, nchunks);
                sOff[i] = rr < R && all.l > 0.f ? probe_offset(all.m, 1.0f / all.l) : -INFINITY;
            }
        }
        __syncthreads();
#pragma unroll
        for (int rb = 0; rb < RB; ++rb)
#pragma unroll
            for (int r = 0; r < 16; ++r) {
                const int in = wave * 32 * RB + rb * 32 + 8 * (r >> 2) + 4 * lh + (r & 3), rr = row_base + in;
                coff[rb][r] = sOff[in];
                const uint32_t enc = rr < R ? (uint32_t)(rr / grp + 1) : 0u;
                if (r & 1) pvis[rb][r >> 1] |= enc << 16; else pvis[rb][r >> 1] = enc;
            }
    }

    constexpr int KCH = PKV * L::CPRK / NT;
    static_assert(KCH >= 1, "a key tile gives every thread at least one 16-byte chunk");
    const int kc = tid % L::CPRK, kr = tid / L::CPRK;
    const bf16_t* Kg = (const bf16_t*)a.k + seq_row0 * a.Hkv * (int64_t)D;
    u32x4 rk[KCH];
    auto load_tile = [&](int t) {
#pragma unroll
        for (int i = 0; i < KCH; ++i) {
            int64_t key = key_begin + (int64_t)t * PKV + kr + (NT / L::CPRK) * i;
            if (key >= a.N) key = a.N - 1;
            rk[i] = *reinterpret_cast<const u32x4*>(Kg + (key * a.Hkv + g) * (int64_t)D + kc * 8);
        }
    };
    auto store_tile = [&](int stage) {
#pragma unroll
        for (int i = 0; i < KCH; ++i) *reinterpret_cast<u32x4*>(sK[stage] + L::koff(kr + (NT / L::CPRK) * i, kc)) = rk[i];
    };

    RowStats first[RB], pair[RB];   // pass 1: the chunk's first two tiles, the two in hand
#pragma unroll
    for (int rb = 0; rb < RB; ++rb) first[rb] = pair[rb] = NO_KEYS;

    const int64_t first_masked = a.N - a.P + 1;   // candidates from here on are hidden from some probe row
    if (n_tiles > 0) { load_tile(0); store_tile(0); }
    __syncthreads();
    for (int t = 0; t < n_tiles; ++t) {
        if (t + 1 < n_tiles) load_tile(t + 1);
        const char* sk = sK[t & 1];
        const int64_t key0 = key_begin + (int64_t)t * PKV;
        const bool need_mask = key0 + PKV > first_masked || key0 + PKV > a.N;
        if (PASS == 1) {
            if (t == 2) {
#pragma unroll
                for (int rb = 0; rb < RB; ++rb) first[rb] = pair[rb];
            }
#pragma unroll
            for (int rb = 0; rb < RB; ++rb) {
                f32x16 s[2];
#pragma unroll
                for (int kb = 0; kb < 2; ++kb) {
#pragma unroll
                    for (int r = 0; r < 16; ++r) s[kb][r] = 0.f;
#pragma unroll
                    for (int ks = 0; ks < KS; ++ks) {
                        bf16x8 kf = *reinterpret_cast<const bf16x8*>(sk + L::koff(kb * 32 + l32, 2 * ks + lh));
                        s[kb] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(kf, qf[rb][ks], s[kb], 0, 0, 0);
                    }
                }
                // lane: probe row = column l32; keys = kb*32 + 8*(r/4) + 4*lh + r%4
                const int vis_rel = vis_last[rb] - (int)key0 - 4 * lh;   // against literals: no thresholds in registers
                float mx = -INFINITY;
#pragma unroll
                for (int kb = 0; kb < 2; ++kb)
#pragma unroll
                    for (int r = 0; r < 16; ++r) {
                        float v = s[kb][r];
                        if (need_mask && kb * 32 + 8 * (r >> 2) + (r & 3) > vis_rel) v = -INFINITY;
                        s[kb][r] = v;
                        mx = fmaxf(mx, v);
                    }
                const auto mh = __builtin_amdgcn_permlane32_swap(__float_as_uint(mx), __float_as_uint(mx), false, false);   // both halves' values
                mx = fmaxf(__uint_as_float(mh[0]), __uint_as_float(mh[1]));
                const float ref = mx == -INFINITY ? 0.f : mx;
                float sum = 0.f;
#pragma unroll
                for (int kb = 0; kb < 2; ++kb)
#pragma unroll
                    for (int r = 0; r < 16; ++r) sum += __builtin_amdgcn_exp2f(s[kb][r] - ref);
                const auto sh = __builtin_amdgcn_permlane32_swap(__float_as_uint(sum), __float_as_uint(sum), false, false);
                const RowStats tile{mx, __uint_as_float(sh[0]) + __uint_as_float(sh[1])};
                pair[rb] = t & 1 ? join(pair[rb], tile) : tile;
                __builtin_amdgcn_sched_barrier(0);   // as in pass 2
            }
        } else {
            float ksum[2] = {0.f, 0.f};
#pragma unroll
            for (int rb = 0; rb < RB; ++rb) {
#pragma unroll
                for (int kb = 0; kb < 2; ++kb) {
                    f32x16 s = coff[rb];
#pragma unroll
                    for (int ks = 0; ks < KS; ++ks) {
                        bf16x8 kf = *reinterpret_cast<const bf16x8*>(sk + L::koff(kb * 32 + l32, 2 * ks + lh));
                        s = __builtin_amdgcn_mfma_f32_32x32x16_bf16(qf[rb][ks], kf, s, 0, 0, 0);
                    }
                    // lane: key = column kb*32 + l32; rows = rb*32 + 8*(r/4) + 4*lh + r%4
                    const int krel = (int)(key0 + kb * 32 + l32 - (a.N - a.P));   // position inside the probe window (< 0: before it)
#pragma unroll
                    for (int r = 0; r < 16; ++r) {
                        float pv = __builtin_amdgcn_exp2f(s[r]);
                        if (need_mask && krel >= (int)((pvis[rb][r >> 1] >> (16 * (r & 1))) & 0xffffu)) pv = 0.f;
                        ksum[kb] += pv;
                    }
                    // one block at a time: interleaved, the blocks' accumulators and exponentials do not fit the registers
                    __builtin_amdgcn_sched_barrier(0);
                }
            }
#pragma unroll
            for (int kb = 0; kb < 2; ++kb) {
                float v = ksum[kb] + __shfl_xor(ksum[kb], 32);
                if (lh == 0) sRed[wave][kb * 32 + l32] = v;
            }
            __syncthreads();
            if (tid < PKV) {
                int64_t key = key0 + tid;
                if (key < a.N) {
                    float tot = sRed[0][tid];
#pragma unroll
                    for (int wv = 1; wv < NWV; ++wv) tot += sRed[wv][tid];   // fixed order
                    a.partial[((int64_t)blockIdx.z * a.Hkv + g) * Np + seq_row0 + key] = tot;
                }
            }
        }
        if (t + 1 < n_tiles) store_tile((t + 1) & 1);
        __syncthreads();
    }
    if (PASS == 1) {
#pragma unroll
        for (int rb = 0; rb < RB; ++rb) {
            const RowStats all = n_tiles > 2 ? join(first[rb], pair[rb]) : pair[rb];
            int rr = row_base + wave * 32 * RB + rb * 32 + l32;
            if (lh == 0) {
                float* o = stats_part + (((int64_t)blockIdx.x * a.Hkv + g) * Rp + rr) * 2;
                o[0] = all.m;
                o[1] = all.l;
            }
        }
    }
}

// stats[g][rr] = (M, 1/L) over the chunks; padded rows rr >= R get (huge, 0).  JOIN_LANES lanes per (g, rr), neighbouring lanes
// neighbouring rows (fixed order: deterministic).
__global__ void __launch_bounds__(256) probe_combine_kernel(const float* __restrict__ stats_part, float* __restrict__ stats,
                                                            int nchunks, int chunk_keys, int Hkv, int Rp, int R, ProbeSegments seg) {
    constexpr int ROWS = 64 / JOIN_LANES;   // per wavefront
    const int lane = threadIdx.x & 63, part = lane / ROWS;
    const int i = (blockIdx.x * 4 + (threadIdx.x >> 6)) * ROWS + lane % ROWS;
    const int per_seq = Hkv * Rp, b = i / per_seq;   // Rp is a multiple of ROWS: a wavefront's rows are one sequence's
    if (b >= (seg.n > 0 ? seg.n : 1)) return;
    const int g = (i - b * per_seq) / Rp, rr = i % Rp;
    if (seg.n > 0) {
        const int64_t c0 = seg.chunk[b];
        nchunks = (int)(seg.chunk[b + 1] - c0);
        stats_part += c0 * per_seq * 2;
    }
    const float* sp = stats_part + ((int64_t)g * Rp + rr) * 2;
    const int64_t step = (int64_t)per_seq * 2;
    auto chunk = [&](int c) {
        const float2 v = *reinterpret_cast<const float2*>(sp + (c < nchunks ? c : nchunks - 1) * step);
        return c < nchunks ? RowStats{v.x, v.y} : NO_KEYS;
    };
    auto join_groups = [&](auto pg) {
        constexpr int PG = decltype(pg)::value, AHEAD = 8;   // groups whose loads are in flight together
        RowStats acc = NO_KEYS;
        for (int q = part; q * PG < nchunks; q += AHEAD * JOIN_LANES) {
            RowStats gs[AHEAD][PG];
#pragma unroll
            for (int u = 0; u < AHEAD; ++u)
#pragma unroll
                for (int e = 0; e < PG; ++e) gs[u][e] = chunk((q + u * JOIN_LANES) * PG + e);   // beyond the last: no keys
#pragma unroll
            for (int u = 0; u < AHEAD; ++u) acc = join(acc, group_of<PG>(gs[u]));
        }
        return acc;
    };
    RowStats acc = chunk_keys == CHUNK_MAX ? join_groups(std::integral_constant<int, 1>{})
                   : chunk_keys == CHUNK_MAX / 2 ? join_groups(std::integral_constant<int, 2>{}) : join_groups(std::integral_constant<int, 4>{});
    for (int off = JOIN_LANES / 2; off > 0; off >>= 1) {
        const RowStats other{__shfl_xor(acc.m, off * ROWS), __shfl_xor(acc.l, off * ROWS)};
        acc = join(acc, other);
    }
    if (part == 0) {   // padded rows weigh nothing
        stats[2 * i] = rr < R ? acc.m : 1e30f;
        stats[2 * i + 1] = rr < R && acc.l > 0.f ? 1.0f / acc.l : 0.f;
    }
}

__global__ void probe_final_kernel(const float* __restrict__ part, float* __restrict__ S, int64_t N, int64_t Np, int nparts,
                                   float inv_rows) {
    int64_t n = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (n >= N) return;
    float acc = 0.f;
    for (int g = 0; g < nparts; ++g) acc += part[(int64_t)g * Np + n];   // (row group, kv head) in order
    S[n] = acc * inv_rows;
}

// probe rows per kv head, padded to whole wavefronts' shares: a multiple of 128 up to 512, of 512 (row groups) beyond
constexpr int PROBE_GROUP_ROWS = 512;
static inline int probe_rp(int P, int H, int Hkv) {
    const int R = P * (H / Hkv), Rp = (R + 127) / 128 * 128;
    return Rp <= PROBE_GROUP_ROWS ? Rp : (Rp + PROBE_GROUP_ROWS - 1) / PROBE_GROUP_ROWS * PROBE_GROUP_ROWS;
}
static inline int probe_groups(int Rp) { return (Rp + PROBE_GROUP_ROWS - 1) / PROBE_GROUP_ROWS; }

// Keys per chunk.  A workgroup fetches its probe rows (64 KB for 256 of 128 elements) and then works tile by tile, so long chunks are the
// cheaper ones once every CU has one; below that the time is the chain of tiles.  64 probe rows, 8 kv heads, both passes: 333 candidates
// 256 -> 64 keys 25 -> 15 us; 8192 candidates (256 workgroups) 256 and 64 keys the same.
constexpr int64_t PROBE_FILL = 256;
int probe_chunk_keys(int64_t N, int P, int H, int Hkv) {
    const int64_t per_chunk = (int64_t)Hkv * probe_groups(probe_rp(P, H, Hkv));
    int keys = CHUNK_MAX;
    while (keys > PKV && (N + keys - 1) / keys * per_chunk < PROBE_FILL) keys >>= 1;
    return keys;
}

size_t probe_scratch_floats(int64_t N, int P, int H, int Hkv) {
    // generic path: stats [P*H, 2].  Matrix-core path: stats_part [nchunks][Hkv][Rp][2] + stats [Hkv][Rp][2]
    // + part [groups][Hkv][Np].  It serves every call of up to N candidates and P rows: one whose chunks were shortened has fewer than
    // twice PROBE_FILL workgroups, and one of 64-key chunks has no more of them than N gives.
    int64_t Np = (N + 255) / 256 * 256;
    const int64_t longest = (N + CHUNK_MAX - 1) / CHUNK_MAX * Hkv, all = (N + PKV - 1) / PKV * Hkv;
    const int64_t filled = 2 * PROBE_FILL + Hkv < all ? 2 * PROBE_FILL + Hkv : all;
    const int64_t chunks_hkv = longest > filled ? longest : filled;
    int64_t Rp = probe_rp(P, H, Hkv);
    const size_t windowed = (size_t)(2 * (int64_t)P * H + 64) + (size_t)(chunks_hkv * Rp * 2 + Hkv * Rp * 2 + probe_groups((int)Rp) * Hkv * Np + 256);
    const size_t single = probe_p1_scratch_floats(N, H);   // the single-row probe uses the same region from its start
    return windowed > single ? windowed : single;
}

bool probe_mfma_supported(const ProbeArgs& a) {
    if (a.d != 128 && a.d != 64) return false;
    if (a.N <= 0 || a.P <= 0 || a.H % a.Hkv != 0) return false;
    if (a.P >= 65535) return false;   // window rows are kept in 16 bits (pass 2)
    auto al = [](const void* p) { return (reinterpret_cast<uintptr_t>(p) & 15u) == 0; };
    return al(a.qp) && al(a.k);
}

// chunks, statistics rows and result rows of one sequence or of a batch
struct ProbePlan { int64_t Np, chunks, max_chunks; int nseq, keys; };
static ProbePlan probe_plan(const ProbeArgs& a, const ProbeSegments& seg) {
    const int64_t Np = (a.N + 255) / 256 * 256;
    if (seg.n > 0) return ProbePlan{Np, seg.chunks, seg.max_chunks, seg.n, seg.chunk_keys};
    const int keys = probe_chunk_keys(a.N, a.P, a.H, a.Hkv);
    const int64_t chunks = (a.N + keys - 1) / keys;
    return ProbePlan{Np, chunks, chunks, 1, keys};
}

template <int D, int RB, int NWV = 4>
static hipError_t launch_probe_t(const ProbeArgs& a, const ProbeSegments& seg, int Rp, hipStream_t s) {
    const ProbePlan pl = probe_plan(a, seg);
    const int nchunks = (int)pl.chunks;
    const int R = a.P * (a.H / a.Hkv);
    float* stats_part = a.partial;
    float* stats = stats_part + (size_t)nchunks * a.Hkv * Rp * 2;
    float* part = stats + (size_t)pl.nseq * a.Hkv * Rp * 2;
    ProbeArgs b = a;
    b.partial = part;
    const float want = attention_mfma_q_scale(D);
    const float qmul = (a.q_scale != 0.f) ? want / a.q_scale : want;   // exactly 1 when the producer applied `want`
    const int groups = probe_groups(Rp);
    dim3 grid(nchunks, a.Hkv, groups), block(256), pblock(64 * NWV);
    probe_mfma_kernel<D, RB, 1, NWV><<<grid, pblock, 0, s>>>(b, Rp, pl.Np, qmul, pl.keys, nchunks, stats_part, nullptr, seg);
    const bool fold = pl.max_chunks <= FOLD_CHUNKS;
    if (!fold) probe_combine_kernel<<<dim3((unsigned)(pl.nseq * a.Hkv * Rp / 32)), block, 0, s>>>(stats_part, stats, nchunks, pl.keys, a.Hkv, Rp, R, seg);
    probe_mfma_kernel<D, RB, 2, NWV><<<grid, pblock, 0, s>>>(b, Rp, pl.Np, qmul, pl.keys, nchunks, stats_part, fold ? nullptr : stats, seg);
    probe_final_kernel<<<dim3((unsigned)((a.N + 255) / 256)), block, 0, s>>>(part, a.S, a.N, pl.Np, groups * a.Hkv, 1.0f / (float)(a.P * a.H));
    return hipGetLastError();
}

static hipError_t launch_probe_any(const ProbeArgs& a, const ProbeSegments& seg, hipStream_t s) {
    const int Rp = probe_rp(a.P, a.H, a.Hkv);
    const int rb = Rp / 128;
    if (a.d == 128) {
        if (rb == 1) return launch_probe_t<128, 1>(a, seg, Rp, s);
        if (rb == 2) return launch_probe_t<128, 2>(a, seg, Rp, s);
        if (rb == 3) return launch_probe_t<128, 3>(a, seg, Rp, s);
        return launch_probe_t<128, 2, 8>(a, seg, Rp, s);   // 512 rows (per group): 8 wavefronts x 64 rows keep two wavefronts per SIMD
    }
    if (rb == 1) return launch_probe_t<64, 1>(a, seg, Rp, s);
    if (rb == 2) return launch_probe_t<64, 2>(a, seg, Rp, s);
    if (rb == 3) return launch_probe_t<64, 3>(a, seg, Rp, s);
    return launch_probe_t<64, 2, 8>(a, seg, Rp, s);
}

hipError_t launch_probe_mfma(const ProbeArgs& a, hipStream_t s) { return launch_probe_any(a, ProbeSegments{nullptr, nullptr, 0, 0, 0, 0}, s); }

size_t probe_batch_scratch_floats(const ProbeArgs& a, const ProbeSegments& seg) {
    const ProbePlan pl = probe_plan(a, seg);
    const int Rp = probe_rp(a.P, a.H, a.Hkv);
    return (size_t)(pl.chunks + pl.nseq) * a.Hkv * Rp * 2 + (size_t)probe_groups(Rp) * a.Hkv * pl.Np;
}

hipError_t launch_probe_mfma_batched(const ProbeArgs& a, const ProbeSegments& seg, hipStream_t s) {
    if (seg.n < 1 || seg.chunks < 1 || (seg.chunk_keys != PKV && seg.chunk_keys != 2 * PKV && seg.chunk_keys != CHUNK_MAX) || seg.chunks > 0x7fffffff || (int64_t)seg.n * a.Hkv * probe_rp(a.P, a.H, a.Hkv) > 0x7fffffff) return hipErrorInvalidValue;
    return launch_probe_any(a, seg, s);
}

__global__ void probe_rows_kernel(const int64_t* __restrict__ off, int P, int64_t total, int32_t* __restrict__ idx) {
    const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (i < total) idx[i] = (int32_t)(off[i / P + 1] - P + i % P);
}
hipError_t launch_probe_rows(const int64_t* off, int n, int P, int32_t* idx, hipStream_t s) {
    const int64_t total = (int64_t)n * P;
    if (total <= 0) return hipSuccess;
    probe_rows_kernel<<<dim3((unsigned)((total + 255) / 256)), dim3(256), 0, s>>>(off, P, total, idx);
    return hipGetLastError();
}

}  // namespace spts
