// Small kernels around the contractions: mask compaction, log-sum-exp merge, generation-level log
// ratios, group advantages, loss/coefficients/diagnostics.  All HBM- or latency-bound; every
// reduction uses a fixed tree so results are bitwise reproducible (no atomics on data).
#include <cmath>

#include "rapid_internal.h"

namespace rapid {

namespace {

constexpr int WAVE = 64;

__device__ inline double wave_sum(double v) {
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o, WAVE);
    return v;
}
__device__ inline double wave_max(double v) {
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) v = fmax(v, __shfl_xor(v, o, WAVE));
    return v;
}
__device__ inline int wave_sum_i(int v) {
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o, WAVE);
    return v;
}

// block-wide reductions for up to 1024 threads; `sm` holds >= 16 doubles
__device__ inline double block_sum(double v, double* sm) {
    v = wave_sum(v);
    const int w = threadIdx.x / WAVE, nw = (blockDim.x + WAVE - 1) / WAVE;
    __syncthreads();
    if ((threadIdx.x & (WAVE - 1)) == 0) sm[w] = v;
    __syncthreads();
    double r = 0.0;
    for (int i = 0; i < nw; ++i) r += sm[i];
    return r;
}
__device__ inline double block_max(double v, double* sm) {
    v = wave_max(v);
    const int w = threadIdx.x / WAVE, nw = (blockDim.x + WAVE - 1) / WAVE;
    __syncthreads();
    if ((threadIdx.x & (WAVE - 1)) == 0) sm[w] = v;
    __syncthreads();
    double r = sm[0];
    for (int i = 1; i < nw; ++i) r = fmax(r, sm[i]);
    return r;
}

// K sums with the two barriers of one (`sm` holds >= 16 K doubles); the same bits as K calls of block_sum
template <int K>
__device__ inline void block_sums(double (&v)[K], double* sm) {
    const int w = threadIdx.x / WAVE, nw = (blockDim.x + WAVE - 1) / WAVE;
#pragma unroll
    for (int k = 0; k < K; ++k) v[k] = wave_sum(v[k]);
    __syncthreads();
    if ((threadIdx.x & (WAVE - 1)) == 0)
#pragma unroll
        for (int k = 0; k < K; ++k) sm[w * K + k] = v[k];
    __syncthreads();
#pragma unroll
    for (int k = 0; k < K; ++k) v[k] = 0.0;
    for (int i = 0; i < nw; ++i)
#pragma unroll
        for (int k = 0; k < K; ++k) v[k] += sm[i * K + k];
}
// Threads for a block that takes N entries with a stride of blockDim: waves without an entry would only wait at the
// barriers and add zeros.  (64 generations, one wave instead of 16: coefficients 7.2 -> 3.4 us with block_sums, plan 8.9 ->
// 6.3 us.)
inline unsigned block_threads(int64_t N, unsigned most) {
    return N < most ? (unsigned)((N + WAVE - 1) / WAVE * WAVE) : most;
}

// ------------------------------------------------------------------ compaction of the padding mask
// Lengths and plan here, the rows in rows.hip: two launches for a small batch, three for the others.  A small batch's call is a
// matter of launches, and these have next to nothing to do.

// One block per generation; its waves take stretches of the sequence of the same length.  One wave where a sequence has
// fewer than 512 positions: 256 positions are about four trips to memory, and a second wave costs a barrier.
inline unsigned row_threads(int64_t T) { return WAVE * (T < 512 ? 1u : T < 256 * 16 ? (unsigned)(T / 256) : 16u); }
struct Stretch { int64_t begin, end; };
__device__ inline Stretch wave_stretch(int64_t T) {
    const int64_t span = (T + blockDim.x - 1) / blockDim.x * WAVE, begin = threadIdx.x / WAVE * span;
    return {begin, begin + span < T ? begin + span : T};
}
// the wave's valid tokens in its stretch (all lanes get the sum)
__device__ inline int count_valid(const uint8_t* mask, int64_t row0, int64_t T, const Stretch& s) {
    const int lane = threadIdx.x & (WAVE - 1);
    const uint8_t* row = mask + row0;
    int cnt = 0;
    if ((T & 3) == 0 && ((uintptr_t)mask & 3) == 0) {
#pragma unroll 4
        for (int64_t t = s.begin / 4 + lane; t < s.end / 4; t += WAVE) {
            const uint32_t w = ((const uint32_t*)row)[t];
            cnt += __popc((((w & 0x7f7f7f7fu) + 0x7f7f7f7fu) | w) & 0x80808080u);   // top bit of every byte that is not 0
        }
    } else {
#pragma unroll 4
        for (int64_t t = s.begin + lane; t < s.end; t += WAVE) cnt += row[t] != 0;
    }
    return wave_sum_i(cnt);
}

// Number of valid tokens of each generation; the blocks together clear the plan's counters.
template <bool ONE_WAVE>
__global__ __launch_bounds__(ONE_WAVE ? WAVE : 1024) void seq_len_kernel(const uint8_t* __restrict__ mask, int64_t N, int64_t T,
                                                       int32_t* __restrict__ seq_len, ZeroWords z) {
    const int64_t n = blockIdx.x;
    int cnt = count_valid(mask, n * T, T, ONE_WAVE ? Stretch{0, T} : wave_stretch(T));
#pragma unroll
    for (int k = 0; k < 2; ++k)
        for (int64_t i = n * blockDim.x + threadIdx.x; i < z.n[k]; i += N * blockDim.x) z.p[k][i] = 0;
    if constexpr (!ONE_WAVE) {
        __shared__ int s_cnt[16];
        if (threadIdx.x % WAVE == 0) s_cnt[threadIdx.x / WAVE] = cnt;
        __syncthreads();
        cnt = 0;
        for (unsigned w = 0; w < blockDim.x / WAVE; ++w) cnt += s_cnt[w];
    }
    if (threadIdx.x == 0) seq_len[n] = cnt;
}

// exclusive prefix sum of v [N] -> cu [N + 1] by a block of up to 1024 threads; returns the total to every thread
__device__ __forceinline__ int block_scan(const int32_t* v, int64_t N, int32_t* cu) {
    constexpr int PER = 8;   // consecutive entries per thread: 8192 per sweep of the block
    __shared__ int s_wave[16];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    int carry = 0;
    for (int64_t base = 0; base < N; base += blockDim.x * PER) {
        const int64_t n0 = base + (int64_t)threadIdx.x * PER;
        int e[PER], mine = 0;
#pragma unroll
        for (int u = 0; u < PER; ++u) {
            e[u] = n0 + u < N ? v[n0 + u] : 0;
            mine += e[u];
        }
        int incl = mine;     // inclusive scan of the threads' sums: within the wave, then over the waves
#pragma unroll
        for (int o = 1; o < 64; o <<= 1) {
            const int up = __shfl_up(incl, o, WAVE);
            if (lane >= o) incl += up;
        }
        __syncthreads();
        if (lane == 63) s_wave[wave] = incl;
        __syncthreads();
        int before = 0, total = 0;
        for (int w = 0; w < (int)blockDim.x / 64; ++w) {
            before += w < wave ? s_wave[w] : 0;
            total += s_wave[w];
        }
        int run = carry + before + incl - mine;
#pragma unroll
        for (int u = 0; u < PER; ++u) {
            if (n0 + u < N && cu) cu[n0 + u] = run;
            run += e[u];
        }
        carry += total;
    }
    if (threadIdx.x == 0 && cu) cu[N] = carry;
    return carry;
}

// Generations whose coefficient dLoss/dlogp is zero whatever the log-probs turn out to be: every reward of the
// group is exactly 0 (then the weighted baseline of Eq. (5) is 0 too, A_n = R_n - b = 0, in every baseline mode;
// likewise the normalised advantage of the clipped surrogate), or the caller's coefficient override is 0.
// Their rows get no gradient: dHidden rows are zero and they add nothing to dW, so the two gradient
// contractions can leave them out.  A generation with a group id outside [0, K) is never idle.
//
// The plan of a batch, by one block: where each group lies (runs), which generations are idle, the prefix sums of the
// lengths, and either the counters of one region (tab NULL) or the chunk table.
// Thread 0 walks the runs of equal group id in order and fills chunk after chunk; then all threads
// give every generation its chunk and first compact row.
// With idle generations (cu_live = prefix sum of the other generations' lengths) a chunk's
// rows are ordered: the generations that carry gradient first, in batch order, then the idle ones, so that the
// two gradient contractions stop at CH_LIVE.
// runs[k] = number of maximal runs of group id k, runs[K + k] / runs[2K + k] = begin / end of (the last of) them,
// runs[3K] = 1 if some group has more than one run.  With one run per group, which is how a sampler that draws G
// generations per prompt lays a batch out, the per-group pass below visits each generation once instead of once
// per group.
//
// IN_LDS: N and K at most PLAN_LDS; what the plan makes for itself stays in the LDS, so that the steps between its
// barriers are not trips to memory.  LENGTHS: it counts the generations' tokens too, a launch less; one block reads the
// whole mask then, which up to PLAN_MASK positions takes it no longer than the launch would (whole steps with either: 64 x 250 positions 92
// and 94 us, 216 x 104 122 and 122, 560 x 53 145 and 141, 1024 x 31 155 and 150).  Else seq_len_kernel has counted them, and has cleared runs and live_group
// where they are in memory.
constexpr int PLAN_LDS = 1024, PLAN_MASK = 16384;
template <bool IN_LDS, bool LENGTHS>
__global__ __launch_bounds__(1024) void plan_kernel(PlanArgs a, const uint8_t* __restrict__ mask, int64_t T) {
    static_assert(IN_LDS || !LENGTHS, "lengths are counted into the LDS");
    constexpr int L = IN_LDS ? PLAN_LDS : 0;
    __shared__ int s_status;
    __shared__ int32_t s_len[L + 1], s_cu[L + 1], s_live_len[L + 1], s_cu_live[L + 1], s_live_group[L + 1], s_run_first[L + 1],
        s_run_end[L + 1], s_run_count[L + 1], s_gid[L + 1];
    const int64_t N = a.N, K = a.K;
    const int32_t* const gid = IN_LDS ? s_gid : a.gid;
    int32_t* const seq_len = IN_LDS ? s_len : a.seq_len;
    int32_t* const cu = IN_LDS ? s_cu : a.cu;
    int32_t* const len_live = IN_LDS ? s_live_len : a.idle.len_live;
    int32_t* const cu_live_out = IN_LDS ? s_cu_live : a.idle.cu_live;
    int32_t* const live_group = IN_LDS ? s_live_group : a.idle.live_group;
    int32_t* const run_count = IN_LDS ? s_run_count : a.runs;
    int32_t* const run_first = IN_LDS ? s_run_first : a.runs + K;
    int32_t* const run_end = IN_LDS ? s_run_end : a.runs + 2 * K;
    __shared__ int s_split;      // some group has more than one run
    if (threadIdx.x == 0) s_split = 0;
    const bool by_reward = a.idle.idle && !a.idle.coef_override;
    float my_reward = 0.f;       // in the LDS a thread has one generation at most
    if constexpr (IN_LDS) {
        if (by_reward && threadIdx.x < N) my_reward = a.idle.rewards[threadIdx.x];
        for (int k = threadIdx.x; k < K; k += blockDim.x) s_live_group[k] = s_run_count[k] = s_run_first[k] = s_run_end[k] = 0;
        if (a.gid)
            for (int n = threadIdx.x; n < N; n += blockDim.x) s_gid[n] = a.gid[n];
    }
    if constexpr (LENGTHS) {
        // 2^lanes_log2 lanes per generation, eight loads of each in flight
        const bool words = (T & 3) == 0 && ((uintptr_t)mask & 3) == 0;
        const int per = (int)(words ? T / 4 : T), lanes_log2 = per <= 64 ? 3 : per <= 128 ? 4 : per <= 256 ? 5 : 6, lanes = 1 << lanes_log2;
        for (int64_t n = threadIdx.x >> lanes_log2; n < N; n += blockDim.x >> lanes_log2) {
            const uint8_t* row = mask + n * T;
            int cnt = 0;
            if (words) {
#pragma unroll 8
                for (int t = threadIdx.x & (lanes - 1); t < per; t += lanes) {
                    const uint32_t w = ((const uint32_t*)row)[t];
                    cnt += __popc((((w & 0x7f7f7f7fu) + 0x7f7f7f7fu) | w) & 0x80808080u);
                }
            } else {
#pragma unroll 8
                for (int t = threadIdx.x & (lanes - 1); t < per; t += lanes) cnt += row[t] != 0;
            }
            for (int o = lanes >> 1; o > 0; o >>= 1) cnt += __shfl_xor(cnt, o, WAVE);
            if ((threadIdx.x & (lanes - 1)) == 0) {
                s_len[n] = cnt;
                a.seq_len[n] = cnt;
            }
        }
    } else if constexpr (IN_LDS) {
        for (int n = threadIdx.x; n < N; n += blockDim.x) s_len[n] = a.seq_len[n];
    }
    __syncthreads();
    if (a.runs || by_reward) {
        for (int64_t n = threadIdx.x; n < N; n += blockDim.x) {
            const int32_t g = gid[n], before = n > 0 ? gid[n - 1] : -1, after = n < N - 1 ? gid[n + 1] : -1;
            // a reward that is not finite counts as 0 in the estimator as well; equal values from several threads
            const float R = IN_LDS ? my_reward : by_reward ? a.idle.rewards[n] : 0.f;
            if (g < 0 || g >= K) continue;
            if (a.runs) {
                if (before != g) {
                    if (atomicAdd(&run_count[g], 1) > 0) s_split = 1;
                    run_first[g] = (int32_t)n;
                }
                if (after != g) run_end[g] = (int32_t)(n + 1);
            }
            if (isfinite(R) && R != 0.f) live_group[g] = 1;
        }
        __syncthreads();
        if (a.runs) {
            if constexpr (IN_LDS) {
                for (int k = threadIdx.x; k < K; k += blockDim.x) {
                    a.runs[k] = s_run_count[k];
                    a.runs[K + k] = s_run_first[k];
                    a.runs[2 * K + k] = s_run_end[k];
                }
            }
            if (threadIdx.x == 0) a.runs[3 * K] = s_split;
        }
    }
    if (a.idle.idle) {
        for (int64_t n = threadIdx.x; n < N; n += blockDim.x) {
            bool z;
            if (a.idle.coef_override) {
                z = a.idle.coef_override[n] == 0.f;
            } else {
                const int32_t g = gid[n];
                z = g >= 0 && g < K && live_group[g] == 0;
            }
            a.idle.idle[n] = z ? 1 : 0;
            len_live[n] = z ? 0 : seq_len[n];
        }
        __syncthreads();
    }
    const int32_t* cu_live = a.idle.idle ? cu_live_out : nullptr;
    const int64_t total = block_scan(seq_len, N, cu);
    if (a.idle.idle) block_scan(len_live, N, cu_live_out);
    if (threadIdx.x == 0 && a.lam_state) a.lam_state[0] = -INFINITY;
    if (!a.tab) {
        if (threadIdx.x == 0 && a.counts) {
            a.counts[CNT_M] = (int32_t)total;
            a.counts[CNT_MR] = (int32_t)((total + ROW_TILE - 1) / ROW_TILE * ROW_TILE);
        }
        if constexpr (IN_LDS) {
            __syncthreads();
            for (int n = threadIdx.x; n <= N; n += blockDim.x) a.cu[n] = s_cu[n];
        }
        return;
    }
    __syncthreads();
    const int64_t Rcap = a.Rcap;
    const int Cmax = a.Cmax;
    int32_t* tab = a.tab;
    if (threadIdx.x == 0) {
        int status = 0, c = 0;
        int64_t placed = 0;
        auto close = [&](int64_t g0, int64_t g1, int64_t rows) {
            if (rows > Rcap) rows = Rcap;
            int32_t* e = tab + (int64_t)c * CH_WORDS;
            e[CH_G0] = (int32_t)g0; e[CH_G1] = (int32_t)g1; e[CH_ROWS] = (int32_t)rows;
            e[CH_M] = (int32_t)((int64_t)c * Rcap + rows);
            e[CH_MR] = (int32_t)((int64_t)c * Rcap + (rows + ROW_TILE - 1) / ROW_TILE * ROW_TILE);
            int64_t live = cu_live ? (int64_t)cu_live[g1] - (int64_t)cu_live[g0] : rows;
            if (live > rows) live = rows;           // only when the chunk was cut short (its outputs are unusable then)
            e[CH_LIVE] = (int32_t)((int64_t)c * Rcap + live);
            e[CH_LIVER] = (int32_t)((int64_t)c * Rcap + (live + ROW_TILE - 1) / ROW_TILE * ROW_TILE);
            e[7] = 0;
            placed += rows;
            ++c;
        };
        if (Cmax == 1) {
            if (total > Rcap) status |= RAPID_STATUS_TOKEN_BOUND;
            close(0, N, total);
        } else {
            int64_t chunk_g0 = 0, chunk_rows = 0, run0 = 0;
            int run_gid = gid[0];
            bool full = false;
            for (int64_t n = 1; n <= N && !full; ++n) {
                if (n < N && gid[n] == run_gid) continue;
                const int64_t rows = (int64_t)cu[n] - (int64_t)cu[run0];   // the run [run0, n)
                if (rows > Rcap) status |= RAPID_STATUS_GROUP_LAYOUT;      // placed alone, cut at Rcap
                if (run0 > chunk_g0 && chunk_rows + rows > Rcap) {
                    if (c == Cmax - 1) {            // no chunk left: the rest of the batch is left out
                        status |= RAPID_STATUS_TOKEN_BOUND;
                        full = true;
                        break;
                    }
                    close(chunk_g0, run0, chunk_rows);
                    chunk_g0 = run0;
                    chunk_rows = 0;
                }
                chunk_rows += rows;
                run0 = n;
                if (n < N) run_gid = gid[n];
            }
            close(chunk_g0, run0, chunk_rows);      // run0 == N unless the chunks ran out
        }
        while (c < Cmax) close(N, N, 0);            // chunks that stay empty (close() counts c up)
        a.counts[CNT_M] = (int32_t)placed;
        a.counts[CNT_MR] = (int32_t)((placed + ROW_TILE - 1) / ROW_TILE * ROW_TILE);
        s_status = status;
    }
    __syncthreads();
    for (int64_t n = threadIdx.x; n < N; n += blockDim.x) {
        int c = -1;
        int64_t g0 = 0, g1 = N;
        for (int k = 0; k < Cmax; ++k) {
            if (Cmax > 1) { g0 = tab[k * CH_WORDS + CH_G0]; g1 = tab[k * CH_WORDS + CH_G1]; }
            if (n >= g0 && n < g1) { c = k; break; }
        }
        a.gen_chunk[n] = c;
        int64_t row0 = -1;
        if (c >= 0) {
            const int64_t before = (int64_t)cu[n] - (int64_t)cu[g0];            // tokens of the chunk's earlier generations
            if (cu_live) {
                const int64_t live_before = (int64_t)cu_live[n] - (int64_t)cu_live[g0];
                const int64_t live_all = (int64_t)cu_live[g1] - (int64_t)cu_live[g0];
                // (an idle generation without tokens has no row to place)
                row0 = (int64_t)c * Rcap + (len_live[n] != seq_len[n] ? live_all + (before - live_before) : live_before);
            } else {
                row0 = (int64_t)c * Rcap + before;
            }
            // Past the chunk's end (the chunk was cut short): left out.  Its rows would be the next chunk's, or lie behind the last.
            if (row0 >= (int64_t)(c + 1) * Rcap) row0 = -1;
        }
        a.gen_row0[n] = (int32_t)row0;
    }
    if (threadIdx.x == 0 && a.dev_status) {
        const int status = s_status | (Cmax > 1 && s_split ? RAPID_STATUS_GROUP_LAYOUT : 0);
        if (status) atomicOr(a.dev_status, status);
    }
}

// The rows' positions, tokens and generations where rows_by_position_kernel does not find them (launch_compact_rows); one block
// per generation.
// A wave's loop is a chain of trips to memory, so it takes 4 x 64 positions at a time, mask and tokens together, and the
// waves of the sequence share it (each counts its stretch first).  One wave, one load after the other: 1 x 131 072
// positions 500 us, 19 now.
template <bool ONE_WAVE>
__global__ __launch_bounds__(ONE_WAVE ? WAVE : 1024) void row_index_kernel(RowsArgs a) {
    const int64_t n = blockIdx.x, T = a.T;
    const int lane = threadIdx.x & (WAVE - 1);
    if (a.tokc)
        for (int64_t e = n; e < a.entries; e += a.N)
            for (int j = a.limits[e * a.stride + CNT_M] + (int)threadIdx.x; j < a.limits[e * a.stride + CNT_MR]; j += blockDim.x) {
                a.tokc[j] = 0;
                a.seqc[j] = 0;
            }
    int64_t base = a.first_row[n];
    const bool left_out = base < 0;
    const int64_t limit = left_out ? 0 : (base / a.region + 1) * a.region;
    const Stretch s = ONE_WAVE ? Stretch{0, T} : wave_stretch(T);
    if constexpr (!ONE_WAVE) {
        __shared__ int s_cnt[16];
        const int cnt = count_valid(a.mask, n * T, T, s), wave = threadIdx.x / WAVE;
        if (lane == 0) s_cnt[wave] = cnt;
        __syncthreads();
        for (int w = 0; w < wave; ++w) base += s_cnt[w];
    }
    bool bad = false;
    constexpr int U = 4;
    for (int64_t t0 = s.begin; t0 < s.end; t0 += U * WAVE) {
        bool v[U];
        int tok[U];
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int64_t t = t0 + u * WAVE + lane;
            v[u] = t < s.end && a.mask[n * T + t] != 0;
            tok[u] = t < s.end && a.tokc ? a.tokens[n * T + t] : 0;
        }
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int64_t t = t0 + u * WAVE + lane, i = n * T + t;
            if (t0 + u * WAVE >= s.end) break;
            const unsigned long long b = __ballot(v[u]);
            const int64_t j = base + __popcll(b & ((1ull << lane) - 1ull));
            if (v[u] && !left_out && j < limit) {
                a.row_index[j] = (int32_t)i;
                if (a.tokc) {
                    const bool in = tok[u] >= 0 && tok[u] < a.V;
                    bad = bad || !in;
                    a.tokc[j] = in ? tok[u] : 0;
                    a.seqc[j] = (int32_t)n;
                }
            } else if (t < s.end) {
                if (a.zero_a) a.zero_a[i] = 0.f;
                if (a.zero_b) a.zero_b[i] = 0.f;
            }
            base += __popcll(b);
        }
    }
    if (bad && a.dev_status) atomicOr(a.dev_status, RAPID_STATUS_BAD_TOKEN);
}

__global__ void f32_add_kernel(const float* __restrict__ src, float* __restrict__ dst, int64_t n) {
    int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n) dst[i] += src[i];
}

__global__ void fill_f32_kernel(float* p, int64_t n, float v) {
    int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n) p[i] = v;
}

// lse[j] = log sum_p part_sum[p][j] exp(part_max[p][j]) ; logp = zy - lse, scattered to [N,T].
// A block of NW waves takes 32 columns (a line of each slot): half a wave, one column per lane, is one of 2 NW groups
// that fold P / (2 NW) slots each, then the (max, sum) pairs of a column are merged in a fixed tree: the two of a
// wave in registers, the waves through LDS.  A group's loads are a chain of batches, each a trip to memory: with 4
// groups per column a few hundred rows took 50 us at P = 1188, with 32 groups 13; 74 000 rows 166 and 138.
// With few slots most of 32 groups are empty and their waves are all the time goes into; 131 072 rows, with the
// sampled tokens' logits, 1 / 4 / 16 waves: P = 2 33 / 36 / 53 us, P = 16 34 / 37 / 55, P = 32 38 / 38 / 55, P = 128 58 / 54 / 61,
// P = 256 83 / 79 / 83; 300 rows: P = 16 12 us with any, P = 128 20 / 14 / 13, P = 256 28 / 16 / 13.
// How P is shared out depends on P alone: every call forms a row's sum in the same order.
struct MaxSum { float mx; double acc; };
// the lower-numbered operand first
__device__ inline MaxSum merge_pair(const MaxSum& a, const MaxSum& b) {
    MaxSum r;
    r.mx = fmaxf(a.mx, b.mx);
    r.acc = 0.0;
    if (a.acc > 0.0) r.acc += a.acc * (double)__expf(a.mx - r.mx);
    if (b.acc > 0.0) r.acc += b.acc * (double)__expf(b.mx - r.mx);
    return r;
}
// Slots [p_begin, p_end) of a column, one after the other with a running maximum; a slot without a positive sum counts for
// nothing.  The loads of a batch of UN are in flight together (a matter of time alone), and its exponentials do not wait for
// each other: the running maximum is known in front of every slot, and a slot takes one exponential, of the sum so far if it
// raises the maximum and of its own sum if not.
template <int UN>
__device__ __forceinline__ MaxSum fold_slots(const float* __restrict__ part_max, const float* __restrict__ part_sum, int p_begin, int p_end,
                                             int64_t ld_part, int64_t jl) {
    MaxSum m{-INFINITY, 0.0};
    for (int p0 = p_begin; p0 < p_end; p0 += UN) {
        float pm[UN], ps[UN], e[UN];
        bool up[UN];
#pragma unroll
        for (int u = 0; u < UN; ++u) {
            const int64_t at = (int64_t)(p0 + u < p_end ? p0 + u : p_end - 1) * ld_part + jl;
            pm[u] = part_max[at];
            ps[u] = part_sum[at];
        }
#pragma unroll
        for (int u = 0; u < UN; ++u) {
            const bool counts = p0 + u < p_end && ps[u] > 0.f;
            up[u] = counts && pm[u] > m.mx;
            e[u] = counts ? __expf(up[u] ? m.mx - pm[u] : pm[u] - m.mx) : 1.f;
            if (!counts) ps[u] = 0.f;
            if (up[u]) m.mx = pm[u];
        }
#pragma unroll
        for (int u = 0; u < UN; ++u) m.acc = up[u] ? fma(m.acc, (double)e[u], (double)ps[u]) : fma((double)ps[u], (double)e[u], m.acc);
    }
    return m;
}
template <int NW>
__global__ __launch_bounds__(64 * NW) void merge_lse_kernel(const float* __restrict__ part_max, const float* __restrict__ part_sum, int P,
                                 int64_t ld_part, const float* __restrict__ zy,
                                 const int32_t* __restrict__ row_index, const int32_t* __restrict__ counts,
                                 int64_t row0, float* __restrict__ lse_c, float* __restrict__ logp_out,
                                 float* __restrict__ lse_out) {
    constexpr int GROUPS = 2 * NW;
    __shared__ float s_mx[NW][32];
    __shared__ double s_acc[NW][32];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, q = wave * 2 + (lane >> 5), col = lane & 31;
    const int64_t jl = (int64_t)blockIdx.x * 32 + col;
    const int64_t j = row0 + jl;
    const int M = counts[CNT_M];
    if (row0 + (int64_t)blockIdx.x * 32 >= M) return;
    const bool live = j < M;
    // The weights exp(pm - mx) are fp32 (relative error 1e-7, far below the fp32 rounding of the
    // partial sums themselves), the accumulation fp64.
    MaxSum m{-INFINITY, 0.0};
    const int p_begin = (int)((int64_t)P * q / GROUPS), p_end = (int)((int64_t)P * (q + 1) / GROUPS);
    if (live) m = fold_slots<10>(part_max, part_sum, p_begin, p_end, ld_part, jl);
    auto merge_halves = [&]() {   // both partners compute the same pair
        const MaxSum o{__shfl_xor(m.mx, 32, 64), __shfl_xor(m.acc, 32, 64)};
        m = lane < 32 ? merge_pair(m, o) : merge_pair(o, m);
    };
    merge_halves();
    const int g = lane >> 5;
    if constexpr (NW > 1) {
        if (lane < 32) {
            s_mx[wave][col] = m.mx;
            s_acc[wave][col] = m.acc;
        }
        __syncthreads();
        if (wave != 0) return;
        constexpr int H = NW / 2;   // wave 0: its halves fold the results of the first and of the second half of the waves
        m = MaxSum{s_mx[g * H][col], s_acc[g * H][col]};
#pragma unroll
        for (int w = 1; w < H; ++w) m = merge_pair(m, MaxSum{s_mx[g * H + w][col], s_acc[g * H + w][col]});
        merge_halves();
    }
    if (!live || g != 0) return;
    const double lse = (double)m.mx + log(m.acc);
    const float lse_f = (float)lse;
    lse_c[j] = lse_f;
    const int32_t pos = row_index[j];
    logp_out[pos] = (float)((double)zy[j] - lse);
    if (lse_out) lse_out[pos] = lse_f;
}

// The same for few rows and many slots (what merge_lse_kernel<16> does, same order): 8 columns per block and a thread for each
// of the 32 groups, so that four times as many compute units read the partials, twice as many slots ahead.  P = 1188, d = 64: 290
// rows 11.6 -> 8.8 us; with 2200 rows the kernel above takes 11.4.
__global__ __launch_bounds__(256) void merge_lse_few_kernel(const float* __restrict__ part_max, const float* __restrict__ part_sum, int P,
                                 int64_t ld_part, const float* __restrict__ zy,
                                 const int32_t* __restrict__ row_index, const int32_t* __restrict__ counts,
                                 int64_t row0, float* __restrict__ lse_c, float* __restrict__ logp_out,
                                 float* __restrict__ lse_out) {
    constexpr int GROUPS = 32, COLS = 8;
    __shared__ float s_mx[GROUPS][COLS];
    __shared__ double s_acc[GROUPS][COLS];
    const int col = threadIdx.x % COLS, q = threadIdx.x / COLS;
    const int64_t jl = (int64_t)blockIdx.x * COLS + col, j = row0 + jl;
    const int M = counts[CNT_M];
    if (j - col >= M) return;
    const bool live = j < M;
    MaxSum m{-INFINITY, 0.0};
    if (live) m = fold_slots<20>(part_max, part_sum, (int)((int64_t)P * q / GROUPS), (int)((int64_t)P * (q + 1) / GROUPS), ld_part, jl);
    s_mx[q][col] = m.mx;
    s_acc[q][col] = m.acc;
    __syncthreads();
    auto at = [&](int g) { return MaxSum{s_mx[g][col], s_acc[g][col]}; };
    if (q < 16) m = merge_pair(at(2 * q), at(2 * q + 1));
    __syncthreads();
    if (q < 16) { s_mx[q][col] = m.mx; s_acc[q][col] = m.acc; }
    __syncthreads();
    if (q >= 2) return;
    m = at(8 * q);
#pragma unroll
    for (int w = 1; w < 8; ++w) m = merge_pair(m, at(8 * q + w));
    const MaxSum o{__shfl_down(m.mx, COLS, 64), __shfl_down(m.acc, COLS, 64)};
    if (q != 0 || !live) return;
    m = merge_pair(m, o);
    const double lse = (double)m.mx + log(m.acc);
    const float lse_f = (float)lse;
    lse_c[j] = lse_f;
    const int32_t pos = row_index[j];
    logp_out[pos] = (float)((double)zy[j] - lse);
    if (lse_out) lse_out[pos] = lse_f;
}

// one block per generation: token-level log ratios and their sum over the generation; for the
// token-level outer weight also sum_t c_{n,t} and max_t log c_{n,t} of the generation's valid tokens
// (c = the token's ratio, clipped at eta if clip_tokens), tsum/tmax may be NULL.
// A wave's loop is a chain of trips to memory (4 x 64 positions each), so the waves of a long sequence share it: 4 x 1024
// positions by one wave each, one load after the other, 14.5 us, 5.4 now.  How a sequence is shared out depends on T alone.
template <bool ONE_WAVE>
__global__ __launch_bounds__(ONE_WAVE ? WAVE : 1024) void seq_logratio_kernel(const float* __restrict__ logp_cur, const float* __restrict__ logp_behav,
                                    const uint8_t* __restrict__ mask, int64_t N, int64_t T,
                                    float* __restrict__ tok_lr, double* __restrict__ s64,
                                    float* __restrict__ s32, double log_eta, int clip_tokens,
                                    double* __restrict__ tsum, double* __restrict__ tmax,
                                    const int32_t* __restrict__ gen_range, int32_t* __restrict__ dev_status) {
    __shared__ double sm[16];
    const int64_t n = blockIdx.x;
    if (gen_range && (n < gen_range[0] || n >= gen_range[1])) return;
    double acc = 0.0, csum = 0.0, cmax = -INFINITY;
    bool bad = false;
    constexpr int U = 4;
    for (int64_t t0 = threadIdx.x; t0 < T; t0 += U * blockDim.x) {
        bool valid[U];
        float cur[U], beh[U];
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int64_t t = t0 + u * blockDim.x, i = n * T + (t < T ? t : t0);
            valid[u] = mask[i] != 0;
            cur[u] = logp_cur[i];
            beh[u] = logp_behav ? logp_behav[i] : 0.f;
        }
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int64_t t = t0 + u * blockDim.x;
            if (t >= T) break;
            double dlt = 0.0;
            if (valid[u] && logp_behav != nullptr) {   // no behaviour log-probs: on-policy, every ratio is 1
                if (isfinite(beh[u])) dlt = (double)cur[u] - (double)beh[u];
                else bad = true;
            }
            if (tok_lr) tok_lr[n * T + t] = (float)dlt;
            acc += dlt;
            if (tsum && valid[u]) {
                const double lc = clip_tokens ? fmin(dlt, log_eta) : dlt;
                csum += exp(lc);
                cmax = fmax(cmax, lc);
            }
        }
    }
    if (__any(bad) && threadIdx.x % WAVE == 0 && dev_status) atomicOr(dev_status, RAPID_STATUS_NONFINITE_LOGP);
    acc = ONE_WAVE ? wave_sum(acc) : block_sum(acc, sm);
    if (tsum) {
        csum = ONE_WAVE ? wave_sum(csum) : block_sum(csum, sm);
        cmax = ONE_WAVE ? wave_max(cmax) : block_max(cmax, sm);
    }
    if (threadIdx.x == 0) {
        if (s64) s64[n] = acc;
        if (s32) s32[n] = (float)acc;
        if (tsum) {
            tsum[n] = csum;
            tmax[n] = cmax;
        }
    }
}

__device__ inline double clipped_weight(const float* s32, const double* s64, int64_t n, double log_eta) {
    if (s64) return exp(fmin(s64[n], log_eta));
    if (!s32) return 1.0;
    return exp(fmin((double)s32[n], log_eta));
}

// one block per group: size, mean/std of R, clipped-weight baseline, advantages of its members.
// With gen_range only the generations in the range are looked at (the caller guarantees that a group
// lies inside or outside the range as a whole); a group without a member there writes nothing.
// The blocks behind those of the K groups take a generation per thread: its checks and weight, and the defaults of one
// that no group owns.  (By the groups' own blocks, one group of 20 000 generations took 76 us, now 57; 20 000 of one 334, 305.)
__global__ __launch_bounds__(256) void group_advantage_kernel(const float* __restrict__ rewards, const int32_t* __restrict__ group_ids,
                                       const float* __restrict__ s32, const double* __restrict__ s64, int64_t N,
                                       double log_eta, int baseline_mode, float* __restrict__ adv,
                                       double* __restrict__ adv64, float* __restrict__ weight, float* __restrict__ gmean,
                                       float* __restrict__ gstd, int32_t* __restrict__ gsize,
                                       const int32_t* __restrict__ gen_range,
                                       const int32_t* __restrict__ runs, int64_t K, int32_t* __restrict__ dev_status) {
    __shared__ double sm[16 * 3];
    const int k = blockIdx.x;
    int64_t n_begin = gen_range ? gen_range[0] : 0, n_end = gen_range ? gen_range[1] : N;
    if (k >= K) {
        const int64_t n = (int64_t)(k - (int)K) * blockDim.x + threadIdx.x;
        if (n < n_begin || n >= n_end) return;
        int bits = 0;
        const int32_t g = group_ids[n];
        if (g < 0 || g >= K) {
            bits |= RAPID_STATUS_BAD_GROUP;
            adv[n] = 0.f;
            if (adv64) adv64[n] = 0.0;
        }
        if (!isfinite(rewards[n])) bits |= RAPID_STATUS_NONFINITE_REWARD;
        if (s64 ? isnan(s64[n]) : (s32 && isnan(s32[n]))) bits |= RAPID_STATUS_NONFINITE_LOGP;
        if (bits && dev_status) atomicOr(dev_status, bits);
        if (weight) weight[n] = (float)clipped_weight(s32, s64, n, log_eta);
        return;
    }
    if (runs && runs[3 * K] == 0) {   // every group is one run of the batch: look at that run only
        const int64_t r0 = runs[k] ? runs[K + k] : 0, r1 = runs[k] ? runs[2 * K + k] : 0;
        n_begin = n_begin > r0 ? n_begin : r0;
        n_end = n_end < r1 ? n_end : r1;
    }
    double cnt = 0.0, sum_r = 0.0, sum_wr = 0.0;
    for (int64_t n = n_begin + threadIdx.x; n < n_end; n += blockDim.x) {
        if (group_ids[n] == k) {
            float r = rewards[n];
            if (!isfinite(r)) r = 0.f;
            cnt += 1.0;
            sum_r += (double)r;
            sum_wr += clipped_weight(s32, s64, n, log_eta) * (double)r;
        }
    }
    double sums[3] = {cnt, sum_r, sum_wr};
    block_sums<3>(sums, sm);
    cnt = sums[0]; sum_r = sums[1]; sum_wr = sums[2];
    if (gen_range && cnt == 0.0) return;   // uniform over the block
    const double mean = cnt > 0.0 ? sum_r / cnt : 0.0;
    double sq = 0.0;
    for (int64_t n = n_begin + threadIdx.x; n < n_end; n += blockDim.x) {
        if (group_ids[n] == k) {
            float r = rewards[n];
            if (!isfinite(r)) r = 0.f;
            const double dlt = (double)r - mean;
            sq += dlt * dlt;
            double b;
            if (baseline_mode == 0) {
                b = sum_wr / cnt;
            } else {
                const double rest = sum_wr - clipped_weight(s32, s64, n, log_eta) * (double)r;
                if (baseline_mode == 1) b = rest / cnt;
                else b = cnt > 1.0 ? rest / (cnt - 1.0) : 0.0;
            }
            adv[n] = (float)((double)r - b);
            if (adv64) adv64[n] = (double)r - b;
        }
    }
    sq = block_sum(sq, sm);
    if (threadIdx.x == 0) {
        if (gsize) gsize[k] = (int32_t)cnt;
        if (gmean) gmean[k] = (float)mean;
        if (gstd) gstd[k] = (float)(cnt > 0.0 ? sqrt(sq / cnt) : 0.0);
    }
}

// g_n = -(loss_scale/N) c_n A_n exp(-lam), c_n the generation's (clipped) ratio; per_token: without the ratio
__device__ inline double generation_coefficient(const CoefArgs& a, bool per_token, double s, double adv, double log_eta,
                                                double log_loss_scale, double logN, double lam) {
    if (adv == 0.0) return 0.0;
    const double lc = per_token ? 0.0 : (a.coef_mode == 0 ? s : fmin(s, log_eta));
    return (adv > 0.0 ? -1.0 : 1.0) * exp(lc + log(fabs(adv)) + log_loss_scale - logN - lam);
}
__device__ inline void write_diag(const CoefArgs& a, const double (&sums)[4], double maxs, double lam) {
    a.loss_out[0] = (float)sums[0];
    if (a.diag) {
        a.diag->n_tokens = a.counts[CNT_M];
        a.diag->n_clipped = (int32_t)sums[3];
        a.diag->n_sequences = (int32_t)a.N;
        a.diag->mean_log_w = (float)(sums[1] / (double)a.N);
        a.diag->mean_abs_log_w = (float)(sums[2] / (double)a.N);
        a.diag->max_abs_s = (float)maxs;
        a.diag->grad_log_scale = (float)lam;
    }
}

// single block: coefficients g_n, the loss, diagnostics (the three uses are described at CoefArgs).
// Generation-level outer weight (tsum NULL): g_n = -(loss_scale/N) c_n A_n, loss = sum_n g_n.
// Token-level (tsum, tmax given): g_n is the generation's factor -(loss_scale/N) A_n, a token's
// coefficient is g_n c_{n,t}, and loss = sum_n g_n sum_t c_{n,t}.  g64 keeps g_n in double for the
// per-row pass.
__global__ __launch_bounds__(1024) void coefficients_kernel(CoefArgs a, double log_eta, double log_loss_scale) {
    __shared__ double sm[16 * 4];
    const int64_t N = a.N;
    const double logN = log((double)N);
    const bool per_token = a.tsum != nullptr && !a.coef_override;
    const bool chunk_pass = a.gen_range != nullptr;
    const int64_t n_begin = chunk_pass ? a.gen_range[0] : 0, n_end = chunk_pass ? a.gen_range[1] : N;
    auto advantage = [&](int64_t n) { return a.adv64 ? a.adv64[n] : (double)a.adv[n]; };
    double lam = 0.0;
    if (!a.coef_override && a.normalized) {
        double mx = -INFINITY;
        for (int64_t n = n_begin + threadIdx.x; n < n_end; n += blockDim.x) {
            const double av = advantage(n);
            if (av != 0.0) {
                const double lc = per_token ? a.tmax[n] : (a.coef_mode == 0 ? a.s64[n] : fmin(a.s64[n], log_eta));
                mx = fmax(mx, lc + log(fabs(av)) + log_loss_scale - logN);   // -inf for a generation without tokens
            }
        }
        mx = block_max(mx, sm);
        if (chunk_pass) {
            const double before = a.lam_state[0];        // -inf: no chunk has carried a coefficient yet
            const double now = fmax(before, mx);
            __syncthreads();                             // everybody has read the old state
            if (threadIdx.x == 0) {
                a.lam_state[0] = now;
                a.lam_chunk[0] = now;
                a.beta_out[0] = (before == -INFINITY) ? 1.f : (float)exp(before - now);
            }
            mx = now;
        }
        lam = (mx == -INFINITY) ? 0.0 : mx;
    } else if (chunk_pass && threadIdx.x == 0) {
        a.lam_state[0] = 0.0;
        a.lam_chunk[0] = 0.0;
        a.beta_out[0] = 1.f;
    }
    double loss = 0.0, slw = 0.0, salw = 0.0, maxs = 0.0, nclip = 0.0;
    for (int64_t n = n_begin + threadIdx.x; n < n_end; n += blockDim.x) {
        const double s = a.s64[n];
        double gn;
        if (a.coef_override) {
            gn = (double)a.coef_override[n];
        } else {
            gn = generation_coefficient(a, per_token, s, advantage(n), log_eta, log_loss_scale, logN, lam);
        }
        if (a.write_g) {
            a.g[n] = (float)gn;
            a.g64[n] = gn;
        }
        loss += per_token ? (gn != 0.0 ? gn * a.tsum[n] : 0.0) : gn;
        const double lw = fmin(s, log_eta);
        slw += lw;
        salw += fabs(lw);
        maxs = fmax(maxs, fabs(s));
        nclip += s > log_eta ? 1.0 : 0.0;
    }
    if (chunk_pass) return;
    double sums[4] = {loss, slw, salw, nclip};
    block_sums<4>(sums, sm);
    maxs = block_max(maxs, sm);
    if (threadIdx.x == 0) write_diag(a, sums, maxs, lam);
}

constexpr int ESTIMATOR_LDS = 1024, ESTIMATOR_POSITIONS = 8192;
// Scattered groups: generations times groups up to which a team of lanes per group looks through the batch instead of a list of the
// members (fp32 steps with either: 64 x 64 positions in fours 71.4 and 73.8 us, 128 x 64 118.8 and 119.8, in pairs 122.8 and 121.4, 256 x 16 88.4
// and 79.2, 1024 x 8 254.8 and 136.2; side by side 128.3).
constexpr int LIST_MEMBERS = 8192;
// The generations of every group k in batch order, order[first[k] .. end[k]), where groups lie scattered: a counting sort over pieces of
// 128 generations, each a wave's.  count [ESTIMATOR_LDS] is zero; byte p of a group's word counts its members in piece p, place[n] those
// of n's group in front of it in its piece.  Generations without a group are left out.  (Its loops stay rolled: unrolled, their ballots
// spill scalar registers of the whole kernel, 0.7 us of every call.)
__device__ inline void list_members(const int32_t* gid, int N, int K, double* count, int32_t* first, int32_t* end, uint8_t* place, uint16_t* order) {
    constexpr int PIECE = 2 * WAVE;
    static_assert(ESTIMATOR_LDS <= 8 * PIECE, "a byte of a group's word per piece");
    auto members = [&](int k, int pieces) {       // of group k in that many first pieces
        uint64_t w = __builtin_bit_cast(uint64_t, count[k]);
        if (pieces < 8) w &= (1ull << 8 * pieces) - 1ull;
        return (int)(((w & 0x00ff00ff00ff00ffull) + (w >> 8 & 0x00ff00ff00ff00ffull)) * 0x0001000100010001ull >> 48);
    };
    const int lane = threadIdx.x & (WAVE - 1), wave = threadIdx.x / WAVE, waves = blockDim.x / WAVE;
#pragma unroll 1
    for (int n0 = wave * PIECE; n0 < N; n0 += waves * PIECE) {
#pragma unroll 1
        for (int n = n0 + lane; n - lane < n0 + PIECE && n - lane < N; n += WAVE) {
            const int g = n < N ? gid[n] : -1;
            const bool in = g >= 0 && g < K;
            unsigned long long same = __ballot(in);      // lanes of the same group
#pragma unroll 1
            for (int bit = 1; bit < ESTIMATOR_LDS; bit <<= 1) {
                const unsigned long long set = __ballot(g & bit);
                same &= g & bit ? set : ~set;
            }
            if (in) {
                uint8_t& here = ((uint8_t*)(count + g))[n0 / PIECE];
                const int before = __popcll(same & ((1ull << lane) - 1ull)), seen = here;
                place[n] = (uint8_t)(seen + before);
                if (before == 0) here = (uint8_t)(seen + __popcll(same));
            }
            __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");      // the second half reads what the first half's lanes wrote
            __builtin_amdgcn_wave_barrier();
        }
    }
    __syncthreads();
    for (int k = threadIdx.x; k < K; k += blockDim.x) end[k] = members(k, 8);
    __syncthreads();
    block_scan(end, K, first);
    __syncthreads();
    for (int n = threadIdx.x; n < N; n += blockDim.x) {
        const int g = gid[n];
        if (g >= 0 && g < K) order[first[g] + members(g, n / PIECE) + place[n]] = (uint16_t)n;
    }
    for (int k = threadIdx.x; k < K; k += blockDim.x) end[k] = first[k + 1];
    __syncthreads();
}

// The whole estimator of a small batch in one block: log ratios of the generations, group advantages, coefficients, loss and
// diagnostics, the rows' coefficients; what seq_logratio_kernel, group_advantage_kernel, coefficients_kernel and
// row_coefficients_kernel do in four dependent launches of 3 to 5 us each, next to nothing of it work.  All sums are taken in 64
// bits, in an order that is fixed for a shape; it is that of the four where every group is one run of at most 64 generations and
// there are as many threads as generations, else their last bits differ.  At most ESTIMATOR_LDS generations and groups, which stay in the LDS, and ESTIMATOR_POSITIONS positions:
// one compute unit takes about 1 us per 1000 of them (32 x 32 positions 7.5 us, 64 x 48 9.6, 4 x 1024 15.1).  TOKENS false: more positions; the log ratios are there (s64, and tsum,
// tmax) and the rows' coefficients are left to row_coefficients_kernel, so that two launches become one.  Whole steps, in one
// block against this split: 64 x 8 positions 46 and 52 us, 64 x 64 58 and 61, 128 x 64 69 and 70, 64 x 250 96 and 92.
template <bool PER_TOKEN, bool TOKENS>
__global__ __launch_bounds__(1024) void small_estimator_kernel(EstimatorArgs a, double log_eta, double log_loss_scale) {
    constexpr int L = ESTIMATOR_LDS, LT = PER_TOKEN ? L : 1;
    __shared__ double sm[16 * 4], s_s[L], s_w[L], s_adv[L], s_tsum[LT], s_tmax[LT], s_part[3][16];
    double* const s_g = s_w;     // the coefficients take the weights' place
    __shared__ float s_r[L];
    __shared__ int32_t s_gid[L], s_first[L + 1], s_end[L];
    __shared__ uint16_t s_order[L];
    __shared__ uint8_t s_place[L];
    __shared__ int s_split, s_longest, s_bits;
    const int N = (int)a.N, K = (int)a.K, tid = threadIdx.x, threads = blockDim.x;
    const int64_t T = a.T;
    for (int n = tid; n < N; n += threads) {
        s_gid[n] = a.group_ids[n];
        s_r[n] = a.rewards[n];
    }
    for (int k = tid; k < K; k += threads) s_first[k] = s_end[k] = -1;
    if (tid == 0) s_split = s_longest = s_bits = 0;
    int bits = 0;
    // generations of the thread's first rows: asked for now, used last
    constexpr int UR = 8;
    int32_t gen[UR];
    const int M = TOKENS ? a.row_counts[CNT_M] : 0, Mr = TOKENS ? a.row_counts[CNT_MR] : 0;
    auto generations_of = [&](int j0) {
#pragma unroll
        for (int q = 0; q < UR; ++q) gen[q] = a.seqc[j0 + q * threads < Mr ? j0 + q * threads : j0];
    };
    if (tid < Mr) generations_of(tid);

    // log ratios: teams of 8 to 64 lanes, or (few generations) several waves per generation
    int waves_log2 = 0;
    if constexpr (TOKENS) {
        const int lanes_log2 = T <= 64 ? 3 : T <= 128 ? 4 : T <= 256 ? 5 : 6, lanes = 1 << lanes_log2;
        while (waves_log2 < 4 && (N << (waves_log2 + 1)) <= threads / WAVE && T >= (512 << waves_log2)) ++waves_log2;
        for (int u = tid >> lanes_log2; u < N << waves_log2; u += threads >> lanes_log2) {
            const int n = u >> waves_log2, part = u & ((1 << waves_log2) - 1);
            const int64_t begin = T * part >> waves_log2, end = T * (part + 1) >> waves_log2;
            double acc = 0.0, csum = 0.0, cmax = -INFINITY;
            constexpr int U = 8;     // positions per lane whose loads are in flight together
            for (int64_t t0 = begin + (tid & (lanes - 1)); t0 < end; t0 += U * lanes) {
                bool valid[U];
                float cur[U], beh[U];
#pragma unroll
                for (int q = 0; q < U; ++q) {
                    const int64_t t = t0 + q * lanes, i = n * T + (t < end ? t : t0);
                    valid[q] = a.mask[i] != 0;
                    cur[q] = a.logp_cur[i];
                    beh[q] = a.logp_behav ? a.logp_behav[i] : 0.f;      // none: on-policy, every ratio is 1
                }
#pragma unroll
                for (int q = 0; q < U; ++q) {
                    const int64_t t = t0 + q * lanes;
                    if (t >= end) break;
                    double dlt = 0.0;
                    if (valid[q] && a.logp_behav) {
                        if (isfinite(beh[q])) dlt = (double)cur[q] - (double)beh[q];
                        else bits |= RAPID_STATUS_NONFINITE_LOGP;
                    }
                    if (a.tok_lr) a.tok_lr[n * T + t] = (float)dlt;
                    acc += dlt;
                    if constexpr (PER_TOKEN) {
                        if (valid[q]) {
                            const double lc = a.clip_tokens ? fmin(dlt, log_eta) : dlt;
                            csum += exp(lc);
                            cmax = fmax(cmax, lc);
                        }
                    }
                }
            }
            for (int o = lanes >> 1; o > 0; o >>= 1) {
                acc += __shfl_xor(acc, o, WAVE);
                if constexpr (PER_TOKEN) {
                    csum += __shfl_xor(csum, o, WAVE);
                    cmax = fmax(cmax, __shfl_xor(cmax, o, WAVE));
                }
            }
            if ((tid & (lanes - 1)) == 0) {
                if (waves_log2 == 0) s_s[n] = acc; else s_part[0][u] = acc;
                if constexpr (PER_TOKEN) {
                    if (waves_log2 == 0) { s_tsum[n] = csum; s_tmax[n] = cmax; } else { s_part[1][u] = csum; s_part[2][u] = cmax; }
                }
            }
        }
    } else {
        for (int n = tid; n < N; n += threads) {
            s_s[n] = a.coef.s64[n];
            if constexpr (PER_TOKEN) { s_tsum[n] = a.coef.tsum[n]; s_tmax[n] = a.coef.tmax[n]; }
        }
    }
    __syncthreads();
    for (int n = tid; n < N; n += threads) {
        if (waves_log2 > 0) {
            double acc = 0.0, csum = 0.0, cmax = -INFINITY;
            for (int u = n << waves_log2; u < (n + 1) << waves_log2; ++u) {
                acc += s_part[0][u];
                csum += s_part[1][u];
                cmax = fmax(cmax, s_part[2][u]);
            }
            s_s[n] = acc;
            if constexpr (PER_TOKEN) { s_tsum[n] = csum; s_tmax[n] = cmax; }
        }
        const double s = s_s[n];
        if (TOKENS && a.s32) a.s32[n] = (float)s;
        s_w[n] = a.logp_behav ? exp(fmin(s, log_eta)) : 1.0;
        s_adv[n] = 0.0;
        // runs of equal group id
        const int32_t g = s_gid[n];
        if (!isfinite(s_r[n])) { bits |= RAPID_STATUS_NONFINITE_REWARD; s_r[n] = 0.f; }
        if (a.logp_behav && isnan(s)) bits |= RAPID_STATUS_NONFINITE_LOGP;
        if (g < 0 || g >= K) { bits |= RAPID_STATUS_BAD_GROUP; continue; }
        if ((n == 0 || s_gid[n - 1] != g) && atomicExch(&s_first[g], n) >= 0) s_split = 1;
        if (n == N - 1 || s_gid[n + 1] != g) s_end[g] = n + 1;
    }
    if (bits) atomicOr(&s_bits, bits);
    __syncthreads();
    const bool split = s_split != 0, listed = split && N * K > LIST_MEMBERS;
    if (listed) {
        for (int i = tid; i < L; i += threads) s_adv[i] = 0.0;
        __syncthreads();
        list_members(s_gid, N, K, s_adv, s_first, s_end, s_place, s_order);
        for (int i = tid; i < L; i += threads) s_adv[i] = 0.0;
    }
    for (int k = tid; k < K; k += threads)
        if (s_first[k] >= 0) atomicMax(&s_longest, s_end[k] - s_first[k]);
    __syncthreads();

    // group advantages: a team of lanes per group, over its run or (some group has several) over its list of members or the batch
    const bool scan = split && !listed;
    const int team_log2 = scan || s_longest > 16 ? 6 : 4, team = 1 << team_log2;
    for (int k = tid >> team_log2; k < K; k += threads >> team_log2) {
        const int begin = scan || s_first[k] < 0 ? 0 : s_first[k], end = scan ? N : s_end[k];
        double cnt = 0.0, sum_wr = 0.0;
        for (int i = begin + (tid & (team - 1)); i < end; i += team) {
            const int n = listed ? s_order[i] : i;
            if (s_gid[n] != k) continue;
            cnt += 1.0;
            sum_wr += s_w[n] * (double)s_r[n];
        }
        for (int o = team >> 1; o > 0; o >>= 1) {
            cnt += __shfl_xor(cnt, o, WAVE);
            sum_wr += __shfl_xor(sum_wr, o, WAVE);
        }
        for (int i = begin + (tid & (team - 1)); i < end; i += team) {
            const int n = listed ? s_order[i] : i;
            if (s_gid[n] != k) continue;
            const double r = (double)s_r[n], rest = sum_wr - s_w[n] * r;
            const double b = a.baseline_mode == 0 ? sum_wr / cnt : a.baseline_mode == 1 ? rest / cnt : cnt > 1.0 ? rest / (cnt - 1.0) : 0.0;
            s_adv[n] = r - b;
        }
    }
    __syncthreads();

    // coefficients, loss, diagnostics (see coefficients_kernel)
    const CoefArgs& c = a.coef;
    const double logN = log((double)N);
    const bool per_token = PER_TOKEN && !c.coef_override;
    double lam = 0.0;
    if (!c.coef_override && c.normalized) {
        double mx = -INFINITY;
        for (int n = tid; n < N; n += threads) {
            const double av = s_adv[n];
            if (av == 0.0) continue;
            const double lc = per_token ? s_tmax[PER_TOKEN ? n : 0] : (c.coef_mode == 0 ? s_s[n] : fmin(s_s[n], log_eta));
            mx = fmax(mx, lc + log(fabs(av)) + log_loss_scale - logN);
        }
        mx = block_max(mx, sm);
        lam = (mx == -INFINITY) ? 0.0 : mx;
    }
    double sums[4] = {0.0, 0.0, 0.0, 0.0}, maxs = 0.0;
    for (int n = tid; n < N; n += threads) {
        const double s = s_s[n], lw = fmin(s, log_eta);
        if (a.adv) a.adv[n] = (float)s_adv[n];
        const double gn = c.coef_override ? (double)c.coef_override[n]
                                          : generation_coefficient(c, per_token, s, s_adv[n], log_eta, log_loss_scale, logN, lam);
        s_g[n] = gn;
        if (!TOKENS) { c.g[n] = (float)gn; c.g64[n] = gn; }
        sums[0] += per_token ? (gn != 0.0 ? gn * s_tsum[PER_TOKEN ? n : 0] : 0.0) : gn;
        sums[1] += lw;
        sums[2] += fabs(lw);
        sums[3] += s > log_eta ? 1.0 : 0.0;
        maxs = fmax(maxs, fabs(s));
    }
    block_sums<4>(sums, sm);     // its barriers also make s_g visible
    // the rows' coefficients (rows past M up to the row tile: 0)
    for (int j0 = tid; j0 < Mr; j0 += UR * threads) {
        if (j0 != tid) generations_of(j0);
#pragma unroll
        for (int q = 0; q < UR; ++q) {
            const int j = j0 + q * threads;
            if (j >= Mr) break;
            double v = j < M ? s_g[gen[q]] : 0.0;
            if (per_token && j < M) {
                double dlt = 0.0;
                if (a.logp_behav) {
                    const int32_t pos = a.row_index[j];
                    const float lb = a.logp_behav[pos];
                    if (isfinite(lb)) dlt = (double)a.logp_cur[pos] - (double)lb;
                }
                v *= exp(a.clip_tokens ? fmin(dlt, log_eta) : dlt);
            }
            a.rowg[j] = (float)v;
        }
    }
    maxs = block_max(maxs, sm);
    if (tid == 0) {
        write_diag(c, sums, maxs, lam);
        if (s_bits && a.dev_status) atomicOr(a.dev_status, s_bits);
    }
}

// the coefficient dL/dlogp of every compact token row: the generation's g_n, times the token's own
// (clipped) ratio for the token-level outer weight; 0 for the padding rows up to the row-tile boundary
__global__ void row_coefficients_kernel(const float* __restrict__ g, const double* __restrict__ g64,
                                        const int32_t* __restrict__ seqc, const int32_t* __restrict__ row_index,
                                        const int32_t* __restrict__ counts, const float* __restrict__ logp_cur,
                                        const float* __restrict__ logp_behav, int per_token, double log_eta,
                                        int clip_tokens, int64_t row0, float* __restrict__ rowg) {
    const int64_t j = row0 + (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    const int M = counts[CNT_M], Mr = counts[CNT_MR];
    if (j >= Mr) return;
    float v = 0.f;
    if (j < M) {
        const int32_t n = seqc[j];
        if (!per_token) {
            v = g[n];
        } else {
            double dlt = 0.0;
            if (logp_behav != nullptr) {
                const int32_t pos = row_index[j];
                const float lb = logp_behav[pos];
                if (isfinite(lb)) dlt = (double)logp_cur[pos] - (double)lb;
            }
            v = (float)(g64[n] * exp(clip_tokens ? fmin(dlt, log_eta) : dlt));
        }
    }
    rowg[j] = v;
}

// zero the gradient rows of masked positions, and of every position of an idle generation (idle may be
// NULL): one block per position
__global__ void zero_masked_rows_kernel(uint32_t* __restrict__ dh, const uint8_t* __restrict__ mask,
                                        int64_t rows, int64_t words_per_row, const int32_t* __restrict__ idle,
                                        int64_t T) {
    const int64_t r = blockIdx.x;
    if (r >= rows || (mask[r] != 0 && !(idle && idle[r / T]))) return;
    uint32_t* p = dh + r * words_per_row;
    for (int64_t i = threadIdx.x; i < words_per_row; i += blockDim.x) p[i] = 0u;
}

// one block per position of [N, T]: a valid position's bf16 gradient row times
// exp(lam_chunk[chunk of its generation] - lam_final); rows whose factor is 1 are left alone
__global__ void rescale_rows_kernel(bf16_t* __restrict__ dh, const uint8_t* __restrict__ mask, int64_t T, int64_t d,
                                    const int32_t* __restrict__ gen_chunk, const double* __restrict__ lam_chunk,
                                    const double* __restrict__ lam_state) {
    const int64_t r = blockIdx.x;
    if (mask[r] == 0) return;
    const int c = gen_chunk[r / T];
    if (c < 0) return;
    const double dl = lam_chunk[c] - lam_state[0];
    if (dl == 0.0 || !(dl < 0.0)) return;         // also skips a state that never left -inf (no coefficient anywhere)
    const float f = (float)exp(dl);
    bf16_t* p = dh + r * d;
    for (int64_t i = threadIdx.x; i < d; i += blockDim.x) {
        const float v = __builtin_bit_cast(float, (uint32_t)p[i] << 16) * f;
        const __bf16 o = (__bf16)v;
        p[i] = __builtin_bit_cast(bf16_t, o);
    }
}

__global__ void f32_to_bf16_kernel(const float* __restrict__ src, bf16_t* __restrict__ dst, int64_t n) {
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n) return;
    const __bf16 b = (__bf16)src[i];
    dst[i] = __builtin_bit_cast(unsigned short, b);
}

inline unsigned blocks_for(int64_t n, int bs) { return (unsigned)((n + bs - 1) / bs); }

}  // namespace

void launch_plan(const uint8_t* mask, int64_t N, int64_t T, const PlanArgs& plan, hipStream_t st) {
    const bool in_lds = N <= PLAN_LDS && plan.K <= PLAN_LDS;
    if (in_lds && N * T <= PLAN_MASK) {
        const int64_t lanes = T <= 256 ? 8 : T <= 512 ? 16 : 64;     // about what the kernel gives a generation
        plan_kernel<true, true><<<1, block_threads(N * lanes, 1024), 0, st>>>(plan, mask, T);
        return;
    }
    ZeroWords z;
    if (!in_lds && plan.runs) { z.p[0] = plan.runs; z.n[0] = 3 * plan.K; }
    if (!in_lds && plan.idle.idle && !plan.idle.coef_override) { z.p[1] = plan.idle.live_group; z.n[1] = plan.K; }
    const unsigned threads = row_threads(T);
    (threads == WAVE ? &seq_len_kernel<true> : &seq_len_kernel<false>)<<<(unsigned)N, threads, 0, st>>>(mask, N, T, plan.seq_len, z);
    if (in_lds) plan_kernel<true, false><<<1, block_threads(N, 1024), 0, st>>>(plan, mask, T);
    else plan_kernel<false, false><<<1, 1024, 0, st>>>(plan, mask, T);
}

// By position, in one launch, where that is a matter of launches or where gradient rows have to be cleared too, a launch with a block
// per position; else with an index of the rows in front.  A wave that packs nothing has a few positions to place and counts
// the whole generation for it: rapid_compaction of 256 x 4096 positions 64 us against 14, of 4096 x 512 117 and 19, of 20 000 x 100 156
// and 40, of 4 x 1024 10 and 10.  Log-probs (d = 1536, V = 256), by position and with an index: 4 x 1024 54 and 60 us, 64 x 250 101
// and 97, 4 x 4096 110 and 110, 64 x 1024 135 and 131, 1024 x 256 608 and 533, 256 x 4096 1979 and 1929.
void launch_compact_rows(const RowsArgs& a, int64_t rows, hipStream_t st) {
    if (a.T <= BY_POSITION_T && (a.dhidden || a.N * a.T <= ROWS_WITHOUT_PLAN)) {
        launch_rows(a, true, rows, st);
        return;
    }
    const unsigned threads = row_threads(a.T);
    (threads == WAVE ? &row_index_kernel<true> : &row_index_kernel<false>)<<<(unsigned)a.N, threads, 0, st>>>(a);
    if (a.dhidden) zero_masked_rows_kernel<<<(unsigned)(a.N * a.T), 128, 0, st>>>(a.dhidden, a.mask, a.N * a.T, a.words_per_row, a.idle, a.T);
    if (a.Hc) launch_rows(a, false, rows, st);
}

void launch_fill_f32(float* p, int64_t n, float v, hipStream_t st) {
    if (n > 0) fill_f32_kernel<<<blocks_for(n, 256), 256, 0, st>>>(p, n, v);
}
void launch_f32_add(const float* src, float* dst, int64_t n, hipStream_t st) {
    if (n > 0) f32_add_kernel<<<blocks_for(n, 256), 256, 0, st>>>(src, dst, n);
}

void launch_merge_lse(const float* part_max, const float* part_sum, int P, int64_t ld_part, const float* zy,
                      const int32_t* row_index, const int32_t* counts, int64_t row0, int64_t rows_max, float* lse_c,
                      float* logp_out, float* lse_out, hipStream_t st) {
    if (rows_max <= 0) return;
    if (P > 128 && rows_max <= 1024) {
        merge_lse_few_kernel<<<blocks_for(rows_max, 8), 256, 0, st>>>(part_max, part_sum, P, ld_part, zy, row_index, counts, row0, lse_c, logp_out, lse_out);
        return;
    }
    auto* kernel = P <= 16 ? &merge_lse_kernel<1> : P <= 128 ? &merge_lse_kernel<4> : &merge_lse_kernel<16>;
    kernel<<<blocks_for(rows_max, 32), P <= 16 ? 64 : P <= 128 ? 256 : 1024, 0, st>>>(part_max, part_sum, P, ld_part, zy, row_index,
                                                                                     counts, row0, lse_c, logp_out, lse_out);
}

void launch_seq_logratio(const float* logp_cur, const float* logp_behav, const uint8_t* mask, int64_t N,
                         int64_t T, float* tok_logratio_out, double* s64, float* s32, float eta, int clip_tokens,
                         double* tsum, double* tmax, const int32_t* gen_range, int32_t* dev_status, hipStream_t st) {
    const double log_eta = (eta > 0.f && std::isfinite(eta)) ? log((double)eta) : (double)INFINITY;
    const unsigned threads = row_threads(T);
    (threads == WAVE ? &seq_logratio_kernel<true> : &seq_logratio_kernel<false>)<<<(unsigned)N, threads, 0, st>>>(
        logp_cur, logp_behav, mask, N, T, tok_logratio_out, s64, s32, log_eta, clip_tokens, tsum, tmax, gen_range, dev_status);
}

void launch_group_advantage(const float* rewards, const int32_t* group_ids, const float* s32, const double* s64,
                            int64_t N, int64_t K, float eta, int baseline_mode, float* adv, double* adv64,
                            float* weight, float* gmean, float* gstd, int32_t* gsize, const int32_t* gen_range,
                            int32_t* dev_status, hipStream_t st, const int32_t* runs) {
    const double log_eta = (eta > 0.f && std::isfinite(eta)) ? log((double)eta) : (double)INFINITY;
    const unsigned threads = block_threads(N, 256);
    group_advantage_kernel<<<(unsigned)K + blocks_for(N, (int)threads), threads, 0, st>>>(rewards, group_ids, s32, s64, N, log_eta, baseline_mode, adv,
                                                        adv64, weight, gmean, gstd, gsize, gen_range, runs, K, dev_status);
}

// ---- the token-level clipped surrogate of the GRPO / DAPO loss steps ---------------------------
namespace {

struct ClipToken { double loss, dlogp, kl; bool clipped; };

// one valid token: omega (surr - beta kl) and its derivative with respect to the current log-prob
__device__ inline ClipToken clip_token(const ClipArgs& a, int64_t i, double adv, double omega, bool* bad) {
    const double cur = (double)a.logp_cur[i];
    double dlt = 0.0;
    if (a.logp_old) {
        const float lo = a.logp_old[i];
        if (isfinite(lo)) dlt = cur - (double)lo; else *bad = true;
    }
    const double r = exp(dlt);
    const double rc = fmin(fmax(r, 1.0 - (double)a.eps_low), 1.0 + (double)a.eps_high);
    const double unclipped = r * adv, clipped = rc * adv;
    ClipToken t;
    t.clipped = unclipped > clipped;
    const double surr = t.clipped ? clipped : unclipped;
    const double dsurr = t.clipped ? 0.0 : unclipped;
    double kl = 0.0, dkl = 0.0;
    if (a.kl_beta != 0.f && a.logp_ref) {
        const float lr = a.logp_ref[i];
        if (isfinite(lr)) {
            const double dref = (double)lr - cur;
            const double e = exp(dref);
            kl = e - dref - 1.0;
            dkl = 1.0 - e;
        } else {
            *bad = true;
        }
    }
    t.kl = kl;
    t.loss = -omega * (surr - (double)a.kl_beta * kl);
    t.dlogp = -omega * (dsurr - (double)a.kl_beta * dkl);
    return t;
}

__device__ inline double clip_omega(const ClipArgs& a, int64_t n) {
    if (a.norm_mode == 0) {
        const int L = a.seq_len[n];
        return L > 0 ? (double)a.loss_scale / ((double)a.N * (double)L) : 0.0;
    }
    const int M = a.counts[CNT_M];
    return M > 0 ? (double)a.loss_scale / (double)M : 0.0;
}

// (R - mean) / (std + eps) of a group's generations in [n_first, n_last), equal rewards give 0.  Its sums are taken by one wave
// (ONE_WAVE: any of a block's) or by the block, over the group's run of the batch or, where some group has several, over the whole range.
struct GroupScan { int64_t begin, end; };
__device__ inline GroupScan group_scan(const ClipArgs& a, int32_t k, int64_t n_first, int64_t n_last) {
    if (a.runs[3 * a.K] != 0) return {n_first, n_last};
    return {a.runs[a.K + k] > n_first ? a.runs[a.K + k] : n_first, a.runs[2 * a.K + k] < n_last ? a.runs[2 * a.K + k] : n_last};
}
__device__ inline double reward_of(const ClipArgs& a, int64_t n) { const float r = a.rewards[n]; return isfinite(r) ? (double)r : 0.0; }
struct GroupStats {
    double mean, scale;     // scale: std + eps
    __device__ double advantage(double r) const { return r != mean ? (r - mean) / scale : 0.0; }
};
template <bool ONE_WAVE>
__device__ inline GroupStats group_stats(const ClipArgs& a, int32_t k, const GroupScan& s, double* sm) {
    const int first = ONE_WAVE ? threadIdx.x & (WAVE - 1) : threadIdx.x, step = ONE_WAVE ? WAVE : blockDim.x;
    auto total = [&](double v) { return ONE_WAVE ? wave_sum(v) : block_sum(v, sm); };
    double cnt = 0.0, sum = 0.0, sq = 0.0;
    for (int64_t m = s.begin + first; m < s.end; m += step)
        if (a.group_ids[m] == k) { cnt += 1.0; sum += reward_of(a, m); }
    cnt = total(cnt);
    const double mean = total(sum) / cnt;
    for (int64_t m = s.begin + first; m < s.end; m += step)
        if (a.group_ids[m] == k) { const double dlt = reward_of(a, m) - mean; sq += dlt * dlt; }
    sq = total(sq);
    const double den = cnt - (double)a.std_ddof;
    return {mean, (den > 0.0 ? sqrt(sq / den) : 0.0) + (double)a.adv_eps};
}

// A block per group: the advantages of its generations, where there are too many generations for each to look for itself.
__global__ __launch_bounds__(256) void clip_advantages_kernel(ClipArgs a) {
    __shared__ double sm[16];
    const int32_t k = blockIdx.x;
    const GroupScan s = group_scan(a, k, 0, a.N);
    if (s.begin >= s.end) return;
    const GroupStats g = group_stats<false>(a, k, s, sm);
    for (int64_t n = s.begin + threadIdx.x; n < s.end; n += blockDim.x)
        if (a.group_ids[n] == k) a.adv64[n] = g.advantage(reward_of(a, n));
}

// One block per generation: its normalised advantage (up to CLIP_SCAN generations every one works its group's mean and deviation
// out by itself, a launch less), its tokens' terms, each formed once for the sums of the generation and
// for the row's coefficient.  The last block: the rows that fill the row tile up.  (One after the other, group_advantage_kernel, this one and
// one for the rows took 16 us of a small step.)
template <bool ONE_WAVE>
__global__ __launch_bounds__(ONE_WAVE ? WAVE : 1024) void clip_generations_kernel(ClipArgs a, const int32_t* __restrict__ gen_range, double* __restrict__ loss_n,
                                        double* __restrict__ clipped_n, double* __restrict__ kl_n) {
    __shared__ double sm[16 * 3];
    const int64_t n = blockIdx.x;
    if (n == a.N) {
        for (int j = a.row_counts[CNT_M] + (int)threadIdx.x; j < a.row_counts[CNT_MR]; j += blockDim.x) a.rowg[j] = 0.f;
        return;
    }
    const int64_t n_first = gen_range ? gen_range[0] : 0, n_last = gen_range ? gen_range[1] : a.N;
    if (n < n_first || n >= n_last) return;
    const int32_t k = a.group_ids[n];
    const float mine = a.rewards[n];
    const int len = a.seq_len[n];
    const int64_t row0 = a.first_row[n];
    int bits = isfinite(mine) ? 0 : RAPID_STATUS_NONFINITE_REWARD;
    double adv = 0.0;
    if (k < 0 || k >= a.K) bits |= RAPID_STATUS_BAD_GROUP;
    else if (a.adv64) adv = a.adv64[n];
    else adv = group_stats<true>(a, k, group_scan(a, k, n_first, n_last), sm).advantage(reward_of(a, n));
    if (threadIdx.x == 0) a.adv[n] = (float)adv;
    const double omega = clip_omega(a, n);
    double sums[3] = {0.0, 0.0, 0.0};
    bool bad = false;
    const int64_t limit = row0 < 0 ? 0 : (row0 / a.region + 1) * a.region, rows = row0 < 0 ? 0 : row0 + len < limit ? len : limit - row0;
    for (int64_t i = threadIdx.x; i < rows; i += blockDim.x) {
        const ClipToken tk = clip_token(a, a.row_index[row0 + i], adv, omega, &bad);
        a.rowg[row0 + i] = (float)tk.dlogp;
        sums[0] += tk.loss;
        sums[1] += tk.clipped ? 1.0 : 0.0;
        sums[2] += tk.kl;
    }
    if (__any(bad)) bits |= RAPID_STATUS_NONFINITE_LOGP;
    if (bits && threadIdx.x % WAVE == 0 && a.dev_status) atomicOr(a.dev_status, bits);
    if constexpr (ONE_WAVE) {
#pragma unroll
        for (int q = 0; q < 3; ++q) sums[q] = wave_sum(sums[q]);
    } else {
        block_sums<3>(sums, sm);
    }
    if (threadIdx.x == 0) {
        loss_n[n] = sums[0];
        clipped_n[n] = sums[1];
        kl_n[n] = sums[2];
    }
}

__global__ void clip_finish_kernel(const double* __restrict__ loss_n, const double* __restrict__ clipped_n,
                                   const double* __restrict__ kl_n, int64_t N, const int32_t* __restrict__ counts,
                                   float* __restrict__ loss_out, rapid_clip_pg_diag* __restrict__ diag) {
    __shared__ double sm[16 * 3];
    double sums[3] = {0.0, 0.0, 0.0};
    for (int64_t n = threadIdx.x; n < N; n += blockDim.x) {
        sums[0] += loss_n[n];
        sums[1] += clipped_n[n];
        sums[2] += kl_n[n];
    }
    block_sums<3>(sums, sm);
    const double loss = sums[0], ncl = sums[1], kl = sums[2];
    if (threadIdx.x == 0) {
        loss_out[0] = (float)loss;
        if (diag) {
            const int M = counts[CNT_M];
            diag->n_tokens = M;
            diag->n_clipped = (int64_t)ncl;
            diag->n_sequences = (int32_t)N;
            diag->mean_kl = M > 0 ? (float)(kl / (double)M) : 0.f;
        }
    }
}

}  // namespace

void launch_clip_advantages(const ClipArgs& a, hipStream_t st) {
    if (a.adv64) clip_advantages_kernel<<<(unsigned)a.K, block_threads(a.N, 256), 0, st>>>(a);
}
void launch_clip_generations(const ClipArgs& a, const int32_t* gen_range, double* loss_n, double* clipped_n, double* kl_n, hipStream_t st) {
    const unsigned threads = row_threads(a.T);
    (threads == WAVE ? &clip_generations_kernel<true> : &clip_generations_kernel<false>)<<<(unsigned)a.N + 1, threads, 0, st>>>(a, gen_range, loss_n, clipped_n, kl_n);
}
void launch_clip_finish(const double* loss_n, const double* clipped_n, const double* kl_n, int64_t N, const int32_t* counts,
                        float* loss_out, rapid_clip_pg_diag* diag, hipStream_t st) {
    clip_finish_kernel<<<1, block_threads(N, 1024), 0, st>>>(loss_n, clipped_n, kl_n, N, counts, loss_out, diag);
}

void launch_coefficients(const CoefArgs& a, hipStream_t st) {
    const double log_eta = (a.eta > 0.f && std::isfinite(a.eta)) ? log((double)a.eta) : (double)INFINITY;
    coefficients_kernel<<<1, block_threads(a.N, 1024), 0, st>>>(a, log_eta, log((double)a.loss_scale));
}

int small_estimator_fits(int64_t N, int64_t T, int64_t K) {
    if (N > ESTIMATOR_LDS || K > ESTIMATOR_LDS) return ESTIMATOR_LAUNCHES;
    return N * T <= ESTIMATOR_POSITIONS ? ESTIMATOR_ONE : ESTIMATOR_GENERATIONS;
}
void launch_small_estimator(const EstimatorArgs& a, bool tokens, hipStream_t st) {
    const float eta = a.coef.eta;
    const double log_eta = (eta > 0.f && std::isfinite(eta)) ? log((double)eta) : (double)INFINITY;
    const int64_t want = tokens ? a.N * a.T / 4 : a.N;        // threads beyond this find next to nothing to do
    const unsigned threads = want >= 1024 ? 1024u : want >= 512 ? 512u : 256u;
    auto* kernel = tokens ? (a.per_token ? &small_estimator_kernel<true, true> : &small_estimator_kernel<false, true>)
                          : (a.per_token ? &small_estimator_kernel<true, false> : &small_estimator_kernel<false, false>);
    kernel<<<1, threads, 0, st>>>(a, log_eta, log((double)a.coef.loss_scale));
}

void launch_row_coefficients(const float* g, const double* g64, const int32_t* seqc, const int32_t* row_index,
                             const int32_t* counts, const float* logp_cur, const float* logp_behav, int per_token,
                             float eta, int clip_tokens, int64_t row0, int64_t rows_max, float* rowg, hipStream_t st) {
    const double log_eta = (eta > 0.f && std::isfinite(eta)) ? log((double)eta) : (double)INFINITY;
    if (rows_max > 0)
        row_coefficients_kernel<<<blocks_for(rows_max, 256), 256, 0, st>>>(g, g64, seqc, row_index, counts, logp_cur,
                                                                           logp_behav, per_token, log_eta,
                                                                           clip_tokens, row0, rowg);
}

void launch_rescale_rows(void* dhidden, const uint8_t* mask, int64_t N, int64_t T, int64_t d, const int32_t* gen_chunk,
                         const double* lam_chunk, const double* lam_state, hipStream_t st) {
    rescale_rows_kernel<<<(unsigned)(N * T), 128, 0, st>>>((bf16_t*)dhidden, mask, T, d, gen_chunk, lam_chunk, lam_state);
}

// master -= lr * grad; optionally also the updated weights in the contraction dtype
__global__ void sgd_step_kernel(float* __restrict__ master, const float* __restrict__ grad, int64_t n, float lr,
                                void* __restrict__ w_out, int dtype) {
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n) return;
    const float w = master[i] - lr * grad[i];
    master[i] = w;
    if (w_out) {
        if (dtype == RAPID_DTYPE_BF16) {
            const __bf16 r = (__bf16)w;
            ((bf16_t*)w_out)[i] = __builtin_bit_cast(bf16_t, r);
        } else {
            ((float*)w_out)[i] = w;
        }
    }
}
void launch_sgd_step(float* master, const float* grad, int64_t n, float lr, void* w_out, int dtype, hipStream_t st) {
    if (n > 0) sgd_step_kernel<<<blocks_for(n, 256), 256, 0, st>>>(master, grad, n, lr, w_out, dtype);
}

// AdamW: bias corrections 1 - beta^step are formed on the host in double
__global__ void adamw_step_kernel(float* __restrict__ master, const float* __restrict__ grad, float* __restrict__ m,
                                  float* __restrict__ v, int64_t n, float lr, float beta1, float beta2, float eps,
                                  float weight_decay, float inv_bc1, float inv_bc2, void* __restrict__ w_out, int dtype) {
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n) return;
    const float g = grad[i];
    const float mi = beta1 * m[i] + (1.f - beta1) * g;
    const float vi = beta2 * v[i] + (1.f - beta2) * g * g;
    m[i] = mi;
    v[i] = vi;
    const float w0 = master[i];
    const float w = w0 - lr * ((mi * inv_bc1) / (sqrtf(vi * inv_bc2) + eps) + weight_decay * w0);
    master[i] = w;
    if (w_out) {
        if (dtype == RAPID_DTYPE_BF16) {
            const __bf16 r = (__bf16)w;
            ((bf16_t*)w_out)[i] = __builtin_bit_cast(bf16_t, r);
        } else {
            ((float*)w_out)[i] = w;
        }
    }
}
void launch_adamw_step(float* master, const float* grad, float* m, float* v, int64_t n, float lr, float beta1, float beta2,
                       float eps, float weight_decay, int64_t step, void* w_out, int dtype, hipStream_t st) {
    const float inv_bc1 = (float)(1.0 / (1.0 - pow((double)beta1, (double)step)));
    const float inv_bc2 = (float)(1.0 / (1.0 - pow((double)beta2, (double)step)));
    if (n > 0)
        adamw_step_kernel<<<blocks_for(n, 256), 256, 0, st>>>(master, grad, m, v, n, lr, beta1, beta2, eps, weight_decay,
                                                              inv_bc1, inv_bc2, w_out, dtype);
}

void launch_f32_to_bf16(const float* src, bf16_t* dst, int64_t n, hipStream_t st) {
    if (n > 0) f32_to_bf16_kernel<<<blocks_for(n, 256), 256, 0, st>>>(src, dst, n);
}

}  // namespace rapid
