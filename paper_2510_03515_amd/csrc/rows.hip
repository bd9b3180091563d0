// The pass over the hidden rows in front of the logits: compacts the valid positions of the batch, packs their hidden rows
// (normalised, if asked for) into the zero-padded operand of the contractions, forms the logit of each row's sampled
// token, and clears what belongs to the other positions.
//
// One launch, a wave per position (or few): a small batch's call is a matter of launches, and this replaces five of them
// (index of the rows, copy, sampled tokens' logits, gradient rows without gradient, zeros of the per-token outputs) that
// took 3 to 5 us each for next to nothing (64 x 48 positions at d = 256: 14 us in all, 7.8 now); a large batch reads its
// hidden rows once instead of twice.  A wave finds the compact row of its first position by counting the mask from the start
// of the generation, 16 bytes per lane and load wherever the mask starts (T / 1024 loads and one for the edges), or, without a plan,
// of the batch; where that does not pay (launch_compact_rows) the rows are indexed by row_index_kernel first and the waves here
// take compact rows.
#include "rapid_internal.h"
#include "row_math.h"

namespace rapid {

namespace {

enum { PACK_NONE = 0, PACK_COPY, PACK_RMS };
constexpr int U = 4;     // 16-byte chunks per lane whose loads are in flight together

__device__ inline void zero_row(void* p, int64_t words) {
    const int lane = threadIdx.x & 63;
    if (words % 4 == 0) {
        uint4* q = (uint4*)p;
        for (int64_t i = lane; i < words / 4; i += 64) q[i] = make_uint4(0u, 0u, 0u, 0u);
    } else {
        uint32_t* q = (uint32_t*)p;
        for (int64_t i = lane; i < words; i += 64) q[i] = 0u;
    }
}

// Hc[j] = hidden row `pos` (normalised with RMS: formed in fp64 and rounded to bf16 once, because which of two neighbouring bf16
// values an element becomes is a decision, and taken from an fp32 product it would fall the other way than the exact value's
// for about one element in 40 000, each moving its row's log-prob by ~1e-4), zeros up to Cpad; and
// zy[j] = inv_temp <Hc[j], W[token]>: fp32, chunk c of 8 elements by lane c % 64, then a fixed tree over the lanes.  W has a
// token's weights in a row, or (GATHER) in a column: 64 bytes are then read for each, which a small batch can afford;
// the sum is formed in the same order.  refz (optional): the reference of a storing forward, zy minus the position's
// ref_logp (zy alone without ref_logp or where that value is not finite).
template <int PACK, bool GATHER>
__device__ __forceinline__ void pack_row(const RowsArgs& a, int64_t j, int64_t pos, int token) {
    const int lane = threadIdx.x & 63;
    const int64_t live = a.d / 8, chunks = a.Cpad / 8;
    const uint4* src = (const uint4*)(a.hidden + pos * a.d);
    uint4* dst = (uint4*)(a.Hc + j * a.ldk);
    const bf16_t* w = a.W + (GATHER ? (int64_t)token : (int64_t)token * a.ldw);
    double inv = 1.0;
    if constexpr (PACK == PACK_RMS) {
        double ss = 0.0;
        for (int64_t base = 0; base < live; base += 64 * U) {
            uint4 v[U];
#pragma unroll
            for (int u = 0; u < U; ++u) {
                if (base + u * 64 >= live) break;
                const int64_t c = base + u * 64 + lane;
                v[u] = src[c < live ? c : live - 1];
            }
#pragma unroll
            for (int u = 0; u < U; ++u) {
                if (base + u * 64 + lane >= live) break;
                float x[8];
                unpack8(v[u], x);
#pragma unroll
                for (int e = 0; e < 8; ++e) ss = fma((double)x[e], (double)x[e], ss);
            }
        }
#pragma unroll
        for (int o = 32; o > 0; o >>= 1) ss += __shfl_xor(ss, o, 64);
        inv = 1.0 / sqrt(ss / (double)a.d + (double)a.rms_eps);
        if (lane == 0) a.inv_rms[j] = (float)inv;
    }
    float acc = 0.f;
    for (int64_t base = 0; base < chunks; base += 64 * U) {
        // Lanes past the end repeat the row's last chunk and drop it: a branch around a load would keep it from being in
        // flight with the others.  (Sets of 64 chunks that lie past the end are left out, by a branch that all lanes take.)
        uint4 h[U], g[U];
        uint32_t wv[U][GATHER ? 8 : 4];
#pragma unroll
        for (int u = 0; u < U; ++u) {
            if (base + u * 64 >= live) break;
            const int64_t c = base + u * 64 + lane < live ? base + u * 64 + lane : live - 1;
            h[u] = src[c];
            if constexpr (PACK == PACK_RMS) g[u] = *(const uint4*)(a.rms_weight + c * 8);
            if constexpr (GATHER) {
                const bf16_t* e = w + c * 8 * a.ldw;
#pragma unroll
                for (int i = 0; i < 8; ++i) wv[u][i] = e[i * a.ldw];
            } else {
                *(uint4*)wv[u] = ((const uint4*)w)[c];
            }
        }
#pragma unroll
        for (int u = 0; u < U; ++u) {
            if (base + u * 64 >= chunks) break;
            const int64_t c = base + u * 64 + lane;
            if (c >= live) {
                if (c < chunks) dst[c] = make_uint4(0u, 0u, 0u, 0u);
                continue;
            }
            float hf[8];
            unpack8(h[u], hf);
            if constexpr (PACK == PACK_RMS) {
                float gf[8];
                unpack8(g[u], gf);
#pragma unroll
                for (int e = 0; e < 8; ++e) hf[e] = round_for_bf16((double)hf[e] * inv * (double)gf[e]);
                h[u] = pack8(hf);
                unpack8(h[u], hf);
            }
            dst[c] = h[u];
#pragma unroll
            for (int e = 0; e < 8; ++e) {
                const float wf = GATHER ? __builtin_bit_cast(float, wv[u][GATHER ? e : 0] << 16)
                                        : __builtin_bit_cast(float, e % 2 ? wv[u][e / 2] & 0xffff0000u : wv[u][e / 2] << 16);
                acc = fmaf(hf[e], wf, acc);
            }
        }
    }
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) acc += __shfl_xor(acc, o, 64);
    if (lane == 0) {
        const float z = acc * a.inv_temp;
        a.zy[j] = z;
        if (a.refz) {
            float lb = a.ref_logp ? a.ref_logp[pos] : 0.f;
            if (!isfinite(lb)) lb = 0.f;
            a.refz[j] = z - lb;
        }
    }
}

// rows that fill a region's last row tile up: token 0, zeros
__device__ __forceinline__ void fill_row(const RowsArgs& a, int64_t j, bool pack) {
    if ((threadIdx.x & 63) == 0 && a.tokc) {
        a.tokc[j] = 0;
        a.seqc[j] = 0;
    }
    if (pack) zero_row(a.Hc + j * a.ldk, a.Cpad / 2);
}

// the wave's valid positions among the first n of `mask`: 16-byte words, and one lane each for the bytes in front of the first
// and behind the last of them
__device__ __forceinline__ int count_before(const uint8_t* mask, int n) {
    const int lane = threadIdx.x & 63;
    const int align = (int)(-(uintptr_t)mask & 15), head = align < n ? align : n, words = (n - head) >> 4;
    auto bytes = [](uint32_t w) { return __popc((((w & 0x7f7f7f7fu) + 0x7f7f7f7fu) | w) & 0x80808080u); };   // top bit of every byte that is not 0
    int cnt = 0;
#pragma unroll 4
    for (int c = lane; c < words; c += 64) {
        const uint4 w = ((const uint4*)(mask + head))[c];
        cnt += bytes(w.x) + bytes(w.y) + bytes(w.z) + bytes(w.w);
    }
    const int edge = lane < 16 ? lane : head + words * 16 + lane - 16;
    if (lane < 16 ? lane < head : lane < 32 && edge < n) cnt += mask[edge] != 0;
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) cnt += __shfl_xor(cnt, o, 64);
    return cnt;
}

// Compact rows: generation n's valid positions, in order, take the rows from first_row[n] on (a negative first row: the
// generation was left out).  They come in regions of `region` rows, and a generation never writes past the end of the region its
// first row lies in.  Token ids out of range are flagged and replaced by 0.
// A wave takes `per_wave` (at most 64) consecutive positions of one generation; the blocks behind those of the positions fill
// the regions' last row tiles up (16 blocks per region).
template <int PACK, bool GATHER>
__global__ __launch_bounds__(256) void rows_by_position_kernel(RowsArgs a, int per_wave, int blocks_per_generation) {
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, waves = blockDim.x >> 6;
    const int64_t N = a.N, T = a.T;
    const int64_t b = blockIdx.x, main_blocks = N * blocks_per_generation;
    if (b >= main_blocks) {
        const int64_t e = (b - main_blocks) / 16, part = (b - main_blocks) % 16;
        int64_t M, end;
        if (a.first_row) {
            M = a.limits[e * a.stride + CNT_M];
            end = a.limits[e * a.stride + CNT_MR];
        } else {
            M = count_before(a.mask, (int)(N * T));
            end = (M + ROW_TILE - 1) / ROW_TILE * ROW_TILE;
            if (part == 0 && threadIdx.x == 0) {
                a.counts_out[CNT_M] = (int32_t)M;
                a.counts_out[CNT_MR] = (int32_t)end;
            }
        }
        for (int64_t j = M + part * waves + wave; j < end; j += 16 * waves) fill_row(a, j, PACK != PACK_NONE);
        return;
    }
    const int64_t n = b / blocks_per_generation;
    const int64_t t0 = ((b - n * blocks_per_generation) * waves + wave) * per_wave;
    if (t0 >= T) return;
    const uint8_t* row = a.mask + n * T;
    const int64_t first = a.first_row ? a.first_row[n] : 0, i_mine = n * T + t0 + lane;
    const bool here = lane < per_wave && t0 + lane < T, valid = here && row[t0 + lane] != 0;
    int tok = valid && a.tokc ? a.tokens[i_mine] : 0;
    const bool idle = a.idle && a.idle[n];
    // valid positions in front of t0, of the generation or (no plan) of the batch
    const int before = a.first_row ? count_before(row, (int)t0) : count_before(a.mask, (int)(n * T + t0));
    const unsigned long long votes = __ballot(valid);
    const int64_t limit = first < 0 ? 0 : (first / a.region + 1) * a.region;
    const int64_t j_mine = first + before + __popcll(votes & ((1ull << lane) - 1ull));
    const bool placed = valid && first >= 0 && j_mine < limit;
    if (placed) {
        if (a.row_index) a.row_index[j_mine] = (int32_t)i_mine;
        if (a.tokc) {
            if (tok < 0 || tok >= a.V) {
                tok = 0;
                if (a.dev_status) atomicOr(a.dev_status, RAPID_STATUS_BAD_TOKEN);
            }
            a.tokc[j_mine] = tok;
            a.seqc[j_mine] = (int32_t)n;
        }
    } else if (here) {
        if (a.zero_a) a.zero_a[i_mine] = 0.f;
        if (a.zero_b) a.zero_b[i_mine] = 0.f;
    }
    const unsigned long long rows = __ballot(placed);
    for (int i = 0; i < per_wave && t0 + i < T; ++i) {
        if constexpr (PACK != PACK_NONE) {
            if ((rows >> i) & 1ull) pack_row<PACK, GATHER>(a, __shfl(j_mine, i, 64), n * T + t0 + i, __shfl(tok, i, 64));
        }
        if (a.dhidden && (idle || !((votes >> i) & 1ull))) zero_row(a.dhidden + (n * T + t0 + i) * a.words_per_row, a.words_per_row);
    }
}

// a wave per compact row, of all regions; row_index and tokc are filled in
template <int PACK, bool GATHER>
__global__ __launch_bounds__(256) void rows_by_row_kernel(RowsArgs a) {
    const int64_t j = (int64_t)blockIdx.x * 4 + (threadIdx.x >> 6);
    const int32_t* lim = a.limits + j / a.region * a.stride;
    if (j >= lim[CNT_MR]) return;
    if (j < lim[CNT_M]) pack_row<PACK, GATHER>(a, j, a.row_index[j], a.tokc[j]);
    else fill_row(a, j, true);
}

template <int PACK, bool GATHER>
void launch_t(const RowsArgs& a, bool by_position, int64_t rows, hipStream_t st) {
    if (by_position) {
        // small batches: a wave per position, all trips side by side; without rows to pack there is next to nothing per position
        const int per_wave = PACK == PACK_NONE ? 16 : a.N * a.T <= 32768 ? 1 : 4;
        // blocks of no more waves than a generation has work for: a launch holds less than 2^32 threads (a block of four waves for each
        // generation of a few positions would be refused from 16.8 M generations on)
        const int64_t wanted = (a.T + per_wave - 1) / per_wave;
        const int waves = wanted < 4 ? (int)wanted : 4;
        const int64_t per_generation = (wanted + waves - 1) / waves, fill = a.tokc ? (int64_t)a.entries * 16 : 0;
        rows_by_position_kernel<PACK, GATHER><<<(unsigned)(a.N * per_generation + fill), 64 * waves, 0, st>>>(a, per_wave, (int)per_generation);
    } else if constexpr (PACK != PACK_NONE) {
        rows_by_row_kernel<PACK, GATHER><<<(unsigned)((rows + 3) / 4), 256, 0, st>>>(a);
    }
}

}  // namespace

void launch_rows(const RowsArgs& a, bool by_position, int64_t rows, hipStream_t st) {
    if (!a.Hc) launch_t<PACK_NONE, false>(a, by_position, rows, st);
    else if (a.rms_weight) a.gather ? launch_t<PACK_RMS, true>(a, by_position, rows, st) : launch_t<PACK_RMS, false>(a, by_position, rows, st);
    else a.gather ? launch_t<PACK_COPY, true>(a, by_position, rows, st) : launch_t<PACK_COPY, false>(a, by_position, rows, st);
}

}  // namespace rapid
