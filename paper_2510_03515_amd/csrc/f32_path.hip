// fp32 path: the same pipeline for float inputs, built from one strided contraction on the fp64 matrix
// instruction plus two row-wise kernels over a materialised row chunk of logits.  It is the accuracy path
// (tolerance 1e-5).
#include <type_traits>

#include "rapid_internal.h"

namespace rapid {

namespace {

typedef double f64x4 __attribute__((ext_vector_type(4)));

// One operand of a contraction: element (o, k) at p[omap(o) * so + kmap(k) * sk].
struct F64Operand {
    const float* p;
    int64_t so, sk;
    const int32_t *omap, *kmap;   // optional index maps, already offset
};

// C[i][j] (+)= alpha sum_k A(i, k) B(j, k) on the fp64 matrix instruction (v_mfma_f64_16x16x4_f64): the operands are
// fp32 in memory and are widened on the way into LDS, the accumulators are fp64.  Bound by the fp64 matrix rate: the
// instruction on its own, from registers, sustains 47 TFLOP/s; 4096 rows x V = 4096 x d = 256 run at 45 (logits), 48
// (dHidden) and 40 (dW).  (A fused multiply-add per lane on a 16 x 16 tile, which this replaces, ran at 12: an LDS read
// and a conversion per operand and product.)
// A workgroup of 4 waves owns TI x TJ of C.  SPLIT: every wave works on the whole tile but on a quarter of the
// contraction index (groups of 4 dealt round robin) and the four sums are added in wave order at the end; that is
// for shapes with too few tiles to fill the chip.  Otherwise the waves share the tile 2 x 2 and each element is
// summed in the order of k whatever the tile size, so the logits of a row do not depend on which size ran.
// KA / KB: the operand is contiguous along k (else along its outer index); MA / MB: its k goes through the map.
// These are template arguments because a branch around a load keeps the loads of a step from being in flight together.
// Global loads run two steps ahead of the MFMAs (two register sets; a step's MFMAs take less than a trip to memory).
// LDS rows are KS + 2 doubles apart (an odd multiple of 16 bytes): a fragment read is free of bank conflicts.
template <int TI, int TJ, int KS, bool SPLIT>
constexpr int f64_lds_bytes() { return (2 * (TI + TJ) * (KS + 2) + (SPLIT ? 4 * TI * TJ : 0)) * 8; }
template <int TI, int TJ, int KS, bool SPLIT, bool KA, bool KB, bool MA, bool MB>
__device__ __forceinline__ void f64_work(const F64Operand& A, const F64Operand& B, const F32Gemm& g, unsigned tile_i, unsigned tile_j, double* lds) {
    constexpr int WI = SPLIT ? TI / 16 : TI / 32, WJ = SPLIT ? TJ / 16 : TJ / 32, LD = KS + 2;
    constexpr int QA = TI * KS / 256, QB = TJ * KS / 256;   // elements per thread and step
    static_assert(KS <= 64 && 256 % KS == 0 && 256 % TI == 0 && 256 % TJ == 0, "thread layout of the loads");
    double *const As[2] = {lds, lds + TI * LD}, *const Bs[2] = {lds + 2 * TI * LD, lds + (2 * TI + TJ) * LD};
    int64_t I = g.I, Kd = g.Kd;
    if (g.counts) {
        const int64_t M = g.counts[CNT_M], left = M > g.i0 ? M - g.i0 : 0;
        if (g.skip_last && left <= g.I) return;   // what this launch would form is still in C
        if (g.limit_k) Kd = left < Kd ? left : Kd;
        else I = left < I ? left : I;
    }
    const int64_t ib = (int64_t)tile_i * TI, jb = (int64_t)tile_j * TJ;
    if (ib >= I) return;
    if (g.limit_k && Kd == 0 && g.beta) return;
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;

    // Thread's share of a step: consecutive threads along whichever index is contiguous in memory.  The outer index
    // of a thread's element q stays the same over the steps, so its address is formed (and its map read) once and
    // then advanced; rows past the end repeat the last one (their sums are not stored).
    auto outer = [&](bool kc, int T, int q) { const int e = tid + 256 * q; return kc ? e / KS : e % T; };
    auto inner = [&](bool kc, int T, int q) { const int e = tid + 256 * q; return kc ? e % KS : e / T; };
    auto first = [&](const F64Operand& X, bool kc, bool map, int T, int q, int64_t base, int64_t limit) {
        int64_t o = base + outer(kc, T, q);
        o = o < limit ? o : limit - 1;
        return X.p + (X.omap ? (int64_t)X.omap[o] : o) * X.so + (map ? 0 : inner(kc, T, q) * X.sk);
    };
    const float* pa[QA];
    const float* pb[QB];
#pragma unroll
    for (int q = 0; q < QA; ++q) pa[q] = first(A, KA, MA, TI, q, ib, I);
#pragma unroll
    for (int q = 0; q < QB; ++q) pb[q] = first(B, KB, MB, TJ, q, jb, g.J);
    const int64_t step_a = KS * A.sk, step_b = KS * B.sk;
    float ra[2][QA], rb[2][QB];
    // mapped operand: the map's entries are read one step before the elements they lead to
    int32_t next[MA ? QA : MB ? QB : 1];
    auto fetch_map = [&](int64_t k0) {
#pragma unroll
        for (int q = 0; q < (MA ? QA : MB ? QB : 0); ++q) {
            const int64_t k = k0 + (MA ? inner(KA, TI, q) : inner(KB, TJ, q));
            next[q] = (MA ? A.kmap : B.kmap)[k < Kd ? k : Kd - 1];
        }
    };
    auto fetch_whole = [&](auto set, int64_t k0) {
#pragma unroll
        for (int q = 0; q < QA; ++q) {
            if constexpr (MA) ra[set][q] = pa[q][(int64_t)next[q] * A.sk];
            else { ra[set][q] = *pa[q]; pa[q] += step_a; }
        }
#pragma unroll
        for (int q = 0; q < QB; ++q) {
            if constexpr (MB) rb[set][q] = pb[q][(int64_t)next[q] * B.sk];
            else { rb[set][q] = *pb[q]; pb[q] += step_b; }
        }
        fetch_map(k0 + KS);
    };
    auto fetch = [&](auto set, int64_t k0) {   // also the last step, which may be short, and steps that do not exist
        if (k0 + KS <= Kd) { fetch_whole(set, k0); return; }
        if (k0 >= Kd) return;
#pragma unroll
        for (int q = 0; q < QA; ++q) {
            const int64_t k = k0 + inner(KA, TI, q);
            ra[set][q] = k < Kd ? pa[q][MA ? (int64_t)next[q] * A.sk : 0] : 0.f;
        }
#pragma unroll
        for (int q = 0; q < QB; ++q) {
            const int64_t k = k0 + inner(KB, TJ, q);
            rb[set][q] = k < Kd ? pb[q][MB ? (int64_t)next[q] * B.sk : 0] : 0.f;
        }
    };
    auto stage = [&](auto set) {
#pragma unroll
        for (int q = 0; q < QA; ++q) As[set][outer(KA, TI, q) * LD + inner(KA, TI, q)] = (double)ra[set][q];
#pragma unroll
        for (int q = 0; q < QB; ++q) Bs[set][outer(KB, TJ, q) * LD + inner(KB, TJ, q)] = (double)rb[set][q];
    };

    f64x4 acc[WI][WJ];
#pragma unroll
    for (int x = 0; x < WI; ++x)
#pragma unroll
        for (int y = 0; y < WJ; ++y) acc[x][y] = f64x4{0.0, 0.0, 0.0, 0.0};
    const int wi = SPLIT ? 0 : (wave & 1) * (WI * 16), wj = SPLIT ? 0 : (wave >> 1) * (WJ * 16);
    const int fo = lane & 15, fk = lane >> 4;   // fragment: row (or column) lane % 16, contraction index lane / 16
    auto multiply = [&](auto set) {
#pragma unroll
        for (int kk = 0; kk < KS / 4; kk += SPLIT ? 4 : 1) {
            const int k = (kk + (SPLIT ? wave : 0)) * 4 + fk;
            double a[WI], b[WJ];
#pragma unroll
            for (int x = 0; x < WI; ++x) a[x] = As[set][(wi + x * 16 + fo) * LD + k];
#pragma unroll
            for (int y = 0; y < WJ; ++y) b[y] = Bs[set][(wj + y * 16 + fo) * LD + k];
#pragma unroll
            for (int x = 0; x < WI; ++x)
#pragma unroll
                for (int y = 0; y < WJ; ++y) acc[x][y] = __builtin_amdgcn_mfma_f64_16x16x4f64(a[x], b[y], acc[x][y], 0, 0, 0);
        }
    };
    const std::integral_constant<int, 0> s0;
    const std::integral_constant<int, 1> s1;
    if (Kd > 0) fetch_map(0);
    fetch(s0, 0);
    fetch(s1, KS);
    if (Kd > 0) stage(s0);
    __syncthreads();
    // step k0 is in LDS, step k0 + KS in registers
    int64_t k0 = 0;
    for (; k0 + 4 * KS <= Kd; k0 += 2 * KS) {
        fetch_whole(s0, k0 + 2 * KS);
        multiply(s0);
        stage(s1);
        __syncthreads();
        fetch_whole(s1, k0 + 3 * KS);
        multiply(s1);
        stage(s0);
        __syncthreads();
    }
    for (; k0 < Kd; k0 += 2 * KS) {
        fetch(s0, k0 + 2 * KS);
        multiply(s0);
        if (k0 + KS >= Kd) break;
        stage(s1);
        __syncthreads();
        fetch(s1, k0 + 3 * KS);
        multiply(s1);
        if (k0 + 2 * KS >= Kd) break;
        stage(s0);
        __syncthreads();
    }

    // element (i, j) of a block sits in lane (i % 4) * 16 + j, register i / 4
    auto write = [&](int64_t i, int64_t j, double sum) {
        if (i >= I || j >= g.J) return;
        const int64_t r = g.c_rows ? (int64_t)g.c_rows[g.i0 + i] : i;
        float* p = g.C + r * g.sc_i + j * g.sc_j;
        const double v = sum * (double)g.alpha;
        *p = (float)(g.beta ? (double)*p + v : v);
    };
    if constexpr (SPLIT) {
        double* const sum = lds + 2 * (TI + TJ) * LD;      // [4][TI * TJ]
#pragma unroll
        for (int x = 0; x < WI; ++x)
#pragma unroll
            for (int y = 0; y < WJ; ++y)
#pragma unroll
                for (int v = 0; v < 4; ++v) sum[wave * (TI * TJ) + (x * 16 + v * 4 + fk) * TJ + y * 16 + fo] = acc[x][y][v];
        __syncthreads();
        for (int e = tid; e < TI * TJ; e += 256)
            write(ib + e / TJ, jb + e % TJ, (sum[e] + sum[TI * TJ + e]) + (sum[2 * TI * TJ + e] + sum[3 * TI * TJ + e]));
    } else {
#pragma unroll
        for (int x = 0; x < WI; ++x)
#pragma unroll
            for (int y = 0; y < WJ; ++y)
#pragma unroll
                for (int v = 0; v < 4; ++v) write(ib + wi + x * 16 + v * 4 + fk, jb + wj + y * 16 + fo, acc[x][y][v]);
    }
}

template <int TI, int TJ, int KS, bool SPLIT, bool KA, bool KB, bool MA, bool MB>
__global__ __launch_bounds__(256) void f64_mfma_kernel(F64Operand A, F64Operand B, F32Gemm g) {
    __shared__ double lds[f64_lds_bytes<TI, TJ, KS, SPLIT>() / 8];
    f64_work<TI, TJ, KS, SPLIT, KA, KB, MA, MB>(A, B, g, blockIdx.y, blockIdx.x, lds);
}

// dHidden and dW of a small shape side by side: two chains of a few trips to memory each that do not depend on each
// other (640 rows x V = 1000 x d = 64: 10.9 and 8.8 us one after the other, 12.6 to 14.0 together).  The first h_blocks blocks are dHidden's.
template <bool KB, bool MA>
__global__ __launch_bounds__(256) void f64_pair_kernel(F64Operand hA, F64Operand hB, F32Gemm h, unsigned h_cols, unsigned h_blocks,
                                                       F64Operand wA, F64Operand wB, F32Gemm w, unsigned w_cols) {
    __shared__ double lds[f64_lds_bytes<16, 16, 64, true>() / 8];
    const unsigned b = blockIdx.x;
    if (b < h_blocks) f64_work<16, 16, 64, true, true, KB, false, false>(hA, hB, h, b / h_cols, b % h_cols, lds);
    else f64_work<16, 16, 64, true, false, false, MA, !MA>(wA, wB, w, (b - h_blocks) / w_cols, (b - h_blocks) % w_cols, lds);
}

__device__ inline double block_reduce(double v, double* sm, bool is_max) {
    for (int o = 32; o > 0; o >>= 1) {
        const double u = __shfl_xor(v, o, 64);
        v = is_max ? fmax(v, u) : v + u;
    }
    const int w = threadIdx.x >> 6, nw = blockDim.x >> 6;
    __syncthreads();
    if ((threadIdx.x & 63) == 0) sm[w] = v;
    __syncthreads();
    double r = sm[0];
    for (int q = 1; q < nw; ++q) r = is_max ? fmax(r, sm[q]) : r + sm[q];
    return r;
}

// one block per chunk row: lse over the V logits, log-prob of the sampled token.  PER > 0: V <= 256 PER, the row is loaded once
// and stays in registers (in two passes over it 640 rows x V = 1000 took 6.2 us, now 4.8; 4096 rows x 4096 34.6 -> 28.0).  Past 16 per
// thread the gain goes on (4096 rows x 6144 49.5 us in two passes, 37.0 with 24 per thread; x 8192 62 and 46 with 32).
template <int PER>
__global__ __launch_bounds__(256) void f32_row_lse_kernel(const float* __restrict__ z, int64_t V, int64_t m0,
                                   const int32_t* __restrict__ tokc, const int32_t* __restrict__ row_index,
                                   const int32_t* __restrict__ counts, float* __restrict__ lse_c,
                                   float* __restrict__ logp_out, float* __restrict__ lse_out) {
    __shared__ double sm[16];
    const int64_t jl = blockIdx.x, j = m0 + jl;
    if (j >= counts[CNT_M]) return;
    const float* row = z + jl * V;
    const int32_t pos = row_index[j], tok = tokc[j];
    double mx = -INFINITY, sum = 0.0;
    if constexpr (PER > 0) {
        float v[PER];
#pragma unroll
        for (int i = 0; i < PER; ++i) {
            const int at = threadIdx.x + 256 * i;
            v[i] = row[at < V ? at : V - 1];
        }
#pragma unroll
        for (int i = 0; i < PER; ++i)
            if (threadIdx.x + 256 * i < V) mx = fmax(mx, (double)v[i]);
        mx = block_reduce(mx, sm, true);
#pragma unroll
        for (int i = 0; i < PER; ++i)
            if (threadIdx.x + 256 * i < V) sum += exp((double)v[i] - mx);
    } else {
        for (int64_t v = threadIdx.x; v < V; v += blockDim.x) mx = fmax(mx, (double)row[v]);
        mx = block_reduce(mx, sm, true);
        for (int64_t v = threadIdx.x; v < V; v += blockDim.x) sum += exp((double)row[v] - mx);
    }
    sum = block_reduce(sum, sm, false);
    if (threadIdx.x == 0) {
        const double lse = mx + log(sum);
        lse_c[j] = (float)lse;
        logp_out[pos] = (float)((double)row[tok] - lse);
        if (lse_out) lse_out[pos] = (float)lse;
    }
}

__global__ void f32_dz_kernel(float* __restrict__ z, int64_t V, int64_t m0, const int32_t* __restrict__ tokc,
                              const float* __restrict__ lse_c, const float* __restrict__ rowg, float inv_temp,
                              const int32_t* __restrict__ counts) {
    const int64_t jl = blockIdx.x, j = m0 + jl;
    if (j >= counts[CNT_M]) return;
    float* row = z + jl * V;
    const double lse = (double)lse_c[j];
    const double gj = (double)rowg[j] * (double)inv_temp;
    const int tok = tokc[j];
    for (int64_t v = threadIdx.x; v < V; v += blockDim.x) {
        const double p = exp((double)row[v] - lse);
        row[v] = (float)(gj * ((v == tok ? 1.0 : 0.0) - p));
    }
}

// Tile: 64 x 64 where that gives every CU two workgroups (a SIMD needs two waves at least to keep the instruction
// going: 35 TFLOP/s with one, 46 with two), else 32 x 32, else (dHidden and dW of small shapes, fewer tiles than CUs)
// 16 x 16 with the contraction shared out over the waves: 10 us for 640 rows x V = 1000 x d = 64, 31 us before.
int64_t tiles_of(const F32Gemm& g, int T) { return ((g.I + T - 1) / T) * ((g.J + T - 1) / T); }
bool tile_64(const F32Gemm& g) { return tiles_of(g, 64) >= 512; }
bool tile_32(const F32Gemm& g) { return tiles_of(g, 32) >= 256 || !g.may_split; }
template <bool KA, bool KB, bool MA, bool MB>
void launch_tiles(const F64Operand& A, const F64Operand& B, const F32Gemm& g, hipStream_t st) {
    auto grid = [&](int T) { return dim3((unsigned)((g.J + T - 1) / T), (unsigned)((g.I + T - 1) / T)); };
    if (tile_64(g)) f64_mfma_kernel<64, 64, 16, false, KA, KB, MA, MB><<<grid(64), 256, 0, st>>>(A, B, g);
    else if (tile_32(g)) f64_mfma_kernel<32, 32, 32, false, KA, KB, MA, MB><<<grid(32), 256, 0, st>>>(A, B, g);
    else f64_mfma_kernel<16, 16, 64, true, KA, KB, MA, MB><<<grid(16), 256, 0, st>>>(A, B, g);
}
struct F64Call { F64Operand A, B; F32Gemm g; };
F64Call f64_call(const F32Gemm& in) {
    F64Call c{{in.A, in.sa_i, in.sa_k, in.a_imap ? in.a_imap + in.i0 : nullptr, in.a_kmap ? in.a_kmap + in.i0 : nullptr},
              {in.B, in.sb_j, in.sb_k, nullptr, nullptr}, in};
    if (in.sc_i == 1 && in.limit_k) {   // C is contiguous along i: form its transpose, so that a store covers whole lines
        const F64Operand t = c.A; c.A = c.B; c.B = t;
        c.g.I = in.J; c.g.J = in.I;
        c.g.sc_i = in.sc_j; c.g.sc_j = 1;
    }
    return c;
}

}  // namespace

void launch_f32_gemm(const F32Gemm& in, hipStream_t st) {
    if (in.I <= 0 || in.J <= 0) return;
    const F64Call c = f64_call(in);
    if (c.A.kmap) launch_tiles<false, false, true, false>(c.A, c.B, c.g, st);        // dW: both operands contiguous along their outer index
    else if (c.B.kmap) launch_tiles<false, false, false, true>(c.A, c.B, c.g, st);
    else if (c.B.sk == 1) launch_tiles<true, true, false, false>(c.A, c.B, c.g, st);
    else launch_tiles<true, false, false, false>(c.A, c.B, c.g, st);
}

void launch_f32_gemm_pair(const F32Gemm& dh, const F32Gemm& dw, hipStream_t st) {
    const F64Call h = f64_call(dh), w = f64_call(dw);
    auto small = [](const F32Gemm& g) { return g.I > 0 && g.J > 0 && !tile_64(g) && !tile_32(g); };
    if (!small(h.g) || !small(w.g)) {
        launch_f32_gemm(dh, st);
        launch_f32_gemm(dw, st);
        return;
    }
    auto cols = [](const F32Gemm& g) { return (unsigned)((g.J + 15) / 16); };
    const unsigned nh = (unsigned)tiles_of(h.g, 16), nw = (unsigned)tiles_of(w.g, 16);
    auto* kernel = h.B.sk == 1 ? (w.A.kmap ? &f64_pair_kernel<true, true> : &f64_pair_kernel<true, false>)
                               : (w.A.kmap ? &f64_pair_kernel<false, true> : &f64_pair_kernel<false, false>);
    kernel<<<nh + nw, 256, 0, st>>>(h.A, h.B, h.g, cols(h.g), nh, w.A, w.B, w.g, cols(w.g));
}

void launch_f32_row_lse(const float* z, int64_t V, int64_t rows, int64_t m0, const int32_t* tokc,
                        const int32_t* row_index, const int32_t* counts, float* lse_c, float* logp_out,
                        float* lse_out, hipStream_t st) {
    if (rows <= 0) return;
    auto* kernel = V <= 1024 ? &f32_row_lse_kernel<4> : V <= 2048 ? &f32_row_lse_kernel<8> : V <= 4096 ? &f32_row_lse_kernel<16> : &f32_row_lse_kernel<0>;
    kernel<<<(unsigned)rows, 256, 0, st>>>(z, V, m0, tokc, row_index, counts, lse_c, logp_out, lse_out);
}

void launch_f32_dz(float* z, int64_t V, int64_t rows, int64_t m0, const int32_t* tokc, const float* lse_c,
                   const float* rowg, float inv_temp, const int32_t* counts, hipStream_t st) {
    if (rows > 0) f32_dz_kernel<<<(unsigned)rows, 256, 0, st>>>(z, V, m0, tokc, lse_c, rowg, inv_temp, counts);
}

}  // namespace rapid
