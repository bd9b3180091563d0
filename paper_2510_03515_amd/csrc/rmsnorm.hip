// Final RMSNorm folded into the operand pack of the fused call (not part of the paper's method: its
// path starts at the hidden state; the Qwen2.5 models it trains end in this norm, and the pack pass
// reads every hidden row anyway).  Forward (rows.hip): the packed, zero-padded bf16 operand holds
// h = x * weight / sqrt(mean(x^2) + eps) instead of a copy of x.  Backward: the dHidden kernel has
// written dL/dh (bf16) into the caller's dhidden buffer; here it becomes dL/dweight (fixed-order partial sums) and, in place,
// dL/dx.
#include "rapid_internal.h"
#include "row_math.h"

namespace rapid {

namespace {

__device__ inline float wave_sum_f(float v) {
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o, 64);
    return v;
}

// sum over the 256 threads of a block, same value in every thread, fixed order
__device__ inline float block_sum_f(float v, float* sm) {
    v = wave_sum_f(v);
    __syncthreads();
    if ((threadIdx.x & 63) == 0) sm[threadIdx.x / 64] = v;
    __syncthreads();
    return (sm[0] + sm[1]) + (sm[2] + sm[3]);
}

// dweight partials: part[b][k] = sum of dh[row][k] x[row][k] inv_rms[row] over the valid compact rows of row block b (a block
// without rows writes nothing).
// A row is read twice over (for the sum over its columns, and for what follows from it) and its partial sums want a
// register per column, so up to 2048 columns a wave does all of it for a few rows at a time, holding a row in registers: x
// and dh are read once.  A thread of a block of 512 rows going down its columns took 0.4 us per row: 334 us for 18 000 rows at
// d = 2048 and with the second pass over the rows and the sum over the blocks 391, now 61; a step of 880 tokens at d = 1592,
// V = 6667 took 426 us, now 193.
template <int C>     // 16-byte chunks per lane
__global__ __launch_bounds__(256) void rmsnorm_backward_kernel(const bf16_t* __restrict__ x, bf16_t* __restrict__ dh, int64_t d,
                                                               const bf16_t* __restrict__ weight, const int32_t* __restrict__ row_index,
                                                               const int32_t* __restrict__ counts, const float* __restrict__ inv_rms,
                                                               float* __restrict__ part, int64_t row0, int per_wave) {
    extern __shared__ float s_part[];     // [4][d]
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int64_t block0 = row0 + (int64_t)blockIdx.x * 4 * per_wave;
    const int M = counts[CNT_M];
    if (block0 >= M) return;
    const int chunks = (int)(d / 8);
    float w[C][8], acc[C][8];
#pragma unroll
    for (int i = 0; i < C; ++i) {
        unpack8(*(const uint4*)(weight + min(lane + i * 64, chunks - 1) * 8), w[i]);
#pragma unroll
        for (int e = 0; e < 8; ++e) acc[i][e] = 0.f;
    }
    const int64_t first = block0 + wave * per_wave, end = first + per_wave < M ? first + per_wave : M;
    uint4 xv[C], gv[C], next_x[C], next_g[C];
    int64_t pos = 0, next_pos = 0;
    float inv = 0.f, next_inv = 0.f;
    auto request = [&](int64_t r) {       // the next row, one row ahead
        next_pos = row_index[r];
        next_inv = inv_rms[r];
#pragma unroll
        for (int i = 0; i < C; ++i) {
            const int64_t at = next_pos * d + min(lane + i * 64, chunks - 1) * 8;
            next_x[i] = *(const uint4*)(x + at);
            next_g[i] = *(const uint4*)(dh + at);
        }
    };
    if (first < end) request(first);
    for (int64_t r = first; r < end; ++r) {
        pos = next_pos;
        inv = next_inv;
#pragma unroll
        for (int i = 0; i < C; ++i) { xv[i] = next_x[i]; gv[i] = next_g[i]; }
        if (r + 1 < end) request(r + 1);
        bf16_t* gr = dh + pos * d;
        float t = 0.f;
#pragma unroll
        for (int i = 0; i < C; ++i) {
            if (lane + i * 64 >= chunks) break;
            float xf[8], gf[8];
            unpack8(xv[i], xf);
            unpack8(gv[i], gf);
#pragma unroll
            for (int e = 0; e < 8; ++e) {
                t = fmaf(gf[e] * w[i][e], xf[e], t);
                acc[i][e] = fmaf(gf[e] * inv, xf[e], acc[i][e]);
            }
        }
        t = wave_sum_f(t);
        const float k3 = inv * inv * inv * t / (float)d;
#pragma unroll
        for (int i = 0; i < C; ++i) {
            if (lane + i * 64 >= chunks) break;
            float xf[8], gf[8], o[8];
            unpack8(xv[i], xf);
            unpack8(gv[i], gf);
#pragma unroll
            for (int e = 0; e < 8; ++e) o[e] = inv * w[i][e] * gf[e] - xf[e] * k3;
            *(uint4*)(gr + (lane + i * 64) * 8) = pack8(o);
        }
    }
    if (!part) return;
#pragma unroll
    for (int i = 0; i < C; ++i) {
        if (lane + i * 64 >= chunks) break;
        float* s = s_part + wave * d + (lane + i * 64) * 8;
        *(float4*)s = make_float4(acc[i][0], acc[i][1], acc[i][2], acc[i][3]);
        *(float4*)(s + 4) = make_float4(acc[i][4], acc[i][5], acc[i][6], acc[i][7]);
    }
    __syncthreads();
    for (int k = threadIdx.x; k < d; k += 256)
        part[blockIdx.x * d + k] = (s_part[k] + s_part[d + k]) + (s_part[2 * d + k] + s_part[3 * d + k]);
}

// the same partials for wider rows: block (b, cb) goes down `rows` rows, 8 columns per thread
__global__ __launch_bounds__(256) void rmsnorm_dweight_partial_kernel(const bf16_t* __restrict__ x, const bf16_t* __restrict__ dh,
                                                                      int64_t d, const int32_t* __restrict__ row_index,
                                                                      const int32_t* __restrict__ counts,
                                                                      const float* __restrict__ inv_rms,
                                                                      float* __restrict__ part, int64_t row0, int rows) {
    const int64_t c = (int64_t)blockIdx.y * blockDim.x + threadIdx.x;   // 8-column chunk
    const int64_t r0 = row0 + (int64_t)blockIdx.x * rows;              // row blocks along x: no 65535 limit
    const int M = counts[CNT_M];
    if (c * 8 >= d || r0 >= M) return;
    float acc[8] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
    const int64_t r1 = r0 + rows < M ? r0 + rows : M;
#pragma unroll 4
    for (int64_t r = r0; r < r1; ++r) {
        const int64_t pos = row_index[r];
        float xv[8], gv[8];
        unpack8(*(const uint4*)(x + pos * d + c * 8), xv);
        unpack8(*(const uint4*)(dh + pos * d + c * 8), gv);
        const float inv = inv_rms[r];
#pragma unroll
        for (int e = 0; e < 8; ++e) acc[e] = fmaf(gv[e] * inv, xv[e], acc[e]);
    }
    float* o = part + (int64_t)blockIdx.x * d + c * 8;
#pragma unroll
    for (int e = 0; e < 8; ++e) o[e] = acc[e];
}

// dweight[k] = sum over the row blocks that hold rows, of every region: 16 waves share a column's blocks, then their sums are
// added in wave order (fp64)
__global__ __launch_bounds__(1024) void rmsnorm_dweight_reduce_kernel(const float* __restrict__ part, int64_t d, int rows,
                                                                      const int32_t* __restrict__ counts, int stride, int regions,
                                                                      int64_t region_rows, int64_t blocks_per_region,
                                                                      float* __restrict__ dweight) {
    __shared__ double sm[16][64];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int64_t k = (int64_t)blockIdx.x * 64 + lane;
    double acc = 0.0;
    if (k < d) {
        for (int g = 0; g < regions; ++g) {
            const int64_t held = counts[g * stride + CNT_M] - g * region_rows, n = (held + rows - 1) / rows;
            const float* p = part + g * blocks_per_region * d + k;
#pragma unroll 8
            for (int64_t b = wave; b < n; b += 16) acc += (double)p[b * d];
        }
    }
    sm[wave][lane] = acc;
    __syncthreads();
    if (wave != 0 || k >= d) return;
    for (int w = 1; w < 16; ++w) acc += sm[w][lane];
    dweight[k] = (float)acc;
}

// in place, one block per valid compact row: dh -> dx = r (w dh) - x r^3 sum_k(dh_k w_k x_k) / d
__global__ __launch_bounds__(256) void rmsnorm_dx_kernel(const bf16_t* __restrict__ x, bf16_t* __restrict__ dh, int64_t d,
                                                         const bf16_t* __restrict__ weight,
                                                         const int32_t* __restrict__ row_index,
                                                         const int32_t* __restrict__ counts,
                                                         const float* __restrict__ inv_rms, int64_t r0) {
    __shared__ float sm[4];
    const int64_t r = r0 + blockIdx.x;
    if (r >= counts[CNT_M]) return;
    const int64_t pos = row_index[r];
    const bf16_t* xr = x + pos * d;
    bf16_t* gr = dh + pos * d;
    const int64_t chunks = d / 8;
    float t = 0.f;
    for (int64_t c = threadIdx.x; c < chunks; c += blockDim.x) {
        float xv[8], gv[8], wv[8];
        unpack8(*(const uint4*)(xr + c * 8), xv);
        unpack8(*(const uint4*)(gr + c * 8), gv);
        unpack8(*(const uint4*)(weight + c * 8), wv);
#pragma unroll
        for (int e = 0; e < 8; ++e) t = fmaf(gv[e] * wv[e], xv[e], t);
    }
    t = block_sum_f(t, sm);   // also orders every thread's reads of the row before the writes below
    const float inv = inv_rms[r];
    const float k3 = inv * inv * inv * t / (float)d;
    for (int64_t c = threadIdx.x; c < chunks; c += blockDim.x) {
        float xv[8], gv[8], wv[8], o[8];
        unpack8(*(const uint4*)(xr + c * 8), xv);
        unpack8(*(const uint4*)(gr + c * 8), gv);
        unpack8(*(const uint4*)(weight + c * 8), wv);
#pragma unroll
        for (int e = 0; e < 8; ++e) o[e] = inv * wv[e] * gv[e] - xv[e] * k3;
        *(uint4*)(gr + c * 8) = pack8(o);
    }
}

}  // namespace

void launch_rmsnorm_backward(const bf16_t* x, bf16_t* dh, int64_t d, const bf16_t* weight, const int32_t* row_index,
                             const int32_t* counts, int stride, int regions, int64_t region_rows, const float* inv_rms, float* part,
                             size_t part_bytes, float* part_512, float* dweight, hipStream_t st) {
    const int C = (int)((d / 8 + 63) / 64);
    // One pass up to 4 chunks per lane, two past them.  The gain does not end there: with 7 chunks per lane 880 rows at d = 3584 take
    // 15 us instead of 20, 40 000 181 instead of 296.
    const bool narrow = C <= 4;
    // Rows per block: few for a small batch, whose rows then go side by side; more if the partial sums would not fit.  Both kernels
    // at d = 1536 with 8, 16, 32 and 64 rows: 880 rows 11, 13, 18 and 27 us, 3000 14, 15, 19 and 29, 8192 23, 20, 21 and 29, 16 384 39,
    // 33, 31 and 33, 40 000 88, 82, 82 and 94.
    int rows = narrow ? ((int64_t)regions * region_rows <= 8192 ? 8 : 32) : 32;
    auto blocks = [&]() { return (region_rows + rows - 1) / rows; };
    while (rows < 512 && (size_t)(blocks() * regions * d) * 4 > part_bytes) rows *= 2;
    if ((size_t)(blocks() * regions * d) * 4 > part_bytes) part = part_512;      // thousands of small regions, each with a block of its own
    for (int g = 0; g < regions; ++g) {
        const int32_t* cnt = counts + (int64_t)g * stride;
        const int64_t row0 = g * region_rows;
        float* p = dweight ? part + g * blocks() * d : nullptr;
        if (narrow) {
            auto* kernel = C == 1 ? &rmsnorm_backward_kernel<1> : C == 2 ? &rmsnorm_backward_kernel<2> : C == 3 ? &rmsnorm_backward_kernel<3> : &rmsnorm_backward_kernel<4>;
            kernel<<<(unsigned)blocks(), 256, (size_t)d * 16, st>>>(x, dh, d, weight, row_index, cnt, inv_rms, p, row0, rows / 4);
            continue;
        }
        if (p) rmsnorm_dweight_partial_kernel<<<dim3((unsigned)blocks(), (unsigned)((d / 8 + 255) / 256)), 256, 0, st>>>(x, dh, d, row_index, cnt, inv_rms, p, row0, rows);
        rmsnorm_dx_kernel<<<(unsigned)region_rows, 256, 0, st>>>(x, dh, d, weight, row_index, cnt, inv_rms, row0);
    }
    if (dweight)
        rmsnorm_dweight_reduce_kernel<<<(unsigned)((d + 63) / 64), 1024, 0, st>>>(part, d, rows, counts, stride, regions, region_rows, blocks(), dweight);
}

}  // namespace rapid
