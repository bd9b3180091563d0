// Final RMSNorm folded into the operand pack of the fused call (not part of the paper's method: its
// path starts at the hidden state; the Qwen2.5 models it trains end in this norm, and the pack pass
// reads every hidden row anyway).  Forward (rows.hip): the packed, zero-padded bf16 operand holds
// h = x * weight / sqrt(mean(x^2) + eps) instead of a copy of x.  Backward: the dHidden kernel has
// written dL/dh (bf16) into the caller's dhidden buffer; two passes over the valid rows turn it into
// dL/dweight (fixed-order partial sums) and, in place, dL/dx.
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

// dweight partials: block (rb, cb) sums dh[row][k] x[row][k] inv_rms[row] over the valid compact rows
// row0 + rb*RB .. +RB for the 8 columns of each of its threads; part[rb][k] (a block without rows writes nothing:
// `part` is zeroed beforehand)
constexpr int RB = 512;
__global__ __launch_bounds__(256) void rmsnorm_dweight_partial_kernel(const bf16_t* __restrict__ x, const bf16_t* __restrict__ dh,
                                                                      int64_t d, const int32_t* __restrict__ row_index,
                                                                      const int32_t* __restrict__ counts,
                                                                      const float* __restrict__ inv_rms,
                                                                      float* __restrict__ part, int64_t row0) {
    const int64_t c = (int64_t)blockIdx.y * blockDim.x + threadIdx.x;   // 8-column chunk
    const int64_t r0 = row0 + (int64_t)blockIdx.x * RB;                // row blocks along x: no 65535 limit
    const int M = counts[CNT_M];
    if (c * 8 >= d || r0 >= M) return;   // the reduction reads the blocks that hold tokens only
    float acc[8] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
    const int64_t r1 = r0 + RB < M ? r0 + RB : M;
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

// dweight[k] = sum over all row blocks, in block order (fp64 accumulate; blocks without rows hold zeros)
__global__ void rmsnorm_dweight_reduce_kernel(const float* __restrict__ part, int64_t d, int64_t nblk,
                                              float* __restrict__ dweight) {
    const int64_t k = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (k >= d) return;
    double acc = 0.0;
    for (int64_t b = 0; b < nblk; ++b) acc += (double)part[b * d + k];
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

int64_t rmsnorm_dweight_blocks(int64_t rows_max) { return (rows_max + RB - 1) / RB; }

void launch_rmsnorm_backward(const bf16_t* x, bf16_t* dh, int64_t d, const bf16_t* weight, const int32_t* row_index,
                             const int32_t* counts, const float* inv_rms, int64_t row0, int64_t rows_max, float* part,
                             hipStream_t st) {
    if (rows_max <= 0) return;
    if (part) {
        dim3 grid((unsigned)rmsnorm_dweight_blocks(rows_max), (unsigned)((d / 8 + 255) / 256));
        rmsnorm_dweight_partial_kernel<<<grid, 256, 0, st>>>(x, dh, d, row_index, counts, inv_rms, part, row0);
    }
    rmsnorm_dx_kernel<<<(unsigned)rows_max, 256, 0, st>>>(x, dh, d, weight, row_index, counts, inv_rms, row0);
}

void launch_rmsnorm_dweight_reduce(const float* part, int64_t d, int64_t nblk, float* dweight, hipStream_t st) {
    rmsnorm_dweight_reduce_kernel<<<(unsigned)((d + 255) / 256), 256, 0, st>>>(part, d, nblk, dweight);
}

}  // namespace rapid
