// Operand packing for the MFMA kernels (hidden rows: rows.hip): zero-padded, tile-aligned bf16 copies of W, unless the batch is
// small enough to read it in place, with its contraction index contiguous, so that the hot loops need no bounds
// checks.  These kernels are pure HBM copies (read once, write once).
#include "rapid_internal.h"

namespace rapid {

namespace {

// one block per destination row; 16-byte chunks (ld_dst, Cpad multiples of 8; src rows 16 B aligned
// when C % 8 == 0, otherwise the element path is taken)
__global__ void copy_pad_bf16_kernel(const bf16_t* __restrict__ src, int64_t ld_src, bf16_t* __restrict__ dst,
                                     int64_t ld_dst, int64_t R, int64_t C, int64_t Cpad, int vec_ok) {
    const int64_t r = blockIdx.x;
    bf16_t* drow = dst + r * ld_dst;
    const bool live = r < R;
    const bf16_t* srow = src + (live ? r : 0) * ld_src;
    if (vec_ok) {
        const int64_t chunks = Cpad / 8, live_chunks = C / 8;
        for (int64_t c = threadIdx.x; c < chunks; c += blockDim.x) {
            uint4 v = make_uint4(0u, 0u, 0u, 0u);
            if (live && c < live_chunks) v = *(const uint4*)(srow + c * 8);
            *(uint4*)(drow + c * 8) = v;
        }
    } else {
        for (int64_t c = threadIdx.x; c < Cpad; c += blockDim.x)
            drow[c] = (live && c < C) ? srow[c] : (bf16_t)0;
    }
}

// 64x64 tile through LDS: dst[c][r] = src[r][c], row-major or (RB > 0) in tile blocks as block_rows_bf16_kernel
// lays them out (a 64 x 64 tile is then 8 KiB of consecutive memory).  16-byte global accesses on both sides when the
// shapes allow (vec: ld_src, ld_dst multiples of 8, 16-byte aligned bases), elements otherwise.
// LDS rows are 66 elements (33 banks) apart: the transposed read of 8 rows x 8 columns per 64 lanes
// is conflict free.
__global__ __launch_bounds__(256) void transpose_pad_bf16_kernel(const bf16_t* __restrict__ src, int64_t ld_src,
                                                                 bf16_t* __restrict__ dst, int64_t ld_dst, int64_t R,
                                                                 int64_t C, int64_t Rpad, int64_t Cpad, int vec, int RB) {
    __shared__ bf16_t tile[64][66];
    const int64_t rb = (int64_t)blockIdx.x * 64, cb = (int64_t)blockIdx.y * 64;
    auto at = [&](int64_t c, int64_t r) {
        return RB ? dst + (c / RB * (Rpad / 64) + r / 64) * (RB * 64) + c % RB * 64 + r % 64 : dst + c * ld_dst + r;
    };
    if (vec) {
        for (int t = threadIdx.x; t < 512; t += 256) {          // 64 rows x 8 chunks of 8 columns
            const int rr = t >> 3, q = t & 7;
            const int64_t r = rb + rr, c = cb + q * 8;
            uint4 v = make_uint4(0u, 0u, 0u, 0u);
            if (r < R && c + 8 <= C) {
                v = *(const uint4*)(src + r * ld_src + c);
            } else if (r < R && c < C) {
                bf16_t e[8];
                for (int i = 0; i < 8; ++i) e[i] = c + i < C ? src[r * ld_src + c + i] : (bf16_t)0;
                v = *(const uint4*)e;
            }
            uint32_t* p = (uint32_t*)&tile[rr][q * 8];          // 4-byte aligned: row stride 132 bytes
            p[0] = v.x; p[1] = v.y; p[2] = v.z; p[3] = v.w;
        }
        __syncthreads();
        for (int t = threadIdx.x; t < 512; t += 256) {          // 64 destination rows x 8 chunks of 8
            const int cc = t >> 3, q = t & 7;
            const int64_t c = cb + cc, r = rb + q * 8;
            if (c >= Cpad || r >= Rpad) continue;
            bf16_t e[8];
#pragma unroll
            for (int i = 0; i < 8; ++i) e[i] = tile[q * 8 + i][cc];
            if (r + 8 <= Rpad) {
                *(uint4*)at(c, r) = *(const uint4*)e;
            } else {
                for (int i = 0; i < 8 && r + i < Rpad; ++i) *at(c, r + i) = e[i];
            }
        }
        return;
    }
    const int tx = threadIdx.x & 63, ty = threadIdx.x >> 6;   // 256 threads: 64 x 4
    for (int rr = ty; rr < 64; rr += 4) {
        const int64_t r = rb + rr, c = cb + tx;
        bf16_t v = 0;
        if (r < R && c < C) v = src[r * ld_src + c];
        tile[rr][tx] = v;
    }
    __syncthreads();
    for (int cc = ty; cc < 64; cc += 4) {
        const int64_t c = cb + cc, r = rb + tx;
        if (c < Cpad && r < Rpad) *at(c, r) = tile[tx][cc];
    }
}

}  // namespace

void launch_copy_pad_bf16(const bf16_t* src, int64_t ld_src, bf16_t* dst, int64_t ld_dst, int64_t R, int64_t C, int64_t Rpad,
                          int64_t Cpad, hipStream_t st) {
    if (Rpad <= 0) return;
    const int vec_ok = (C % 8 == 0) && (ld_src % 8 == 0) && (((uintptr_t)src) % 16 == 0);
    copy_pad_bf16_kernel<<<(unsigned)Rpad, 256, 0, st>>>(src, ld_src, dst, ld_dst, R, C, Cpad, vec_ok);
}

// [R, C] (row stride ld) -> tile-blocked [Rpad, Cpad] (multiples of RB and 64, zero padded): block (rt, kt) holds rows
// rt*RB .. +RB, columns kt*64 .. +64 as RB contiguous 128-byte rows; blocks ordered (rt, kt).
__global__ __launch_bounds__(256) void block_rows_bf16_kernel(const bf16_t* __restrict__ src, int64_t ld, bf16_t* __restrict__ dst,
                                                              int64_t R, int64_t C, int RB, int64_t KT, int vec) {
    const int64_t rt = blockIdx.y, kt = blockIdx.x;
    bf16_t* d = dst + (rt * KT + kt) * RB * 64;
#pragma unroll 8
    for (int t = threadIdx.x; t < RB * 8; t += 256) {
        const int64_t r = rt * RB + (t >> 3), c = kt * 64 + (t & 7) * 8;
        uint4 v = make_uint4(0u, 0u, 0u, 0u);
        if (r < R && c < C) {
            const bf16_t* s = src + r * ld + c;
            if (vec && c + 8 <= C) {
                v = *(const uint4*)s;
            } else {
                bf16_t e[8];
                for (int i = 0; i < 8; ++i) e[i] = c + i < C ? s[i] : (bf16_t)0;
                v = *(const uint4*)e;
            }
        }
        *(uint4*)(d + (int64_t)t * 8) = v;
    }
}
void launch_block_rows_bf16(const bf16_t* src, int64_t ld, bf16_t* dst, int64_t R, int64_t C, int64_t Rpad, int64_t Cpad, int RB,
                            hipStream_t st) {
    dim3 grid((unsigned)(Cpad / 64), (unsigned)(Rpad / RB));
    const int vec = (ld % 8 == 0) && (((uintptr_t)src) % 16 == 0);
    block_rows_bf16_kernel<<<grid, 256, 0, st>>>(src, ld, dst, R, C, RB, Cpad / 64, vec);
}

void launch_transpose_blocks_bf16(const bf16_t* src, int64_t ld_src, bf16_t* dst, int64_t R, int64_t C, int64_t Rpad, int64_t Cpad,
                                  int RB, hipStream_t st) {
    dim3 grid((unsigned)((Rpad + 63) / 64), (unsigned)((Cpad + 63) / 64));
    const int vec = (ld_src % 8 == 0) && (((uintptr_t)src) % 16 == 0);
    transpose_pad_bf16_kernel<<<grid, 256, 0, st>>>(src, ld_src, dst, 0, R, C, Rpad, Cpad, vec, RB);
}

void launch_transpose_pad_bf16(const bf16_t* src, int64_t ld_src, bf16_t* dst, int64_t ld_dst, int64_t R,
                               int64_t C, int64_t Rpad, int64_t Cpad, hipStream_t st) {
    if (Rpad <= 0 || Cpad <= 0) return;
    dim3 grid((unsigned)((Rpad + 63) / 64), (unsigned)((Cpad + 63) / 64));
    const int vec = (ld_src % 8 == 0) && (ld_dst % 8 == 0) && (((uintptr_t)src) % 16 == 0) && (((uintptr_t)dst) % 16 == 0);
    transpose_pad_bf16_kernel<<<grid, 256, 0, st>>>(src, ld_src, dst, ld_dst, R, C, Rpad, Cpad, vec, 0);
}

}  // namespace rapid
