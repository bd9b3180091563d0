// Operand packing for the MFMA kernels (hidden rows: rows.hip): zero-padded, tile-aligned bf16 copies of W, unless the batch is
// small enough to read it in place, with its contraction index contiguous, so that the hot loops need no bounds
// checks.  These kernels are pure HBM copies (read once, write once).
#include "rapid_internal.h"

namespace rapid {

namespace {

// 16 bytes from where only the element's 2-byte alignment is given, as rows of an odd vocabulary have it
struct Unaligned16 { uint32_t w[4]; } __attribute__((packed, aligned(2)));
__device__ __forceinline__ uint4 load16(const bf16_t* p) {
    const Unaligned16 u = *(const Unaligned16*)p;
    return make_uint4(u.w[0], u.w[1], u.w[2], u.w[3]);
}

// elements c .. c + 8 of a row of C elements, zeros past its end
__device__ __forceinline__ uint4 load_chunk(const bf16_t* row, int64_t c, int64_t C) {
    if (c + 8 <= C) return load16(row + c);
    bf16_t e[8];
    for (int i = 0; i < 8; ++i) e[i] = c + i < C ? row[c + i] : (bf16_t)0;
    return *(const uint4*)e;
}

// one block per destination row; 16-byte chunks (dst rows are 16-byte aligned, Cpad a multiple of 8)
__global__ void copy_pad_bf16_kernel(const bf16_t* __restrict__ src, int64_t ld_src, bf16_t* __restrict__ dst,
                                     int64_t ld_dst, int64_t R, int64_t C, int64_t Cpad) {
    const int64_t r = blockIdx.x;
    const bool live = r < R;
    const bf16_t* srow = src + (live ? r : 0) * ld_src;
    for (int64_t c = threadIdx.x; c < Cpad / 8; c += blockDim.x)
        *(uint4*)(dst + r * ld_dst + c * 8) = live ? load_chunk(srow, c * 8, C) : make_uint4(0u, 0u, 0u, 0u);
}

// 64x64 tile through LDS: dst[c][r] = src[r][c], row-major or (RB > 0) in tile blocks as block_rows_bf16_kernel
// lays them out (a 64 x 64 tile is then 8 KiB of consecutive memory).  16-byte global accesses on both sides, unaligned ones where the
// rows are (element by element d = 232, V = 135922 took 43 us, 30 now).
// LDS rows are 66 elements (33 banks) apart: the transposed read of 8 rows x 8 columns per 64 lanes
// is conflict free.
__global__ __launch_bounds__(256) void transpose_pad_bf16_kernel(const bf16_t* __restrict__ src, int64_t ld_src,
                                                                 bf16_t* __restrict__ dst, int64_t ld_dst, int64_t R,
                                                                 int64_t C, int64_t Rpad, int64_t Cpad, int RB) {
    __shared__ bf16_t tile[64][66];
    const int64_t rb = (int64_t)blockIdx.x * 64, cb = (int64_t)blockIdx.y * 64;
    auto at = [&](int64_t c, int64_t r) {
        return RB ? dst + (c / RB * (Rpad / 64) + r / 64) * (RB * 64) + c % RB * 64 + r % 64 : dst + c * ld_dst + r;
    };
    for (int t = threadIdx.x; t < 512; t += 256) {          // 64 rows x 8 chunks of 8 columns
        const int rr = t >> 3, q = t & 7;
        const int64_t r = rb + rr, c = cb + q * 8;
        const uint4 v = r < R ? load_chunk(src + r * ld_src, c, C) : make_uint4(0u, 0u, 0u, 0u);
        uint32_t* p = (uint32_t*)&tile[rr][q * 8];          // 4-byte aligned: row stride 132 bytes
        p[0] = v.x; p[1] = v.y; p[2] = v.z; p[3] = v.w;
    }
    __syncthreads();
    for (int t = threadIdx.x; t < 512; t += 256) {          // 64 destination rows x 8 chunks of 8 (Rpad is a multiple of 64)
        const int cc = t >> 3, q = t & 7;
        const int64_t c = cb + cc, r = rb + q * 8;
        if (c >= Cpad) continue;
        bf16_t e[8];
#pragma unroll
        for (int i = 0; i < 8; ++i) e[i] = tile[q * 8 + i][cc];
        *(uint4*)at(c, r) = *(const uint4*)e;
    }
}

// Both packed copies of W at once, a tile of 64 x 64 per block: Wvd [Vpad, ldk] (columns below dpad), the operand of the logits
// kernels, and the tile blocks of RB rows x 64 that dHidden reads ([dpadR, Vpad], see block_rows_bf16_kernel).  W is read
// once, and a small head's two launches (4 us each) are one: d = 1536, V = 151936 335 -> 250 us.
template <bool VD>     // W is stored [V, d], else [d, V]
__global__ __launch_bounds__(256) void pack_both_bf16_kernel(const bf16_t* __restrict__ W, int64_t d, int64_t V, bf16_t* __restrict__ Wvd,
                                                             int64_t ldk, int64_t dpad, bf16_t* __restrict__ blocks, int64_t dpadR, int RB,
                                                             int64_t KT) {
    __shared__ bf16_t tile[64][66];       // rows 33 banks apart: the transposed read is conflict free
    const int64_t v0 = (int64_t)blockIdx.x * 64, d0 = (int64_t)blockIdx.y * 64;
    auto at_block = [&](int64_t dd, int64_t v) { return blocks + (dd / RB * KT + v / 64) * (RB * 64) + dd % RB * 64 + v % 64; };
    auto at_row = [&](int64_t v, int64_t dd) { return Wvd + v * ldk + dd; };
    for (int t = threadIdx.x; t < 512; t += 256) {
        const int rr = t >> 3, q = t & 7;
        const int64_t v = VD ? v0 + rr : v0 + q * 8, dd = VD ? d0 + q * 8 : d0 + rr;
        const uint4 x = VD ? (v < V ? load_chunk(W + v * d, dd, d) : make_uint4(0u, 0u, 0u, 0u))
                           : (dd < d ? load_chunk(W + dd * V, v, V) : make_uint4(0u, 0u, 0u, 0u));
        if (VD) { if (dd < dpad) *(uint4*)at_row(v, dd) = x; }
        else { if (dd < dpadR) *(uint4*)at_block(dd, v) = x; }
        uint32_t* p = (uint32_t*)&tile[rr][q * 8];
        p[0] = x.x; p[1] = x.y; p[2] = x.z; p[3] = x.w;
    }
    __syncthreads();
    for (int t = threadIdx.x; t < 512; t += 256) {
        const int cc = t >> 3, q = t & 7;
        bf16_t e[8];
#pragma unroll
        for (int i = 0; i < 8; ++i) e[i] = tile[q * 8 + i][cc];
        const int64_t v = VD ? v0 + q * 8 : v0 + cc, dd = VD ? d0 + cc : d0 + q * 8;
        if (VD) { if (dd < dpadR) *(uint4*)at_block(dd, v) = *(const uint4*)e; }
        else { if (dd < dpad) *(uint4*)at_row(v, dd) = *(const uint4*)e; }
    }
}

}  // namespace

void launch_copy_pad_bf16(const bf16_t* src, int64_t ld_src, bf16_t* dst, int64_t ld_dst, int64_t R, int64_t C, int64_t Rpad,
                          int64_t Cpad, hipStream_t st) {
    if (Rpad <= 0) return;
    copy_pad_bf16_kernel<<<(unsigned)Rpad, 256, 0, st>>>(src, ld_src, dst, ld_dst, R, C, Cpad);
}

// [R, C] (row stride ld) -> tile-blocked [Rpad, Cpad] (multiples of RB and 64, zero padded): block (rt, kt) holds rows
// rt*RB .. +RB, columns kt*64 .. +64 as RB contiguous 128-byte rows; blocks ordered (rt, kt).
__global__ __launch_bounds__(256) void block_rows_bf16_kernel(const bf16_t* __restrict__ src, int64_t ld, bf16_t* __restrict__ dst,
                                                              int64_t R, int64_t C, int RB, int64_t KT) {
    const int64_t rt = blockIdx.y, kt = blockIdx.x;
    bf16_t* d = dst + (rt * KT + kt) * RB * 64;
#pragma unroll 8
    for (int t = threadIdx.x; t < RB * 8; t += 256) {
        const int64_t r = rt * RB + (t >> 3), c = kt * 64 + (t & 7) * 8;
        const uint4 v = r < R ? load_chunk(src + r * ld, c, C) : make_uint4(0u, 0u, 0u, 0u);
        *(uint4*)(d + (int64_t)t * 8) = v;
    }
}
void launch_block_rows_bf16(const bf16_t* src, int64_t ld, bf16_t* dst, int64_t R, int64_t C, int64_t Rpad, int64_t Cpad, int RB,
                            hipStream_t st) {
    dim3 grid((unsigned)(Cpad / 64), (unsigned)(Rpad / RB));
    block_rows_bf16_kernel<<<grid, 256, 0, st>>>(src, ld, dst, R, C, RB, Cpad / 64);
}

void launch_transpose_blocks_bf16(const bf16_t* src, int64_t ld_src, bf16_t* dst, int64_t R, int64_t C, int64_t Rpad, int64_t Cpad,
                                  int RB, hipStream_t st) {
    dim3 grid((unsigned)((Rpad + 63) / 64), (unsigned)((Cpad + 63) / 64));
    transpose_pad_bf16_kernel<<<grid, 256, 0, st>>>(src, ld_src, dst, 0, R, C, Rpad, Cpad, RB);
}

void launch_transpose_pad_bf16(const bf16_t* src, int64_t ld_src, bf16_t* dst, int64_t ld_dst, int64_t R,
                               int64_t C, int64_t Rpad, int64_t Cpad, hipStream_t st) {
    if (Rpad <= 0 || Cpad <= 0) return;
    dim3 grid((unsigned)((Rpad + 63) / 64), (unsigned)((Cpad + 63) / 64));
    transpose_pad_bf16_kernel<<<grid, 256, 0, st>>>(src, ld_src, dst, ld_dst, R, C, Rpad, Cpad, 0);
}

void launch_pack_both_bf16(const bf16_t* W, bool vd, int64_t d, int64_t V, bf16_t* Wvd, int64_t ldk, int64_t dpad, bf16_t* blocks,
                           int64_t dpadR, int RB, int64_t Vpad, hipStream_t st) {
    const dim3 grid((unsigned)(Vpad / 64), (unsigned)(((dpad > dpadR ? dpad : dpadR) + 63) / 64));
    (vd ? &pack_both_bf16_kernel<true> : &pack_both_bf16_kernel<false>)<<<grid, 256, 0, st>>>(W, d, V, Wvd, ldk, dpad, blocks, dpadR, RB, Vpad / 64);
}

}  // namespace rapid
