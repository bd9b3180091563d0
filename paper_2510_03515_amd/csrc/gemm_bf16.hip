// bf16 MFMA contractions of the hot path for gfx950 (CDNA4): one tiled main loop (two operand
// layouts) and four epilogues.
//   fwd_lse : logits tile  -> per-slot (max, sum exp) of the streaming log-softmax + gathered logit
//   dz      : logits tile  -> dz = g (onehot - softmax) / temperature, written as bf16
//   dh      : dH = dz . W^T          (contraction over the vocabulary)
//   dw      : dW (+)= H^T . dz       (contraction over the tokens of a row chunk)
//
// Tiling.  C[i][j] = sum_k A(i,k) B(j,k); operands are zero padded to whole tiles, so the loop has
// no bounds checks, but for W read in place (a small batch), whose addresses are clamped to the matrix (see
// Loader).  A workgroup of NWI x NWJ 64-lane waves owns a 256 x 256 tile (the largest whose
// fp32 accumulators a CU's registers hold, which minimises L2 -> LDS bytes per flop), each wave
// WI x WJ blocks of 32 x 32 computed with v_mfma_f32_32x32x16_bf16 (a lane feeds 8 consecutive k of
// one row).  The default is 2 x 4 waves of 128 x 64, two waves per SIMD.  K advances 64 elements
// per step through two LDS stages of 64 KiB (one barrier per step); operand tiles arrive by
// global_load_lds_dwordx4 (memory -> LDS without passing through registers; consecutive lanes fill
// consecutive 16-byte slots, so the LDS swizzle is applied to the global address).  The kernels
// are persistent: one workgroup per CU walks tile ids that are mapped to tiles so that the
// workgroups resident on an XCD (ids equal mod 8) own neighbouring tiles and share operand panels
// in that XCD's L2.
//
// LDS layouts (both conflict-free for a 256-byte LDS cycle, checked with SQ_LDS_BANK_CONFLICT):
//  * row-major operands ([row][k], k contiguous): a tile row of a step is 128 bytes = 8 chunks of
//    16 bytes; chunk c of row r sits at position c ^ ((r >> 1) & 7); fragments are read with
//    ds_read_b128.
//  * k-major operands ([k][column]; both of dW, whose contraction index is the token row, and W in place where
//    its other index is the contiguous one): see the comment above KMajor below; fragments are read with the LDS transpose read.
//
// Accumulator layout of a 32 x 32 block (lane l, register v): j = l % 32,
// i = 8 (v / 4) + 4 (l / 32) + v % 4: a lane owns runs of 4 consecutive i for one j, so every
// epilogue keeps j = the token row (per-lane scalars: lse, coefficient, token id, output row) and
// stores 4 consecutive i with one 8- or 16-byte access.
#include <atomic>
#include <type_traits>
#include <utility>

#include "rapid_internal.h"

namespace rapid {

namespace {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef __bf16 bf16x4 __attribute__((ext_vector_type(4)));
typedef float f32x16 __attribute__((ext_vector_type(16)));
typedef unsigned u32x4 __attribute__((ext_vector_type(4)));
typedef short s16x4 __attribute__((ext_vector_type(4)));
typedef short s16x8 __attribute__((ext_vector_type(8)));

constexpr float LOG2E = 1.4426950408889634f;

// Geometry of a workgroup: NWI x NWJ waves, each owning WI x WJ blocks of 32 x 32.
// 2 x 4 waves of 128 x 64 is the default (two waves per SIMD, which lets the hardware overlap one
// wave's LDS, barrier and memory-issue waits with the other's MFMAs at the price of 1.5x the LDS
// fragment reads); 2 x 2 waves of 128 x 128 (one wave per SIMD, 256 accumulator registers per lane)
// and 2 x 8 waves of 128 x 32 are selectable.
template <int NWI_, int NWJ_, int WI_, int WJ_>
struct Geo {
    static constexpr int NWI = NWI_, NWJ = NWJ_, WI = WI_, WJ = WJ_;
    static constexpr int NW = NWI * NWJ, NT = 64 * NW;
    static constexpr int BI = NWI * WI * 32, BJ = NWJ * WJ * 32;
    // A k-major operand of 192 (or 224) columns is loaded as 256 (a request then covers whole rows; the last columns are
    // not used), so an LDS stage has room for a power of two.
    static constexpr int LI = BI > 128 ? 256 : BI, LJ = BJ > 128 ? 256 : BJ;
    static constexpr int STAGE_BYTES = (LI + LJ) * 128;
    static constexpr int LDS_BYTES = 2 * STAGE_BYTES;
};

// Barrier without the memory fence of __syncthreads; the loops place their own waits before it.
__device__ __forceinline__ void lds_barrier() {
    asm volatile("" ::: "memory");
    __builtin_amdgcn_s_barrier();
    asm volatile("" ::: "memory");
}

template <int WI, int WJ>
struct Frags {
    bf16x8 a[WI], b[WJ];
};

// LDS fragment reads and their waits are issued by hand.  With direct memory -> LDS loads in the
// loop the compiler's wait insertion falls back to lgkmcnt(0) before every MFMA block, which also
// waits for the reads just issued for the NEXT sub-step and so undoes the software pipelining.
// LDS reads of a wave complete in order, so "at most n reads outstanding" after issuing the next
// sub-step's n reads means exactly "the current sub-step's fragments have arrived".
__device__ __forceinline__ uint32_t lds_addr(const char* p) {
    return (uint32_t)(uintptr_t)(__attribute__((address_space(3))) const char*)p;
}
template <int OFF>
__device__ __forceinline__ bf16x8 ds_read128(uint32_t addr) {
    bf16x8 v;
    asm volatile("ds_read_b128 %0, %1 offset:%2" : "=v"(v) : "v"(addr), "n"(OFF) : "memory");
    return v;
}
template <int OFF>
__device__ __forceinline__ s16x4 ds_read_tr64(uint32_t addr) {
    s16x4 v;
    asm volatile("ds_read_b64_tr_b16 %0, %1 offset:%2" : "=v"(v) : "v"(addr), "n"(OFF) : "memory");
    return v;
}
__device__ __forceinline__ void ds_write64(uint32_t addr, uint2 v) {
    asm volatile("ds_write_b64 %0, %1" ::"v"(addr), "v"(__builtin_bit_cast(unsigned long, v)) : "memory");
}
// waits until at most N LDS reads are outstanding, and makes the fragments depend on the wait
template <int N, int WI, int WJ>
__device__ __forceinline__ void wait_frags(Frags<WI, WJ>& f) {
    asm volatile("s_waitcnt lgkmcnt(%0)" ::"n"(N < 15 ? N : 15) : "memory");
#pragma unroll
    for (int ib = 0; ib < WI; ++ib) asm volatile("" : "+v"(f.a[ib]));
#pragma unroll
    for (int jb = 0; jb < WJ; ++jb) asm volatile("" : "+v"(f.b[jb]));
}

template <int WI, int WJ>
__device__ __forceinline__ void mma_block(const Frags<WI, WJ>& f, f32x16 (&acc)[WI][WJ]) {
#pragma unroll
    for (int ib = 0; ib < WI; ++ib)
#pragma unroll
        for (int jb = 0; jb < WJ; ++jb)
            acc[ib][jb] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(f.a[ib], f.b[jb], acc[ib][jb], 0, 0, 0);
}

// One MFMA block of a K step that also carries half of the step's tile-load requests (HALF = 0 / 1),
// one request after every few MFMAs.  A memory instruction holds its wave at issue until the memory
// pipeline accepts it, and that pipeline takes most of a step to accept a whole stage; requests
// bunched at the top of the step kept every wave out of its MFMAs for hundreds of cycles, spread out
// they are accepted at once and the SIMD's other wave fills the gaps.
// A wave makes T requests per step, numbered in the order `request(r)` is to be called; the block with
// HALF = 0 carries the first half of them, request_first_half makes the same ones without MFMAs.
template <class S, int HALF, int T, class F>
__device__ __forceinline__ void mma_block_requesting(const Frags<S::WI, S::WJ>& f, f32x16 (&acc)[S::WI][S::WJ],
                                                     F&& request) {
    constexpr int NB = S::WI * S::WJ;
#pragma unroll
    for (int ib = 0; ib < S::WI; ++ib)
#pragma unroll
        for (int jb = 0; jb < S::WJ; ++jb) {
            acc[ib][jb] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(f.a[ib], f.b[jb], acc[ib][jb], 0, 0, 0);
            const int slot = HALF * NB + ib * S::WJ + jb;
#pragma unroll
            for (int r = 0; r < T; ++r)
                if (r * 2 * NB / T == slot) {
                    __builtin_amdgcn_sched_barrier(0);
                    request(r);
                    __builtin_amdgcn_sched_barrier(0);
                }
        }
}
template <class S, int T, class F>
__device__ __forceinline__ void request_first_half(F&& request) {
    constexpr int NB = S::WI * S::WJ;
#pragma unroll
    for (int r = 0; r < T; ++r)
        if (r * 2 * NB / T < NB) request(r);
}
__device__ __forceinline__ void load_to_lds_16(const char* gp, char* lp) {
    __builtin_amdgcn_global_load_lds((const __attribute__((address_space(1))) void*)gp,
                                     (__attribute__((address_space(3))) void*)lp, 16, 0, 0);
}

// Scheduling fence: nothing is moved across it.  The K step is written in the order that software-
// pipelines it (fragments of the next sub-step are requested before the MFMAs of the current one,
// tile requests sit between given MFMAs) and the fences keep that order.
__device__ __forceinline__ void fence() { __builtin_amdgcn_sched_barrier(0); }

struct NoPace {
    __device__ __forceinline__ void operator()(int) const {}
};

// Keeps all workgroups of a launch within a few K steps of each other, so that a W panel one XCD
// has pulled through the memory-side cache is still there when the others ask for it.  Every
// `every` K steps thread 0 counts its workgroup in and polls, a bounded number of times, until the
// others of the round have arrived; the rest of the workgroup meets it at the next barrier.  Purely
// a pacing hint: nothing depends on it, a poll that runs out sets the counter's top bit, which
// satisfies every later target, and the kernel goes on unpaced.
struct GridPace {
    unsigned* ctr;      // arrival counter, zero at launch
    unsigned base;      // arrivals of the rounds before this tile
    unsigned n;         // workgroups that work on a tile in this round
    int every;          // K steps between meetings (power of two), 0 = off
    __device__ __forceinline__ void operator()(int kt) const {
        if (every == 0 || ((kt + 1) & (every - 1)) != 0) return;
        if (threadIdx.x == 0) {
            const unsigned target = base + n * (unsigned)((kt + 1) / every);
            __hip_atomic_fetch_add(ctr, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            int polls = 0;
            while (__hip_atomic_load(ctr, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) < target) {
                if (++polls == 256) {
                    __hip_atomic_fetch_or(ctr, 0x80000000u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                    break;
                }
                __builtin_amdgcn_s_sleep(8);
            }
        }
    }
};

// ---- contraction index major operands ("k-major") ---------------------------------------------
// For dW = H^T dz both operands are stored with the contraction index (the token row) as the slow
// dimension: A(k, i) = dz[row k][column i], B(k, j) = H[row k][column j].  A K step is 64 rows of
// 2 COLS bytes; it goes to LDS row by row (direct loads, 16-byte chunks) and the MFMA fragments are
// read with ds_read_b64_tr_b16, the LDS transpose read of gfx950: in each group of 16 lanes, lane
// l receives element (l % 4) of the 8-byte pieces addressed by lanes l/4, l/4 + 4, l/4 + 8,
// l/4 + 12 of the group.  Pointing lane s of a group at row (s / 4), columns 4 (s % 4) .. + 3
// therefore hands lane l column l and 4 consecutive rows: exactly the per-lane slice of an MFMA
// operand (row of the operand = column of the tile, 4 of its 8 k values).
// A row is cut into 64-byte segments and segment g of row r is kept at position g ^ (r % SEGS),
// so that the four rows one transpose read touches per 32 lanes fall on different banks.
template <int COLS, int NW, int STEP = 64>         // STEP: rows (contraction indices) per K step
struct KMajor {
    static constexpr int ROW_BYTES = COLS * 2;
    static constexpr int CPR = COLS / 8;          // 16-byte chunks per row
    static constexpr int RPI = 64 / CPR;          // rows covered by one wave-wide load instruction
    static constexpr int ROUNDS = STEP / (NW * RPI);
    static constexpr int ROUND_ROWS = NW * RPI;
    static constexpr int SEGS = CPR / 4;          // 64-byte segments per row
    static constexpr int TILE_BYTES = STEP * ROW_BYTES;
};

template <int OFF>
__device__ __forceinline__ bf16x8 read_tr_frag(uint32_t a0, uint32_t a1) {
    const s16x4 lo = ds_read_tr64<OFF>(a0);
    const s16x4 hi = ds_read_tr64<OFF>(a1);
    const s16x8 v = __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7);
    return __builtin_bit_cast(bf16x8, v);
}

// xa / xb: this lane's LDS byte offsets (two half-fragments per block) within a stage, sub-step 0
template <int KS, class S>
__device__ __forceinline__ void load_frags_kmajor(Frags<S::WI, S::WJ>& f, uint32_t cur, const int (&xa)[S::WI][2],
                                                  const int (&xb)[S::WJ][2]) {
    constexpr int OA = KS * 16 * KMajor<S::BI, S::NW>::ROW_BYTES, OB = KS * 16 * KMajor<S::BJ, S::NW>::ROW_BYTES;
#pragma unroll
    for (int ib = 0; ib < S::WI; ++ib) f.a[ib] = read_tr_frag<OA>(cur + xa[ib][0], cur + xa[ib][1]);
#pragma unroll
    for (int jb = 0; jb < S::WJ; ++jb) f.b[jb] = read_tr_frag<OB>(cur + xb[jb][0], cur + xb[jb][1]);
}

// One operand of a contraction, seen from a tile: element (outer index o, contraction index k) at p[o * ld + k], or, if
// the contraction index is the slow one ("k-major"), at p[k * ld + o].  `step` is the distance of two K steps in bytes.
// outer_left, k_left: how many outer and contraction indices exist from here on (both >= 1; looked at only for an
// operand that is read in place, not from a zero-padded copy).
struct Operand {
    const bf16_t* p;
    int64_t ld, step;
    int outer_left = 0;
    int64_t k_left = 0;
};

// How a wave requests one K step of a tile with EXT outer indices from an operand, and where in the LDS it goes.
// CLAMP: requests past the end of a matrix that is read in place repeat its last row or chunk instead.  What a
// repeated outer index contributes is dropped by the epilogues; a repeated contraction index meets a zero of the other
// operand (packed hidden rows and dz are zero there).
template <class S, int EXT, bool KM, bool CLAMP>
struct Loader {
    using K = KMajor<EXT, S::NW>;
    static constexpr int ROUNDS = KM ? K::ROUNDS : EXT / (8 * S::NW);           // requests per wave and step
    static constexpr int ROUND = KM ? K::ROUND_ROWS : 8 * S::NW;                // rows between two of them
    static constexpr int LDS_ROUND = KM ? K::ROUND_ROWS * K::ROW_BYTES : 8 * S::NW * 128;
    static constexpr int NV = CLAMP ? ROUNDS : 1;
    const char* g;          // wave-uniform (scalar registers)
    int64_t ld2;            // bytes
    uint32_t voff[NV];      // lane's offset from g (CLAMP: for every request; else of the first one)
    int row0, col;          // CLAMP: lane's row of round 0, and its first element within a row
    int lds_wave;           // byte offset of the wave's first request within the operand's stage
    int64_t k_left;
    __device__ __forceinline__ Loader(const Operand& o, int wave, int lane) {
        ld2 = o.ld * 2; k_left = o.k_left;
        if (KM) {       // lane l of a request covers chunk slot l % CPR of row l / CPR of its band
            const int lrow = lane / K::CPR, pos = lane % K::CPR, row = wave * K::RPI + lrow;
            col = (((pos >> 2) ^ (row & (K::SEGS - 1))) * 4 + (pos & 3)) * 8;
            lds_wave = wave * K::RPI * K::ROW_BYTES;
            row0 = row;
            if (CLAMP) { g = (const char*)o.p; col = min(col, o.outer_left - 8); }
            else { g = (const char*)(o.p + (int64_t)(wave * K::RPI) * o.ld); voff[0] = (uint32_t)(lrow * ld2 + col * 2); }
        } else {        // lane l of a request covers row l / 8 of the wave's 8-row band and the chunk that belongs at slot l % 8
            col = ((lane & 7) ^ ((((wave & 1) << 2) + (lane >> 4)) & 7)) * 8;
            lds_wave = wave * 8 * 128;
            row0 = wave * 8 + (lane >> 3);
            if (CLAMP) {
                g = (const char*)o.p;
#pragma unroll
                for (int r = 0; r < NV; ++r) voff[r] = (uint32_t)(min(row0 + r * ROUND, o.outer_left - 1) * ld2 + col * 2);
            } else {
                g = (const char*)(o.p + (int64_t)(wave * 8) * o.ld);
                voff[0] = (uint32_t)((lane >> 3) * ld2 + col * 2);
            }
        }
    }
    // CLAMP: offsets for K step `kt` (only the last one may be short; every step is treated alike: no branch in the loop)
    __device__ __forceinline__ void at_step(int kt) {
        if (!CLAMP) return;
        const int64_t left = k_left - (int64_t)kt * 64;
        const int here = left < 64 ? (int)left : 64;
        if (KM) {
#pragma unroll
            for (int r = 0; r < NV; ++r) voff[r] = (uint32_t)min(row0 + r * ROUND, here - 1) * (uint32_t)ld2 + (uint32_t)(col * 2);
        } else {
            const int c = min(col, here - 8);   // the rows' share of voff stays, the chunk's is replaced
            const uint32_t move = (uint32_t)((c - last_col) * 2);
#pragma unroll
            for (int r = 0; r < NV; ++r) voff[r] += move;
            last_col = c;
        }
    }
    int last_col = 0;
    __device__ __forceinline__ void start() { last_col = col; at_step(0); }
    __device__ __forceinline__ void request(int r, char* stage) const {
        if (CLAMP) load_to_lds_16(g + voff[r], stage + lds_wave + r * LDS_ROUND);
        else load_to_lds_16(g + (int64_t)(r * ROUND) * ld2 + voff[0], stage + lds_wave + r * LDS_ROUND);
    }
};

// Where a lane reads its MFMA fragments of an operand: blocks of 32 outer indices from block `first` on.
template <class S, int EXT, int NB, bool KM>
struct Reader {
    using K = KMajor<EXT, S::NW>;
    static constexpr int READS = KM ? 2 * NB : NB;    // LDS reads per sub-step
    int x[KM ? NB : 4][2];    // k-major: byte offsets of a block's two half fragments; else x[sub-step][0]
    __device__ __forceinline__ Reader(int lane, int first, int base) {
        if constexpr (KM) {
            // lane l of a transpose read addresses row 8 (l / 32) + (l % 16) / 4 (+ 4 for the second half of the fragment,
            // + 16 per sub-step), 8 bytes at column 32 b + 16 ((l / 16) % 2) + 4 (l % 4)
            const int q = (lane & 15) >> 2;
            const int sub_bytes = (2 * ((lane >> 4) & 1) + ((lane & 3) >> 1)) * 16 + 8 * (lane & 1);
#pragma unroll
            for (int h = 0; h < 2; ++h) {
                const int row = 8 * (lane >> 5) + q + 4 * h;
                const int at = base + row * K::ROW_BYTES + sub_bytes;
#pragma unroll
                for (int n = 0; n < NB; ++n) x[n][h] = at + (((first + n) ^ ((4 * h + q) & (K::SEGS - 1))) * 64);
            }
        } else {
#pragma unroll
            for (int ks = 0; ks < 4; ++ks)
                x[ks][0] = base + (first * 32 + (lane & 31)) * 128 + (((ks * 2 + (lane >> 5)) ^ ((lane >> 1) & 7)) * 16);
        }
    }
    template <int KS, int... N>
    __device__ __forceinline__ void load_seq(bf16x8 (&f)[NB], uint32_t stage, std::integer_sequence<int, N...>) const {
        if constexpr (KM) ((f[N] = read_tr_frag<KS * 16 * K::ROW_BYTES>(stage + x[N][0], stage + x[N][1])), ...);
        else ((f[N] = ds_read128<N * (32 * 128)>(stage + x[KS][0])), ...);
    }
    template <int KS>
    __device__ __forceinline__ void load(bf16x8 (&f)[NB], uint32_t stage) const {
        load_seq<KS>(f, stage, std::make_integer_sequence<int, NB>{});
    }
};

// acc = sum over `ktiles` steps of 64 of A(i, k) B(j, k) for the tile the two operands point at.
// AK / BK: the operand is k-major; CLAMP: A is read in place (see Loader).  TAIL: of B's outer indices only the first live_j
// matter; waves without any of them leave acc 0.
// first_requested: prefetch_tile has requested step 0.
template <class S, bool AK, bool BK, bool CLAMP, bool TAIL = false, class Pace = NoPace>
__device__ __forceinline__ void mainloop(const Operand& A, const Operand& B, int ktiles, char* lds, f32x16 (&acc)[S::WI][S::WJ],
                                         Pace pace = Pace(), int live_j = 0, bool first_requested = false) {
    constexpr int WI = S::WI, WJ = S::WJ, B_STAGE = S::LI * 128;
    constexpr int EA = AK ? S::LI : S::BI, EB = BK ? S::LJ : S::BJ;     // outer indices that are loaded
    const int tid = threadIdx.x;
    const int lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int wave_i = wave % S::NWI, wave_j = wave / S::NWI;
    Loader<S, EA, AK, CLAMP> la(A, wave, lane);
    Loader<S, EB, BK, false> lb(B, wave, lane);
    const Reader<S, EA, WI, AK> ra(lane, wave_i * WI, 0);
    const Reader<S, EB, WJ, BK> rb(lane, wave_j * WJ, B_STAGE);

#pragma unroll
    for (int ib = 0; ib < WI; ++ib)
#pragma unroll
        for (int jb = 0; jb < WJ; ++jb)
#pragma unroll
            for (int v = 0; v < 16; ++v) acc[ib][jb][v] = 0.f;

    if (ktiles <= 0) return;

    constexpr int NRA = Loader<S, EA, AK, CLAMP>::ROUNDS, NRB = Loader<S, EB, BK, false>::ROUNDS, T = NRA + NRB;
    char* dst = lds;        // stage the requests go to
    auto request = [&](int r) {
        if (r < NRA) la.request(r, dst); else lb.request(r - NRA, dst + B_STAGE);
    };
    // A workgroup runs tile after tile: everybody must be done with the LDS stages of the tile before
    // (its last reads, its trailing requests, a staged epilogue) before they are filled again.
    la.start();
    if (!first_requested) {
        lds_barrier();
#pragma unroll
        for (int r = 0; r < T; ++r) request(r);
    }
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    lds_barrier();

    // One K step on stage `cur` = kt % 2 (its first fragments f0 were read at the end of the step before,
    // and the first half of tile kt+1 was requested there too):
    //   read f1 (sub-step 1) | MFMA f0 + second half of the requests for tile kt+1
    //   read f0 (sub-step 2) | MFMA f1
    //   read f1 (sub-step 3) | MFMA f0
    //   wait: own requests landed, own reads of `cur` done; barrier
    //   read f0 of tile kt+1 | MFMA f1 + first half of the requests for tile kt+2 (into `cur`)
    // After the barrier tile kt+1 is complete and nobody reads `cur` any more.  Steps past the last
    // tile re-request the last tile into the idle stage, which keeps the loop free of branches and
    // every address in bounds.  (Skipping those requests with a uniform branch each was tried: the logits
    // kernels, where they are 6 % of the memory -> LDS traffic, got 2 % slower and dHidden 5 %.)
    Frags<WI, WJ> f0, f1;
    constexpr int NR = Reader<S, EA, WI, AK>::READS + Reader<S, EB, WJ, BK>::READS;   // LDS reads per sub-step
    auto advance = [&](bool more, int kt) {
        la.g += more ? A.step : 0;
        lb.g += more ? B.step : 0;
        la.at_step(kt);
    };
    dst = lds + S::STAGE_BYTES;
    if constexpr (TAIL) {
        if (wave_j * (WJ * 32) >= live_j) {     // the wave only makes its share of the requests (those that others read)
            const int read_j = (live_j + WJ * 32 - 1) / (WJ * 32) * (WJ * 32);     // a wave with tokens reads its whole share
            auto requests = [&](int kt) {
                advance(kt < ktiles, kt < ktiles ? kt : ktiles - 1);
#pragma unroll
                for (int r = 0; r < T; ++r)
                    if (r < NRA || (r - NRA) * (8 * S::NW) < read_j) request(r);
            };
            requests(1);
            for (int kt = 0; kt < ktiles; ++kt) {
                asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
                lds_barrier();
                dst = lds + (kt & 1) * S::STAGE_BYTES;
                requests(kt + 2);
            }
            asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
            return;
        }
    }
    {
        const uint32_t l0 = lds_addr(lds);
        ra.template load<0>(f0.a, l0);
        rb.template load<0>(f0.b, l0);
        advance(ktiles > 1, ktiles > 1 ? 1 : 0);
        request_first_half<S, T>(request);   // of tile 1
        // A register that an LDS read (issued from inline assembly) is still writing must not meet
        // a compiler-made copy, and copies appear where control flow splits or joins: every read is
        // therefore waited for in the block that issued it.
        wait_frags<0>(f0);
    }
    for (int kt = 0; kt < ktiles; ++kt) {
        char* cur = lds + (kt & 1) * S::STAGE_BYTES;
        char* nxt = lds + ((kt + 1) & 1) * S::STAGE_BYTES;
        const uint32_t lc = lds_addr(cur), ln = lds_addr(nxt);
        fence();
        ra.template load<1>(f1.a, lc);
        rb.template load<1>(f1.b, lc);
        fence();
        dst = nxt;
        mma_block_requesting<S, 1, T>(f0, acc, request);
        fence();
        ra.template load<2>(f0.a, lc);
        rb.template load<2>(f0.b, lc);
        wait_frags<NR>(f1);
        fence();
        mma_block<WI, WJ>(f1, acc);
        fence();
        ra.template load<3>(f1.a, lc);
        rb.template load<3>(f1.b, lc);
        wait_frags<NR>(f0);
        fence();
        mma_block<WI, WJ>(f0, acc);
        fence();
        wait_frags<0>(f1);
        asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
        lds_barrier();
        pace(kt);   // no LDS read or tile request is in flight here
        ra.template load<0>(f0.a, ln);
        rb.template load<0>(f0.b, ln);
        fence();
        const bool more = kt + 2 < ktiles;
        advance(more, more ? kt + 2 : ktiles - 1);
        dst = cur;
        mma_block_requesting<S, 0, T>(f1, acc, request);
        fence();
        wait_frags<0>(f0);
    }
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");   // the requests for steps that do not exist
}

// Requests step 0 of a tile into LDS stage 0, for a mainloop call that is told so: right after the mainloop of the tile
// before, whose epilogue then covers the trip to memory (and must keep to stage 1).  No barrier is needed: nobody reads
// the stages any more for values that count, and a wave fills the same bytes of a stage in every step.
template <class S, bool AK, bool BK, bool CLAMP>
__device__ __forceinline__ void prefetch_tile(const Operand& A, const Operand& B, char* lds) {
    constexpr int EA = AK ? S::LI : S::BI, EB = BK ? S::LJ : S::BJ;
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    Loader<S, EA, AK, CLAMP> la(A, wave, lane);
    const Loader<S, EB, BK, false> lb(B, wave, lane);
    la.start();
#pragma unroll
    for (int r = 0; r < Loader<S, EA, AK, CLAMP>::ROUNDS; ++r) la.request(r, lds);
#pragma unroll
    for (int r = 0; r < Loader<S, EB, BK, false>::ROUNDS; ++r) lb.request(r, lds + S::LI * 128);
}

// The same contraction (same fragments, same order of summation: same bits) with three LDS stages for A, whose steps are
// requested two ahead, beside two for B.  For a batch of few rows: W streams through the chip once and every step of it
// comes from HBM, a longer trip than a step takes, while the few hidden rows are in the L2.  All 160 KiB of LDS.
// A group of requests is B's step k and A's step k + 1, in this order, so "all but the last NRA have landed" leaves A's
// step under way.
template <class S>
constexpr int deep_lds_bytes() { return (3 * S::LI + 2 * S::LJ) * 128; }
template <class S, bool AK, bool CLAMP, bool TAIL>
__device__ __forceinline__ void mainloop_deep(const Operand& A, const Operand& B, int ktiles, char* lds, f32x16 (&acc)[S::WI][S::WJ],
                                              int live_j, bool first_requested) {
    constexpr int WI = S::WI, WJ = S::WJ, A_STAGE = S::LI * 128, B_STAGE = S::LJ * 128, B0 = 3 * A_STAGE;
    constexpr int EA = AK ? S::LI : S::BI, EB = S::BJ;
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int wave_i = wave % S::NWI, wave_j = wave / S::NWI;
    Loader<S, EA, AK, CLAMP> la(A, wave, lane);
    Loader<S, EB, false, false> lb(B, wave, lane);
    const Reader<S, EA, WI, AK> ra(lane, wave_i * WI, 0);
    const Reader<S, EB, WJ, false> rb(lane, wave_j * WJ, 0);
    constexpr int NRA = Loader<S, EA, AK, CLAMP>::ROUNDS, NRB = Loader<S, EB, false, false>::ROUNDS, T = NRA + NRB;
#pragma unroll
    for (int ib = 0; ib < WI; ++ib)
#pragma unroll
        for (int jb = 0; jb < WJ; ++jb)
#pragma unroll
            for (int v = 0; v < 16; ++v) acc[ib][jb][v] = 0.f;

    char *dst_a = lds, *dst_b = lds + B0;
    auto request = [&](int r) {
        if (r < NRB) lb.request(r, dst_b); else la.request(r - NRB, dst_a);
    };
    int step_a = 0;                                 // step that la stands at (steps past the last one repeat it, into idle stages)
    auto advance_a = [&]() {
        if (step_a + 1 < ktiles) { ++step_a; la.g += A.step; }
        la.at_step(step_a);
    };
    la.start();
    if (!first_requested) {
        lds_barrier();      // see mainloop
#pragma unroll
        for (int r = 0; r < T; ++r) request(r);     // B's and A's step 0
    }
    advance_a();
    dst_a = lds + A_STAGE;
    if (!first_requested) {
#pragma unroll
        for (int r = 0; r < NRA; ++r) la.request(r, dst_a);
    }
    asm volatile("s_waitcnt vmcnt(%0)" ::"n"(NRA) : "memory");
    lds_barrier();
    int a_cur = 0, a_fill = 2;                      // A's stages: of step kt, and of the step requested next
    // the group for step kt + 1: B's step kt + 1 and A's step kt + 2
    auto next_group = [&](int kt) {
        lb.g += kt + 1 < ktiles ? B.step : 0;
        advance_a();
        dst_b = lds + B0 + ((kt + 1) & 1) * B_STAGE;
        dst_a = lds + a_fill * A_STAGE;
        a_fill = a_fill == 2 ? 0 : a_fill + 1;
    };
    next_group(0);
    if constexpr (TAIL) {
        if (wave_j * (WJ * 32) >= live_j) {         // see mainloop
            const int read_j = (live_j + WJ * 32 - 1) / (WJ * 32) * (WJ * 32);
            auto requests = [&]() {
#pragma unroll
                for (int r = 0; r < T; ++r)
                    if (r >= NRB || r * (8 * S::NW) < read_j) request(r);
            };
            requests();
            for (int kt = 0; kt < ktiles; ++kt) {
                asm volatile("s_waitcnt vmcnt(%0)" ::"n"(NRA) : "memory");
                lds_barrier();
                next_group(kt + 1);
                requests();
            }
            asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
            return;
        }
    }
    Frags<WI, WJ> f0, f1;
    constexpr int NR = Reader<S, EA, WI, AK>::READS + Reader<S, EB, WJ, false>::READS;
    {
        ra.template load<0>(f0.a, lds_addr(lds));
        rb.template load<0>(f0.b, lds_addr(lds + B0));
        request_first_half<S, T>(request);
        wait_frags<0>(f0);
    }
    for (int kt = 0; kt < ktiles; ++kt) {
        const int a_next = a_cur == 2 ? 0 : a_cur + 1;
        const uint32_t ca = lds_addr(lds + a_cur * A_STAGE), na = lds_addr(lds + a_next * A_STAGE);
        const uint32_t cb = lds_addr(lds + B0 + (kt & 1) * B_STAGE), nb = lds_addr(lds + B0 + ((kt + 1) & 1) * B_STAGE);
        fence();
        ra.template load<1>(f1.a, ca);
        rb.template load<1>(f1.b, cb);
        fence();
        mma_block_requesting<S, 1, T>(f0, acc, request);
        fence();
        ra.template load<2>(f0.a, ca);
        rb.template load<2>(f0.b, cb);
        wait_frags<NR>(f1);
        fence();
        mma_block<WI, WJ>(f1, acc);
        fence();
        ra.template load<3>(f1.a, ca);
        rb.template load<3>(f1.b, cb);
        wait_frags<NR>(f0);
        fence();
        mma_block<WI, WJ>(f0, acc);
        fence();
        wait_frags<0>(f1);
        asm volatile("s_waitcnt vmcnt(%0)" ::"n"(NRA) : "memory");
        lds_barrier();
        ra.template load<0>(f0.a, na);
        rb.template load<0>(f0.b, nb);
        fence();
        next_group(kt + 1);
        mma_block_requesting<S, 0, T>(f1, acc, request);
        fence();
        wait_frags<0>(f0);
        a_cur = a_next;
    }
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
}
// the requests before the loop, for the next tile (see prefetch_tile; the epilogue that covers them keeps off the LDS)
template <class S, bool AK, bool CLAMP>
__device__ __forceinline__ void prefetch_tile_deep(const Operand& A, const Operand& B, int ktiles, char* lds) {
    constexpr int EA = AK ? S::LI : S::BI;
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    Loader<S, EA, AK, CLAMP> la(A, wave, lane);
    const Loader<S, S::BJ, false, false> lb(B, wave, lane);
    la.start();
#pragma unroll
    for (int r = 0; r < Loader<S, S::BJ, false, false>::ROUNDS; ++r) lb.request(r, lds + 3 * S::LI * 128);
#pragma unroll
    for (int r = 0; r < Loader<S, EA, AK, CLAMP>::ROUNDS; ++r) la.request(r, lds);
    if (ktiles > 1) la.g += A.step;
    la.at_step(ktiles > 1 ? 1 : 0);
#pragma unroll
    for (int r = 0; r < Loader<S, EA, AK, CLAMP>::ROUNDS; ++r) la.request(r, lds + S::LI * 128);
}

// The same contraction with K steps of 32 rows through NST LDS stages (NST x 32 rows = the same LDS as two
// steps of 64), the requests NST - 1 steps ahead of the MFMAs: the streamed operand of dW comes from HBM, and
// one step of lead is less than a trip there.  Same LDS layout per row, same fragments, same order of
// summation per accumulator: identical results.
template <class S, int NST>
__device__ __forceinline__ void mainloop_kmajor32(const bf16_t* __restrict__ A, int64_t lda, const bf16_t* __restrict__ B,
                                                  int64_t ldb, int ksteps, char* lds, f32x16 (&acc)[S::WI][S::WJ]) {
    constexpr int WI = S::WI, WJ = S::WJ;
    using KA = KMajor<S::BI, S::NW, 32>;
    using KB = KMajor<S::BJ, S::NW, 32>;
    static_assert(KA::ROUNDS >= 1 && KB::ROUNDS >= 1, "a wave instruction must not span more than a step");
    constexpr int STAGE = KA::TILE_BYTES + KB::TILE_BYTES, D = NST - 1, T = KA::ROUNDS + KB::ROUNDS;
    static_assert(NST * STAGE <= S::LDS_BYTES, "stages must fit the kernel's LDS");
    const int tid = threadIdx.x;
    const int lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int wave_i = wave % S::NWI, wave_j = wave / S::NWI;

    auto lane_voff = [&](int cpr, int segs, int rpi, int64_t ld) -> uint32_t {
        const int lrow = lane / cpr, p = lane % cpr;
        const int row_low = (wave * rpi + lrow) & (segs - 1);
        const int gseg = (p >> 2) ^ row_low;
        return (uint32_t)(((int64_t)lrow * ld + (gseg * 4 + (p & 3)) * 8) * 2);
    };
    const uint32_t voff_a = lane_voff(KA::CPR, KA::SEGS, KA::RPI, lda);
    const uint32_t voff_b = lane_voff(KB::CPR, KB::SEGS, KB::RPI, ldb);
    const char* ga = (const char*)(A + (int64_t)(wave * KA::RPI) * lda) + voff_a;
    const char* gb = (const char*)(B + (int64_t)(wave * KB::RPI) * ldb) + voff_b;
    const int64_t round_a = (int64_t)KA::ROUND_ROWS * lda * 2, round_b = (int64_t)KB::ROUND_ROWS * ldb * 2;
    const int64_t step_a = 32 * lda * 2, step_b = 32 * ldb * 2;
    const int lds_wave_a = wave * KA::RPI * KA::ROW_BYTES;
    const int lds_wave_b = KA::TILE_BYTES + wave * KB::RPI * KB::ROW_BYTES;

    const int q = (lane & 15) >> 2;
    const int sub_bytes = (2 * ((lane >> 4) & 1) + ((lane & 3) >> 1)) * 16 + 8 * (lane & 1);
    const int rowpart = 8 * (lane >> 5) + q;
    int xa[WI][2], xb[WJ][2];
#pragma unroll
    for (int r = 0; r < 2; ++r) {
        const int sw = 4 * r + q;   // low bits of the row this lane addresses in half r
        const int base_a = (rowpart + 4 * r) * KA::ROW_BYTES + ((((wave_i * WI) ^ (sw & (KA::SEGS - 1))) * 64)) + sub_bytes;
        const int base_b = KA::TILE_BYTES + (rowpart + 4 * r) * KB::ROW_BYTES +
                           ((((wave_j * WJ) ^ (sw & (KB::SEGS - 1))) * 64)) + sub_bytes;
#pragma unroll
        for (int ib = 0; ib < WI; ++ib) xa[ib][r] = base_a ^ (ib * 64);
#pragma unroll
        for (int jb = 0; jb < WJ; ++jb) xb[jb][r] = base_b ^ (jb * 64);
    }

#pragma unroll
    for (int ib = 0; ib < WI; ++ib)
#pragma unroll
        for (int jb = 0; jb < WJ; ++jb)
#pragma unroll
            for (int v = 0; v < 16; ++v) acc[ib][jb][v] = 0.f;
    if (ksteps <= 0) return;

    int src_step = 0;       // K step the next requests fetch (clamped to the last one), and the stage they go to
    char* dst;
    auto request = [&](int r) {
        if (r < KA::ROUNDS)
            load_to_lds_16(ga + src_step * step_a + r * round_a, dst + lds_wave_a + r * (KA::ROUND_ROWS * KA::ROW_BYTES));
        else
            load_to_lds_16(gb + src_step * step_b + (r - KA::ROUNDS) * round_b,
                           dst + lds_wave_b + (r - KA::ROUNDS) * (KB::ROUND_ROWS * KB::ROW_BYTES));
    };
    lds_barrier();   // see mainloop
#pragma unroll
    for (int st = 0; st < D; ++st) {
        dst = lds + st * STAGE;
        src_step = st < ksteps ? st : ksteps - 1;
#pragma unroll
        for (int r = 0; r < T; ++r) request(r);
    }
    asm volatile("s_waitcnt vmcnt(%0)" ::"n"((D - 1) * T) : "memory");   // step 0 has landed
    lds_barrier();
    Frags<WI, WJ> f0, f1;
    load_frags_kmajor<0, S>(f0, lds_addr(lds), xa, xb);
    wait_frags<0>(f0);
    int cur_i = 0, fil_i = D;
    for (int kt = 0; kt < ksteps; ++kt) {
        const uint32_t lc = lds_addr(lds + cur_i * STAGE);
        const int nxt_i = cur_i + 1 == NST ? 0 : cur_i + 1;
        const uint32_t ln = lds_addr(lds + nxt_i * STAGE);
        fence();
        load_frags_kmajor<1, S>(f1, lc, xa, xb);
        fence();
        dst = lds + fil_i * STAGE;
        src_step = kt + D < ksteps ? kt + D : ksteps - 1;
        mma_block_requesting<S, 0, 2 * T>(f0, acc, request);   // the T requests for step kt + D, spread over the MFMAs
        fence();
        wait_frags<0>(f1);
        asm volatile("s_waitcnt vmcnt(%0)" ::"n"((D - 1) * T) : "memory");   // own requests for step kt + 1 have landed
        lds_barrier();
        load_frags_kmajor<0, S>(f0, ln, xa, xb);
        fence();
        mma_block<WI, WJ>(f1, acc);
        fence();
        wait_frags<0>(f0);
        cur_i = nxt_i;
        fil_i = fil_i + 1 == NST ? 0 : fil_i + 1;
    }
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");   // the requests for steps that do not exist
}

// Workgroup id -> tile.  Hardware deals consecutive workgroup ids round-robin to the 8 XCDs (each
// with its own L2), so id % 8 picks the XCD and id / 8 the position in that XCD's contiguous share
// of a grouped order: GI tiles along i for one j, then the next j, ... so that workgroups resident
// together on an XCD re-use each other's operand panels out of L2.
struct TileId { int ti, tj; bool valid; };
// position `vid` of the grouped order -> tile
__device__ __forceinline__ TileId tile_of_vid(int vid, int tilesI, int tilesJ, int GI) {
    const int total = tilesI * tilesJ;
    TileId t;
    t.valid = vid < total;
    const int group_sz = GI * tilesJ;
    const int grp = vid / group_sz;
    const int first_i = grp * GI;
    const int gi = min(GI, tilesI - first_i);
    const int rem = vid - grp * group_sz;
    t.ti = first_i + rem % gi;
    t.tj = rem / gi;
    return t;
}
__device__ __forceinline__ TileId map_tile(int pid, int tilesI, int tilesJ, int GI) {
    const int per = (tilesI * tilesJ + 7) / 8;
    return tile_of_vid((pid & 7) * per + (pid >> 3), tilesI, tilesJ, GI);
}

__host__ __device__ inline int ids_for(int tilesI, int tilesJ) { return (int)(((int64_t)tilesI * tilesJ + 7) / 8 * 8); }
// The kernels are persistent: one workgroup per CU (LDS admits no more) walks the ids
// blockIdx.x, blockIdx.x + gridDim.x, ...; gridDim.x is a multiple of 8, so a workgroup stays on its
// XCD's share of the order and the workgroups of an XCD stay on neighbouring tiles.  This saves the
// launch gap between workgroups and the dispatch of the ids whose tiles hold no token rows.
std::atomic<int> g_num_cu{256};
inline unsigned grid_for(int tilesI, int tilesJ) {
    const int ids = ids_for(tilesI, tilesJ), cus = g_num_cu.load() / 8 * 8;
    return (unsigned)(ids < cus ? ids : cus);
}

// The head as the first operand of the logits kernels (tile ti of 256 vocabulary entries, contraction over d) and of
// dHidden (tile ti of the hidden dimension, contraction over the vocabulary from K step k0 on): from the packed copy, or
// in place, where one of the two layouts has its contraction index last and the other is read k-major.
template <class S, int WM>
__device__ __forceinline__ Operand logits_w(const WInPlace& w, const bf16_t* packed, int64_t ldk, int ti) {
    if (WM == W_PACKED) return Operand{packed + (int64_t)ti * S::BI * ldk, ldk, 128};
    const int64_t v0 = (int64_t)ti * S::BI;
    if (WM == W_VD) return Operand{w.W + v0 * w.d, w.d, 128, (int)(w.V - v0), w.d};
    return Operand{w.W + v0, w.V, w.V * (K_TILE * 2), (int)(w.V - v0), w.d};
}
template <class S, int WM>
__device__ __forceinline__ Operand dh_w(const WInPlace& w, int ti, int k0) {
    const int64_t d0 = (int64_t)ti * S::BI, v0 = (int64_t)k0 * K_TILE;
    if (WM == W_VD) return Operand{w.W + v0 * w.d + d0, w.d, w.d * (K_TILE * 2), (int)(w.d - d0), w.V - v0};
    return Operand{w.W + d0 * w.V + v0, w.V, 128, (int)(w.d - d0), w.V - v0};
}

template <class S>
struct Lane {
    int lane, wave, wave_i, wave_j, hi, lj;
    __device__ __forceinline__ Lane() {
        lane = threadIdx.x & 63;
        wave = threadIdx.x >> 6;
        wave_i = wave % S::NWI;
        wave_j = wave / S::NWI;
        hi = lane >> 5;
        lj = lane & 31;
    }
};

__device__ __forceinline__ uint2 pack_bf16x4(float a, float b, float c, float d) {
    bf16x4 r;
    r[0] = (__bf16)a; r[1] = (__bf16)b; r[2] = (__bf16)c; r[3] = (__bf16)d;
    return __builtin_bit_cast(uint2, r);
}

// A 256 x 256 tile of bf16 values leaves through LDS so that it reaches memory as whole 256-byte row
// segments, 32 token rows per wave at a time.  Each wave owns a private region for them (128 columns, 256 bytes per
// row).  A lane writes its runs of 4 consecutive
// columns (8 bytes) at 16-byte chunk c ^ (row % 16) of the row, then the wave reads the region back
// row-wise, 16 lanes x 16 bytes per row, and stores 4 full rows per instruction.  The stores are
// streamed (non-temporal): the destination is far larger than the L2s and must not push the
// operand panels out.  `value(ib, jb, v)` is the element the lane holds in accumulator register v of
// block (ib, jb); `out` points at (first row of the wave, first column of the wave) of the tile.
// All waves must be done with both LDS stages (barrier) before the call.
template <class S, class F>
__device__ __forceinline__ void store_tile_through_lds(char* lds, const Lane<S>& L, bf16_t* out, int64_t ld, F&& value) {
    constexpr int WI = S::WI, WJ = S::WJ;
    static_assert(WI == 4, "laid out for 128 columns (256 bytes) per wave row");
    const uint32_t region = lds_addr(lds) + L.wave * (32 * 256), lrow = region + L.lj * 256 + L.hi * 8;
    const int rx = L.lj & 15;
    // read back row-wise: lane l covers chunk l % 16 of row 4 t + l / 16
    const int c = L.lane & 15, r4 = L.lane >> 4;
    bf16_t* o = out + (int64_t)r4 * ld + c * 8;
#pragma unroll
    for (int jb = 0; jb < WJ; ++jb) {
#pragma unroll
        for (int ib = 0; ib < WI; ++ib)
#pragma unroll
            for (int q = 0; q < 4; ++q)
                ds_write64(lrow + (((ib * 4 + q) ^ rx) * 16),
                           pack_bf16x4(value(ib, jb, q * 4), value(ib, jb, q * 4 + 1), value(ib, jb, q * 4 + 2), value(ib, jb, q * 4 + 3)));
        // LDS accesses of a wave complete in order.  All by hand: the compiler would wait for a prefetch into the other
        // stage before it touches the LDS.
        bf16x8 v[8];
#pragma unroll
        for (int tt = 0; tt < 8; ++tt) v[tt] = ds_read128<0>(region + (tt * 4 + r4) * 256 + ((c ^ ((tt * 4 + r4) & 15)) * 16));
        asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
#pragma unroll
        for (int tt = 0; tt < 8; ++tt) asm volatile("" : "+v"(v[tt]));
#pragma unroll
        for (int tt = 0; tt < 8; ++tt)
            __builtin_nontemporal_store(__builtin_bit_cast(u32x4, v[tt]), (u32x4*)(o + (int64_t)(jb * 8 + tt) * 4 * ld));
    }
}

// ragged last vocabulary tile: the columns that do not exist become -infinity
template <class S>
__device__ __forceinline__ void mask_padding(f32x16 (&acc)[S::WI][S::WJ], int n_valid, int hi) {
    if (n_valid >= S::WI * 32) return;
#pragma unroll
    for (int ib = 0; ib < S::WI; ++ib)
#pragma unroll
        for (int jb = 0; jb < S::WJ; ++jb)
#pragma unroll
            for (int v = 0; v < 16; ++v) {
                const int rel = ib * 32 + (v >> 2) * 8 + hi * 4 + (v & 3);
                acc[ib][jb][v] = rel < n_valid ? acc[ib][jb][v] : -INFINITY;
            }
}

// ------------------------------------------------------------------------------------- fwd_lse
// STORE: also keep, for a backward that reloads them instead of recomputing the logits, the tile's
// scaled probabilities u[j][v] = exp(z[j][v] - r[j]) in bf16 in a.zc.  The reference r[j] (a.refz) is
// known before the sweep, so the row's log-sum-exp is not needed to write u, and the backward needs
// one factor per row, -g exp(r - lse), instead of a pass over the stored tile.  r is the logit of
// the row's sampled token minus its behaviour log-prob: the behaviour policy's log-sum-exp, moved by
// the token's own drift, so u is close to the probability itself; without behaviour log-probs it is
// the sampled token's logit and u = p_v / p_y.  The exponent is clamped at 2^115 (a logit 79 above
// the reference); a clamp sets RAPID_STATUS_LOGIT_RANGE.
//
// Epilogue of a logits tile: per token row j (one lane pair) the max and the sum of exponentials over this
// wave's 128 vocabulary columns.  The logit of the sampled token is gathered by a separate small kernel,
// so the per-element work is one max, one fma, one exp and one add (STORE: and one multiply).
template <class S>
__device__ __forceinline__ void load_references(const FwdArgs& a, int64_t j_tile, int M, float (&ref)[S::WJ]) {
    const Lane<S> L;
#pragma unroll
    for (int jb = 0; jb < S::WJ; ++jb) {
        const int64_t j = j_tile + (L.wave_j * S::WJ + jb) * 32 + L.lj;
        ref[jb] = a.refz[j < M ? j : M - 1];
        if (j >= M) ref[jb] = 0.f;      // rows past the last token: zero logits
    }
}
template <class S, bool STORE>
__device__ __forceinline__ void fwd_epilogue(const FwdArgs& a, const TileId& t, int64_t j_tile, int M, char* lds,
                                             f32x16 (&acc)[S::WI][S::WJ], const float (&ref)[S::WJ]) {
    constexpr int WI = S::WI, WJ = S::WJ;
    const Lane<S> L;
    const int i_base = t.ti * S::BI + L.wave_i * (WI * 32);
    const int n_valid = (int)a.V - i_base;          // columns of this wave that exist (>= 128: all)
    const int64_t slot = (int64_t)t.ti * S::NWI + L.wave_i;
    const float zs = a.inv_temp * LOG2E;            // inv_temp > 0: max commutes with the scaling
    mask_padding<S>(acc, n_valid, L.hi);
    float m[WJ], nm[WJ], l[WJ];
#pragma unroll
    for (int jb = 0; jb < WJ; ++jb) {
        float mx = -INFINITY;
#pragma unroll
        for (int ib = 0; ib < WI; ++ib)
#pragma unroll
            for (int v = 0; v < 16; ++v) mx = fmaxf(mx, acc[ib][jb][v]);
        mx = fmaxf(mx, __shfl_xor(mx, 32, 64));
        m[jb] = mx;
        nm[jb] = (mx == -INFINITY) ? 0.f : -mx * zs;
        l[jb] = 0.f;
    }
    if (STORE) {
        float f[WJ];   // exp(wave maximum - reference): turns exp(z - maximum) into exp(z - reference)
        bool clamped = false;
#pragma unroll
        for (int jb = 0; jb < WJ; ++jb) {
            const float r2 = ref[jb] * LOG2E;
            float e2 = m[jb] * zs - r2;                        // -inf for a wave of padding columns only
            if (e2 > 115.f) { e2 = 115.f; clamped = true; }
            f[jb] = __builtin_amdgcn_exp2f(e2);
        }
        if (clamped && a.dev_status) atomicOr(a.dev_status, RAPID_STATUS_LOGIT_RANGE);
        lds_barrier();     // every wave is done with the stage that is used below; a prefetch into the other one goes on
        store_tile_through_lds<S>(lds, L,
                                  a.zc + (j_tile - a.zc_row0 + L.wave_j * (WJ * 32)) * a.ldz + (int64_t)t.ti * S::BI + L.wave_i * (WI * 32),
                                  a.ldz, [&](int ib, int jb, int v) {
                                      const float e = __builtin_amdgcn_exp2f(fmaf(acc[ib][jb][v], zs, nm[jb]));
                                      l[jb] += e;
                                      return e * f[jb];
                                  });
    } else {
#pragma unroll
        for (int jb = 0; jb < WJ; ++jb)
#pragma unroll
            for (int ib = 0; ib < WI; ++ib)
#pragma unroll
                for (int v = 0; v < 16; ++v) l[jb] += __builtin_amdgcn_exp2f(fmaf(acc[ib][jb][v], zs, nm[jb]));
    }
#pragma unroll
    for (int jb = 0; jb < WJ; ++jb) {
        const int64_t j = j_tile + L.wave_j * (WJ * 32) + jb * 32 + L.lj;
        const float ls = l[jb] + __shfl_xor(l[jb], 32, 64);
        if (L.hi == 0) {
            a.part_max[slot * a.ld_part + (j - a.part_row0)] = m[jb] * a.inv_temp;
            a.part_sum[slot * a.ld_part + (j - a.part_row0)] = ls;
        }
    }
}

// one workgroup per CU on 256 x 256 tiles: the logits tile on MFMA, then the epilogue above
template <class S, bool STORE, int WM, bool DEEP = false>
__global__ __launch_bounds__(S::NT) void fwd_lse_kernel(FwdArgs a) {
    constexpr int WI = S::WI, WJ = S::WJ;
    extern __shared__ __attribute__((aligned(128))) char lds[];
    const int M = a.counts[CNT_M], Mr = a.counts[CNT_MR];
    if (a.row0 >= Mr) return;
    // the order (and with it the split over the XCDs) covers the row tiles that hold tokens only
    const int tilesM = min(a.tilesM * (256 / S::BJ), (int)((Mr - a.row0 + S::BJ - 1) / S::BJ));
    const int per = ids_for(a.tilesV, tilesM) / 8, wgs = gridDim.x / 8, x = blockIdx.x & 7, w = blockIdx.x >> 3;
    // The last row tile is the cheaper the fewer tokens it holds (waves without any do no products: 260 to 300 tokens at
    // d = 1536, V = 151936 241 -> 212 us a call, 16 to 100 tokens 174 -> 153 us).  Where a round of workgroups covers whole groups of the
    // order, a workgroup would meet the same row tile in every round: it moves on by one row tile per round then.
    const int turn = wgs % (a.gi * tilesM) == 0 ? a.gi : 0;
    auto tile = [&](int r) {        // of round r; once there is none, later rounds have none either
        const int pos = r * wgs + (w + r * turn) % wgs;
        TileId t = tile_of_vid(x * per + pos, a.tilesV, tilesM, a.gi);
        t.valid = t.valid && r * wgs < per && pos < per;
        return t;
    };
    auto opW = [&](const TileId& t) { return logits_w<S, WM>(a.w, a.Wvd, a.ldk, t.ti); };
    auto opH = [&](const TileId& t) { return Operand{a.Hc + (a.row0 + (int64_t)t.tj * S::BJ) * a.ldk, a.ldk, 128}; };
    // The next tile's first step is on its way while this tile's epilogue runs (in stage 1, if its waves' regions fit): a
    // trip to memory per tile of d / 64 steps.  The kernel's time without and with it, three runs of each in turn: d = 256
    // 573-580 -> 553-558 us, 290 tokens at d = 1536 180 -> 176 us, d = 896 18.56 -> 18.39 ms, d = 1536 28.26 -> 28.12 ms (the chip is near
    // its power limit there); a whole step changes by less than its spread.
    // In-place reads with a store have no registers left for it (11 spilled; small head's forward 15.5 -> 17.6 us).
    constexpr bool AHEAD = !STORE || (!DEEP && WM == W_PACKED && S::NW * (32 * 256) <= S::STAGE_BYTES);
    TileId t = tile(0);
    for (int r = 0; t.valid; ++r) {
        const int64_t j_tile = a.row0 + (int64_t)t.tj * S::BJ;   // first token row of the tile
        const int live = (int)min((int64_t)S::BJ, M - j_tile);
        f32x16 acc[WI][WJ];
        float ref[WJ];
        if (STORE && AHEAD) load_references<S>(a, j_tile, M, ref);
        const int ktiles = (int)(a.dpad / K_TILE);
        if constexpr (DEEP) mainloop_deep<S, WM == W_DV, WM != W_PACKED, true>(opW(t), opH(t), ktiles, lds, acc, live, AHEAD && r > 0);
        else mainloop<S, WM == W_DV, false, WM != W_PACKED, true>(opW(t), opH(t), ktiles, lds, acc, NoPace(), live, AHEAD && r > 0);
        const TileId next = tile(r + 1);
        if (STORE && !AHEAD) load_references<S>(a, j_tile, M, ref);
        if (STORE && AHEAD) {     // they are here: the compiler shall see that before the requests below
#pragma unroll
            for (int jb = 0; jb < WJ; ++jb) asm volatile("" : "+v"(ref[jb]));
        }
        if (AHEAD && next.valid) {
            if constexpr (DEEP) prefetch_tile_deep<S, WM == W_DV, WM != W_PACKED>(opW(next), opH(next), ktiles, lds);
            else prefetch_tile<S, WM == W_DV, false, WM != W_PACKED>(opW(next), opH(next), lds);
        }
        if (STORE || (int)(threadIdx.x >> 6) / S::NWI * (WJ * 32) < live)      // else: no token of this wave's
            fwd_epilogue<S, STORE>(a, t, j_tile, M, lds + (AHEAD ? S::STAGE_BYTES : 0), acc, ref);
        t = next;
    }
}

// ---------------------------------------------------------------- fwd_lse, two workgroups per CU
// The tiles of the logits kernels are short (K = d is a few dozen steps) and end in an epilogue the MFMA
// pipe does not take part in (max, exp, sum over the accumulators; STORE: the staged store).  With one
// workgroup per CU nothing else is resident to use the pipe meanwhile.  This variant runs TWO workgroups
// of 4 waves per CU, each on a 256 (vocabulary) x 128 (token rows) tile, so one workgroup's epilogue and
// tile fill overlap the other's main loop.  Each wave still owns 128 x 64 (the same fragments per MFMA as
// the 8-wave kernel).  For two workgroups to fit, K advances 32 per step through three LDS stages of
// 24 KiB (72 KiB per workgroup).  Half-line rows would double the L2 requests, so W comes from a copy that
// is blocked per (256-row tile, K step): 16 KiB contiguous, already in the LDS order, and a request is a
// straight 1 KiB copy; the hidden rows stay row-major (half a line per row and step, a third of the bytes).
//
// LDS layout of a stage: 256 W rows, then 128 hidden rows, 64 bytes each = 4 chunks of 16 bytes; chunk c of
// row r sits at position c ^ ((r >> 2) & 3), which makes the ds_read_b128 fragment reads conflict free
// (16 consecutive lanes = 16 consecutive rows of one chunk index cover 256 distinct bytes).
template <int NWJ_, int NSTAGE_, int WJ_ = 2>
struct FwdK32 {
    using S = Geo<2, NWJ_, 4, WJ_>;                // 2 x NWJ waves of 128 x (32 WJ): a 256 x (32 WJ NWJ) tile
    static constexpr int K_STEP = 32, NSTAGE = NSTAGE_, NW = 2 * NWJ_;
    static constexpr int A_BYTES = 256 * 64, B_BYTES = S::BJ * 64, STAGE = A_BYTES + B_BYTES;
    static constexpr int LDS_BYTES = STAGE * NSTAGE;
    static constexpr int RA = 16 / NW, RB = S::BJ / 16 / NW, R = RA + RB;   // 1 KiB requests per wave and step
};
using Fwd2 = FwdK32<2, 3>;   // two workgroups per CU: 4 waves, 256 x 128, 72 KiB
using Fwd3 = FwdK32<4, 4>;   // one workgroup per CU: 8 waves, 256 x 256, 128 KiB, requests three steps ahead
using Fwd4 = FwdK32<2, 4, 4>;   // the same with 4 waves of 128 x 128 (a third fewer LDS fragment reads per MFMA)

// acc = W_tile . H_tile^T over `ksteps` steps of 32.  wblk: the tile's first block of the blocked copy of W
// (ksteps blocks of 16 KiB follow each other); B: first hidden row of the tile, row-major, ldb elements.
// The requests run NSTAGE - 1 steps ahead of the MFMAs.
template <class F2>
__device__ __forceinline__ void mainloop32(const char* __restrict__ wblk, const bf16_t* __restrict__ B, int64_t ldb,
                                           int ksteps, char* lds, f32x16 (&acc)[4][F2::S::WJ]) {
    using S = typename F2::S;
    constexpr int WI = 4, WJ = S::WJ, NW = F2::NW, RA = F2::RA, R = F2::R, NST = F2::NSTAGE, D = NST - 1;
    const int tid = threadIdx.x;
    const int lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int wave_i = wave & 1, wave_j = wave >> 1;

    // requests: 1 KiB each; request r of a wave is unit r NW + wave of its operand (W: linear; hidden rows: 16 rows)
    const char* ga = wblk + wave * 1024 + lane * 16;
    const int gchunk = (lane & 3) ^ ((lane >> 4) & 3);            // chunk that belongs at slot lane % 4 of row lane / 4
    const char* gb = (const char*)(B + (int64_t)(wave * 16 + (lane >> 2)) * ldb + gchunk * 8);
    const int64_t b_round = (int64_t)(16 * NW) * ldb * 2;         // the wave's next 16 rows
    const int dst_wave = wave * 1024;

    // fragment reads
    const int frow = lane & 31, fhi = lane >> 5;
    const int x0 = (fhi ^ ((frow >> 2) & 3)) * 16, x1 = x0 ^ 32;  // chunk 2 ks + fhi at its swizzled position
    const int a_off = (wave_i * 128 + frow) * 64;
    const int b_off = F2::A_BYTES + (wave_j * (WJ * 32) + frow) * 64;

#pragma unroll
    for (int ib = 0; ib < WI; ++ib)
#pragma unroll
        for (int jb = 0; jb < WJ; ++jb)
#pragma unroll
            for (int v = 0; v < 16; ++v) acc[ib][jb][v] = 0.f;
    if (ksteps <= 0) return;

    int src_step = 0;       // K step the next requests fetch (clamped to the last one: the loop has no branches
    char* dst;              // and every address stays in bounds), and the stage they go to
    auto request = [&](int r) {
        if (r < RA)
            load_to_lds_16(ga + (int64_t)src_step * F2::A_BYTES + r * (NW * 1024), dst + dst_wave + r * (NW * 1024));
        else
            load_to_lds_16(gb + (int64_t)src_step * 64 + (r - RA) * b_round,
                           dst + F2::A_BYTES + dst_wave + (r - RA) * (NW * 1024));
    };
    auto read_frags = [&](Frags<WI, WJ>& f, const char* stage, int x) {
        const uint32_t la = lds_addr(stage) + a_off + x, lb = lds_addr(stage) + b_off + x;
        f.a[0] = ds_read128<0>(la); f.a[1] = ds_read128<2048>(la); f.a[2] = ds_read128<4096>(la); f.a[3] = ds_read128<6144>(la);
        f.b[0] = ds_read128<0>(lb); f.b[1] = ds_read128<2048>(lb);
        if constexpr (WJ == 4) { f.b[2] = ds_read128<4096>(lb); f.b[3] = ds_read128<6144>(lb); }
    };

    // everybody is done with the stages of the tile before (reads, trailing requests, a staged epilogue)
    lds_barrier();
#pragma unroll
    for (int st = 0; st < D; ++st) {                  // steps 0 .. D-1 into stages 0 .. D-1
        dst = lds + st * F2::STAGE;
        src_step = st < ksteps ? st : ksteps - 1;
#pragma unroll
        for (int r = 0; r < R; ++r) request(r);
    }
    asm volatile("s_waitcnt vmcnt(%0)" ::"n"((D - 1) * R) : "memory");   // step 0 has landed (loads complete in order)
    lds_barrier();
    Frags<WI, WJ> f0, f1;
    read_frags(f0, lds, x0);
    wait_frags<0>(f0);
    // One K step on stage `cur` (its first fragments f0 are in registers):
    //   read f1 (second half of the step) | MFMA f0 + the requests for step kt+D into stage (kt+D) % NSTAGE
    //   wait: own reads of `cur` done, own requests for step kt+1 landed; barrier
    //   read f0 of step kt+1              | MFMA f1
    // The stage the requests go to was read during step kt-1, and everybody passed the barrier at the end of it.
    int cur_i = 0, fil_i = D;
    for (int kt = 0; kt < ksteps; ++kt) {
        char* cur = lds + cur_i * F2::STAGE;
        const int nxt_i = cur_i + 1 == NST ? 0 : cur_i + 1;
        char* nxt = lds + nxt_i * F2::STAGE;
        fence();
        read_frags(f1, cur, x1);
        fence();
        dst = lds + fil_i * F2::STAGE;
        src_step = kt + D < ksteps ? kt + D : ksteps - 1;
        mma_block_requesting<S, 0, 2 * R>(f0, acc, request);   // the R requests spread over the 8 MFMAs
        fence();
        wait_frags<0>(f1);
        asm volatile("s_waitcnt vmcnt(%0)" ::"n"((D - 1) * R) : "memory");
        lds_barrier();
        read_frags(f0, nxt, x0);
        fence();
        mma_block<WI, WJ>(f1, acc);
        fence();
        wait_frags<0>(f0);
        cur_i = nxt_i;
        fil_i = fil_i + 1 == NST ? 0 : fil_i + 1;
    }
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");   // the requests for steps that do not exist
}

template <class F2, bool STORE>
__global__ __launch_bounds__(64 * F2::NW, (F2::NW == 4 && F2::S::WJ == 2) ? 2 : 1) void fwd_lse2_kernel(FwdArgs a) {
    using S = typename F2::S;
    extern __shared__ __attribute__((aligned(128))) char lds[];
    const int M = a.counts[CNT_M], Mr = a.counts[CNT_MR];
    if (a.row0 >= Mr) return;
    // the order covers the row tiles that hold tokens only
    const int tilesM = min(a.tilesM * (256 / S::BJ), (int)((Mr - a.row0 + S::BJ - 1) / S::BJ));
    const int ksteps = (int)(a.dpad / F2::K_STEP);
    for (int pid = blockIdx.x, ids = ids_for(a.tilesV, tilesM); pid < ids; pid += gridDim.x) {
        const TileId t = map_tile(pid, a.tilesV, tilesM, a.gi);
        if (!t.valid) continue;
        const int64_t j_tile = a.row0 + (int64_t)t.tj * S::BJ;
        f32x16 acc[4][S::WJ];
        mainloop32<F2>((const char*)a.WvdB + (int64_t)t.ti * ksteps * F2::A_BYTES, a.Hc + j_tile * a.ldk, a.ldk, ksteps, lds, acc);
        float ref[S::WJ];
        if (STORE) load_references<S>(a, j_tile, M, ref);
        fwd_epilogue<S, STORE>(a, t, j_tile, M, lds, acc, ref);
    }
}

// W as the two-workgroup forward reads it: for every 256-row tile and K step of 32 a 16 KiB block, row r's
// chunk c (8 elements) at position c ^ ((r >> 2) & 3) of the row's 64 bytes.  One thread per 16-byte chunk.
__global__ void block_w32_kernel(const bf16_t* __restrict__ Wvd, int64_t ldk, bf16_t* __restrict__ out, int64_t Vpad,
                                 int64_t dpad) {
    const int64_t o = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;   // destination chunk
    const int64_t ksteps = dpad / 32, total = Vpad * ksteps * 4;
    if (o >= total) return;
    const int64_t tile = o / (ksteps * 1024), rem = o % (ksteps * 1024);
    const int64_t ks = rem / 1024;
    const int within = (int)(rem % 1024), row = within >> 2, pos = within & 3;
    const int c = pos ^ ((row >> 2) & 3);
    const uint4 v = *(const uint4*)(Wvd + (tile * 256 + row) * ldk + ks * 32 + c * 8);
    *(uint4*)(out + o * 8) = v;
}

// ------------------------------------------------------------------------------------------ dz
template <class S, int WM>
__global__ __launch_bounds__(S::NT) void dz_kernel(DzArgs a) {
    constexpr int WI = S::WI, WJ = S::WJ;
    extern __shared__ __attribute__((aligned(128))) char lds[];
    const int M = a.counts[CNT_M], Mr = a.counts[CNT_MR];
    if (a.m0 >= Mr) return;
    const int tilesM = min(a.tilesM * (256 / S::BJ), (int)((Mr - a.m0 + S::BJ - 1) / S::BJ));   // row tiles that hold tokens
    for (int pid = blockIdx.x, ids = ids_for(a.tilesV, tilesM); pid < ids; pid += gridDim.x) {
    const TileId t = map_tile(pid, a.tilesV, tilesM, a.gi);
    if (!t.valid) continue;
    f32x16 acc[WI][WJ];
    mainloop<S, WM == W_DV, false, WM != W_PACKED>(logits_w<S, WM>(a.w, a.Wvd, a.ldk, t.ti),
                                                   Operand{a.Hc + (int64_t)t.tj * S::BJ * a.ldk, a.ldk, 128}, (int)(a.dpad / K_TILE), lds, acc);
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");   // the spare tile request of the last step
    __syncthreads();                                    // every wave is done with both stages
    // dz = -g p here; the +g of the sampled token's column is added by a separate small kernel, so
    // the per-element work is one fma, one exp, one multiply and half a convert.  Rows past the last token are
    // zero (they may belong to generations without gradient, whose logits are any size: exp of one of them
    // times g = 0 would be NaN), columns past V too (dHidden may meet repeated weights there).
    const Lane<S> L;
    const int64_t i_base = (int64_t)t.ti * S::BI + L.wave_i * (WI * 32);
    const int64_t jl_base = (int64_t)t.tj * S::BJ + L.wave_j * (WJ * 32);   // row in chunk
    const float zs = a.inv_temp * LOG2E;
    if (a.m0 + jl_base + WJ * 32 > M) {
#pragma unroll
        for (int jb = 0; jb < WJ; ++jb) {
            const bool live = a.m0 + jl_base + jb * 32 + L.lj < M;
#pragma unroll
            for (int ib = 0; ib < WI; ++ib)
#pragma unroll
                for (int v = 0; v < 16; ++v) acc[ib][jb][v] = live ? acc[ib][jb][v] : 0.f;
        }
    }
    mask_padding<S>(acc, (int)(a.V - i_base), L.hi);
    float ngj[WJ], nlse[WJ];
#pragma unroll
    for (int jb = 0; jb < WJ; ++jb) {
        const int64_t j = a.m0 + jl_base + jb * 32 + L.lj;
        const bool live = j < M;
        ngj[jb] = live ? -a.rowg[j] * a.inv_temp : 0.f;
        nlse[jb] = live ? -a.lse_c[j] * LOG2E : 0.f;
    }
    store_tile_through_lds<S>(lds, L, a.dz + jl_base * a.ldz + i_base, a.ldz, [&](int ib, int jb, int v) {
        return ngj[jb] * __builtin_amdgcn_exp2f(fmaf(acc[ib][jb][v], zs, nlse[jb]));
    });
    }
}

// ------------------------------------------------------------------------------- sharing out tiles
// The tiles of dHidden are long (the contraction runs over the whole vocabulary) and few, those of dW are few if the
// head is small: a launch has a handful of rounds of one tile per workgroup, or less than one, and a last round that
// is only partly filled would leave most of the chip idle for a whole tile.  So the rem tiles of the last, partial
// round are not dealt out tile by tile: the contraction of each is cut into S equal segments, and the rem x S
// (segment, tile) units, in that order, are dealt to the XCDs in contiguous shares.  An XCD thus works on one or a few
// segments of all those tiles and reads only those stretches of the operands: they come from memory about once,
// however few rows there are.  A workgroup leaves the fp32 accumulators of a unit in `part`, and a second kernel adds
// the S pieces of a tile in segment order and stores the result, which does not depend on timing.
// Measured, dHidden: d = 1536, V = 151936, about 2200 rows: 1.73 ms when a launch had no more workgroups than tiles,
// 0.76 ms now; d = 256, V = 4096, 1800 rows: 104 -> 21 us, dW there 49 -> 29 us with the second pass; dW of d = 896, 73 000
// rows, whose last round was a third full: 18.8 -> 17.1 ms.
constexpr int MAX_UNITS = 512;      // partial tiles a launch may leave (part_bytes)
struct TileShare {     // how a launch of `grid` workgroups works through `total` tiles
    int wgs, full_rounds, rem, segs, unit_share;
    bool cut;
    __device__ __forceinline__ TileShare(int total, int grid, int ktiles, bool can_cut) {
        wgs = grid / 8; full_rounds = total / grid; rem = total - full_rounds * grid;
        // S with the shortest last round, counted in K steps of a workgroup: the segments of its units, about 5 steps for
        // filling the pipeline and storing the accumulators, and the second pass over 256 KiB per unit (1 / 25 step each).
        // In whole numbers (25 S times the cost), so that the kernel that cuts and the one that adds the pieces agree.
        segs = 1;
        int64_t best = 25 * ((int64_t)ktiles + 4);
        if (can_cut && rem > 0) {
            for (int sg = 2; sg <= 64 && rem * sg <= MAX_UNITS && sg * 4 <= ktiles; sg += sg < 8 ? 1 : sg / 4) {
                const int rounds = (rem * sg + grid - 1) / grid;
                const int64_t cost = 25 * (int64_t)rounds * (ktiles + 5 * sg) + rem * sg * sg;
                if (cost * segs < best * sg) { best = cost; segs = sg; }
            }
        }
        cut = segs > 1;
        unit_share = (rem * segs + 7) / 8;
    }
};

// the accumulators as they are: register r of thread tid at part[unit][r][tid]
template <class S>
__device__ __forceinline__ void store_unit(float* part, int unit, const f32x16 (&acc)[S::WI][S::WJ]) {
    int64_t off = (int64_t)unit * (S::BI * S::BJ) + threadIdx.x;
#pragma unroll
    for (int ib = 0; ib < S::WI; ++ib)
#pragma unroll
        for (int jb = 0; jb < S::WJ; ++jb) {
            asm volatile("" : "+v"(off));   // one address per block of 16 stores, formed here and not ahead of the loops
#pragma unroll
            for (int v = 0; v < 16; ++v) part[off + v * S::NT] = acc[ib][jb][v];
            off += 16 * S::NT;
        }
}
// sum[16] = block (ib, jb) of tile tpos of the cut round, its pieces added in segment order (one after the other, 42 pieces
// of a tile were 23 us of trips to memory)
template <class S>
__device__ __forceinline__ void sum_units(const float* part, const TileShare& sh, int tpos, int ib, int jb, float (&sum)[16]) {
#pragma unroll
    for (int v = 0; v < 16; ++v) sum[v] = 0.f;
    const float* in = part + (int64_t)tpos * (S::BI * S::BJ) + threadIdx.x + (int64_t)((ib * S::WJ + jb) * 16) * S::NT;
    const int64_t next = (int64_t)sh.rem * (S::BI * S::BJ);
    auto add = [&](auto pieces) {      // that many pieces, their loads in flight together
        constexpr int P = decltype(pieces)::value;
        float got[P][16];
#pragma unroll
        for (int p = 0; p < P; ++p)
#pragma unroll
            for (int v = 0; v < 16; ++v) got[p][v] = in[p * next + v * S::NT];
#pragma unroll
        for (int p = 0; p < P; ++p)
#pragma unroll
            for (int v = 0; v < 16; ++v) sum[v] += got[p][v];
        in += P * next;
    };
    int seg = 0;
    for (; seg + 4 <= sh.segs; seg += 4) add(std::integral_constant<int, 4>{});
    for (; seg < sh.segs; ++seg) add(std::integral_constant<int, 1>{});
}

// ------------------------------------------------------------------------------------------ dh
// K steps: the vocabulary rounded up to whole steps (in the packed copy and in dz zeros follow)
__device__ __forceinline__ int dh_ksteps(const DhArgs& a) { return (int)((a.w.V + K_TILE - 1) / K_TILE); }

// row tiles that hold tokens (tilesM counts 256 rows each)
template <class S>
__device__ __forceinline__ int dh_row_tiles(const DhArgs& a, int M) {
    return (int)min((int64_t)a.tilesM * (256 / S::BJ), (M - a.m0 + S::BJ - 1) / S::BJ);
}

// stores a tile of dHidden: accumulators times the row factor (if any), bf16, to the rows' positions
template <class S>
__device__ __forceinline__ void dh_store(const DhArgs& a, const TileId& t, int M, const f32x16 (&acc)[S::WI][S::WJ]) {
    constexpr int WI = S::WI, WJ = S::WJ;
    const Lane<S> L;
    const int64_t i_base = (int64_t)t.ti * S::BI + L.wave_i * (WI * 32);
#pragma unroll
    for (int jb = 0; jb < WJ; ++jb) {
        const int64_t j = a.m0 + (int64_t)t.tj * S::BJ + L.wave_j * (WJ * 32) + jb * 32 + L.lj;
        if (j >= M) continue;
        bf16_t* out = a.dhidden + (int64_t)a.row_index[j] * a.d;
        const float cj = a.rowc ? a.rowc[j] : 1.f;   // cached ratios: the row's -g p_y / temperature
#pragma unroll
        for (int ib = 0; ib < WI; ++ib)
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                const int64_t i0 = i_base + ib * 32 + q * 8 + L.hi * 4;
                if (i0 < a.d)
                    *(uint2*)(out + i0) = pack_bf16x4(cj * acc[ib][jb][q * 4], cj * acc[ib][jb][q * 4 + 1],
                                                      cj * acc[ib][jb][q * 4 + 2], cj * acc[ib][jb][q * 4 + 3]);
            }
    }
}

// acc = the tile's contraction over the K steps [k0, k1)
template <class S, int WM, class Pace>
__device__ __forceinline__ void dh_contract(const DhArgs& a, const TileId& t, int k0, int k1, char* lds,
                                            f32x16 (&acc)[S::WI][S::WJ], Pace pace) {
    const Operand z{a.dz + (int64_t)t.tj * S::BJ * a.ldv + (int64_t)k0 * K_TILE, a.ldv, 128};
    if constexpr (WM != W_PACKED) {
        mainloop<S, WM == W_VD, false, true, false, Pace>(dh_w<S, WM>(a.w, t.ti, k0), z, k1 - k0, lds, acc, pace);
        return;
    }
    const Operand w = a.WdvB ? Operand{a.WdvB + ((int64_t)t.ti * (a.Vpad / K_TILE) + k0) * (S::BI * 64), 64, S::BI * 128}   // tile-blocked copy
                             : Operand{a.Wdv + (int64_t)t.ti * S::BI * a.ldv + (int64_t)k0 * K_TILE, a.ldv, 128};
    mainloop<S, false, false, false, false, Pace>(w, z, k1 - k0, lds, acc, pace);
}

// what workgroup `block` of `grid` does
template <class S, int WM>
__device__ __forceinline__ void dh_work(const DhArgs& a, int block, int grid, char* lds) {
    constexpr int WI = S::WI, WJ = S::WJ;
    const int tilesD = (int)(a.dpadR / S::BI);
    const int M = a.counts[CNT_M];
    if (a.m0 >= M) return;
    // the order (and with it the split over the XCDs) covers the row tiles that hold tokens only: a
    // short last chunk would otherwise leave whole XCDs with nothing but empty tiles
    const int tilesM = dh_row_tiles<S>(a, M);
    const int x = block & 7, w = block >> 3;
    const int ktiles = dh_ksteps(a);
    const TileShare sh(tilesD * tilesM, grid, ktiles, a.part != nullptr);
    const int gi = a.gi > 0 ? a.gi : tilesD;
    GridPace pace{a.pace, 0u, (unsigned)grid, a.pace ? a.pace_every : 0};   // see GridPace
    const unsigned meetings = (unsigned)(ktiles / (pace.every ? pace.every : 1));
    for (int round = 0; round < sh.full_rounds; ++round) {
        const TileId t = tile_of_vid((x * sh.full_rounds + round) * sh.wgs + w, tilesD, tilesM, gi);
        f32x16 acc[WI][WJ];
        pace.base = meetings * (unsigned)(grid * round);
        dh_contract<S, WM, GridPace>(a, t, 0, ktiles, lds, acc, pace);
        dh_store<S>(a, t, M, acc);
    }
    // the last round: unit u = (segment u / rem, tile u % rem); the accumulators of a cut tile go to part[u]
    pace.base = meetings * (unsigned)(grid * sh.full_rounds);
    pace.n = (unsigned)sh.rem;
    for (int pos = w; pos < sh.unit_share; pos += sh.wgs) {
        const int u = x * sh.unit_share + pos;
        if (u >= sh.rem * sh.segs) break;
        const int seg = u / sh.rem, tpos = u - seg * sh.rem;
        const int k0 = (int)((int64_t)ktiles * seg / sh.segs), k1 = (int)((int64_t)ktiles * (seg + 1) / sh.segs);
        const TileId t = tile_of_vid(sh.full_rounds * grid + tpos, tilesD, tilesM, gi);
        f32x16 acc[WI][WJ];
        if (!sh.cut) {
            dh_contract<S, WM, GridPace>(a, t, k0, k1, lds, acc, pace);
            dh_store<S>(a, t, M, acc);
            continue;
        }
        dh_contract<S, WM, NoPace>(a, t, k0, k1, lds, acc, NoPace());
        store_unit<S>(a.part, u, acc);
    }
}
template <class S, int WM>
__global__ __launch_bounds__(S::NT) void dh_kernel(DhArgs a) {
    extern __shared__ __attribute__((aligned(128))) char lds[];
    dh_work<S, WM>(a, blockIdx.x, gridDim.x, lds);
}

// adds the pieces of the tiles that dh_work cut (grid_of_dh: the number of its workgroups) and stores
// them; workgroup (tpos, block) does the 32 x 32 block `block` of every wave of tile tpos of the last round
template <class S>
__device__ __forceinline__ void dh_add_pieces(const DhArgs& a, int grid_of_dh, int tpos, int block) {
    constexpr int WJ = S::WJ, WI = S::WI;
    const int tilesD = (int)(a.dpadR / S::BI);
    const int M = a.counts[CNT_M];
    if (a.m0 >= M) return;
    const int tilesM = dh_row_tiles<S>(a, M);
    const TileShare sh(tilesD * tilesM, grid_of_dh, dh_ksteps(a), true);
    const int ib = block / WJ, jb = block % WJ;
    if (!sh.cut || tpos >= sh.rem) return;
    const TileId t = tile_of_vid(sh.full_rounds * grid_of_dh + tpos, tilesD, tilesM, a.gi > 0 ? a.gi : tilesD);
    const Lane<S> L;
    const int64_t i_base = (int64_t)t.ti * S::BI + L.wave_i * (WI * 32) + ib * 32;
    const int64_t j = a.m0 + (int64_t)t.tj * S::BJ + L.wave_j * (WJ * 32) + jb * 32 + L.lj;
    if (j >= M) return;
    float sum[16];
    sum_units<S>(a.part, sh, tpos, ib, jb, sum);
    bf16_t* out = a.dhidden + (int64_t)a.row_index[j] * a.d;
    const float cj = a.rowc ? a.rowc[j] : 1.f;
#pragma unroll
    for (int q = 0; q < 4; ++q) {
        const int64_t i0 = i_base + q * 8 + L.hi * 4;
        if (i0 < a.d)
            *(uint2*)(out + i0) = pack_bf16x4(cj * sum[q * 4], cj * sum[q * 4 + 1], cj * sum[q * 4 + 2], cj * sum[q * 4 + 3]);
    }
}

template <class S>
__global__ __launch_bounds__(S::NT) void dh_reduce_kernel(DhArgs a, int grid_of_dh) {
    dh_add_pieces<S>(a, grid_of_dh, blockIdx.x, blockIdx.y);
}

// ------------------------------------------------------------------------------------------ dw
// dW is stored [d, V] or [V, d]; i is the index that is contiguous in memory (VD: the hidden dimension, else the
// vocabulary), so a lane's runs of 4 consecutive i are consecutive words of a row in either layout.
typedef float f32x4u __attribute__((ext_vector_type(4), aligned(4)));      // rows need not start on 16 bytes
typedef unsigned short u16x4u __attribute__((ext_vector_type(4), aligned(2)));
__device__ __forceinline__ u16x4u round4(const f32x4u& v) {
    u16x4u h;
#pragma unroll
    for (int r = 0; r < 4; ++r) h[r] = __builtin_bit_cast(unsigned short, (__bf16)v[r]);
    return h;
}
// 4 consecutive elements at offset `off` = j ld + i of dW, the first `n` of which exist (n <= 0: none):
// value = old * scale + sum if beta; to fp32 dW or, with a.dW16, rounded to it
struct DwOut {
    float* dW; bf16_t* dW16; int64_t ld; int nI, nJ; float scale; bool beta;
    __device__ __forceinline__ DwOut(const DwArgs& a, bool vd)
        : dW(a.dW), dW16(a.dW16), ld(vd ? a.d : a.V), nI((int)(vd ? a.d : a.V)), nJ((int)(vd ? a.V : a.d)),
          scale((a.beta && a.beta_scale) ? a.beta_scale[0] : 1.f), beta(a.beta != 0) {}
    __device__ __forceinline__ f32x4u old(int64_t off, int n) const {
        f32x4u c = {0.f, 0.f, 0.f, 0.f};
        if (!beta || n <= 0) return c;
        const float* p = dW + off;
        if (n >= 4) return *(const f32x4u*)p;
        for (int r = 0; r < n; ++r) c[r] = p[r];
        return c;
    }
    __device__ __forceinline__ void put(int64_t off, int n, const f32x4u& c, const f32x4u& sum) const {
        if (n <= 0) return;
        f32x4u o;
#pragma unroll
        for (int r = 0; r < 4; ++r) o[r] = c[r] * scale + sum[r];
        if (dW16) {
            const u16x4u h = round4(o);
            bf16_t* p = dW16 + off;
            if (n >= 4) { *(u16x4u*)p = h; return; }
            for (int r = 0; r < n; ++r) p[r] = h[r];
            return;
        }
        float* p = dW + off;
        if (n >= 4) { *(f32x4u*)p = o; return; }
        for (int r = 0; r < n; ++r) p[r] = o[r];
    }
};

// A tile of dW leaves through LDS: straight from the accumulators a store instruction would touch 32 rows, 32 bytes of
// each, and a tile of 256 KiB is a third of this kernel's time when there are few rows to contract.  Each wave owns a
// region of 32 rows j x IBW * 32 columns i.  Measured, d = 1536, V = 151936: added to a [V, d] gradient, about 2100 rows,
// 1.67 -> 1.06 ms; [d, V] without the addition, 13 000 rows, 2 % faster.  All waves must be done with both LDS stages (barrier) before the call.
template <class S>
__device__ __forceinline__ void dw_store(char* lds, const DwOut& out, int64_t i_tile, int64_t j_tile, const f32x16 (&acc)[S::WI][S::WJ]) {
    constexpr int fit = S::LDS_BYTES / S::NW / (32 * 128);                          // blocks of 32 x 32 floats per wave
    constexpr int pow2 = S::WI & -S::WI;                                            // largest power of two that divides WI
    constexpr int IBW = fit >= pow2 ? pow2 : fit >= pow2 / 2 ? pow2 / 2 : 1;
    constexpr int C = IBW * 8, R = 64 / C, T = 32 / R;                              // 16-byte chunks per row; rows per access
    static_assert(fit >= 1 && S::WI % IBW == 0 && C <= 64, "region");
    const Lane<S> L;
    constexpr int U = T < 8 ? T : 8;                                                // accesses in flight together
    char* region = lds + L.wave * (IBW * 32 * 128);
    const int c = L.lane % C, rr = L.lane / C;
    const int64_t step = R * out.ld;
    const bool inside = i_tile + S::BI <= out.nI && j_tile + S::BJ <= out.nJ;
#pragma unroll
    for (int jb = 0; jb < S::WJ; ++jb)
#pragma unroll
        for (int i0 = 0; i0 < S::WI; i0 += IBW) {
            char* row = region + L.lj * (C * 16);
#pragma unroll
            for (int ib = 0; ib < IBW; ++ib)
#pragma unroll
                for (int q = 0; q < 4; ++q)
                    *(float4*)(row + (((ib * 8 + q * 2 + L.hi) ^ (L.lj & (C - 1))) * 16)) =
                        make_float4(acc[i0 + ib][jb][q * 4], acc[i0 + ib][jb][q * 4 + 1], acc[i0 + ib][jb][q * 4 + 2],
                                    acc[i0 + ib][jb][q * 4 + 3]);
            const int j = (int)j_tile + (L.wave_j * S::WJ + jb) * 32 + rr, i = (int)i_tile + (L.wave_i * S::WI + i0) * 32 + c * 4;
            int64_t off = (int64_t)j * out.ld + i;
            auto value = [&](int t) {
                const int r = t * R + rr;
                const float4 v = *(const float4*)(region + r * (C * 16) + ((c ^ (r & (C - 1))) * 16));
                return f32x4u{v.x, v.y, v.z, v.w};
            };
            // rolled: the accumulators of the other blocks leave no registers for all of a region's rows at once
            if (inside) {   // no branch between the accesses of a batch, so that they are in flight together
#pragma unroll 1
                for (int t0 = 0; t0 < T; t0 += U, off += U * step) {
                    f32x4u cur[U];
                    if (out.beta) {
#pragma unroll
                        for (int t = 0; t < U; ++t) cur[t] = *(const f32x4u*)(out.dW + off + t * step);
                    } else {
#pragma unroll
                        for (int t = 0; t < U; ++t) cur[t] = f32x4u{0.f, 0.f, 0.f, 0.f};
                    }
#pragma unroll
                    for (int t = 0; t < U; ++t) cur[t] = cur[t] * out.scale + value(t0 + t);
                    if (out.dW16) {
#pragma unroll
                        for (int t = 0; t < U; ++t) __builtin_nontemporal_store(round4(cur[t]), (u16x4u*)(out.dW16 + off + t * step));
                    } else {
#pragma unroll
                        for (int t = 0; t < U; ++t) __builtin_nontemporal_store(cur[t], (f32x4u*)(out.dW + off + t * step));
                    }
                }
            } else {
#pragma unroll 1
                for (int t = 0; t < T; ++t, off += step) {
                    const int n = j + t * R < out.nJ ? out.nI - i : 0;
                    const f32x4u cur = out.old(off, n);
                    out.put(off, n, cur, value(t));
                }
            }
        }
}

template <class S, bool VD, bool DEEP = false>
__device__ __forceinline__ void dw_work(const DwArgs& a, int block, int grid, char* lds) {
    constexpr int WI = S::WI, WJ = S::WJ;
    const int tilesV = (int)(a.Vpad / (VD ? S::BJ : S::BI)), tilesD = (int)(a.dpadR / (VD ? S::BI : S::BJ));
    const int Mr = a.counts[CNT_MR];
    int64_t rows = (int64_t)Mr - a.m0;
    rows = rows < 0 ? 0 : (rows > a.Mc ? a.Mc : rows);
    if (rows == 0 && a.beta && !a.dW16) return;   // nothing to add
    const int x = block & 7, w = block >> 3;
    const int ktiles = (int)(rows / K_TILE);
    const TileShare sh(tilesV * tilesD, grid, ktiles, a.part != nullptr);
    const DwOut out(a, VD);
    auto contract = [&](const TileId& t, int k0, int k1, f32x16 (&acc)[WI][WJ]) {
        const bf16_t* z = a.dz + (int64_t)t.ti * (VD ? S::BJ : S::BI) + (int64_t)k0 * K_TILE * a.ldz;
        const bf16_t* h = a.Hc + (int64_t)t.tj * (VD ? S::BI : S::BJ) + (int64_t)k0 * K_TILE * a.ldH;
        const Operand oz{z, a.ldz, a.ldz * (K_TILE * 2)}, oh{h, a.ldH, a.ldH * (K_TILE * 2)};
        if constexpr (VD) mainloop<S, true, true, false>(oh, oz, k1 - k0, lds, acc);
        else if constexpr (DEEP) mainloop_kmajor32<S, 4>(z, a.ldz, h, a.ldH, (k1 - k0) * 2, lds, acc);
        else mainloop<S, true, true, false>(oz, oh, k1 - k0, lds, acc);
    };
    auto finish = [&](const TileId& t, const f32x16 (&acc)[WI][WJ]) {
        lds_barrier();   // every wave is done with both stages
        dw_store<S>(lds, out, (int64_t)(VD ? t.tj : t.ti) * S::BI, (int64_t)(VD ? t.ti : t.tj) * S::BJ, acc);
    };
    for (int round = 0; round < sh.full_rounds; ++round) {
        const TileId t = tile_of_vid((x * sh.full_rounds + round) * sh.wgs + w, tilesV, tilesD, a.gi);
        f32x16 acc[WI][WJ];
        contract(t, 0, ktiles, acc);
        finish(t, acc);
    }
    for (int pos = w; pos < sh.unit_share; pos += sh.wgs) {   // the last round (see TileShare)
        const int u = x * sh.unit_share + pos;
        if (u >= sh.rem * sh.segs) break;
        const int seg = u / sh.rem, tpos = u - seg * sh.rem;
        const TileId t = tile_of_vid(sh.full_rounds * grid + tpos, tilesV, tilesD, a.gi);
        f32x16 acc[WI][WJ];
        contract(t, (int)((int64_t)ktiles * seg / sh.segs), (int)((int64_t)ktiles * (seg + 1) / sh.segs), acc);
        if (sh.cut) store_unit<S>(a.part, u, acc); else finish(t, acc);
    }
}
template <class S, bool VD, bool DEEP = false>
__global__ __launch_bounds__(S::NT) void dw_kernel(DwArgs a) {
    extern __shared__ __attribute__((aligned(128))) char lds[];
    dw_work<S, VD, DEEP>(a, blockIdx.x, gridDim.x, lds);
}

// adds the pieces of the tiles that dw_work cut and stores them (see dh_add_pieces)
template <class S, bool VD>
__device__ __forceinline__ void dw_add_pieces(const DwArgs& a, int grid_of_dw, int tpos, int block) {
    const int tilesV = (int)(a.Vpad / (VD ? S::BJ : S::BI)), tilesD = (int)(a.dpadR / (VD ? S::BI : S::BJ));
    const int Mr = a.counts[CNT_MR];
    int64_t rows = (int64_t)Mr - a.m0;
    rows = rows < 0 ? 0 : (rows > a.Mc ? a.Mc : rows);
    const TileShare sh(tilesV * tilesD, grid_of_dw, (int)(rows / K_TILE), true);
    const int ib = block / S::WJ, jb = block % S::WJ;
    if (!sh.cut || tpos >= sh.rem) return;
    const TileId t = tile_of_vid(sh.full_rounds * grid_of_dw + tpos, tilesV, tilesD, a.gi);
    const DwOut out(a, VD);
    const Lane<S> L;
    const int i = (VD ? t.tj : t.ti) * S::BI + (L.wave_i * S::WI + ib) * 32 + L.hi * 4;
    const int j = (VD ? t.ti : t.tj) * S::BJ + (L.wave_j * S::WJ + jb) * 32 + L.lj;
    const int64_t off = (int64_t)j * out.ld + i;
    const int left = j < out.nJ ? out.nI - i : 0;
    f32x4u cur[4];
#pragma unroll
    for (int q = 0; q < 4; ++q) cur[q] = out.old(off + q * 8, left - q * 8);
    float sum[16];
    sum_units<S>(a.part, sh, tpos, ib, jb, sum);
#pragma unroll
    for (int q = 0; q < 4; ++q)
        out.put(off + q * 8, left - q * 8, cur[q], f32x4u{sum[q * 4], sum[q * 4 + 1], sum[q * 4 + 2], sum[q * 4 + 3]});
}

template <class S, bool VD>
__global__ __launch_bounds__(S::NT) void dw_reduce_kernel(DwArgs a, int grid_of_dw) {
    dw_add_pieces<S, VD>(a, grid_of_dw, blockIdx.x, blockIdx.y);
}

// dHidden and dW of a small batch side by side: neither fills the chip for longer than it takes to get going, and they do
// not depend on each other.  The first grid_dh workgroups are dHidden's; of their second passes in one launch (dh_dw_reduce_kernel) the
// first tiles_dh columns of the grid.  d = 256, V = 4096, about 1800 tokens: 17.1 and 16.6 us, second passes 7.2 and 6.4, one after the other;
// 20.8 and 9.3 together.
template <class S, int WM, bool VD>
__global__ __launch_bounds__(S::NT, 2) void dh_dw_kernel(DhArgs h, DwArgs w, int grid_dh) {
    extern __shared__ __attribute__((aligned(128))) char lds[];
    if ((int)blockIdx.x < grid_dh) dh_work<S, WM>(h, blockIdx.x, grid_dh, lds);
    else dw_work<S, VD>(w, blockIdx.x - grid_dh, gridDim.x - grid_dh, lds);
}
template <class S, bool VD>
__global__ __launch_bounds__(S::NT) void dh_dw_reduce_kernel(DhArgs h, DwArgs w, int grid_dh, int grid_dw, int tiles_dh) {
    if ((int)blockIdx.x < tiles_dh) dh_add_pieces<S>(h, grid_dh, blockIdx.x, blockIdx.y);
    else dw_add_pieces<S, VD>(w, grid_dw, blockIdx.x - tiles_dh, blockIdx.y);
}

// dz[row][tok_row] += g: the one-hot part of dz = g (onehot - p)
__global__ void token_onehot_kernel(bf16_t* __restrict__ dz, int64_t ldz, int64_t m0, int64_t rows,
                                    const int32_t* __restrict__ tokc, const float* __restrict__ rowg, float inv_temp,
                                    const int32_t* __restrict__ counts) {
    const int64_t jl = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    const int64_t j = m0 + jl;
    if (jl >= rows || j >= counts[CNT_M]) return;
    bf16_t* p = dz + jl * ldz + tokc[j];
    const float cur = (float)__builtin_bit_cast(__bf16, *p);
    const __bf16 r = (__bf16)(cur + rowg[j] * inv_temp);
    *p = __builtin_bit_cast(bf16_t, r);
}

// After a forward that stored u = exp(z - r) (see fwd_lse_kernel), with lse and the row coefficients
// g known: dz[j][v] = (g_j / temperature) (onehot_y[v] - p_v) = c_j u'[j][v], with the row factor
// c_j = -(g_j / temperature) exp(r_j - lse_j) and u' = u except at the sampled token, where
// u'[j][y] = exp(lse_j - r_j) (p_y - 1).  One wave per token row writes c_j (0 past the last
// token), replaces that one element, and scales the row of the packed hidden copy by c_j: dW
// contracts over token rows, so there the factor has to sit on an operand (dHidden applies it to
// its accumulators).  |lse - r| is clamped at 80 (sets RAPID_STATUS_LOGIT_RANGE: such a row's
// gradient is truncated).
__global__ __launch_bounds__(256) void cache_finish_kernel(bf16_t* __restrict__ u, int64_t ldz, bf16_t* __restrict__ Hc,
                                                           int64_t ldk, const int32_t* __restrict__ tokc,
                                                           const float* __restrict__ zy, const float* __restrict__ refz,
                                                           const float* __restrict__ lse_c, const float* __restrict__ rowg,
                                                           float inv_temp, const int32_t* __restrict__ counts,
                                                           int64_t row0, float* __restrict__ rowc,
                                                           int32_t* __restrict__ dev_status) {
    const int64_t j = row0 + (int64_t)blockIdx.x * 4 + (threadIdx.x >> 6);
    const int lane = threadIdx.x & 63;
    const int M = counts[CNT_M], Mr = counts[CNT_MR];
    if (j >= Mr) return;
    float c = 0.f;
    if (j < M) {
        const float lse = lse_c[j];
        float a = lse - refz[j];
        if (!(fabsf(a) <= 80.f)) {
            a = a > 0.f ? 80.f : -80.f;
            if (lane == 0 && dev_status) atomicOr(dev_status, RAPID_STATUS_LOGIT_RANGE);
        }
        c = -rowg[j] * inv_temp * __expf(-a);
        if (lane == 0) {
            const __bf16 r = (__bf16)(__expf(a) * expm1f(zy[j] - lse));   // exp(lse - r) (p_y - 1)
            u[(j - row0) * ldz + tokc[j]] = __builtin_bit_cast(bf16_t, r);
        }
    }
    if (lane == 0) rowc[j] = c;
    uint4* row = (uint4*)(Hc + j * ldk);
    for (int c8 = lane; c8 < ldk / 8; c8 += 64) {
        const uint4 in = row[c8];
        const uint32_t w[4] = {in.x, in.y, in.z, in.w};
        float o[8];
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            o[2 * e] = c * __builtin_bit_cast(float, w[e] << 16);
            o[2 * e + 1] = c * __builtin_bit_cast(float, w[e] & 0xffff0000u);
        }
        const uint2 a0 = pack_bf16x4(o[0], o[1], o[2], o[3]), a1 = pack_bf16x4(o[4], o[5], o[6], o[7]);
        row[c8] = make_uint4(a0.x, a0.y, a1.x, a1.y);
    }
}

// Lets `kernel` use `bytes` of dynamic LDS: once per kernel and device (the attribute belongs to the
// device's copy of the function), not once per launch.  One static bit mask per kernel.
template <auto kernel>
void allow_lds(int bytes) {
    static std::atomic<uint64_t> done{0};
    int dev = 0;
    (void)hipGetDevice(&dev);
    const uint64_t bit = 1ull << (dev & 63);
    if (done.load(std::memory_order_acquire) & bit) return;
    if (hipFuncSetAttribute((const void*)kernel, hipFuncAttributeMaxDynamicSharedMemorySize, bytes) == hipSuccess)
        done.fetch_or(bit, std::memory_order_release);
}

// waves per workgroup: 4 (2 x 2 of 128 x 128), 8 (2 x 4 of 128 x 64) or 16; 0 = each kernel's own
// default: 8 for the logits kernels and dW, 4 for dHidden (measured: its long K loop gains more from
// the 4-wave tile's third fewer LDS reads than it loses in latency hiding)
std::atomic<int> g_waves{0};
static int waves_for(int own_default) {
    const int w = g_waves.load();
    return w ? w : own_default;
}

using G4 = Geo<2, 2, 4, 4>;        // 256 x 256, 4 waves
using G4_I128 = Geo<2, 2, 2, 4>;   // 128 x 256
using G4_J128 = Geo<2, 2, 4, 2>;   // 256 x 128
using G8 = Geo<2, 4, 4, 2>;        // 256 x 256, 8 waves
using G8_I128 = Geo<2, 4, 2, 2>;   // 128 x 256
using G8_J128 = Geo<2, 4, 4, 1>;   // 256 x 128
using G16 = Geo<2, 8, 4, 1>;       // 256 x 256, 16 waves of 128 x 32
using G16_I128 = Geo<2, 8, 2, 1>;  // 128 x 256
using G16_J128 = Geo<4, 4, 2, 1>;  // 256 x 128
// hidden dimension in tiles of 224 or 192 (see hidden_tile)
using G4_I224 = Geo<1, 4, 7, 2>;   // 224 x 256, waves of 224 x 64
using G4_128 = Geo<2, 2, 2, 2>;    // 128 x 128, for a launch with little to contract
using G4_I192 = Geo<2, 2, 3, 4>;   // 192 x 256, waves of 96 x 128
using G4_J192 = Geo<2, 2, 4, 3>;   // 256 x 192

template <class S, int WM, bool DEEP = false>
void launch_fwd_lse_t(const FwdArgs& a, hipStream_t st) {
    constexpr int bytes = DEEP ? deep_lds_bytes<S>() : S::LDS_BYTES;
    const unsigned grid = grid_for(a.tilesV, a.tilesM * (256 / S::BJ));
    if (a.zc) {
        allow_lds<&fwd_lse_kernel<S, true, WM, DEEP>>(bytes);
        fwd_lse_kernel<S, true, WM, DEEP><<<grid, S::NT, bytes, st>>>(a);
    } else {
        allow_lds<&fwd_lse_kernel<S, false, WM, DEEP>>(bytes);
        fwd_lse_kernel<S, false, WM, DEEP><<<grid, S::NT, bytes, st>>>(a);
    }
}
template <class S, int WM>
void launch_dz_t(const DzArgs& a, hipStream_t st) {
    allow_lds<&dz_kernel<S, WM>>(S::LDS_BYTES);
    dz_kernel<S, WM><<<grid_for(a.tilesV, a.tilesM * (256 / S::BJ)), S::NT, S::LDS_BYTES, st>>>(a);
}
// workgroups of a launch that may cut tiles: as many as the chip holds
template <class S>
unsigned grid_of_cut() {
    return (unsigned)(g_num_cu.load() / 8 * 8 * (2 * S::LDS_BYTES <= 160 * 1024 ? 2 : 1));
}
template <class S, int WM>
void launch_dh_t(const DhArgs& a, hipStream_t st) {
    allow_lds<&dh_kernel<S, WM>>(S::LDS_BYTES);
    const int tilesD = (int)(a.dpadR / S::BI);
    DhArgs b = a;
    if ((size_t)MAX_UNITS * S::BI * S::BJ * 4 > a.part_bytes) b.part = nullptr;
    // with scratch for cut tiles a launch of few tiles takes the whole chip as well
    const unsigned grid = b.part ? grid_of_cut<S>() : grid_for(tilesD, a.tilesM * (256 / S::BJ));
    dh_kernel<S, WM><<<grid, S::NT, S::LDS_BYTES, st>>>(b);
    const int64_t tiles = (int64_t)tilesD * a.tilesM * (256 / S::BJ);
    if (b.part) dh_reduce_kernel<S><<<dim3((unsigned)(tiles < grid ? tiles : grid), S::WI * S::WJ), S::NT, 0, st>>>(b, (int)grid);
}
template <class S, bool VD, bool DEEP = false>
void launch_dw_t(const DwArgs& a, hipStream_t st) {
    allow_lds<&dw_kernel<S, VD, DEEP>>(S::LDS_BYTES);
    const int64_t tilesV = a.Vpad / (VD ? S::BJ : S::BI), tilesD = a.dpadR / (VD ? S::BI : S::BJ), tiles = tilesV * tilesD;
    DwArgs b = a;
    if ((size_t)MAX_UNITS * S::BI * S::BJ * 4 > a.part_bytes) b.part = nullptr;
    const unsigned grid = b.part ? grid_of_cut<S>() : grid_for((int)tilesV, (int)tilesD);
    dw_kernel<S, VD, DEEP><<<grid, S::NT, S::LDS_BYTES, st>>>(b);
    if (b.part && tiles % grid != 0)
        dw_reduce_kernel<S, VD><<<dim3((unsigned)(tiles % grid), S::WI * S::WJ), S::NT, 0, st>>>(b, (int)grid);
}

}  // namespace

size_t dh_part_bytes() { return (size_t)MAX_UNITS * 256 * 256 * 4; }
bool default_waves() { return g_waves.load() == 0; }
void set_waves_per_workgroup(int n) { g_waves = (n == 4 || n == 8 || n == 16) ? n : 0; }
void set_cu_count(int n) { g_num_cu = n >= 8 ? n : 8; }


void launch_block_w32(const bf16_t* Wvd, int64_t ldk, bf16_t* out, int64_t Vpad, int64_t dpad, hipStream_t st) {
    const int64_t chunks = Vpad * (dpad / 32) * 4;
    block_w32_kernel<<<(unsigned)((chunks + 255) / 256), 256, 0, st>>>(Wvd, ldk, out, Vpad, dpad);
}
// Logits of a small batch on a small head: tiles of half the token rows where the whole ones would leave half the chip
// without any; same bits (a tile's columns and its order of summation stay the same).
static bool half_tiles(int tilesV, int tilesM) { return (int64_t)tilesV * tilesM <= g_num_cu.load() / 2; }
void launch_fwd_lse(const FwdArgs& a, hipStream_t st) {
    if (a.WvdB && a.k32_mode == 3) {   // one workgroup of 4 waves per CU, K steps of 32 requested three steps ahead
        const unsigned grid = grid_for(a.tilesV, a.tilesM);
        if (a.zc) {
            allow_lds<&fwd_lse2_kernel<Fwd4, true>>(Fwd4::LDS_BYTES);
            fwd_lse2_kernel<Fwd4, true><<<grid, 256, Fwd4::LDS_BYTES, st>>>(a);
        } else {
            allow_lds<&fwd_lse2_kernel<Fwd4, false>>(Fwd4::LDS_BYTES);
            fwd_lse2_kernel<Fwd4, false><<<grid, 256, Fwd4::LDS_BYTES, st>>>(a);
        }
        return;
    }
    if (a.WvdB && a.k32_mode == 2) {   // one workgroup of 8 waves per CU, K steps of 32 requested three steps ahead
        const unsigned grid = grid_for(a.tilesV, a.tilesM);
        if (a.zc) {
            allow_lds<&fwd_lse2_kernel<Fwd3, true>>(Fwd3::LDS_BYTES);
            fwd_lse2_kernel<Fwd3, true><<<grid, 512, Fwd3::LDS_BYTES, st>>>(a);
        } else {
            allow_lds<&fwd_lse2_kernel<Fwd3, false>>(Fwd3::LDS_BYTES);
            fwd_lse2_kernel<Fwd3, false><<<grid, 512, Fwd3::LDS_BYTES, st>>>(a);
        }
        return;
    }
    if (a.WvdB) {   // two workgroups of 4 waves per CU on 256 x 128 tiles
        const int ids = ids_for(a.tilesV, a.tilesM * 2), slots = g_num_cu.load() / 8 * 8 * 2;
        const unsigned grid = (unsigned)(ids < slots ? ids : slots);
        if (a.zc) {
            allow_lds<&fwd_lse2_kernel<Fwd2, true>>(Fwd2::LDS_BYTES);
            fwd_lse2_kernel<Fwd2, true><<<grid, 256, Fwd2::LDS_BYTES, st>>>(a);
        } else {
            allow_lds<&fwd_lse2_kernel<Fwd2, false>>(Fwd2::LDS_BYTES);
            fwd_lse2_kernel<Fwd2, false><<<grid, 256, Fwd2::LDS_BYTES, st>>>(a);
        }
        return;
    }
    if (half_tiles(a.tilesV, a.tilesM)) {
        if (a.w.mode == W_VD) { launch_fwd_lse_t<G8_J128, W_VD>(a, st); return; }
        if (a.w.mode == W_DV) { launch_fwd_lse_t<G8_J128, W_DV>(a, st); return; }
        if (waves_for(8) == 8) { launch_fwd_lse_t<G8_J128, W_PACKED>(a, st); return; }
    }
    // W's steps two ahead (mainloop_deep) where the few rows leave little else to do; a short tile is over before it pays,
    // the steps past its end are fetched for nothing.  Calls at V = 151936, without and with it: 100 tokens at d = 512 64 -> 59 us, d = 1024
    // 105 -> 96, d = 1536 147 -> 134; 290 tokens (two row tiles) d = 512 86 -> 90, d = 768 109 -> 111, d = 1024 144 -> 137,
    // d = 1536 208 -> 195; 900 tokens as before.
    if (a.tilesM <= 2 && a.dpad >= (int64_t)a.tilesM * 8 * K_TILE) {
        if (a.w.mode == W_VD) { launch_fwd_lse_t<G8, W_VD, true>(a, st); return; }
        if (a.w.mode == W_DV) { launch_fwd_lse_t<G8, W_DV, true>(a, st); return; }
    }
    if (a.w.mode == W_VD) { launch_fwd_lse_t<G8, W_VD>(a, st); return; }
    if (a.w.mode == W_DV) { launch_fwd_lse_t<G8, W_DV>(a, st); return; }
    const int w = waves_for(8);
    if (w == 16) launch_fwd_lse_t<G16, W_PACKED>(a, st);
    else if (w == 8) launch_fwd_lse_t<G8, W_PACKED>(a, st);
    else launch_fwd_lse_t<G4, W_PACKED>(a, st);
}
int fwd_slots_per_tile() { return 2; }

void launch_dz(const DzArgs& a, hipStream_t st) {
    const int w = waves_for(8);
    const bool half = half_tiles(a.tilesV, a.tilesM);
    if (half && a.w.mode == W_VD) launch_dz_t<G8_J128, W_VD>(a, st);
    else if (half && a.w.mode == W_DV) launch_dz_t<G8_J128, W_DV>(a, st);
    else if (half && w == 8) launch_dz_t<G8_J128, W_PACKED>(a, st);
    else if (a.w.mode == W_VD) launch_dz_t<G8, W_VD>(a, st);
    else if (a.w.mode == W_DV) launch_dz_t<G8, W_DV>(a, st);
    else if (w == 16) launch_dz_t<G16, W_PACKED>(a, st);
    else if (w == 8) launch_dz_t<G8, W_PACKED>(a, st);
    else launch_dz_t<G4, W_PACKED>(a, st);
    const int64_t rows = (int64_t)a.tilesM * 256;
    token_onehot_kernel<<<(unsigned)((rows + 255) / 256), 256, 0, st>>>(a.dz, a.ldz, a.m0, rows, a.tokc, a.rowg,
                                                                      a.inv_temp, a.counts);
}

void launch_cache_finish(bf16_t* u, int64_t ldz, bf16_t* Hc, int64_t ldk, const int32_t* tokc,
                         const float* zy, const float* refz, const float* lse_c, const float* rowg, float inv_temp,
                         const int32_t* counts, int64_t row0, int64_t rows_max, float* rowc, int32_t* dev_status,
                         hipStream_t st) {
    if (rows_max <= 0) return;
    cache_finish_kernel<<<(unsigned)((rows_max + 3) / 4), 256, 0, st>>>(u, ldz, Hc, ldk, tokc, zy, refz, lse_c, rowg,
                                                                        inv_temp, counts, row0, rowc, dev_status);
}
// A launch whose contraction is short when it is spread over the whole chip leaves 256 KiB of pieces per workgroup behind,
// and passing them through memory twice takes longer than the products do: tiles of 128 x 128 then, which are cut into
// fewer segments (two workgroups share a compute unit).  Measured, dHidden and dW with both tiles, `most` = K steps per
// compute unit with tiles of 256 (upper bounds of the batch): d = 256, V = 4096 (3 steps) 35 -> 26 us and 31 -> 25 us;
// d = 1024, V = 2000 (8) 40 / 40 and 40 -> 32; d = 128, V = 30000 (13) 56 -> 54 and 39 -> 31; d = 768, V = 20000 (15) 56 -> 51, but
// dW, whose 237 tiles fill the chip as they are, 43 -> 47; d = 512, V = 16000 (29) 71 -> 73 and 72 -> 63.
static bool few_steps(int64_t tiles, int64_t ksteps, int most) { return tiles * ksteps <= (int64_t)most * g_num_cu.load(); }
static bool short_dh_steps(int64_t d, int64_t tilesM, int64_t V) { return few_steps((d + 255) / 256 * tilesM, (V + K_TILE - 1) / K_TILE, 16); }
// a packed copy has to be laid out for it, and, with no bound on the rows as reading in place has, half the chip has to be without tiles
bool short_dh_packed(int64_t d, int64_t tilesM, int64_t V) {
    return default_waves() && (d + 255) / 256 * tilesM <= g_num_cu.load() / 2 && short_dh_steps(d, tilesM, V);
}
static bool short_dh(const DhArgs& a) {
    if (!a.part) return false;
    return a.w.mode != W_PACKED ? short_dh_steps(a.d, a.tilesM, a.w.V) : a.dtile == 128 && short_dh_packed(a.d, a.tilesM, a.w.V);
}
static bool short_dw(const DwArgs& a) {
    const int64_t tiles = (a.d + 255) / 256 * (a.Vpad / 256);
    return default_waves() && a.part && tiles <= g_num_cu.load() / 2 && few_steps(tiles, a.Mc / K_TILE, 32);
}
void launch_dh(const DhArgs& a, hipStream_t st) {
    const int w = waves_for(4);
    const bool d256 = a.dtile == 256;   // else 128, or 192 or 224 in the default geometry
    if (short_dh(a)) {
        DhArgs b = a;
        b.dpadR = round_up(a.d, 128);
        a.w.mode == W_VD ? launch_dh_t<G4_128, W_VD>(b, st) : a.w.mode == W_DV ? launch_dh_t<G4_128, W_DV>(b, st) : launch_dh_t<G4_128, W_PACKED>(b, st);
        return;
    }
    if (a.dtile == 224)
        a.w.mode == W_VD ? launch_dh_t<G4_I224, W_VD>(a, st) : a.w.mode == W_DV ? launch_dh_t<G4_I224, W_DV>(a, st) : launch_dh_t<G4_I224, W_PACKED>(a, st);
    else if (a.dtile == 192)
        a.w.mode == W_VD ? launch_dh_t<G4_I192, W_VD>(a, st) : a.w.mode == W_DV ? launch_dh_t<G4_I192, W_DV>(a, st) : launch_dh_t<G4_I192, W_PACKED>(a, st);
    else if (a.w.mode == W_VD) d256 ? launch_dh_t<G4, W_VD>(a, st) : launch_dh_t<G4_I128, W_VD>(a, st);
    else if (a.w.mode == W_DV) d256 ? launch_dh_t<G4, W_DV>(a, st) : launch_dh_t<G4_I128, W_DV>(a, st);
    else if (w == 16) d256 ? launch_dh_t<G16, W_PACKED>(a, st) : launch_dh_t<G16_I128, W_PACKED>(a, st);
    else if (w == 8) d256 ? launch_dh_t<G8, W_PACKED>(a, st) : launch_dh_t<G8_I128, W_PACKED>(a, st);
    else d256 ? launch_dh_t<G4, W_PACKED>(a, st) : launch_dh_t<G4_I128, W_PACKED>(a, st);
}

std::atomic<int> g_dw_deep{0};
void set_dw_deep(int on) { g_dw_deep = on ? 1 : 0; }
void launch_dw(const DwArgs& a, hipStream_t st) {
    const int w = waves_for(8);
    const bool d256 = a.dtile == 256;   // else 128, or 192 in the default geometry
    if (short_dw(a)) {
        DwArgs b = a;
        b.dpadR = round_up(a.d, 128);
        a.w_layout == RAPID_W_VD ? launch_dw_t<G4_128, true>(b, st) : launch_dw_t<G4_128, false>(b, st);
        return;
    }
    if (a.dtile == 192) { a.w_layout == RAPID_W_VD ? launch_dw_t<G4_I192, true>(a, st) : launch_dw_t<G4_J192, false>(a, st); return; }
    if (a.w_layout == RAPID_W_VD) {
        if (w == 16) d256 ? launch_dw_t<G16, true>(a, st) : launch_dw_t<G16_I128, true>(a, st);
        else if (w == 8) d256 ? launch_dw_t<G8, true>(a, st) : launch_dw_t<G8_I128, true>(a, st);
        else d256 ? launch_dw_t<G4, true>(a, st) : launch_dw_t<G4_I128, true>(a, st);
        return;
    }
    if (g_dw_deep.load() && w == 8) {   // K steps of 32 rows, requests three steps ahead
        d256 ? launch_dw_t<G8, false, true>(a, st) : launch_dw_t<G8_J128, false, true>(a, st);
        return;
    }
    if (w == 16) d256 ? launch_dw_t<G16, false>(a, st) : launch_dw_t<G16_J128, false>(a, st);
    else if (w == 8) d256 ? launch_dw_t<G8, false>(a, st) : launch_dw_t<G8_J128, false>(a, st);
    else d256 ? launch_dw_t<G4, false>(a, st) : launch_dw_t<G4_J128, false>(a, st);
}

template <int WM, bool VD>
static void launch_dh_dw_t(const DhArgs& h, const DwArgs& w, hipStream_t st) {
    using S = G4_128;
    allow_lds<&dh_dw_kernel<S, WM, VD>>(S::LDS_BYTES);
    const unsigned each = grid_of_cut<S>() / 2;
    const int64_t tiles_dh = h.dpadR / S::BI * h.tilesM * (256 / S::BJ), tiles_dw = w.Vpad / S::BI * (w.dpadR / S::BJ) % each;
    const unsigned cols_dh = (unsigned)(tiles_dh < each ? tiles_dh : each);
    dh_dw_kernel<S, WM, VD><<<2 * each, S::NT, S::LDS_BYTES, st>>>(h, w, (int)each);
    dh_dw_reduce_kernel<S, VD><<<dim3(cols_dh + (unsigned)tiles_dw, S::WI * S::WJ), S::NT, 0, st>>>(h, w, (int)each, (int)each, (int)cols_dh);
}
// scratch that the pieces of one of the two take
constexpr size_t PAIR_PART = (size_t)MAX_UNITS * G4_128::BI * G4_128::BJ * 4;
// where both take tiles of 128 x 128, two of whose workgroups share a compute unit: one of each
bool dh_dw_together(const DhArgs& h, const DwArgs& w) { return short_dh(h) && short_dw(w) && h.part_bytes >= 2 * PAIR_PART && h.part == w.part; }
void launch_dh_dw(const DhArgs& h, const DwArgs& w, hipStream_t st) {
    DhArgs a = h;
    DwArgs b = w;
    a.dpadR = b.dpadR = round_up(h.d, 128);
    b.part = w.part + PAIR_PART / 4;
    // dW has the layout of the head that dHidden reads in place
    if (h.w.mode == W_VD) launch_dh_dw_t<W_VD, true>(a, b, st);
    else if (h.w.mode == W_DV) launch_dh_dw_t<W_DV, false>(a, b, st);
    else w.w_layout == RAPID_W_VD ? launch_dh_dw_t<W_PACKED, true>(a, b, st) : launch_dh_dw_t<W_PACKED, false>(a, b, st);
}

}  // namespace rapid
