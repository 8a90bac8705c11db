// lagom_gemm: C[M,N] = A[M,K] . B, bf16 inputs, fp32 accumulation on the gfx950 matrix
// cores, the computation whose slow-down the overlap model describes (Sec. 3.2, Fig. 3).
//
// Tiling: one workgroup of 256 threads (4 wavefronts, 2 x 2) owns a 256 x 256 tile of C and
// walks K in steps of 64; each wavefront owns a 128 x 128 block, i.e. 256 fp32 accumulators per
// lane (the whole AGPR file), so one workgroup is resident per compute unit.  Products that at
// most 256 tiles of 128 x 128 or of 256 x 128 cover use those instead: 256 x 256 tiles would
// leave compute units idle (see the small-tile kernels below); still smaller ones split K over a
// workgroup's wavefronts (see "few tiles").
// Workgroup ids are remapped so that the workgroups of one XCD (ids equal modulo 8) cover a
// compact block of tiles and share A/B panels in that XCD's L2.
//
// Fast kernel (64 <= K <= 2^22; described for B stored [N,K] and K a multiple of 64):
//   * v_mfma_f32_16x16x32_bf16, 8 x 8 MFMA tiles per wavefront.  Under random operands the chip
//     is power limited, and this shape costs less energy per flop than 32x32x16: a register-only
//     loop sustains 86 % of the 2.5 PFLOP/s peak at 2.14 GHz with it against 77 % at 1.89 GHz.
//     The MFMAs are inline asm with the accumulators pinned to AGPRs (with the builtin the
//     register allocator copies the 64 accumulator quads around on every iteration).
//   * A and B tiles go from global memory straight into LDS (global_load_lds_dwordx4, scalar base
//     + 32-bit lane offset).  LDS holds five 32 KiB slots used as a ring A0,B0,A1,B1,A2,...: while
//     step kt multiplies the tiles in two slots, the loads of B(kt+1), A(kt+2) and B(kt+2) are in
//     flight, issued so that every load has at least half a step to land before it is needed.
//   * One side instruction per MFMA: a 16x16x32 MFMA keeps the matrix core busy for 16 cycles and
//     takes 4 to issue, so one load, M0 write or ds_read issued right behind it costs nothing,
//     whereas several in a row leave the matrix core idle (measured: 2720 -> 2370 cycles per
//     K-step against 2048 of pure MFMA time).
//   * LDS rows are 128 bytes (64 bf16 = eight 16-byte groups); group g of row r is stored at
//     position g ^ ((r >> 1) & 7).  LDS on gfx950 has 64 banks of 4 bytes, so two rows share a
//     bank line; this swizzle makes the 16 lanes of a ds_read_b128 phase hit 16 distinct
//     16-byte bank groups.
//   * Operand fragments are double buffered in registers (two 32-wide k-slices of 8 + 8
//     fragments); the steady-state loop is branch-free (the last two K-steps, which load nothing
//     or only B, are peeled).
//   * The MFMA is issued with the B fragment as first operand, so a lane ends up holding four
//     consecutive columns of one row of C; results are staged through LDS and written to HBM as
//     16-byte vectors, whole rows of the wavefront's block contiguous.
//   * B stored [K,N] (N a multiple of 8, N <= 2^23) runs the same kernel: the B tile lies in LDS as
//     in memory, 64 rows (k) of 256 columns, and ds_read_b64_tr_b16 transposes while reading: two
//     reads give a lane the 8 consecutive k of one column.  48 instead of 32 LDS reads per K-step,
//     still one per MFMA.
//   * K not a multiple of 64 (kernels of their own): the last step takes the last 64 columns, of which
//     the loop has multiplied some already, and clears those in its operand fragments (in both, so
//     that no stray NaN meets a zero).  Its loads are in flight like any other step's; the rest of K
//     fetched behind the loop with guarded loads cost a memory latency per tile: 4096 x 4096 x 184
//     14.7 -> 13.4 us, x 72 12.7 -> 12.0, 4096 x 4352 x 2056 76.4 -> 74.0.
// General kernel (any K multiple of 8, either B layout, v_mfma_f32_32x32x16_bf16): tiles are
// fetched into registers with bounds checks and zero fill, then stored to LDS ([K,N]: 8 x 8
// blocks transposed in registers first); single buffered.  Slower; used for K < 64 and beyond
// the fast kernel's size limits.
#include <hip/hip_runtime.h>
#include <atomic>
#include <type_traits>
#include "common.h"

namespace {

constexpr int BM = 256, BN = 256, BK = 64, THREADS = 256;
constexpr int VEC_PER_THREAD = (BM * BK / 8) / THREADS;  // 16-byte vectors of one operand tile per thread = 8

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float f32x16 __attribute__((ext_vector_type(16)));
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));

struct GemmArgs {
    const uint16_t* A;
    const uint16_t* B;
    void* C;
    int64_t M, N, K;
    int32_t tiles_m, tiles_n;
    int32_t rows;               // of the blocks that the list of tiles runs through (tile_in_list); 0: the list in columns of 8, XCDs in turn
};

__device__ __forceinline__ uint32_t bf16_round_bits(float f) {
    const uint32_t u = __float_as_uint(f);
    const uint32_t upper = u >> 16, lower = u & 0xffffu;
    const uint32_t r = upper + ((lower > 0x8000u || (lower == 0x8000u && (upper & 1u))) ? 1u : 0u);
    return ((u & 0x7fffffffu) > 0x7f800000u) ? (upper | 0x0040u) : r;
}

// index (in 16-byte units) of group `cg` of row `row` in a swizzled [rows][8] tile
__device__ __forceinline__ int swz(int row, int cg) { return row * 8 + (cg ^ (row & 7)); }

// Workgroup id -> (tile_m, tile_n).  Hardware deals consecutive ids round-robin to the 8 XCDs: XCD x is given the x-th eighth
// of the list of tiles, and the list runs down columns of `rows` tile-rows, so that what an XCD works on at a time is a block of
// tiles that shares A and B panels in its L2.
__device__ __forceinline__ void tile_in_list(int lin, int tiles_m, int tiles_n, int rows, int* tm, int* tn) {
    const int per_group = rows * tiles_n;
    const int grp = lin / per_group;
    const int first_m = grp * rows;
    const int high = tiles_m - first_m < rows ? tiles_m - first_m : rows;
    const int in = lin - grp * per_group;
    *tm = first_m + in % high;
    *tn = in / high;
}
__device__ __forceinline__ void tile_of(int id, const GemmArgs& p, int* tm, int* tn) {
    const int total = p.tiles_m * p.tiles_n, x = id & 7, over = total & 7;
    const int lin = p.rows ? x * (total >> 3) + (x < over ? x : over) + (id >> 3) : id;
    tile_in_list(lin, p.tiles_m, p.tiles_n, p.rows ? p.rows : 8, tm, tn);
}

template <bool B_NK, bool OUT_BF16>
__global__ void __launch_bounds__(THREADS) gemm_bf16_general_kernel(const GemmArgs p) {
    __shared__ u32x4 sA[BM * 8];
    __shared__ u32x4 sB[BN * 8];

    const int tid = threadIdx.x;
    const int lane = tid & 63;
    const int wave = tid >> 6;
    const int wm = wave >> 1, wn = wave & 1;
    int tm, tn;
    tile_of(blockIdx.x, p, &tm, &tn);
    const int64_t m0 = (int64_t)tm * BM, n0 = (int64_t)tn * BN;
    const int64_t M = p.M, N = p.N, K = p.K;

    f32x16 acc[4][4];
#pragma unroll
    for (int i = 0; i < 4; ++i)
#pragma unroll
        for (int j = 0; j < 4; ++j)
#pragma unroll
            for (int v = 0; v < 16; ++v) acc[i][j][v] = 0.0f;

    u32x4 ra[VEC_PER_THREAD], rb[VEC_PER_THREAD];
    const u32x4 zero = {0u, 0u, 0u, 0u};

    auto fetch = [&](int64_t k0) {
#pragma unroll
        for (int i = 0; i < VEC_PER_THREAD; ++i) {
            const int id = tid + THREADS * i;
            const int row = id >> 3, cg = id & 7;
            const int64_t gm = m0 + row, gk = k0 + cg * 8;
            ra[i] = (gm < M && gk < K) ? *reinterpret_cast<const u32x4*>(p.A + gm * K + gk) : zero;
        }
        if (B_NK) {
#pragma unroll
            for (int i = 0; i < VEC_PER_THREAD; ++i) {
                const int id = tid + THREADS * i;
                const int row = id >> 3, cg = id & 7;
                const int64_t gn = n0 + row, gk = k0 + cg * 8;
                rb[i] = (gn < N && gk < K) ? *reinterpret_cast<const u32x4*>(p.B + gn * K + gk) : zero;
            }
        } else {
#pragma unroll
            for (int i = 0; i < VEC_PER_THREAD; ++i) {   // B[K,N]: a thread holds an 8 (k) x 8 (n) block
                const int64_t gk = k0 + (tid & 7) * 8 + i, gn = n0 + (tid >> 3) * 8;
                rb[i] = (gk < K && gn < N) ? *reinterpret_cast<const u32x4*>(p.B + gk * N + gn) : zero;
            }
        }
    };
    auto stage = [&]() {
#pragma unroll
        for (int i = 0; i < VEC_PER_THREAD; ++i) {
            const int id = tid + THREADS * i;
            sA[swz(id >> 3, id & 7)] = ra[i];
        }
        if (B_NK) {
#pragma unroll
            for (int i = 0; i < VEC_PER_THREAD; ++i) {
                const int id = tid + THREADS * i;
                sB[swz(id >> 3, id & 7)] = rb[i];
            }
        } else {
            // Transpose the 8 x 8 block in registers: column e of the block becomes one 16-byte group
            // (8 consecutive k of row n) of the [n][k] tile.  v_perm_b32 picks the low or the high halves
            // of two rows' words.  The 8 lanes tid & 7 of a row n write its 8 different groups.
            const int kb = tid & 7, nv = tid >> 3;
#pragma unroll
            for (int e = 0; e < 8; ++e) {
                u32x4 col;
#pragma unroll
                for (int j = 0; j < 4; ++j)
                    col[j] = __builtin_amdgcn_perm(rb[2 * j + 1][e >> 1], rb[2 * j][e >> 1],
                                                   (e & 1) ? 0x07060302u : 0x05040100u);
                sB[swz(nv * 8 + e, kb)] = col;
            }
        }
    };

    const int64_t ksteps = (K + BK - 1) / BK;
    fetch(0);
    stage();
    __syncthreads();
    for (int64_t kt = 0; kt < ksteps; ++kt) {
        if (kt + 1 < ksteps) fetch((kt + 1) * BK);
#pragma unroll
        for (int kk = 0; kk < BK / 16; ++kk) {
            const int cg = kk * 2 + (lane >> 5);
            bf16x8 a[4], b[4];
#pragma unroll
            for (int t = 0; t < 4; ++t) {
                a[t] = __builtin_bit_cast(bf16x8, sA[swz(wm * 128 + t * 32 + (lane & 31), cg)]);
                b[t] = __builtin_bit_cast(bf16x8, sB[swz(wn * 128 + t * 32 + (lane & 31), cg)]);
            }
#pragma unroll
            for (int i = 0; i < 4; ++i)
#pragma unroll
                for (int j = 0; j < 4; ++j)
                    acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a[i], b[j], acc[i][j], 0, 0, 0);
        }
        __syncthreads();
        if (kt + 1 < ksteps) {
            stage();
            __syncthreads();
        }
    }

    // accumulator element v of a 32x32 tile: row 8*(v/4) + 4*(lane/32) + v%4, column lane%32
#pragma unroll
    for (int i = 0; i < 4; ++i)
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            const int64_t col = n0 + wn * 128 + j * 32 + (lane & 31);
#pragma unroll
            for (int v = 0; v < 16; ++v) {
                const int64_t row = m0 + wm * 128 + i * 32 + 8 * (v >> 2) + 4 * (lane >> 5) + (v & 3);
                if (row < M && col < N) {
                    if (OUT_BF16) reinterpret_cast<uint16_t*>(p.C)[row * N + col] = (uint16_t)bf16_round_bits(acc[i][j][v]);
                    else reinterpret_cast<float*>(p.C)[row * N + col] = acc[i][j][v];
                }
            }
        }
}


// ------------------------------------------------------------------------- fast kernel
typedef float f32x2 __attribute__((ext_vector_type(2)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
constexpr int LDS_SLOTS = 5;                             // ring of operand tiles: A0 B0 A1 B1 A2 ...
constexpr int SLOT_BYTES = BM * BK * 2;                  // 32 KiB: one operand tile
constexpr int FAST_LDS_BYTES = LDS_SLOTS * SLOT_BYTES;   // 160 KiB: all of a compute unit's LDS
constexpr int64_t FAST_MAX_K = int64_t(1) << 22;         // 256 rows x K x 2 bytes must fit a 32-bit lane offset
constexpr int64_t FAST_MAX_N_KN = int64_t(1) << 23;      // B stored [K,N]: so must 128 rows x N x 2 bytes

__device__ __forceinline__ int swz64(int row, int cg) { return row * 8 + (cg ^ ((row >> 1) & 7)); }

// B stored [K,N]: 16-byte group c of row k of a tile sits at position c ^ kn_swz(k).  A transposing read
// touches rows 8q + 4h + r (q, r = 0..3) for one h, 32 bytes in each: the swizzle sends those 16 rows to 16
// different 32-byte windows.
__device__ __forceinline__ int kn_swz(int k) { return (((k >> 3) & 3) << 3) | ((k & 3) << 1); }

// One 16x16x32 MFMA, accumulator pinned to the AGPR file.  Written as inline asm: with the builtin the
// register allocator rotates the 64 accumulator quads through copies on every loop iteration.
#define LAGOM_MFMA_16x16x32(ACC, SRC_A, SRC_B) \
    asm volatile("v_mfma_f32_16x16x32_bf16 %0, %1, %2, %0" : "+a"(ACC) : "v"(SRC_A), "v"(SRC_B))

typedef short s16x4 __attribute__((ext_vector_type(4)));
typedef short s16x8 __attribute__((ext_vector_type(8)));

// 16 bytes of a row of C whose length is no multiple of 16 bytes, `left` elements in front of the row's end: rows start
// off the 16-byte grid, but a global store needs no more than the element's alignment.  Only what crosses the end of the
// row goes element by element.  bf16 result, everything element by element -> this: 3645 x 7797 x 96 58.8 -> 26.4 us,
// 4096 x 4097 x 64 33.7 -> 15.0, 1082 x 4319 x 808 26.0 -> 19.0; fp32 4100 x 4201 x 512 43.2 -> 30.4.
typedef u32x4 u32x4_aligned2 __attribute__((aligned(2)));
typedef uint32_t u32x2_aligned2 __attribute__((ext_vector_type(2), aligned(2)));
template <bool OUT_BF16>
__device__ __forceinline__ void store_ragged(char* out, u32x4 val, int64_t left) {
    constexpr int VEC = OUT_BF16 ? 8 : 4;
    if (left >= VEC) {
        *reinterpret_cast<u32x4_aligned2*>(out) = val;
        return;
    }
#pragma unroll
    for (int k = 0; k < VEC - 1; ++k)
        if (k < left) {
            if (OUT_BF16) reinterpret_cast<uint16_t*>(out)[k] = (uint16_t)(val[k >> 1] >> (16 * (k & 1)));
            else reinterpret_cast<uint32_t*>(out)[k] = val[k];
        }
}

// A store through the L2 to memory: nothing of it is left to be written back when the kernel ends.  (The compiler has no such store of this
// size; behind one of 16 bytes a vector instruction may write its registers two wait states later, which the compiler does not see to.)  For fp32 results of
// products with K split over wavefronts whose rows lie on the 64-byte grid, of which a store fills 64 bytes at a time: us, in the L2 -> through, results in the last-level cache
// | results that are not: 1000 x 960 x 320 5.77 -> 5.32 | 6.61 -> 6.14, 1024 x 1024 x 1024 7.04 -> 6.53 | 8.76 -> 8.24, 512 x 1904 x 1024 [K,N] 7.93 -> 7.46 | 10.1 -> 9.6, 640 x 624 x 136
// 4.31 -> 4.11 | 4.78 -> 4.60, 90 x 5408 x 128 4.19 -> 4.05 | 4.69 -> 4.52, 512 x 496 x 512 3.95 -> 3.87 | 4.84 -> 4.75.  Parts of 64 bytes gain as much in that cache,
// but memory takes them badly: 1000 x 952 x 320 5.75 -> 5.37 | 6.59 -> 7.02, 1000 x 956 x 320 5.77 -> 5.59 | 6.58 -> 7.29, bf16 (32 bytes a store) 1000 x 960 x 320 5.56 -> 5.32 | 6.38 -> 6.69,
// 1000 x 958 x 320 5.58 -> 6.69.  So do rows of 128 and 256 x 128 tiles that end inside lines: past the L2 -> through 2048 x 2040 x 256 fp32 8.21 -> 7.23 | 8.64 ->
// 11.50, 5742 x 1000 x 128 [K,N] 7.78 -> 6.97 | 8.15 -> 10.70, 713 x 5672 x 640 fp32 13.5 -> 12.1 | 14.5 -> 19.6, on the 64-byte grid 2000 x 2000 x 1024 fp32
// 11.2 -> 10.9 | 11.5 -> 13.7.
__device__ __forceinline__ void store_through(char* out, u32x4 val) { asm volatile("global_store_dwordx4 %0, %1, off sc1\n\ts_nop 1" ::"v"(out), "v"(val) : "memory"); }

// Clears an operand fragment in the lanes that do not keep theirs.
template <class FRAG>
__device__ __forceinline__ void keep_frag(FRAG& f, bool keep) {
    typedef uint32_t words __attribute__((ext_vector_type(sizeof(FRAG) / 4)));
    words w = __builtin_bit_cast(words, f);
#pragma unroll
    for (int i = 0; i < (int)(sizeof(FRAG) / 4); ++i) w[i] = keep ? w[i] : 0u;
    f = __builtin_bit_cast(FRAG, w);
    asm volatile("" : "+v"(f));
}
// An MFMA may read a register that a vector instruction wrote only some wait states later, and the compiler does not see
// the MFMAs in the asm statements.
__device__ __forceinline__ void wait_before_mfma() {
    __builtin_amdgcn_sched_barrier(0);
    asm volatile("s_nop 3" ::: "memory");
    __builtin_amdgcn_sched_barrier(0);
}
typedef __attribute__((address_space(3))) char* lds_bytes;

// B_KN = false: B stored [N,K]; true: B stored [K,N], its tiles kept in LDS as 64 rows (k) of 256 columns
// and transposed by the LDS reads.
// K_TAIL: K is not a multiple of 64; the last tile begins at column K - 64, behind the start of the one before it.
template <bool B_KN, bool OUT_BF16, bool K_TAIL>
__device__ __forceinline__ void fast_gemm_body(const GemmArgs& p, int tm, int tn) {
    extern __shared__ u32x4 smem[];   // LDS_SLOTS operand tiles of 2048 16-byte slots
    // Wavefronts of a communication kernel may share this wavefront's SIMD (this kernel leaves them
    // registers): let the instruction arbiter prefer the GEMM.
    __builtin_amdgcn_s_setprio(3);
    const int tid = threadIdx.x;
    const int lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int wm = wave >> 1, wn = wave & 1;
    const int64_t m0 = (int64_t)tm * BM, n0 = (int64_t)tn * BN;
    const int64_t M = p.M, N = p.N, K = p.K;
    const char* smem_bytes = reinterpret_cast<const char*>(smem);

    f32x4 acc[8][8];
#pragma unroll
    for (int i = 0; i < 8; ++i)
#pragma unroll
        for (int j = 0; j < 8; ++j)
#pragma unroll
            for (int v = 0; v < 4; ++v) acc[i][j][v] = 0.0f;

    // Load instruction d (0..7) of an operand tile fills its 16-byte slots [(d*4+wave)*64, +64):
    // lane -> row (d*4+wave)*8 + lane/8, stored group lane%8, i.e. source group (lane%8) ^ ((row>>1)&7).
    // (row>>1)&7 does not depend on d because rows of successive d differ by 32.
    // Addresses are a wave-uniform 64-bit base (first row of the tile, advanced along K) plus a 32-bit
    // byte offset per lane; rows past the edge re-read the last row.
    const int srow = wave * 8 + (lane >> 3);
    const int scg = (lane & 7) ^ ((srow >> 1) & 7);
    const char* base_a = reinterpret_cast<const char*>(p.A + m0 * K);
    // B stored [K,N]: a tile is 64 rows (k) of 512 bytes (256 n = 32 groups).  Load d fills rows
    // 8*d + 2*wave + lane/32, stored group lane%32 holding source group (lane%32) ^ kn_swz(row);
    // groups past the last column re-read the last one.  Successive K-steps are 64 rows of B apart.
    const char* base_b = reinterpret_cast<const char*>(B_KN ? p.B + n0 : p.B + n0 * K);
    const int64_t b_step = B_KN ? 2 * BK * N : 2 * BK;   // bytes from one K-step's tile of B to the next
    uint32_t a_off[8], b_off[8];
#pragma unroll
    for (int d = 0; d < 8; ++d) {
        const int64_t r = srow + 32 * d, last_a = M - 1 - m0, last_b = N - 1 - n0;
        a_off[d] = (uint32_t)(((r < last_a ? r : last_a) * K + scg * 8) * 2);
        if (B_KN) {
            const int krow = 8 * d + 2 * wave + (lane >> 5);
            const int64_t grp = (lane & 31) ^ kn_swz(krow), last_grp = (N - n0) / 8 - 1;
            b_off[d] = (uint32_t)((krow * N + (grp < last_grp ? grp : last_grp) * 8) * 2);
        } else {
            b_off[d] = (uint32_t)(((r < last_b ? r : last_b) * K + scg * 8) * 2);
        }
    }
    // LDS byte address of this wavefront's 1 KiB window of load 0 in slot 0
    const uint32_t lds0 = (uint32_t)(size_t)(__attribute__((address_space(3))) char*)smem + wave * 1024;
    // 16 bytes per lane from global memory straight into LDS: M0 holds the LDS address of lane 0.
    auto load_now = [&](const char* sbase, uint32_t voff, int slot, int d) {
        const uint32_t la = lds0 + slot * SLOT_BYTES + d * 4096;
        asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, %2" ::"s"(la), "v"(voff), "s"(sbase) : "memory");
    };
    // main-loop form in two halves, one MFMA apart (which also is the wait state M0 needs before the load)
    auto set_m0 = [&](uint32_t slot_base, int d) { asm volatile("s_add_i32 m0, %0, %1" ::"s"(slot_base), "n"(d * 4096) : "memory"); };
    // (no immediate offset: the hardware would add it to the LDS address as well)
    auto load_m0 = [&](const char* sbase, uint32_t voff) { asm volatile("global_load_lds_dwordx4 %0, %1" ::"v"(voff), "s"(sbase) : "memory"); };

    const int64_t ksteps = K_TAIL ? (K + BK - 1) / BK : K / BK;
    const int again = K_TAIL ? (int)(ksteps * BK - K) : 0;      // columns of the last tile that the one before it holds as well
    const int64_t again_a = 2 * again, again_b = B_KN ? 2 * again * N : 2 * again;   // in bytes
    // (a K_TAIL product has at least two steps)
    const char* const base_a1 = base_a + BK * 2 - (K_TAIL && ksteps == 2 ? again_a : 0);
    const char* const base_b1 = base_b + b_step - (K_TAIL && ksteps == 2 ? again_b : 0);
    // prologue: A0 -> slot 0, B0 -> slot 1, A1 -> slot 2, first half of B1 -> slot 3
#pragma unroll
    for (int d = 0; d < 8; ++d) load_now(base_a, a_off[d], 0, d);
#pragma unroll
    for (int d = 0; d < 8; ++d) load_now(base_b, b_off[d], 1, d);
    if (ksteps > 1) {
#pragma unroll
        for (int d = 0; d < 8; ++d) load_now(base_a1, a_off[d], 2, d);
#pragma unroll
        for (int d = 0; d < 4; ++d) load_now(base_b1, b_off[d], 3, d);
        asm volatile("s_waitcnt vmcnt(12)" ::: "memory");   // loads complete in issue order: A0 and B0 are in
    } else {
        asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    }
    __builtin_amdgcn_s_barrier();

    // Fragment r of a 32-wide k-slice: lane -> row 16*r + lane%16, 16-byte group 4*slice + lane/16.
    const int arow = wm * 128 + (lane & 15), brow = wn * 128 + (lane & 15), kq = lane >> 4;
    bf16x8 fa[2][8], fb[2][8];
    // B stored [K,N]: fragment j of a k-slice is two transposing reads (h = 0, 1).  In each, lane
    // 16*q + i hands in the address of B[8q + 4h + i/4][16j + 4*(i%4) .. +3] and receives
    // B[8q + 4h + 0..3][16j + i]: together the 8 consecutive k of column 16j + lane%16 that the MFMA
    // pairs with A[row][8q .. 8q+7].  kn_frag[j]: the lane's byte offset for fragment j in a tile's slot;
    // slice and h move it by whole rows (16 KiB, 2 KiB), which the swizzle does not see.
    s16x4 fbh[B_KN ? 2 : 1][B_KN ? 8 : 1][2];
    uint32_t kn_frag[B_KN ? 8 : 1];
    if (B_KN) {
        const int i = lane & 15, r = i >> 2;
        const int krow = 8 * kq + r;                                   // slice 0, h = 0
        const int grp0 = wn * 16 + ((i & 3) >> 1);                     // source group of fragment 0
#pragma unroll
        for (int j = 0; j < 8; ++j)
            kn_frag[j] = (uint32_t)(krow * 512 + (((grp0 + 2 * j) ^ kn_swz(krow)) << 4) + 8 * (i & 1));
    }
    // r: 0..7 = A0..A7, 8..15 = B0..B7; half: which of the two reads of a [K,N] B fragment
    auto read_frag = [&](const u32x4* sa, const u32x4* sb, int ks, int r, int buf, int half) {
        if (r < 8) {
            fa[buf][r] = __builtin_bit_cast(bf16x8, sa[swz64(arow + r * 16, ks * 4 + kq)]);
        } else if (!B_KN) {
            fb[buf][r - 8] = __builtin_bit_cast(bf16x8, sb[swz64(brow + (r - 8) * 16, ks * 4 + kq)]);
        } else {
            typedef s16x4 __attribute__((address_space(3))) * tr_ptr;
            fbh[buf][r - 8][half] = __builtin_amdgcn_ds_read_tr16_b64_v4i16(
                (tr_ptr)((lds_bytes)(const char*)sb + kn_frag[r - 8] + ks * 16384 + half * 2048));
        }
    };
    auto b_frag = [&](int buf, int j) -> bf16x8 {
        if (!B_KN) return fb[buf][j];
        return __builtin_bit_cast(bf16x8, __builtin_shufflevector(fbh[buf][j][0], fbh[buf][j][1], 0, 1, 2, 3, 4, 5, 6, 7));
    };
#pragma unroll
    for (int r = 0; r < 16; ++r) {
        read_frag(smem, smem + SLOT_BYTES / 16, 0, r, 0, 0);
        if (B_KN && r >= 8) read_frag(smem, smem + SLOT_BYTES / 16, 0, r, 0, 1);
    }

    // One K-step = 2 k-slices x 8 groups x 8 MFMAs (group g: A fragment g against the 8 B fragments).
    // MORE1 / MORE2: tiles kt+1 / kt+2 exist (compile-time, so that the steady-state loop has no
    // branches; the last two K-steps are peeled).  Every MFMA is followed by at most one other
    // instruction, which issues while the matrix core works on that MFMA:
    //   loads   one per group, M0 after the group's first MFMA and the load after its third:
    //           groups 0-3 second half of B(kt+1); 4-11 A(kt+2) into the fifth slot; 12-15 first half
    //           of B(kt+2) into the slot A(kt) has just left.
    //   reads   slice 0: two fragments of slice 1 per group; slice 1, groups 4-7: four fragments per
    //           group of slice 0 of tile kt+1, in the order the next step consumes them.
    //   barrier in front of group 12: by then this wavefront holds every fragment of tile kt in
    //           registers and tile kt+1 has landed (the 8 youngest loads, A(kt+2), may still fly), so
    //           after the barrier tile kt's slots are free and tile kt+1 may be read.
    constexpr int kReadOrder[16] = {0, 8, 9, 10, 11, 12, 13, 14, 15, 1, 2, 3, 4, 5, 6, 7};   // A0, B0..B7, A1..A7
    // Byte offsets of the slots of A(kt), B(kt), A(kt+1), B(kt+1), A(kt+2).  Advancing by one K-step moves
    // every role two slots along a ring of five, which is a pure rotation of these five values.
    uint32_t o_a = 0, o_b = SLOT_BYTES, o_a1 = 2 * SLOT_BYTES, o_b1 = 3 * SLOT_BYTES, o_a2 = 4 * SLOT_BYTES;
    const char* g_a = base_a + 2 * (BK * 2);   // &A[m0][(kt+2)*64]
    const char* g_b = base_b1;                 // tile kt+1 of B; tile kt+2 is reached through b_off_next
    uint32_t b_off_next[4];
#pragma unroll
    for (int d = 0; d < 4; ++d) b_off_next[d] = b_off[d] + (uint32_t)b_step;
    // Fragment reads of one k-slice in the order the MFMAs consume them.  [N,K]: 16 reads, A0, B0..B7,
    // A1..A7.  [K,N]: 24 reads, every B fragment being two.
    constexpr int kReads = B_KN ? 24 : 16;
    auto read_nth = [&](const u32x4* sa, const u32x4* sb, int ks, int n, int buf) {
        if (!B_KN) read_frag(sa, sb, ks, kReadOrder[n], buf, 0);
        else if (n == 0) read_frag(sa, sb, ks, 0, buf, 0);
        else if (n <= 16) read_frag(sa, sb, ks, 8 + (n - 1) / 2, buf, (n - 1) & 1);
        else read_frag(sa, sb, ks, n - 16, buf, 0);
    };
    auto step = [&](auto more1_c, auto more2_c) {
        constexpr bool more1 = decltype(more1_c)::value, more2 = decltype(more2_c)::value;
        const u32x4* sa = reinterpret_cast<const u32x4*>(smem_bytes + o_a);
        const u32x4* sb = reinterpret_cast<const u32x4*>(smem_bytes + o_b);
        const u32x4* sa1 = reinterpret_cast<const u32x4*>(smem_bytes + o_a1);
        const u32x4* sb1 = reinterpret_cast<const u32x4*>(smem_bytes + o_b1);
        const uint32_t l_b1 = lds0 + o_b1, l_a2 = lds0 + o_a2, l_a = lds0 + o_a;
#pragma unroll
        for (int ks = 0; ks < 2; ++ks) {
            if (K_TAIL && !more1) {
#pragma unroll
                for (int r = 0; r < 8; ++r) {
                    keep_frag(fa[ks][r], ks * 4 + kq >= again / 8);
                    if (!B_KN) keep_frag(fb[ks][r], ks * 4 + kq >= again / 8);
                    else { keep_frag(fbh[ks][r][0], ks * 4 + kq >= again / 8); keep_frag(fbh[ks][r][1], ks * 4 + kq >= again / 8); }
                }
                wait_before_mfma();
            }
#pragma unroll
            for (int g = 0; g < 8; ++g) {
                const int q = ks * 8 + g;
                if (q == 12) {
                    if (more2) asm volatile("s_waitcnt vmcnt(8)" ::: "memory");
                    else asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
                    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
                    __builtin_amdgcn_s_barrier();
                    __builtin_amdgcn_sched_barrier(0);
                }
#pragma unroll
                for (int j = 0; j < 8; ++j) {
                    // B fragment first: the lane's 4 results are C[row lane%16][4 consecutive columns]
                    LAGOM_MFMA_16x16x32(acc[g][j], b_frag(ks, j), fa[ks][g]);
                    __builtin_amdgcn_sched_barrier(0);
                    if (j == 0) {
                        if (q < 4) { if (more1) set_m0(l_b1, 4 + q); }
                        else if (q < 12) { if (more2) set_m0(l_a2, q - 4); }
                        else { if (more2) set_m0(l_a, q - 12); }
                    }
                    if (j == 2) {
                        if (q < 4) { if (more1) load_m0(g_b, b_off[4 + q]); }
                        else if (q < 12) { if (more2) load_m0(g_a, a_off[q - 4]); }
                        else { if (more2) load_m0(g_b, b_off_next[q - 12]); }
                    }
                    if (ks == 0) {   // slice 1 of this tile: 2 (3) reads per group
                        if (j == 3) read_nth(sa, sb, 1, (kReads / 8) * g, 1);
                        if (j == 5) read_nth(sa, sb, 1, (kReads / 8) * g + 1, 1);
                        if (B_KN && j == 6) read_nth(sa, sb, 1, 3 * g + 2, 1);
                    } else if (more1 && g >= 4) {   // slice 0 of tile kt+1: 4 (6) reads per group
                        if (!B_KN) {
                            if (j & 1) read_nth(sa1, sb1, 0, (g - 4) * 4 + (j >> 1), 0);
                        } else {
                            constexpr int kSlot[8] = {-1, 0, -1, 1, 2, 3, 4, 5};
                            if (kSlot[j] >= 0) read_nth(sa1, sb1, 0, (g - 4) * 6 + kSlot[j], 0);
                        }
                    }
                    __builtin_amdgcn_sched_barrier(0);
                }
            }
        }
        const uint32_t t_a = o_a, t_b = o_b;
        o_a = o_a1; o_b = o_b1; o_a1 = o_a2; o_b1 = t_a; o_a2 = t_b;
        g_a += BK * 2;
        g_b += b_step;
    };
    int kt = 0;
    const int nk = (int)ksteps;
    for (; kt + (K_TAIL ? 3 : 2) < nk; ++kt) step(std::true_type{}, std::true_type{});
    if (K_TAIL && kt + 2 < nk) {     // the step that begins to load the last tile
        g_a -= again_a;
#pragma unroll
        for (int d = 0; d < 4; ++d) b_off_next[d] -= (uint32_t)again_b;
        step(std::true_type{}, std::true_type{});
        g_b -= again_b;
        ++kt;
    }
    if (kt + 1 < nk) { step(std::true_type{}, std::false_type{}); ++kt; }
    if (kt < nk) step(std::false_type{}, std::false_type{});
    // The compiler does not see an MFMA inside the asm statements and therefore adds none of the wait
    // states an accumulator read needs after one: give the last results their cycles here, and make
    // every later use of an accumulator depend on a statement that follows these cycles.
    asm volatile("s_nop 7\n\ts_nop 7\n\ts_nop 7" ::: "memory");
#pragma unroll
    for (int i = 0; i < 8; ++i)
#pragma unroll
        for (int j = 0; j < 8; ++j) asm volatile("" : "+a"(acc[i][j]));
    __builtin_amdgcn_s_barrier();   // every wavefront is past its last LDS read before the slots are reused below

    // Epilogue.  acc[i][j][v] is row 16*i + lane%16, column 16*j + 4*(lane/16) + v of the wavefront's
    // 128 x 128 block.  The block is staged in the wavefront's own 32 KiB of LDS as rows of ROW_BYTES
    // (16-byte group c of row r stored at c ^ (r & 15)) and written out as 16-byte vectors, whole rows
    // of the block contiguous: all 128 rows at once for bf16, 64 rows per pass for fp32.  A wavefront
    // reads back only what it wrote itself, and LDS serves one wavefront's accesses in order, so the
    // passes need no waits between them beyond the data dependencies.
    constexpr int ESZ = OUT_BF16 ? 2 : 4;
    constexpr int PASSES = OUT_BF16 ? 1 : 2;
    constexpr int ROW_BYTES = 128 * ESZ, GROUPS = ROW_BYTES / 16, ROWS_PER_READ = 64 / GROUPS, VEC = 16 / ESZ;
    const int r_in = lane & 15, c_q = 4 * (lane >> 4);
    char* st = reinterpret_cast<char*>(smem) + wave * SLOT_BYTES;
    const bool interior = m0 + BM <= M && n0 + BN <= N;
    const bool vector_ok = (N % VEC) == 0;
    const int rd_row = lane / GROUPS, rd_cv = lane % GROUPS;
    const int64_t gcol = n0 + wn * 128 + rd_cv * VEC;
#pragma unroll
    for (int pass = 0; pass < PASSES; ++pass) {
#pragma unroll
        for (int ii = 0; ii < 8 / PASSES; ++ii)
#pragma unroll
            for (int j = 0; j < 8; ++j) {
                const int i = pass * (8 / PASSES) + ii;
                const int r = ii * 16 + r_in;
                const int cb = (j * 16 + c_q) * ESZ;          // byte offset of the first of four consecutive columns
                char* dst = st + r * ROW_BYTES + (((cb >> 4) ^ (r & 15)) << 4) + (cb & 15);
                if (OUT_BF16) {
                    const bf16x2 lo = __builtin_convertvector(f32x2{acc[i][j][0], acc[i][j][1]}, bf16x2);
                    const bf16x2 hi = __builtin_convertvector(f32x2{acc[i][j][2], acc[i][j][3]}, bf16x2);
                    uint2 v;
                    v.x = __builtin_bit_cast(uint32_t, lo);
                    v.y = __builtin_bit_cast(uint32_t, hi);
                    *reinterpret_cast<uint2*>(dst) = v;
                } else {
                    *reinterpret_cast<f32x4*>(dst) = acc[i][j];
                }
            }
        const int64_t row0 = m0 + wm * 128 + pass * (128 / PASSES) + rd_row;
#pragma unroll
        for (int tb = 0; tb < 4; ++tb) {   // eight reads in flight, then eight stores
            u32x4 val[8];
#pragma unroll
            for (int e = 0; e < 8; ++e) {
                const int r = rd_row + ROWS_PER_READ * (tb * 8 + e);
                val[e] = *reinterpret_cast<const u32x4*>(st + r * ROW_BYTES + ((rd_cv ^ (r & 15)) << 4));
            }
            // Past the L2s, also where rows of C are off the 64-byte grid and two wavefronts write parts of a line.  Into them such products
            // alone are faster (5000 x 5080 x 512 fp32 45 -> 42 us over 16 results, 37 over one), but rows on the grid lose (6400 x 5632 x 2056
            // fp32 132 -> 144, 8192 x 8448 x 256 fp32 73 -> 81), and what runs beside a product finds its data gone from the last-level
            // cache: a 64 MiB gather on 8 channels beside three of 5000 x 5080 x 512 fp32 166 -> 253.
#pragma unroll
            for (int e = 0; e < 8; ++e) {
                const int64_t grow = row0 + ROWS_PER_READ * (tb * 8 + e);
                char* out = reinterpret_cast<char*>(p.C) + (grow * N + gcol) * ESZ;
                if (vector_ok) {
                    if (interior || (grow < M && gcol < N)) __builtin_nontemporal_store(val[e], reinterpret_cast<u32x4*>(out));
                } else if (grow < M) {
                    store_ragged<OUT_BF16>(out, val[e], N - gcol);
                }
            }
        }
    }
}

template <bool OUT_BF16>
__global__ void __launch_bounds__(THREADS) gemm_bf16_nk_kernel(const GemmArgs p) { int tm, tn; tile_of(blockIdx.x, p, &tm, &tn); fast_gemm_body<false, OUT_BF16, false>(p, tm, tn); }
template <bool OUT_BF16>
__global__ void __launch_bounds__(THREADS) gemm_bf16_kn_kernel(const GemmArgs p) { int tm, tn; tile_of(blockIdx.x, p, &tm, &tn); fast_gemm_body<true, OUT_BF16, false>(p, tm, tn); }
// K >= 64 and not a multiple of 64 (kernels of their own: the peeled last step clears fragments; as many registers)
template <bool OUT_BF16>
__global__ void __launch_bounds__(THREADS) gemm_bf16_nk_tail_kernel(const GemmArgs p) { int tm, tn; tile_of(blockIdx.x, p, &tm, &tn); fast_gemm_body<false, OUT_BF16, true>(p, tm, tn); }
template <bool OUT_BF16>
__global__ void __launch_bounds__(THREADS) gemm_bf16_kn_tail_kernel(const GemmArgs p) { int tm, tn; tile_of(blockIdx.x, p, &tm, &tn); fast_gemm_body<true, OUT_BF16, true>(p, tm, tn); }

// ------------------------------------------------------------------------- small-tile kernels
// 128 x 128 x 64 and 256 x 128 x 64 tiles for products with too few 256 x 256 tiles to fill the chip.
// Same workgroup (4 wavefronts, 2 x 2; a wavefront owns NI x 4 MFMA tiles, NI = 4 or 8, i.e. 64 or 128
// accumulators), same LDS-direct loads, row layout and swizzles as the large kernel.  LDS holds a ring of
// A+B tile pairs: five for NI = 4 (a K-step is only 32 MFMAs long, loads run four to five steps ahead),
// three for NI = 8.  One barrier per K-step, in its middle.
constexpr int SBN = 128;
constexpr int S_B_BYTES = SBN * BK * 2;                   // 16 KiB
template <int NI> struct SmallTile {
    static constexpr int BM_ = 32 * NI;                   // rows of a tile
    static constexpr int A_BYTES = BM_ * BK * 2;          // 16 or 32 KiB
    static constexpr int STAGE_BYTES = A_BYTES + S_B_BYTES;
    static constexpr int STAGES = NI == 4 ? 5 : 3;
    static constexpr int AHEAD = STAGES - 1;
    static constexpr int LA = NI, LB = 4;                 // load instructions per wavefront for an A / a B tile
    static_assert(STAGES * STAGE_BYTES <= FAST_LDS_BYTES, "the ring fits the LDS");
};
constexpr int SBM = SmallTile<4>::BM_, MBM = SmallTile<8>::BM_;

// B stored [K,N]: a B tile is 64 rows (k) of 256 bytes (128 n = 16 groups); group c of row k sits at
// c ^ kn_swz128(k), which spreads the rows of a transposing read over the 8 32-byte windows of a row.
__device__ __forceinline__ int kn_swz128(int k) { return (((k >> 3) & 1) << 3) | ((k & 3) << 1); }

// K_TAIL: K is not a multiple of 64, and rows start anywhere between two 128-byte lines: 64 columns of a row reach into two lines, and
// the compute unit's cache, which looks up one line at a time, takes twice the time.  LINES: tile t holds line t of every row
// instead, counted from the one that the row starts in, so a row that starts s groups (of 16 bytes) behind a line has the last s groups of
// K-step t in tile t + 1: the lanes that need those read there.  A group's place in its row in LDS is the one it would have without the
// shift.  One tile more is loaded, and one more has to be there.  The last K-step's columns behind K are cleared in the fragments.  256 x 128 tiles,
// with three in LDS, hold A in lines and B in K-steps.
// Without LINES: the last tile begins at column K - 64 (see the large kernel).
constexpr int LINE = BK * 2;
// How many groups of 16 bytes a row starts behind a line.  Rows 8 apart start alike.
__device__ __forceinline__ int skew(const uint16_t* base, int row, int64_t K) { return (int)(((uintptr_t)base >> 4) + (uint32_t)row * (uint32_t)(K / 8)) & 7; }
enum TileKind { USUAL_TILE, LAST_TILE, END_TILE };
// A lane's offset against its group's in the columns of a K-step, which count from one line in front of them.  Lanes with nothing to load read
// what lies in a line that others of their row read.
struct LinesOf {
    uint32_t usual;             // part of the offset as it is held: the group of K-step t in tile t, or of the one before, if it lies behind the line
    uint32_t first, last, end;  // against that: in tile 0 (nothing in front of the row), in the last K-step's tile, and in the one behind
                                // it, from the same place (nothing behind the row)
    __device__ __forceinline__ LinesOf(bool behind, int group, int last_groups)
        : usual(behind ? 0u : LINE), first(behind ? LINE - 16u * group : 0u),
          last(!behind && group >= last_groups ? 16u * (uint32_t)(last_groups - 1 - group) : 0u),
          end((behind && group < last_groups ? LINE : LINE + 16u * (uint32_t)(last_groups - 1 - group)) - usual) {}
};
template <int NI, bool B_KN, bool OUT_BF16, bool K_TAIL, bool LINES = false>
__device__ __forceinline__ void small_gemm_body(const GemmArgs& p, int tm, int tn) {
    typedef SmallTile<NI> T;
    constexpr int S_STAGES = T::STAGES, S_AHEAD = T::AHEAD, S_STAGE_BYTES = T::STAGE_BYTES, S_OPERAND_BYTES = T::A_BYTES;
    constexpr int LA = T::LA, LB = T::LB, PER_TILE = LA + LB;
    static_assert(!LINES || K_TAIL);
    constexpr bool LINES_B = LINES && !B_KN && NI == 4;
    extern __shared__ u32x4 smem[];
    __builtin_amdgcn_s_setprio(3);
    const int tid = threadIdx.x;
    const int lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int wm = wave >> 1, wn = wave & 1;
    const int64_t m0 = (int64_t)tm * T::BM_, n0 = (int64_t)tn * SBN;
    const int64_t M = p.M, N = p.N, K = p.K;
    const char* smem_bytes = reinterpret_cast<const char*>(smem);

    f32x4 acc[NI][4];
#pragma unroll
    for (int i = 0; i < NI; ++i)
#pragma unroll
        for (int j = 0; j < 4; ++j) acc[i][j] = f32x4{0.f, 0.f, 0.f, 0.f};

    const int nk = (int)(K_TAIL ? (K + BK - 1) / BK : K / BK);
    // load d of an operand tile: rows (d*4 + wave)*8 + lane/8, as in the large kernel
    const int srow = wave * 8 + (lane >> 3);
    const int scg = (lane & 7) ^ ((srow >> 1) & 7);
    const char* g_a = reinterpret_cast<const char*>(p.A + m0 * K) - (LINES ? LINE : 0);
    const char* g_b = reinterpret_cast<const char*>(B_KN ? p.B + n0 : p.B + n0 * K) - (LINES_B ? LINE : 0);
    const int last_groups = (int)(K / 8) - 8 * (nk - 1);
    const LinesOf lines_a(scg + skew(p.A, srow, K) >= 8, scg, last_groups), lines_b(scg + skew(p.B, srow, K) >= 8, scg, last_groups);
    const int64_t b_step = B_KN ? 2 * BK * N : 2 * BK;
    uint32_t a_off[LA], b_off[LB];
#pragma unroll
    for (int d = 0; d < LA; ++d) {
        const int64_t r = srow + 32 * d, last_a = M - 1 - m0;
        a_off[d] = (uint32_t)(((r < last_a ? r : last_a) * K + scg * 8) * 2) + (LINES ? lines_a.usual : 0u);
    }
    uint32_t b_row[LB];          // [K,N] with LINES: to the first row, which rows behind K re-read
    const uint32_t b_past_k = scg < last_groups ? 0u : 16u * (uint32_t)(scg - last_groups + 1);      // [N,K] with LINES of A only: to the last group
#pragma unroll
    for (int d = 0; d < LB; ++d) {
        const int64_t r = srow + 32 * d, last_b = N - 1 - n0;
        if (B_KN) {   // load d fills rows 16*d + 4*wave + lane/16 of the [64][128] tile, stored group lane%16
            const int krow = 16 * d + 4 * wave + (lane >> 4);
            const int64_t grp = (lane & 15) ^ kn_swz128(krow), last_grp = (N - n0) / 8 - 1;
            b_off[d] = (uint32_t)((krow * N + (grp < last_grp ? grp : last_grp) * 8) * 2);
            b_row[d] = krow < 8 * last_groups ? 0u : (uint32_t)(krow * N * 2);
        } else {
            b_off[d] = (uint32_t)(((r < last_b ? r : last_b) * K + scg * 8) * 2) + (LINES_B ? lines_b.usual : 0u);
        }
    }
    const uint32_t lds0 = (uint32_t)(size_t)(__attribute__((address_space(3))) char*)smem + wave * 1024;
    const int nl = LINES ? nk + 1 : nk;         // tiles that are loaded
    const int again = K_TAIL && !LINES ? (int)((int64_t)nk * BK - K) : 0;      // columns of the last tile that the one before it holds as well
    const int64_t again_a = 2 * again, again_b = B_KN ? 2 * again * N : 2 * again;   // in bytes
    // g_a / g_b from the tile in front of `t` to tile t.  (The compiler must not know `t`: it would peel the loop's last
    // iterations for this comparison, and copy accumulators between them.)
    auto is_last = [&](int t) { asm volatile("" : "+s"(t)); return t == nl - 1; };
    auto next_a = [&](int t) { g_a += BK * 2; if (K_TAIL) g_a -= is_last(t) ? (LINES ? LINE : again_a) : 0; };
    auto next_b = [&](int t) { g_b += b_step; if (K_TAIL) g_b -= is_last(t) ? (LINES ? b_step : again_b) : 0; };
    // the lane's offsets in load d of tile t
    auto from_a = [&](TileKind kind, int d) { return a_off[d] + (!LINES || kind == USUAL_TILE ? 0u : kind == LAST_TILE ? lines_a.last : lines_a.end); };
    auto from_b = [&](TileKind kind, int d) {
        if (!LINES || kind == USUAL_TILE) return b_off[d];
        return B_KN ? b_off[d] - b_row[d] : !LINES_B ? b_off[d] - b_past_k : b_off[d] + (kind == LAST_TILE ? lines_b.last : lines_b.end);
    };
    auto kind_of = [&](int t) { return t < nk - 1 ? USUAL_TILE : t == nk - 1 ? LAST_TILE : END_TILE; };
    auto load_tile = [&](int stage) {   // the tile g_a / g_b point at (tile `stage`), then advance them one K-step
        const uint32_t base = lds0 + stage * S_STAGE_BYTES;
        const uint32_t first_a = LINES && stage == 0 ? lines_a.first : 0u, first_b = LINES_B && stage == 0 ? lines_b.first : 0u;
#pragma unroll
        for (int d = 0; d < LA; ++d)
            asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, %2" ::"s"(base + d * 4096), "v"(from_a(kind_of(stage), d) + first_a), "s"(g_a) : "memory");
#pragma unroll
        for (int d = 0; d < LB; ++d)
            asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, %2" ::"s"(base + S_OPERAND_BYTES + d * 4096), "v"(from_b(kind_of(stage), d) + first_b), "s"(g_b) : "memory");
        next_a(stage + 1);
        next_b(stage + 1);
    };

    for (int t = 0; t < S_AHEAD && t < nl; ++t) load_tile(t);
    // Tile t >= AHEAD is loaded in two halves: A behind the barrier of step t-STAGES, B in the first half of
    // step t-AHEAD (g_a / g_b point at the next tile to load of their operand).
    auto set_m0 = [&](uint32_t lds) { asm volatile("s_mov_b32 m0, %0" ::"s"(lds) : "memory"); };
    auto load_m0 = [&](const char* sbase, uint32_t voff) { asm volatile("global_load_lds_dwordx4 %0, %1" ::"v"(voff), "s"(sbase) : "memory"); };
    if (S_AHEAD < nl) {
#pragma unroll
        for (int d = 0; d < LA; ++d)
            asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, %2" ::"s"(lds0 + S_AHEAD * S_STAGE_BYTES + d * 4096), "v"(from_a(kind_of(S_AHEAD), d)), "s"(g_a) : "memory");
        next_a(S_AHEAD + 1);
    }

    const int arow = wm * (16 * NI) + (lane & 15), brow = wn * 64 + (lane & 15), kq = lane >> 4;
    bf16x8 fa[2][NI];
    bf16x8 fb[2][4];             // fragments of the two 32-wide k-slices, read half a K-step before their MFMAs
    s16x4 fbh[B_KN ? 2 : 1][B_KN ? 4 : 1][2];
    // B stored [K,N]: fragment j is two transposing reads (rows 8q + 4h + i/4 of the slice, h = 0, 1; see the
    // large kernel); kn_frag[j] is the lane's byte offset for h = 0 in slice 0
    uint32_t kn_frag[B_KN ? 4 : 1];
    if (B_KN) {
        const int i = lane & 15, krow = 8 * kq + (i >> 2);
        const int grp0 = wn * 8 + ((i & 3) >> 1);
#pragma unroll
        for (int j = 0; j < 4; ++j)
            kn_frag[j] = (uint32_t)(krow * 256 + (((grp0 + 2 * j) ^ kn_swz128(krow)) << 4) + 8 * (i & 1));
    }
    constexpr int UNITS = NI + 4;
    // read unit u of a slice, in the order the MFMAs consume them: A0, B0, B1, B2, B3, A1, A2, ...
    const bool behind_a[2] = {kq + skew(p.A, arow, K) >= 8, 4 + kq + skew(p.A, arow, K) >= 8};     // LINES: the lane's groups lie in the next tile
    const bool behind_b[2] = {kq + skew(p.B, brow, K) >= 8, 4 + kq + skew(p.B, brow, K) >= 8};
    auto read_unit = [&](uint32_t stage_bytes, uint32_t next_bytes, int ks, int u) {
        const u32x4* sa = reinterpret_cast<const u32x4*>(smem_bytes + (LINES && behind_a[ks] ? next_bytes : stage_bytes));
        const u32x4* sb = reinterpret_cast<const u32x4*>(smem_bytes + (LINES_B && behind_b[ks] ? next_bytes : stage_bytes)) + S_OPERAND_BYTES / 16;
        if (u == 0 || u >= 5) {
            const int r = u == 0 ? 0 : u - 4;
            fa[ks][r] = __builtin_bit_cast(bf16x8, sa[swz64(arow + r * 16, ks * 4 + kq)]);
        } else if (!B_KN) {
            fb[ks][u - 1] = __builtin_bit_cast(bf16x8, sb[swz64(brow + (u - 1) * 16, ks * 4 + kq)]);
        } else {
            typedef s16x4 __attribute__((address_space(3))) * tr_ptr;
            const lds_bytes at = (lds_bytes)(const char*)sb + kn_frag[u - 1] + ks * 8192;
            fbh[ks][u - 1][0] = __builtin_amdgcn_ds_read_tr16_b64_v4i16((tr_ptr)at);
            fbh[ks][u - 1][1] = __builtin_amdgcn_ds_read_tr16_b64_v4i16((tr_ptr)(at + 1024));
        }
    };
    auto b_frag = [&](int ks, int j) -> bf16x8 {
        if (!B_KN) return fb[ks][j];
        return __builtin_bit_cast(bf16x8, __builtin_shufflevector(fbh[ks][j][0], fbh[ks][j][1], 0, 1, 2, 3, 4, 5, 6, 7));
    };
    // loads complete in issue order: wait until all but the youngest `tiles` whole tiles have landed
    auto wait_all_but = [&](int tiles) {
        if (tiles >= 3 && S_AHEAD > 3) asm volatile("s_waitcnt vmcnt(%0)" ::"n"(3 * PER_TILE) : "memory");
        else if (tiles >= 2 && S_AHEAD > 2) asm volatile("s_waitcnt vmcnt(%0)" ::"n"(2 * PER_TILE) : "memory");
        else if (tiles >= 1) asm volatile("s_waitcnt vmcnt(%0)" ::"n"(PER_TILE) : "memory");
        else asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    };
    // tile 0 (LINES: and tile 1, or its A half; the A half of tile AHEAD, if any, may fly on as well)
    wait_all_but((nl < S_AHEAD ? nl : S_AHEAD) - (LINES && NI == 4 ? 2 : 1));
    __builtin_amdgcn_s_barrier();
#pragma unroll
    for (int u = 0; u < UNITS; ++u) read_unit(0, S_STAGE_BYTES, 0, u);

    // One K-step = 2 k-slices x 4*NI MFMAs, each MFMA followed by at most one side instruction (a B fragment
    // of the [K,N] layout being two reads):
    //   first half   NI + 4 fragment reads of slice 1; then the B half of tile kt+AHEAD (M0 write and load
    //                alternating)
    //   barrier      behind vmcnt: tile kt+1 has landed for every wavefront; nobody reads tile kt any more
    //                (its fragments are in registers), so its slot can take the A half of tile kt+STAGES
    //   second half  NI + 4 fragment reads of slice 0 of tile kt+1; then the A half of tile kt+STAGES
    // LOAD_B / LOAD_A / NEXT: tiles kt+AHEAD / kt+STAGES / kt+1 exist (compile time: no branch inside a step).
    uint32_t o_cur = 0, o_next = S_STAGE_BYTES, o_b4 = S_AHEAD * S_STAGE_BYTES;   // byte offsets of the slots of tiles kt, kt+1, kt+4
    uint32_t o_third = 2 * S_STAGE_BYTES;       // LINES: of tile kt+2
    auto behind = [&](uint32_t o) { return o + S_STAGE_BYTES == S_STAGES * S_STAGE_BYTES ? 0 : o + S_STAGE_BYTES; };
    int kt = 0;
    auto step = [&](auto load_b_c, auto load_a_c, auto next_c, auto kind_b_c, auto kind_a_c) {
        constexpr TileKind KIND_B = decltype(kind_b_c)::value, KIND_A = decltype(kind_a_c)::value;     // of the tiles it loads
        constexpr bool LOAD_B = decltype(load_b_c)::value, LOAD_A = decltype(load_a_c)::value, NEXT = decltype(next_c)::value;
        const uint32_t l_b = lds0 + o_b4 + S_OPERAND_BYTES, l_a = lds0 + o_cur;
#pragma unroll
        for (int ks = 0; ks < 2; ++ks) {
            if (ks == 1) {
                // issued and not needed yet: the whole tiles kt+2 (LINES: kt+3; of three tiles the B half of kt+2) .. kt+AHEAD that exist
                if (LOAD_B) asm volatile("s_waitcnt vmcnt(%0)" ::"n"(!LINES ? (S_AHEAD - 1) * PER_TILE : S_AHEAD > 2 ? (S_AHEAD - 2) * PER_TILE : LB) : "memory");
                else if (NEXT) wait_all_but(nk - 2 - kt);
                asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
                __builtin_amdgcn_s_barrier();
                __builtin_amdgcn_sched_barrier(0);
            }
            if (K_TAIL && !NEXT) {
                const bool keep = LINES ? ks * 4 + kq < last_groups : ks * 4 + kq >= again / 8;
#pragma unroll
                for (int i = 0; i < NI; ++i) keep_frag(fa[ks][i], keep);
#pragma unroll
                for (int j = 0; j < 4; ++j) {
                    if (!B_KN) keep_frag(fb[ks][j], keep);
                    else { keep_frag(fbh[ks][j][0], keep); keep_frag(fbh[ks][j][1], keep); }
                }
                wait_before_mfma();
            }
#pragma unroll
            for (int i = 0; i < NI; ++i)
#pragma unroll
                for (int j = 0; j < 4; ++j) {
                    const int sl = i * 4 + j;     // slot within the half
                    // B fragment first: a lane holds 4 consecutive columns of one row
                    LAGOM_MFMA_16x16x32(acc[i][j], b_frag(ks, j), fa[ks][i]);
                    __builtin_amdgcn_sched_barrier(0);
                    if (sl < UNITS) {
                        if (ks == 0) read_unit(o_cur, o_next, 1, sl);
                        else if (NEXT) read_unit(o_next, o_third, 0, sl);
                    } else {
                        const int d = (sl - UNITS) >> 1, odd = (sl - UNITS) & 1;
                        if (ks == 0 && LOAD_B && d < LB) { if (odd) load_m0(g_b, from_b(KIND_B, d)); else set_m0(l_b + d * 4096); }
                        if (ks == 1 && LOAD_A && d < LA) { if (odd) load_m0(g_a, from_a(KIND_A, d)); else set_m0(l_a + d * 4096); }
                    }
                    __builtin_amdgcn_sched_barrier(0);
                }
        }
        if (LOAD_B) next_b(kt + S_AHEAD + 1);
        if (LOAD_A) next_a(kt + S_STAGES + 1);
        o_cur = o_next;
        o_next = LINES ? o_third : behind(o_next);
        if (LINES) o_third = behind(o_third);
        o_b4 = behind(o_b4);
        ++kt;
    };
    constexpr std::true_type yes{};
    constexpr std::false_type no{};
    constexpr std::integral_constant<TileKind, USUAL_TILE> usual{};
    constexpr std::integral_constant<TileKind, LAST_TILE> last{};
    constexpr std::integral_constant<TileKind, END_TILE> end{};
    while (kt + S_STAGES < nk - (LINES ? 1 : 0)) step(yes, yes, yes, usual, usual);
    // at most STAGES steps are left (LINES: and the two that load the last tiles), peeled in straight-line code (a loop over step variants makes
    // the register allocator copy accumulators between them, with none of the wait states a copy behind an MFMA needs)
    if (LINES) {
        if (kt + S_STAGES == nk - 1) step(yes, yes, yes, usual, last);
        if (kt + S_STAGES == nk) step(yes, yes, yes, last, end);
    }
    // (tile nk of B in K-steps, of which nothing is read, is not loaded where it would still be under way behind the last step)
    if ((!LINES || LINES_B || S_AHEAD > 2) && kt + S_AHEAD < nl) step(yes, no, yes, end, usual);
    if (kt + 1 < nk) step(no, no, yes, usual, usual);
    if (S_AHEAD > 2) {
        if (kt + 1 < nk) step(no, no, yes, usual, usual);
        if (kt + 1 < nk) step(no, no, yes, usual, usual);
    }
    if (kt < nk) step(no, no, no, usual, usual);
    // wait states behind the last inline-asm MFMA, as in the large kernel
    asm volatile("s_nop 7\n\ts_nop 7\n\ts_nop 7" ::: "memory");
#pragma unroll
    for (int i = 0; i < NI; ++i)
#pragma unroll
        for (int j = 0; j < 4; ++j) asm volatile("" : "+a"(acc[i][j]));
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    __builtin_amdgcn_s_barrier();   // every wavefront is past its last LDS read, and no load is on its way there, before the ring is reused below

    // Epilogue: acc[i][j][v] is row 16*i + lane%16, column 16*j + 4*(lane/16) + v of the wavefront's 16*NI x 64
    // block, staged in the wavefront's own LDS as rows of ROW_BYTES (16-byte group c of row r at c ^ (r % GROUPS))
    // and written out as 16-byte vectors, whole rows of the block contiguous.
    constexpr int ESZ = OUT_BF16 ? 2 : 4;
    constexpr int ROW_BYTES = 64 * ESZ, GROUPS = ROW_BYTES / 16, ROWS_PER_READ = 64 / GROUPS, VEC = 16 / ESZ;
    constexpr int WROWS = 16 * NI;
    static_assert(4 * WROWS * ROW_BYTES <= T::STAGES * T::STAGE_BYTES, "the staging areas fit the ring");
    char* st = reinterpret_cast<char*>(smem) + wave * (WROWS * ROW_BYTES);
    const int r_in = lane & 15, c_q = 4 * (lane >> 4);
#pragma unroll
    for (int i = 0; i < NI; ++i)
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            const int r = i * 16 + r_in;
            const int cb = (j * 16 + c_q) * ESZ;
            char* dst = st + r * ROW_BYTES + (((cb >> 4) ^ (r & (GROUPS - 1))) << 4) + (cb & 15);
            if (OUT_BF16) {
                const bf16x2 lo = __builtin_convertvector(f32x2{acc[i][j][0], acc[i][j][1]}, bf16x2);
                const bf16x2 hi = __builtin_convertvector(f32x2{acc[i][j][2], acc[i][j][3]}, bf16x2);
                uint2 v;
                v.x = __builtin_bit_cast(uint32_t, lo);
                v.y = __builtin_bit_cast(uint32_t, hi);
                *reinterpret_cast<uint2*>(dst) = v;
            } else {
                *reinterpret_cast<f32x4*>(dst) = acc[i][j];
            }
        }
    const int rd_row = lane / GROUPS, rd_cv = lane % GROUPS;
    const int64_t gcol = n0 + wn * 64 + rd_cv * VEC, row0 = m0 + wm * WROWS + rd_row;
    const int rows = gcol < N ? (int)(M - row0 < WROWS ? M - row0 : WROWS) : 0;   // of the block and of C from this lane's first one on
    char* out = reinterpret_cast<char*>(p.C) + (row0 * N + gcol) * ESZ;
    const int64_t rows_on = ROWS_PER_READ * N * ESZ;
    const auto read = [&](int e) {   // ROWS_PER_READ whole rows of the block
        const int r = rd_row + ROWS_PER_READ * e;
        return *reinterpret_cast<const u32x4*>(st + r * ROW_BYTES + ((rd_cv ^ (r & (GROUPS - 1))) << 4));
    };
    if (__builtin_expect(N % VEC == 0, 1)) {
#pragma unroll
        for (int e = 0; e < WROWS / ROWS_PER_READ; ++e, out += rows_on)
            if (ROWS_PER_READ * e < rows) __builtin_nontemporal_store(read(e), reinterpret_cast<u32x4*>(out));
    } else {   // rolled: unrolled, the code alone, which a launch has to fetch, costs 2 to 7 % (3001 x 1001 x 512 8.9 us, so 8.25)
#pragma unroll 1
        for (int e = 0; e < WROWS / ROWS_PER_READ; ++e, out += rows_on)
            if (ROWS_PER_READ * e < rows) store_ragged<OUT_BF16>(out, read(e), N - gcol);
    }
}

template <bool OUT_BF16>
__global__ void __launch_bounds__(THREADS) gemm_bf16_nk128_kernel(const GemmArgs p) { int tm, tn; tile_of(blockIdx.x, p, &tm, &tn); small_gemm_body<4, false, OUT_BF16, false>(p, tm, tn); }
template <bool OUT_BF16>
__global__ void __launch_bounds__(THREADS) gemm_bf16_kn128_kernel(const GemmArgs p) { int tm, tn; tile_of(blockIdx.x, p, &tm, &tn); small_gemm_body<4, true, OUT_BF16, false>(p, tm, tn); }
// 256 x 128 tiles
template <bool OUT_BF16>
__global__ void __launch_bounds__(THREADS) gemm_bf16_nk256x128_kernel(const GemmArgs p) { int tm, tn; tile_of(blockIdx.x, p, &tm, &tn); small_gemm_body<8, false, OUT_BF16, false>(p, tm, tn); }
template <bool OUT_BF16>
__global__ void __launch_bounds__(THREADS) gemm_bf16_kn256x128_kernel(const GemmArgs p) { int tm, tn; tile_of(blockIdx.x, p, &tm, &tn); small_gemm_body<8, true, OUT_BF16, false>(p, tm, tn); }
// K not a multiple of 64, lines of A and B, or of A alone, as they lie in memory
template <bool B_KN, bool OUT_BF16>
__global__ void __launch_bounds__(THREADS) gemm_bf16_lines128_kernel(const GemmArgs p) { int tm, tn; tile_of(blockIdx.x, p, &tm, &tn); small_gemm_body<4, B_KN, OUT_BF16, true, true>(p, tm, tn); }
template <bool B_KN, bool OUT_BF16>
__global__ void __launch_bounds__(THREADS) gemm_bf16_lines256x128_kernel(const GemmArgs p) { int tm, tn; tile_of(blockIdx.x, p, &tm, &tn); small_gemm_body<8, B_KN, OUT_BF16, true, true>(p, tm, tn); }
// K >= 64 and not a multiple of 64
template <bool OUT_BF16>
__global__ void __launch_bounds__(THREADS) gemm_bf16_nk128_tail_kernel(const GemmArgs p) { int tm, tn; tile_of(blockIdx.x, p, &tm, &tn); small_gemm_body<4, false, OUT_BF16, true>(p, tm, tn); }
template <bool OUT_BF16>
__global__ void __launch_bounds__(THREADS) gemm_bf16_kn128_tail_kernel(const GemmArgs p) { int tm, tn; tile_of(blockIdx.x, p, &tm, &tn); small_gemm_body<4, true, OUT_BF16, true>(p, tm, tn); }
template <bool OUT_BF16>
__global__ void __launch_bounds__(THREADS) gemm_bf16_nk256x128_tail_kernel(const GemmArgs p) { int tm, tn; tile_of(blockIdx.x, p, &tm, &tn); small_gemm_body<8, false, OUT_BF16, true>(p, tm, tn); }
template <bool OUT_BF16>
__global__ void __launch_bounds__(THREADS) gemm_bf16_kn256x128_tail_kernel(const GemmArgs p) { int tm, tn; tile_of(blockIdx.x, p, &tm, &tn); small_gemm_body<8, true, OUT_BF16, true>(p, tm, tn); }

// ------------------------------------------------------------------------- large tiles, the last round in small ones
// A product of more than 256 large tiles runs in rounds of 256 (one per compute unit), and the last round costs as much
// as a full one however few tiles are in it: 4100 x 4200 has 289, of which 33 kept 256 compute units waiting.  Here the
// whole rounds are large tiles and what is left over is cut into its 128 x 128 quadrants, which spread over the chip and
// start as the large tiles of the last whole round end.  The large tiles are the first `nlarge` of a list that has the
// tiles inside C first and those its edges cut through last, so quadrants that lie outside C altogether (they return at
// once) are saved too.  Every element is summed in the same order whichever tile holds it.
struct MixedArgs {
    GemmArgs g;                 // tiles_m, tiles_n: 256 x 256
    int32_t full_m, full_n;     // tiles inside C altogether
    int32_t nlarge;             // a multiple of 256
    int32_t per_xcd;            // left-over tiles an XCD takes the quadrants of
};

template <bool B_KN, bool OUT_BF16, bool K_TAIL>
__device__ __forceinline__ void mixed_gemm_body(const MixedArgs& p) {
    const int id = blockIdx.x, x = id & 7;
    const bool large = id < p.nlarge;
    // XCD x: the x-th eighth of the large tiles, then the quadrants of the x-th eighth of the rest, four in a row of one tile
    const int j = (id - p.nlarge) >> 3;
    const int lin = large ? x * (p.nlarge >> 3) + (id >> 3) : p.nlarge + x * p.per_xcd + (j >> 2);
    const int inside = p.full_m * p.full_n, right = p.full_m * (p.g.tiles_n - p.full_n);
    int tm, tn;
    if (lin < inside) tile_in_list(lin, p.full_m, p.full_n, 8, &tm, &tn);
    else if (lin < inside + right) { tm = lin - inside; tn = p.full_n; }
    else { tm = p.full_m; tn = lin - inside - right; }
    if (large) {
        fast_gemm_body<B_KN, OUT_BF16, K_TAIL>(p.g, tm, tn);
        return;
    }
    if (lin >= p.g.tiles_m * p.g.tiles_n) return;
    tm = 2 * tm + (j & 1);
    tn = 2 * tn + ((j >> 1) & 1);
    if ((int64_t)tm * SBM >= p.g.M || (int64_t)tn * SBN >= p.g.N) return;
    small_gemm_body<4, B_KN, OUT_BF16, K_TAIL>(p.g, tm, tn);
}
template <bool OUT_BF16>
__global__ void __launch_bounds__(THREADS) gemm_bf16_nk_mixed_kernel(const MixedArgs p) { mixed_gemm_body<false, OUT_BF16, false>(p); }
template <bool OUT_BF16>
__global__ void __launch_bounds__(THREADS) gemm_bf16_kn_mixed_kernel(const MixedArgs p) { mixed_gemm_body<true, OUT_BF16, false>(p); }
template <bool OUT_BF16>
__global__ void __launch_bounds__(THREADS) gemm_bf16_nk_mixed_tail_kernel(const MixedArgs p) { mixed_gemm_body<false, OUT_BF16, true>(p); }
template <bool OUT_BF16>
__global__ void __launch_bounds__(THREADS) gemm_bf16_kn_mixed_tail_kernel(const MixedArgs p) { mixed_gemm_body<true, OUT_BF16, true>(p); }

// ------------------------------------------------------------------------- few tiles: K split over a workgroup
// Products whose 128 x 128 tiles occupy a small part of the chip.  Each of those tiles is bound by what one compute unit
// loads, so the time is that of (rows + columns of a tile) x K and the idle compute units do not help; here tiles are
// 64 x 64 or smaller, and the wavefronts of a workgroup take the 64-wide slices of K in turn (slice s belongs to
// wavefront s mod WAVES), each summing the whole tile over its slices.  A wavefront has LDS of its own for SETS slices,
// filled by LDS-direct loads in the other kernels' layout, and waits for them by itself: no barrier in the loop.  (Loaded
// straight into fragments, neighbouring lanes read different rows, and the compute unit's cache serves 16 instead of 64
// bytes a cycle.)  The partial tiles are added through LDS in the order of the wavefronts: the result depends on the
// sizes only.
template <int MI, int NJ, int WAVES_, int SETS_> struct SplitTile {
    static constexpr int MI_ = MI, NJ_ = NJ, WAVES = WAVES_, SETS = SETS_;
    static constexpr int TM = 16 * MI, TN = 16 * NJ;
    static constexpr int LA = TM / 8, LB = TN / 8, PER_SET = LA + LB;       // load instructions of a slice, 1 KiB each
    static constexpr int ITEMS = MI * NJ * 64;                              // 16-byte pieces of a partial tile
    static constexpr int LDS_BYTES = WAVES * (SETS * PER_SET * 1024 > ITEMS * 16 ? SETS * PER_SET * 1024 : ITEMS * 16);
    static_assert(LDS_BYTES <= FAST_LDS_BYTES, "the slices in flight fit the LDS");
};

// B stored [K,N]: a slice is 64 rows (k) of TN columns; 16-byte group c of row k sits at c ^ kn_swz_split(k), which sends
// the rows that half a wavefront's transposing read touches to different 32-byte windows of LDS's 256 bytes.
template <int NJ> __device__ __forceinline__ int kn_swz_split(int k) {
    return NJ == 4 ? (((k >> 3) & 1) << 2) | (((k >> 1) & 1) << 1) : ((k >> 3) & 1) << 1;
}

// tile_of() of at most 256 tiles.  A product of 4 us feels two divisions (0.1 us of 512 x 512 x 512): they are multiplications by
// 2^32 / divisor, rounded up, exact as long as dividend x divisor is below 2^32.
struct SplitOrder {
    uint32_t rows, per_group, last;        // tile-rows of a group, its tiles, tile-rows of the last group
    uint32_t by_group, by_rows, by_last;
};
__device__ __forceinline__ void tile_of(uint32_t id, const GemmArgs& p, const SplitOrder& o, int* tm, int* tn) {
    const uint32_t total = p.tiles_m * p.tiles_n, x = id & 7, over = total & 7;
    const uint32_t lin = x * (total >> 3) + (x < over ? x : over) + (id >> 3);
    const uint32_t grp = o.per_group > 1 ? __umulhi(lin, o.by_group) : lin, in = lin - grp * o.per_group;
    const bool last = (grp + 1) * o.rows >= (uint32_t)p.tiles_m;
    const uint32_t high = last ? o.last : o.rows, col = high > 1 ? __umulhi(in, last ? o.by_last : o.by_rows) : in;
    *tm = grp * o.rows + in - col * high;
    *tn = col;
}

template <class T, bool B_KN, bool K_TAIL>
__device__ __forceinline__ void split_gemm_body(const GemmArgs& p, int tm, int tn, bool out_bf16) {
    constexpr int MI = T::MI_, NJ = T::NJ_, WAVES = T::WAVES, SETS = T::SETS, LA = T::LA, LB = T::LB;
    static_assert(!B_KN || NJ == 2 || NJ == 4, "the [K,N] swizzle is for rows of 64 or 128 bytes");
    extern __shared__ u32x4 smem[];            // [wavefront][set][rows of A, B]; then [wavefront][ITEMS]
    __builtin_amdgcn_s_setprio(3);
    const int tid = threadIdx.x, lane = tid & 63, q = lane >> 4, r = lane & 15;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int64_t m0 = (int64_t)tm * T::TM, n0 = (int64_t)tn * T::TN, M = p.M, N = p.N, K = p.K;

    const int slices = (int)((K + BK - 1) / BK);
    const int again = K_TAIL ? (int)((int64_t)slices * BK - K) : 0;    // the last slice begins at K - 64, as in the tiled kernels
    // Load d of an operand: 8 rows of 128 bytes, lane -> row 8*d + lane/8, stored group lane%8 (see the large kernel).
    // Rows past the edge re-read the last one.
    uint32_t a_off[LA], b_off[LB];
#pragma unroll
    for (int d = 0; d < LA; ++d) {
        const int row = 8 * d + (lane >> 3);
        const int64_t last = M - 1 - m0;
        a_off[d] = (uint32_t)(((row < last ? row : last) * K + 8 * ((lane & 7) ^ ((row >> 1) & 7))) * 2);
    }
#pragma unroll
    for (int d = 0; d < LB; ++d) {
        if (B_KN) {   // TN/8 groups a row: lane -> row (512/TN)*d + lane/(TN/8); groups past the last column re-read the last one
            const int krow = (512 / T::TN) * d + lane / LB;
            const int64_t grp = (lane % LB) ^ kn_swz_split<NJ>(krow), last = (N - n0) / 8 - 1;
            b_off[d] = (uint32_t)((krow * N + (grp < last ? grp : last) * 8) * 2);
        } else {
            const int row = 8 * d + (lane >> 3);
            const int64_t last = N - 1 - n0;
            b_off[d] = (uint32_t)(((row < last ? row : last) * K + 8 * ((lane & 7) ^ ((row >> 1) & 7))) * 2);
        }
    }
    const char* const base_a = reinterpret_cast<const char*>(p.A + m0 * K);
    const char* const base_b = reinterpret_cast<const char*>(B_KN ? p.B + n0 : p.B + n0 * K);
    constexpr int SET_BYTES = T::PER_SET * 1024, B_BYTES = LA * 1024;       // B's place in a set
    const uint32_t lds0 = (uint32_t)(size_t)(__attribute__((address_space(3))) char*)smem + wave * (SETS * SET_BYTES);
    const char* const mine = reinterpret_cast<const char*>(smem) + wave * (SETS * SET_BYTES);
    auto load = [&](uint32_t lds, const char* sbase, uint32_t voff) {
        asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, %2" ::"s"(lds), "v"(voff), "s"(sbase) : "memory");
    };
    auto fetch = [&](int set, int slice) {
        // behind the last slice every lane reads the same 16 bytes, for nothing: the waits below count loads
        const bool there = slice < slices;
        const uint32_t mask = there ? ~0u : 0u;
        const int64_t k0 = there ? (K_TAIL && slice == slices - 1 ? K - BK : (int64_t)slice * BK) : 0;
        const char* const from_a = base_a + 2 * k0;
        const char* const from_b = base_b + 2 * (B_KN ? k0 * N : k0);
#pragma unroll
        for (int d = 0; d < LA; ++d) load(lds0 + set * SET_BYTES + d * 1024, from_a, a_off[d] & mask);
#pragma unroll
        for (int d = 0; d < LB; ++d) load(lds0 + set * SET_BYTES + B_BYTES + d * 1024, from_b, b_off[d] & mask);
    };
    f32x4 acc[MI][NJ];
#pragma unroll
    for (int i = 0; i < MI; ++i)
#pragma unroll
        for (int j = 0; j < NJ; ++j) {
            acc[i][j] = f32x4{0.f, 0.f, 0.f, 0.f};
            // Where the compiler sees constants it takes the loop's vectors apart into single registers and puts each together again for
            // the next slice: 64 x 64 tiles then took up to 252 registers (now 152 - 172), and large tiles with such pieces behind
            // them 428 (now 388 and 396, like the other large ones), which channels beside a product did not fit with.
            asm volatile("" : "+v"(acc[i][j]));
        }
    u32x4 fa[2][MI], fb[2][NJ];
    auto read = [&](int set) {
        const u32x4* sa = reinterpret_cast<const u32x4*>(mine + set * SET_BYTES);
        const u32x4* sb = reinterpret_cast<const u32x4*>(mine + set * SET_BYTES + B_BYTES);
#pragma unroll
        for (int h = 0; h < 2; ++h) {
#pragma unroll
            for (int i = 0; i < MI; ++i) fa[h][i] = sa[swz64(16 * i + r, 4 * h + q)];
#pragma unroll
            for (int j = 0; j < NJ; ++j) {
                if (!B_KN) {
                    fb[h][j] = sb[swz64(16 * j + r, 4 * h + q)];
                } else {      // two transposing reads, as in the large kernel
                    typedef s16x4 __attribute__((address_space(3))) * tr_ptr;
                    const int krow = 32 * h + 8 * q + (r >> 2), grp = 2 * j + ((r & 3) >> 1);
                    s16x4 x[2];
#pragma unroll
                    for (int u = 0; u < 2; ++u)
                        x[u] = __builtin_amdgcn_ds_read_tr16_b64_v4i16((tr_ptr)((lds_bytes)(const char*)sb + (krow + 4 * u) * (2 * T::TN) +
                                                                               ((grp ^ kn_swz_split<NJ>(krow + 4 * u)) << 4) + 8 * (r & 1)));
                    fb[h][j] = __builtin_bit_cast(u32x4, __builtin_shufflevector(x[0], x[1], 0, 1, 2, 3, 4, 5, 6, 7));
                }
            }
        }
    };
    auto multiply = [&](int slice) {
        const u32x4 zero = {0u, 0u, 0u, 0u};
#pragma unroll
        for (int h = 0; h < 2; ++h) {
            const bool keep = !K_TAIL || slice < slices - 1 || 4 * h + q >= again / 8;
#pragma unroll
            for (int i = 0; i < MI; ++i)
#pragma unroll
                for (int j = 0; j < NJ; ++j)      // B first: a lane's 4 results are C[row lane%16][4 consecutive columns]
                    acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, keep ? fb[h][j] : zero),
                                                                        __builtin_bit_cast(bf16x8, keep ? fa[h][i] : zero), acc[i][j], 0, 0, 0);
        }
    };
#pragma unroll
    for (int t = 0; t < SETS; ++t) fetch(t, wave + t * WAVES);
    for (int slice = wave; slice < slices;) {
#pragma unroll
        for (int t = 0; t < SETS; ++t) {
            if (t > 0 && slice >= slices) break;
            asm volatile("s_waitcnt vmcnt(%0)" ::"n"((SETS - 1) * T::PER_SET) : "memory");     // loads complete in issue order
            read(t);
            asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");     // the fragments are in registers: the set may be filled again
            __builtin_amdgcn_sched_barrier(0);
            fetch(t, slice + SETS * WAVES);
            multiply(slice);
            slice += WAVES;
        }
    }
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    __syncthreads();       // nothing is in flight into LDS, and nobody reads a slice any more

    f32x4* const partial = reinterpret_cast<f32x4*>(smem);
#pragma unroll
    for (int i = 0; i < MI; ++i)
#pragma unroll
        for (int j = 0; j < NJ; ++j) partial[wave * T::ITEMS + (i * NJ + j) * 64 + lane] = acc[i][j];
    __syncthreads();
    const bool through = T::TM >= 32 && !out_bf16 && (((uintptr_t)p.C | (uintptr_t)(4 * N)) & 63) == 0;
    for (int item = tid; item < T::ITEMS; item += 64 * WAVES) {
        f32x4 x = partial[item];
#pragma unroll
        for (int w = 1; w < WAVES; ++w) x = x + partial[w * T::ITEMS + item];
        const int ij = item >> 6;
        const int64_t row = m0 + 16 * (ij / NJ) + r, col = n0 + 16 * (ij % NJ) + 4 * q;
        if (row >= M || col >= N) continue;
        // element-aligned stores, as in store_ragged
        if (out_bf16) {
            uint16_t* out = reinterpret_cast<uint16_t*>(p.C) + row * N + col;
            u32x2_aligned2 v;
            v[0] = __builtin_bit_cast(uint32_t, __builtin_convertvector(f32x2{x[0], x[1]}, bf16x2));
            v[1] = __builtin_bit_cast(uint32_t, __builtin_convertvector(f32x2{x[2], x[3]}, bf16x2));
            if (col + 4 <= N) *reinterpret_cast<u32x2_aligned2*>(out) = v;
            else
#pragma unroll
                for (int e = 0; e < 3; ++e)
                    if (col + e < N) out[e] = (uint16_t)(v[e >> 1] >> (16 * (e & 1)));
        } else {
            float* out = reinterpret_cast<float*>(p.C) + row * N + col;
            if (through) store_through(reinterpret_cast<char*>(out), __builtin_bit_cast(u32x4, x));
            else if (col + 4 <= N) *reinterpret_cast<u32x4_aligned2*>(out) = __builtin_bit_cast(u32x4, x);
            else
#pragma unroll
                for (int e = 0; e < 3; ++e)
                    if (col + e < N) out[e] = x[e];
        }
    }
}

template <class T, bool B_KN, bool K_TAIL>
__global__ void __launch_bounds__(64 * T::WAVES) gemm_bf16_split_kernel(const GemmArgs p, const SplitOrder order, const int out_bf16) {
    int tm, tn;
    tile_of(blockIdx.x, p, order, &tm, &tn);
    split_gemm_body<T, B_KN, K_TAIL>(p, tm, tn, out_bf16 != 0);
}

// ------------------------------------------------------------------------- large tiles, the last round in split pieces
// As above with 64 x 64 pieces of the left-over tiles, K split over a workgroup's wavefronts: where few tiles are left over, their
// quadrants occupy a part of the chip and each is bound by what one compute unit loads.  The pieces inside C are numbered without
// gaps: a tile at the edge may hold few of them.  Their sums are added wavefront by wavefront, the large tiles' along K: equal rows of A
// give rows of C that may differ in the fp32 sums' rounding where one of them lies in a piece (rel 5e-8).
typedef SplitTile<4, 4, 4, 2> Piece;
struct PiecesArgs {
    GemmArgs g;                 // tiles_m, tiles_n: 256 x 256
    int32_t full_m, full_n;     // tiles inside C altogether
    int32_t nlarge;             // a multiple of 256
    int32_t edge_m, edge_n;     // pieces across a tile that C's lower, right edge cuts through
    int32_t inside, right;      // pieces of the tiles left over inside C and at its right edge; the lower edge's follow
    int32_t first_right, first_low;     // tiles of either edge among the large ones
    int32_t pieces;
    int32_t lead;               // pieces in front of the large tiles, a multiple of 8; the others follow them
};
constexpr int kPiecesAcross = BM / Piece::TM;

template <bool B_KN, bool OUT_BF16, bool K_TAIL>
__device__ __forceinline__ void pieces_gemm_body(const PiecesArgs& p) {
    static_assert(64 * Piece::WAVES == THREADS && BM == BN && Piece::TM == Piece::TN, "pieces and large tiles in one launch");
    const int id = blockIdx.x, x = id & 7, behind = id - p.lead;
    if (behind >= 0 && behind < p.nlarge) {
        const int lin = x * (p.nlarge >> 3) + (behind >> 3), inside = p.full_m * p.full_n, right = p.full_m * (p.g.tiles_n - p.full_n);
        int tm, tn;
        if (lin < inside) tile_in_list(lin, p.full_m, p.full_n, 8, &tm, &tn);
        else if (lin < inside + right) { tm = lin - inside; tn = p.full_n; }
        else { tm = p.full_m; tn = lin - inside - right; }
        fast_gemm_body<B_KN, OUT_BF16, K_TAIL>(p.g, tm, tn);
        return;
    }
    constexpr int A = kPiecesAcross;
    const int over = p.pieces & 7;
    int j = x * (p.pieces >> 3) + (x < over ? x : over) + ((behind < 0 ? id : id - p.nlarge) >> 3);
    int tm, tn;
    if (j < p.inside) {
        tile_in_list(p.nlarge + j / (A * A), p.full_m, p.full_n, 8, &tm, &tn);
        tm = tm * A + j % A;
        tn = tn * A + j / A % A;
    } else if ((j -= p.inside) < p.right) {             // down the strip, then across
        const int rows = (p.full_m - p.first_right) * A;
        tm = p.first_right * A + j % rows;
        tn = p.full_n * A + j / rows;
    } else {                                            // along the strip, edge_m pieces high
        j -= p.right;
        tm = p.full_m * A + j % p.edge_m;
        tn = p.first_low * A + j / p.edge_m;
    }
    split_gemm_body<Piece, B_KN, K_TAIL>(p.g, tm, tn, OUT_BF16);
}
template <bool OUT_BF16>
__global__ void __launch_bounds__(THREADS) gemm_bf16_nk_pieces_kernel(const PiecesArgs p) { pieces_gemm_body<false, OUT_BF16, false>(p); }
template <bool OUT_BF16>
__global__ void __launch_bounds__(THREADS) gemm_bf16_kn_pieces_kernel(const PiecesArgs p) { pieces_gemm_body<true, OUT_BF16, false>(p); }
template <bool OUT_BF16>
__global__ void __launch_bounds__(THREADS) gemm_bf16_nk_pieces_tail_kernel(const PiecesArgs p) { pieces_gemm_body<false, OUT_BF16, true>(p); }
template <bool OUT_BF16>
__global__ void __launch_bounds__(THREADS) gemm_bf16_kn_pieces_tail_kernel(const PiecesArgs p) { pieces_gemm_body<true, OUT_BF16, true>(p); }

// Lets a kernel have a compute unit's whole LDS: set once per kernel (and per device: a process may drive several); a
// failure is not remembered.
template <auto KERNEL>
int allow_lds() {
    static std::atomic<uint64_t> done_on_device{0};
    int dev = 0;
    if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev > 63) dev = 63;
    const uint64_t bit = uint64_t{1} << dev;
    if (dev == 63 || !(done_on_device.load(std::memory_order_acquire) & bit)) {
        const hipError_t attr = hipFuncSetAttribute(reinterpret_cast<const void*>(KERNEL),
                                                    hipFuncAttributeMaxDynamicSharedMemorySize, FAST_LDS_BYTES);
        if (attr != hipSuccess) return lagom::fail(LAGOM_EHIP, "gemm: cannot raise the LDS limit: %s", hipGetErrorString(attr));
        done_on_device.fetch_or(bit, std::memory_order_release);
    }
    return LAGOM_OK;
}

template <auto KERNEL, class ARGS>
int launch_fast(const ARGS& a, dim3 grid, hipStream_t st) {
    if (int rc = allow_lds<KERNEL>()) return rc;
    hipLaunchKernelGGL(KERNEL, grid, dim3(THREADS), FAST_LDS_BYTES, st, a);
    return LAGOM_OK;
}

// The block of tiles that an XCD works on at a time: n tiles, near to square in rows of A and of B; `rows` of them is the height of
// the list's groups, all of (nearly) one height.  (A product of few tile-columns: whole tile-rows, rows = 1.)
struct Block { int32_t rows; int64_t high, across; };
Block block_of(int64_t tiles_m, int64_t tiles_n, int64_t tile_m, int64_t tile_n, int64_t n) {
    const int64_t square = n * tile_n / tile_m;
    int64_t rows = 1;
    while (rows * (rows + 1) < square) ++rows;          // to the nearest of the square root
    if (rows * tiles_n < n) return {1, (n + tiles_n - 1) / tiles_n, tiles_n};
    const int64_t groups = (tiles_m + rows / 2) / rows;
    rows = groups > 1 ? (tiles_m + groups - 1) / groups : tiles_m;
    const int64_t high = rows < n ? rows : n;
    return {(int32_t)rows, high, (n + high - 1) / high};
}
// Up to this K what two XCDs both read is too little to matter, and the orders are the previous ones: columns of 8, dealt out to
// the XCDs only where their number is a multiple of 8, and for split products the shorter side of C first.  us, those orders ->
// blocks:
//   64 x 64 split tiles      1024 x 1024 x 512 6.4 -> 6.3, x 1024 8.3 -> 7.6, x 4096 16.8 -> 15.2; 384 x 512 x 7040 13.7 -> 12.8
//   32 x 32 split tiles      512 x 512 x 512 4.20 -> 4.20, x 4096 9.6 -> 8.9
//   128 x 128 tiles          170 x 6953 x 1448 17.3 -> 16.0; 1152 x 1408 x 3968 26.4 -> 24.9
// Larger tiles, bound by their matrix cores, keep the previous orders for every K: 3484 x 4296 x 2048 50.3 -> 48.2, but 3400 x
// 3400 x 4096 80.0 -> 81.8 and 5632 x 1280 x 7168 91.7 -> 94.0, 26 shapes 0.3 % in the mean.
constexpr int64_t kShortK = 512;
int64_t at_a_time(int64_t tiles) { return tiles < 32 * 8 ? (tiles + 7) / 8 : 32; }      // tiles an XCD's 32 compute units work on
Block tile_block(int64_t tiles_m, int64_t tiles_n, int64_t tile_m, int64_t tile_n, int64_t K) {
    const int64_t tiles = tiles_m * tiles_n, n = at_a_time(tiles);
    if (K > kShortK && tiles % 8 && tile_m == SBM) return block_of(tiles_m, tiles_n, tile_m, tile_n, n);
    if (tiles % 8) return {0, 1, n};
    const int64_t high = tiles_m < 8 ? tiles_m < n ? tiles_m : n : 8 < n ? 8 : n;
    return {8, high, (n + high - 1) / high};
}
// Split products, whose shorter side of C comes first otherwise, take a block where it reads at most 4/5 of what that order does.  us, that
// order -> blocks: 11 x 18 tiles of 64 x 32 at K = 8192 (0.6 of the reading) 19.8 -> 18.7, 16 x 10 of 16 x 32 at 4096 (0.64) 7.6 -> 7.1, 16 x 4 at 8192 (0.8)
// 14.0 -> 13.0; but 24 x 8 tiles of 32 x 32 at K = 8192 (0.91) 12.9 -> 13.5, 13 x 2 of 16 x 32 at 6592 (1.0) 7.5 -> 8.8, 3 x 8 at 4048 (1.2) 7.2 -> 8.2.
Block split_block(int64_t tiles_m, int64_t tiles_n, int64_t tile_m, int64_t tile_n, int64_t K) {
    const int64_t n = at_a_time(tiles_m * tiles_n);
    const bool m_first = tiles_m <= tiles_n;
    const int64_t inner = m_first ? tiles_m : tiles_n, in = inner < n ? inner : n, across = (n + in - 1) / in;
    const Block shorter_first{(int32_t)(m_first ? tiles_m : 1), m_first ? in : across, m_first ? across : in};
    if (K <= kShortK) return shorter_first;
    const Block block = block_of(tiles_m, tiles_n, tile_m, tile_n, n);
    auto reads = [&](const Block& b) { return b.high * tile_m + b.across * tile_n; };
    return 5 * reads(block) <= 4 * reads(shorter_first) ? block : shorter_first;
}

template <class T, bool B_KN, bool K_TAIL>
int launch_split_kernel(const GemmArgs& a, bool out_bf16, hipStream_t st) {
    constexpr auto kernel = gemm_bf16_split_kernel<T, B_KN, K_TAIL>;
    if (int rc = allow_lds<kernel>()) return rc;
    const dim3 grid((unsigned)(a.tiles_m * a.tiles_n));
    const uint32_t rows = (uint32_t)split_block(a.tiles_m, a.tiles_n, T::TM, T::TN, a.K).rows, last = (uint32_t)a.tiles_m - (uint32_t)(a.tiles_m - 1) / rows * rows;
    auto by = [](uint32_t d) { return (uint32_t)(((uint64_t{1} << 32) + d - 1) / d); };        // 2^32 does not fit: not used for d = 1
    const SplitOrder order{rows, rows * (uint32_t)a.tiles_n, last, by(rows * (uint32_t)a.tiles_n), by(rows), by(last)};
    hipLaunchKernelGGL(kernel, grid, dim3(64 * T::WAVES), T::LDS_BYTES, st, a, order, out_bf16 ? 1 : 0);
    return LAGOM_OK;
}
template <class T>
int launch_split(GemmArgs a, bool b_is_nk, bool out_bf16, hipStream_t st) {
    a.tiles_m = (int32_t)((a.M + T::TM - 1) / T::TM);
    a.tiles_n = (int32_t)((a.N + T::TN - 1) / T::TN);
    const bool tail = a.K % BK != 0;
    if (b_is_nk) return tail ? launch_split_kernel<T, false, true>(a, out_bf16, st) : launch_split_kernel<T, false, false>(a, out_bf16, st);
    return tail ? launch_split_kernel<T, true, true>(a, out_bf16, st) : launch_split_kernel<T, true, false>(a, out_bf16, st);
}

constexpr int kRound = 256;         // workgroups in a round: one per compute unit

// The smallest tile that still covers C in one round of workgroups (256 compute units): 128 x 128, else
// 256 x 128, else 256 x 256.  Fewer, larger tiles would leave compute units idle; smaller tiles in several
// rounds lose more to their lower arithmetic intensity than they gain.
enum Tiling { TILE_128x128, TILE_256x128, TILE_256x256 };
Tiling choose_tiling(int64_t M, int64_t N, int64_t K) {
    if (K < BK || K > FAST_MAX_K) return TILE_256x256;
    const int64_t cols = (N + SBN - 1) / SBN;
    if (((M + SBM - 1) / SBM) * cols <= 256) return TILE_128x128;
    if (((M + MBM - 1) / MBM) * cols <= 256) return TILE_256x128;
    return TILE_256x256;
}

// The smallest tile that covers C in one round is the fastest here too, whatever it loads in all: a workgroup's time is that
// of its own loads, (rows + columns of its tile) x K at 60 - 110 GB/s with the launch in it (what follows, divided), less the
// more compute units load.  us, 128 x 128 tiles -> 64 x 64 | 64 x 32 | 32 x 32 | 16 x 32:
//   33 x 1000 x 4096    23.6 -> 11.5 |  8.9 |  6.9 |  5.9 (96 workgroups)     256 x 256 x 8192   43.1 -> 18.7 | 17.7 | 13.0 | 10.9 (128)
//   512 x 512 x 512      6.3 ->  5.6 |  4.7 |  4.1 (256) |  6.3               640 x 640 x 4096   24.5 -> 14.9 | 12.0 (200) | 18.0 | 28.0
//   1024 x 1024 x 4096  25.1 -> 16.8 (256) | 26.8 | 43.8 | 77.1               40 x 8192 x 8192   42.9 -> 24.1 | 22.6 (256) | 27.4 | 31.0
// With fewer slices than wavefronts the additions at the end cost what the split gains: 64 x 64 tiles 5.4 us against 5.3 us at
// 1024 x 1024 x 256 and 5.8 against 5.9 at K = 384; 64 x 32 tiles 4.4 against 5.1 at 640 x 640 x 256, 4.3 against 4.3 at
// K = 128 and 4.3 against 4.1 at K = 64; 32 x 32 tiles 4.1 against 4.1 at 512 x 512 x 64.
struct Split {
    int (*launch)(GemmArgs, bool, bool, hipStream_t);      // null: K is not split
    int tm, tn, threads;
};
template <class T> Split split_with() { return {launch_split<T>, T::TM, T::TN, 64 * T::WAVES}; }
Split choose_split(int64_t M, int64_t N, int64_t K) {
    if (K < BK || K > FAST_MAX_K) return {};
    auto tiles = [&](int64_t tm, int64_t tn) { return ((M + tm - 1) / tm) * ((N + tn - 1) / tn); };
    if (tiles(16, 32) <= kRound) return split_with<SplitTile<1, 2, 8, 3>>();
    if (tiles(32, 32) <= kRound) return split_with<SplitTile<2, 2, 8, 2>>();
    if (K < 2 * BK) return {};
    if (tiles(64, 32) <= kRound && tiles(64, 32) <= tiles(32, 64)) return split_with<SplitTile<4, 2, 4, 3>>();
    if (tiles(32, 64) <= kRound) return split_with<SplitTile<2, 4, 4, 3>>();
    if (tiles(64, 64) <= kRound && K > 4 * BK) return split_with<SplitTile<4, 4, 4, 2>>();
    return {};
}

// A chip full of 128 x 128 tiles takes 0.39 of the time of one full of 256 x 256 tiles, so up to two rounds of quadrants
// are cheaper than one more round of large tiles.  us, large tiles only -> cut: 4096 x N x 4096 with N = 4352 (16 left
// over) 154.9 -> 113.2, 4608 (32) 157.1 -> 116.5, 5120 (64) 158.4 -> 123.0, 6144 (128, two rounds of quadrants) 164.0 ->
// 154.4; 4100 x 4200 x 2048 (33 left over, 65 quadrants) 86.1 -> 64.8; 8192 x 8448 x 8192 (fifth round, 32) 808 -> 733.
constexpr int kMaxQuadrants = 2 * kRound;

// Whether the last round of a product in large tiles is worth cutting into quadrants (their number, else 0), and how.
int choose_mixed(const GemmArgs& g, MixedArgs* out) {
    const int64_t tiles = (int64_t)g.tiles_m * g.tiles_n;
    const int rest = (int)(tiles % kRound);
    if (tiles <= kRound || rest == 0) return 0;
    MixedArgs a{g, (int32_t)(g.M / BM), (int32_t)(g.N / BN), (int32_t)(tiles - rest), (rest + 7) / 8};
    // quadrants that hold something: 4 of a tile inside C, fewer of one that an edge cuts through
    const int64_t inside = (int64_t)a.full_m * a.full_n, right = (int64_t)a.full_m * (g.tiles_n - a.full_n);
    const int halves_m = g.M % BM == 0 || g.M % BM > SBM ? 2 : 1, halves_n = g.N % BN == 0 || g.N % BN > SBN ? 2 : 1;
    int quadrants = 0;
    for (int64_t lin = a.nlarge; lin < tiles; ++lin)
        quadrants += lin < inside ? 4 : lin < inside + right ? 2 * halves_n : halves_m * (lin - inside - right < a.full_n ? 2 : halves_n);
    if (quadrants > kMaxQuadrants) return 0;
    *out = a;
    return quadrants;
}

// Whether what is left over fits one round of pieces, and how.  A round of quadrants takes 0.39 of one of large tiles, one of
// pieces 0.2 - 0.25 however few they are.  us, quadrants -> pieces:
//   4096 x 4352 x 4096 (256 pieces) 112.7 -> 103.5, x 512 24.1 -> 23.6, [K,N] x 1024 38.1 -> 35.6
//   4352 x 4096 x 2048 [K,N] 63.4 -> 58.3, fp32 70.6 -> 64.9
//   4100 x 4200 x 2056 (194 pieces) 75.7 -> 70.8, [K,N] fp32 80.9 -> 75.0
//   4153 x 7768 x 3384 [K,N] 187 -> 182
// Beside communication, which shares the compute units that all the pieces need at once, nothing is gained: makespans with ring
// shares on 8 to 64 channels 0.97 - 1.04 of the quadrants'.  As for a product of its own, 64 x 64 pieces need more than four
// slices of K: 4100 x 4200 x 320 22.5 -> 22.3.
// Half of the chip begins with a piece each, so that its large tiles store a piece's time behind the others': the results of a
// round, stored by all at one moment, cost what the memory takes for them (64 MiB of fp32 results 14 us of 78).  us, all pieces
// behind -> 64 | 128 | 192 in front, bf16, fp32:
//   one round   4100 x 4200 x 2056 [K,N] 68.9 -> 67.2 | 65.0 | 67.4, 75.8 -> 72.8 | 68.6 | 71.6   4352 x 4096 x 2048 [K,N] 61.3 -> 59.4 | 58.7 | 60.1, 66.5 -> 64.6 | 65.6 | 65.9
//               4096 x 4160 x 1024 33.6 -> 31.7 | 31.8 | 31.8, 38.4 -> 34.9 | 35.1 | 35.0         4096 x 4352 x 4096 106.1 -> 106.4 | 105.7 | 106.4, 111.6 -> 111.2 | 108.2 | 110.8
//   two         4100 x 8200 x 1024 66.6 -> 63.5 | 60.8 | 63.8, 77.7 -> 75.7 | 71.1 | 72.5         4153 x 7768 x 3384 180 -> 182 | 182 | 183, 190 -> 191 | 191 | 191
//   three       8200 x 6200 x 2048 166 -> 158 | 155 | 161, 183 -> 174 | 168 | 173                 12300 x 4100 x 1536 136 -> 136 | 137 | 137, 150 -> 150 | 150 | 151
// Beside communication a unit that hosts a channel and begins with a piece ends a piece's time later than it did, and behind a single round
// nothing is left to make up for it.  Makespans beside a ring share of eight 3.1 MiB buffers on 8 | 32 | 64 channels, all behind -> 128 in front, bf16:
//   one round   4100 x 4200 x 2056 [K,N] 253 -> 258 | 123 -> 129 | 95 -> 104    4352 x 4096 x 2048 227 -> 232 | 108 -> 115 | 81 -> 88
//   two, three  4100 x 8200 x 1024 243 -> 240 | 117 -> 113 | 90 -> 86           8200 x 6200 x 2048 296 -> 296 | 193 -> 181 | 171 -> 182
// (with the pieces behind the first 128 large tiles the same).  Quadrants in front of large tiles gain nothing (4096 x 6144 x 2048 fp32 91.4 -> 93.0).
// That is with results in the last-level cache.  With others from call to call, all behind -> 128 in front, bf16, fp32: 4100 x 4200 x 2056 [K,N] 77.0 -> 71.8, 82.5 -> 74.3,
// 4160 x 4224 x 3000 109 -> 100, 112 -> 103, 4096 x 4288 x 1024 38.6 -> 37.5, 42.7 -> 40.7, x 2048 63.3 -> 62.8, 67.2 -> 66.8, 4096 x 4160 x 1024 38.0 -> 37.9, 41.3 -> 42.1, 8200 x 6200 x 2048
// 174 -> 168, 190 -> 181, but not behind a long K, of which the two halves of the chip then load different parts: 4096 x 4160 x 4096 109 -> 113, 113 -> 119 (in the cache 104 ->
// 103, 109 -> 106), 4096 x 4224 x 4096 110 -> 112, 114 -> 117; nor where a full round of pieces goes with a single one: 4352 x 4096 x 2048 [K,N] 65.1 -> 65.1, 70.5 -> 71.2.
constexpr int kLead = kRound / 2, kLeadOfOneRound = kRound * 7 / 8, kLeadMaxK = 3072;
bool choose_pieces(const GemmArgs& g, PiecesArgs* out) {
    const int64_t tiles = (int64_t)g.tiles_m * g.tiles_n;
    const int rest = (int)(tiles % kRound);
    if (g.K <= 4 * BK || tiles <= kRound || rest == 0) return false;
    PiecesArgs a{g, (int32_t)(g.M / BM), (int32_t)(g.N / BN), (int32_t)(tiles - rest), 0, 0, 0, 0, 0, 0, 0, 0};
    auto across = [](int64_t size, int64_t tile) { return (int32_t)((size % tile + Piece::TM - 1) / Piece::TM); };
    a.edge_m = across(g.M, BM);
    a.edge_n = across(g.N, BN);
    const int64_t inside = (int64_t)a.full_m * a.full_n, right = (int64_t)a.full_m * (g.tiles_n - a.full_n);
    const int64_t in_right = a.nlarge - inside, in_low = in_right - right;       // large tiles behind those inside, behind those at the right
    a.first_right = (int32_t)(in_right > 0 ? in_right < right ? in_right : right : 0);
    a.first_low = (int32_t)(in_low > 0 ? in_low : 0);
    const int64_t n_inside = in_right < 0 ? -in_right * kPiecesAcross * kPiecesAcross : 0;
    const int64_t n_right = (right - a.first_right) * kPiecesAcross * a.edge_n;
    int64_t n_low = 0;                                   // the lower edge's tiles, the corner last
    if (g.tiles_m > a.full_m) {
        const int64_t cols = (int64_t)a.full_n * kPiecesAcross + a.edge_n;
        n_low = (cols - (int64_t)a.first_low * kPiecesAcross) * a.edge_m;
    }
    if (n_inside + n_right + n_low > kRound) return false;
    a.inside = (int32_t)n_inside; a.right = (int32_t)n_right; a.pieces = (int32_t)(n_inside + n_right + n_low);
    if (g.K < kLeadMaxK && (a.nlarge > kRound || a.pieces <= kLeadOfOneRound)) a.lead = (a.pieces < kLead ? a.pieces : kLead) & ~7;
    *out = a;
    return true;
}

// 128 x 128 tiles of a product whose K is no multiple of 64, in lines as they lie in memory.  One tile more to load and one more to wait for
// cost 0.8 us, and where A and B lie in the L2s already their lines may as well be asked for twice.  us, 64 columns from wherever they
// begin -> lines, [N,K] | [K,N], whose rows of B begin where they began; inputs in the last-level cache, others from call to call:
//   1053 x 1536 (108 tiles)  x 520  8.7 -> 8.2 | 8.3 -> 8.5    x 776 11.2 -> 9.7  | 10.0 -> 10.2   x 1304 16.0 -> 12.6 | 13.7 -> 13.3
//   200 x 8000 (126)         x 520  8.0 -> 8.2 | 8.1 -> 8.5    x 776 10.9 -> 9.7  | 9.9 -> 10.2    x 1304 15.6 -> 12.5 | 13.4 -> 13.3
//   1024 x 4096 (256)        x 520 10.1 -> 9.1 | 9.2 -> 9.2    x 776 12.2 -> 10.6 | 11.4 -> 10.9   x 1304 17.6 -> 14.6 | 15.4 -> 14.8
// The same inputs from call to call, in the L2s where they fit: 1053 x 1536 x 776 8.8 -> 9.4, x 1544 16.5 -> 13.7 | 14.2 -> 14.8, x 3080 30.9 -> 22.5 |
// 25.2 -> 24.4; 1024 x 4096 x 776 11.1 -> 10.1 | 10.0 -> 10.3, x 3080 33.6 -> 26.4 | 29.2 -> 27.7.  Inputs from HBM: 1053 x 1536 x 776 12.5 -> 11.1 |
// 11.8 -> 11.4, x 3080 39.1 -> 31.0 | 34.9 -> 30.1.
// The same way through products with K split over wavefronts, which then take neighbouring slices and a line more each, gains 7 - 20 % from K = 3000
// on and loses as much up to 2000.
// Rows that start alike gain less: of a K that is a multiple of 16 every fourth row starts at a line, of one that is a multiple of 32 every other one.
// K = 1288 to 7224 in every class, three shapes, others' time = 1: odd multiples of 8 [N,K] 0.68 - 0.82, [K,N] 0.92 - 1.00; of 16 0.71 - 0.87 and 0.94 - 1.02; of 32
// 0.81 - 0.98 and 0.97 - 1.04.
bool lines_pay(int64_t K, bool b_is_nk) { return K >= (b_is_nk ? 640 : 1280) && (b_is_nk || K % 32 != 0); }
// 256 x 128 tiles, of which LDS holds three: A alone in lines, whose loads are half a K-step in front of B's.  us, the same inputs from call
// to call | inputs from HBM:
//   2048 x 4096 (256 tiles)  x 776 17.9 -> 17.4 | 19.6 -> 18.4    x 2056 38.4 -> 34.8 | 48.3 -> 41.8    [K,N] 35.1 -> 33.9 | 43.4 -> 40.2
//   2100 x 2200 (162)        x 776 14.8 -> 15.0 | 19.7 -> 19.6    x 2056 29.8 -> 29.9 | 42.1 -> 40.8    [K,N] 30.6 -> 29.9 | 42.8 -> 40.2
//   713 x 5672 (135)         x 776 16.1 -> 15.7 | 20.7 -> 20.3    x 2056 33.5 -> 30.6 | 42.9 -> 40.4    [K,N] 33.3 -> 31.8 | 43.1 -> 39.9
// x 1032 0.94 - 1.01 ([K,N] 0.96 - 1.03), x 520 0.97 - 1.06, x 1544 0.90 - 1.00.
// Those are odd multiples of 8.  K = 1544 to 6584 in every class, 2048 x 4096, 2100 x 2176, 713 x 5632 and 2966 x 1536, others' time = 1: odd multiples of 8 [N,K]
// 0.88 - 0.96, [K,N] 0.95 - 1.03; of 16 0.89 - 1.01 and 0.97 - 1.08; of 32 0.95 - 1.08 and 1.01 - 1.17.
bool lines_of_a_pay(int64_t K, bool b_is_nk) { return K >= 1536 && K % (b_is_nk ? 32 : 16) != 0; }

constexpr int64_t kMaxDim = 1 << 24;

}  // namespace

namespace lagom {
int check_gemm_args(const void* A, const void* B, const void* C, int64_t M, int64_t N, int64_t K, int out_dt) {
    if (!A || !B || !C) return fail(LAGOM_EINVAL, "null matrix pointer");
    if (M < 1 || N < 1 || K < 1) return fail(LAGOM_EINVAL, "M, N, K must be positive");
    if (M > kMaxDim || N > kMaxDim || K > kMaxDim) return fail(LAGOM_EINVAL, "dimension above 2^24");
    if (K % 8) return fail(LAGOM_EINVAL, "K=%lld must be a multiple of 8", (long long)K);
    if (elem_size(out_dt) == 0) return fail(LAGOM_EINVAL, "unknown output dtype %d", out_dt);
    if (((uintptr_t)A | (uintptr_t)B | (uintptr_t)C) & 15) return fail(LAGOM_EALIGN, "matrix pointer not 16-byte aligned");
    return LAGOM_OK;
}
}  // namespace lagom

extern "C" int lagom_gemm_describe(int64_t M, int64_t N, int64_t K, lagom_dtype out_dt, lagom_gemm_geometry* out) {
    if (!out || M < 1 || N < 1 || K < 1 || lagom::elem_size(out_dt) == 0) return lagom::fail(LAGOM_EINVAL, "bad argument");
    // what lagom_gemm launches for this shape, by the same rules ([K,N] with N above FAST_MAX_N_KN apart, whose kernel has no quadrants)
    const double out_bytes = lagom::elem_size(out_dt);
    auto loads = [&](int64_t rows, int64_t cols) { return (double)(rows + cols) * (double)K * 2.0; };
    out->tb = 1;   // one workgroup per compute unit: LDS, or the general kernel's 256 accumulators a lane
    out->tile_k = BK;
    if (const Split split = choose_split(M, N, K); split.launch) {
        const int64_t tm = (M + split.tm - 1) / split.tm, tn = (N + split.tn - 1) / split.tn;
        out->mu = tm * tn;
        out->tile_m = split.tm; out->tile_n = split.tn; out->threads = split.threads;
        out->d_bytes = loads(split.tm, split.tn) + (double)split.tm * split.tn * out_bytes;
        const Block block = split_block(tm, tn, split.tm, split.tn, K);
        out->d_bytes_past_l2 = loads(block.high * split.tm, block.across * split.tn) / (double)at_a_time(out->mu) + (double)split.tm * split.tn * out_bytes;
        return LAGOM_OK;
    }
    const Tiling tiling = choose_tiling(M, N, K);
    const int64_t bm = tiling == TILE_128x128 ? SBM : BM, bn = tiling == TILE_256x256 ? BN : SBN;
    const int64_t tm = (M + bm - 1) / bm, tn = (N + bn - 1) / bn;
    out->mu = tm * tn;
    out->d_bytes = loads(bm, bn) + (double)bm * bn * out_bytes;
    out->tile_m = (int32_t)bm; out->tile_n = (int32_t)bn; out->threads = THREADS;
    const bool may_cut = tiling == TILE_256x256 && K >= BK && K <= FAST_MAX_K && M <= kMaxDim && N <= kMaxDim;
    const GemmArgs a{nullptr, nullptr, nullptr, M, N, K, (int32_t)tm, (int32_t)tn, 8};
    MixedArgs mixed;
    PiecesArgs cut;
    const bool pieces = may_cut && choose_pieces(a, &cut);
    const int quadrants = may_cut && !pieces ? choose_mixed(a, &mixed) : 0;
    // the block of tiles an XCD works on at a time (32 compute units per XCD): n tiles in r tile-rows and c tile-columns need
    // r A panels and c B panels between them
    const Block block = quadrants || pieces ? Block{8, tm < 8 ? tm : 8, (32 + (tm < 8 ? tm : 8) - 1) / (tm < 8 ? tm : 8)} : tile_block(tm, tn, bm, bn, K);
    out->d_bytes_past_l2 = loads(block.high * bm, block.across * bn) / (double)at_a_time(tm * tn) + (double)bm * bn * out_bytes;
    if (pieces) {      // means over the large tiles and the pieces; a tile's sixteen share its panels, and so does what an XCD takes of a strip
        const double piece_out = (double)Piece::TM * Piece::TN * out_bytes;
        const int64_t n = (cut.pieces + 7) / 8;
        auto of_strip = [&](int64_t high) {      // pieces across, the other way
            high = high < n ? high : n;
            return loads(high * Piece::TM, (n + high - 1) / high * Piece::TN) / (double)n;
        };
        const double past_l2 = (cut.inside ? cut.inside * loads(BM, BN) / (kPiecesAcross * kPiecesAcross) : 0.0) +
                               (cut.right ? cut.right * of_strip((int64_t)(cut.full_m - cut.first_right) * kPiecesAcross) : 0.0) +
                               (cut.pieces > cut.inside + cut.right ? (cut.pieces - cut.inside - cut.right) * of_strip(cut.edge_m) : 0.0);
        out->mu = cut.nlarge + cut.pieces;
        auto mean = [&](double large, double all_pieces) { return (cut.nlarge * large + all_pieces + cut.pieces * piece_out) / (double)out->mu; };
        out->d_bytes = mean(out->d_bytes, cut.pieces * loads(Piece::TM, Piece::TN));
        out->d_bytes_past_l2 = mean(out->d_bytes_past_l2, past_l2);
    }
    if (quadrants) {   // means over the large tiles and the quadrants that hold something; the four of a tile share its panels
        const double quadrant_out = (double)SBM * SBN * out_bytes;
        out->mu = mixed.nlarge + quadrants;
        auto mean = [&](double large, double quadrant) { return (mixed.nlarge * large + quadrants * quadrant) / (double)out->mu; };
        out->d_bytes = mean(out->d_bytes, loads(SBM, SBN) + quadrant_out);
        out->d_bytes_past_l2 = mean(out->d_bytes_past_l2, loads(2 * SBM, 2 * SBN) / 4.0 + quadrant_out);
    }
    return LAGOM_OK;
}

extern "C" int lagom_gemm(const void* A, const void* B, void* C, int64_t M, int64_t N, int64_t K,
                          int b_is_nk, lagom_dtype out_dt, void* hip_stream) {
    if (int rc = lagom::check_gemm_args(A, B, C, M, N, K, out_dt)) return rc;
    if (!b_is_nk && (N % 8)) return lagom::fail(LAGOM_EINVAL, "B stored [K,N] needs N to be a multiple of 8");
    const Tiling tiling = choose_tiling(M, N, K);
    if (const Split split = choose_split(M, N, K); split.launch) {
        const GemmArgs a{static_cast<const uint16_t*>(A), static_cast<const uint16_t*>(B), C, M, N, K, 0, 0, 0};
        if (int rc = split.launch(a, b_is_nk != 0, out_dt == LAGOM_BF16, static_cast<hipStream_t>(hip_stream))) return rc;
        const hipError_t e = hipGetLastError();
        if (e != hipSuccess) return lagom::fail(LAGOM_EHIP, "gemm launch: %s", hipGetErrorString(e));
        return LAGOM_OK;
    }
    if (tiling != TILE_256x256) {
        const int bm = tiling == TILE_128x128 ? SBM : MBM;
        GemmArgs a{static_cast<const uint16_t*>(A), static_cast<const uint16_t*>(B), C, M, N, K,
                   (int32_t)((M + bm - 1) / bm), (int32_t)((N + SBN - 1) / SBN), 0};
        a.rows = tile_block(a.tiles_m, a.tiles_n, bm, SBN, K).rows;
        const dim3 grid((unsigned)(a.tiles_m * a.tiles_n));
        hipStream_t st = static_cast<hipStream_t>(hip_stream);
        const bool bf = out_dt == LAGOM_BF16;
        const bool tail = K % BK != 0;
        int rc;
#define LAGOM_PICK(NAME) (bf ? launch_fast<NAME<true>>(a, grid, st) : launch_fast<NAME<false>>(a, grid, st))
        if (tiling == TILE_128x128 && tail && lines_pay(K, b_is_nk)) {
            if (b_is_nk) rc = bf ? launch_fast<gemm_bf16_lines128_kernel<false, true>>(a, grid, st) : launch_fast<gemm_bf16_lines128_kernel<false, false>>(a, grid, st);
            else rc = bf ? launch_fast<gemm_bf16_lines128_kernel<true, true>>(a, grid, st) : launch_fast<gemm_bf16_lines128_kernel<true, false>>(a, grid, st);
        } else if (tiling == TILE_256x128 && tail && lines_of_a_pay(K, b_is_nk)) {
            if (b_is_nk) rc = bf ? launch_fast<gemm_bf16_lines256x128_kernel<false, true>>(a, grid, st) : launch_fast<gemm_bf16_lines256x128_kernel<false, false>>(a, grid, st);
            else rc = bf ? launch_fast<gemm_bf16_lines256x128_kernel<true, true>>(a, grid, st) : launch_fast<gemm_bf16_lines256x128_kernel<true, false>>(a, grid, st);
        } else if (tiling == TILE_128x128) {
            if (b_is_nk) rc = tail ? LAGOM_PICK(gemm_bf16_nk128_tail_kernel) : LAGOM_PICK(gemm_bf16_nk128_kernel);
            else rc = tail ? LAGOM_PICK(gemm_bf16_kn128_tail_kernel) : LAGOM_PICK(gemm_bf16_kn128_kernel);
        } else {
            if (b_is_nk) rc = tail ? LAGOM_PICK(gemm_bf16_nk256x128_tail_kernel) : LAGOM_PICK(gemm_bf16_nk256x128_kernel);
            else rc = tail ? LAGOM_PICK(gemm_bf16_kn256x128_tail_kernel) : LAGOM_PICK(gemm_bf16_kn256x128_kernel);
        }
#undef LAGOM_PICK
        if (rc) return rc;
        const hipError_t e = hipGetLastError();
        if (e != hipSuccess) return lagom::fail(LAGOM_EHIP, "gemm launch: %s", hipGetErrorString(e));
        return LAGOM_OK;
    }
    GemmArgs a{static_cast<const uint16_t*>(A), static_cast<const uint16_t*>(B), C, M, N, K,
               (int32_t)((M + BM - 1) / BM), (int32_t)((N + BN - 1) / BN), 0};
    a.rows = tile_block(a.tiles_m, a.tiles_n, BM, BN, K).rows;
    const int64_t tiles = (int64_t)a.tiles_m * a.tiles_n;
    if (tiles > (1 << 30)) return lagom::fail(LAGOM_EINVAL, "too many tiles");
    hipStream_t st = static_cast<hipStream_t>(hip_stream);
    const dim3 grid((unsigned)tiles), block(THREADS);
    const bool bf = out_dt == LAGOM_BF16;
    const bool fast = K >= BK && K <= FAST_MAX_K && (b_is_nk || N <= FAST_MAX_N_KN);
    MixedArgs mixed;
    PiecesArgs pieces;
    if (fast && choose_pieces(a, &pieces)) {
        const dim3 both((unsigned)(pieces.nlarge + pieces.pieces));
        const bool tail = K % BK != 0;
        int rc;
#define LAGOM_PICK(NAME) (bf ? launch_fast<NAME<true>>(pieces, both, st) : launch_fast<NAME<false>>(pieces, both, st))
        if (b_is_nk) rc = tail ? LAGOM_PICK(gemm_bf16_nk_pieces_tail_kernel) : LAGOM_PICK(gemm_bf16_nk_pieces_kernel);
        else rc = tail ? LAGOM_PICK(gemm_bf16_kn_pieces_tail_kernel) : LAGOM_PICK(gemm_bf16_kn_pieces_kernel);
#undef LAGOM_PICK
        if (rc) return rc;
    } else if (fast && choose_mixed(a, &mixed)) {
        const dim3 both((unsigned)(mixed.nlarge + 32 * mixed.per_xcd));
        const bool tail = K % BK != 0;
        int rc;
#define LAGOM_PICK(NAME) (bf ? launch_fast<NAME<true>>(mixed, both, st) : launch_fast<NAME<false>>(mixed, both, st))
        if (b_is_nk) rc = tail ? LAGOM_PICK(gemm_bf16_nk_mixed_tail_kernel) : LAGOM_PICK(gemm_bf16_nk_mixed_kernel);
        else rc = tail ? LAGOM_PICK(gemm_bf16_kn_mixed_tail_kernel) : LAGOM_PICK(gemm_bf16_kn_mixed_kernel);
#undef LAGOM_PICK
        if (rc) return rc;
    } else if (fast) {
        int rc;
        if (K % BK == 0) {
            if (b_is_nk) rc = bf ? launch_fast<gemm_bf16_nk_kernel<true>>(a, grid, st) : launch_fast<gemm_bf16_nk_kernel<false>>(a, grid, st);
            else rc = bf ? launch_fast<gemm_bf16_kn_kernel<true>>(a, grid, st) : launch_fast<gemm_bf16_kn_kernel<false>>(a, grid, st);
        } else {
            if (b_is_nk) rc = bf ? launch_fast<gemm_bf16_nk_tail_kernel<true>>(a, grid, st) : launch_fast<gemm_bf16_nk_tail_kernel<false>>(a, grid, st);
            else rc = bf ? launch_fast<gemm_bf16_kn_tail_kernel<true>>(a, grid, st) : launch_fast<gemm_bf16_kn_tail_kernel<false>>(a, grid, st);
        }
        if (rc) return rc;
    } else if (b_is_nk) {
        if (bf) hipLaunchKernelGGL((gemm_bf16_general_kernel<true, true>), grid, block, 0, st, a);
        else hipLaunchKernelGGL((gemm_bf16_general_kernel<true, false>), grid, block, 0, st, a);
    } else {
        if (bf) hipLaunchKernelGGL((gemm_bf16_general_kernel<false, true>), grid, block, 0, st, a);
        else hipLaunchKernelGGL((gemm_bf16_general_kernel<false, false>), grid, block, 0, st, a);
    }
    const hipError_t e = hipGetLastError();
    if (e != hipSuccess) return lagom::fail(LAGOM_EHIP, "gemm launch: %s", hipGetErrorString(e));
    return LAGOM_OK;
}
