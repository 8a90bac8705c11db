// lagom_comm_kernel: the local data-movement step of a chunked collective on gfx950.
//
// Mapping of the paper's three resource parameters (Sec. 2.2, Sec. 3.2) onto CDNA4:
//   NC  channels   -> workgroups of the launch (each occupies wave slots of one CU),
//   NT  threads    -> workgroup size (NT/64 wavefronts),
//   C   chunk size -> the unit of work a channel takes at a time: chunk g of the byte
//                     range is moved by workgroup g mod NC.
// A wavefront's work is a sequence of units of 1 KiB (64 lanes x 16 bytes): unit n of a chunk belongs to
// wavefront n mod (NT/64), and the sequence runs on from chunk to chunk.  The walk over it lives in scalar
// registers, and the loads of the next batch of units are issued before the current batch is added and stored
// (see "the pipelined mover" below), so that a channel is bound by what a compute unit's memory pipeline
// moves (93 - 117 GB/s, loads and stores together) and not by one memory latency per batch.
// With fewer wavefronts it is bound by their instructions, of which one wavefront issues one in five cycles.
// Every byte is touched once, so stores always carry the non-temporal hint (measured on MI355X: +3..7 % and no
// write-allocate traffic in the L2 that a co-running GEMM depends on).  Loads carry it only
// when at least kStreamLoadsFromNC channels have work: with that many channels the
// kernel is bandwidth-bound and streams from HBM (+6..13 %), while with few channels it is
// latency-bound and its sources are usually still in the last-level cache, where the hint
// costs 15..30 %; and so are what a ring's steps read, on any number of channels (launch_steps).
//
// Arithmetic (reduce-copy): fp32 additions in source order, bf16 widened exactly by a
// 16-bit shift, one round-to-nearest-even at the store.  Only additions are used, so no
// fused operation can change the rounding.
#include <hip/hip_runtime.h>
#include <atomic>
#include <type_traits>
#include <utility>
#include "common.h"

namespace {

// How a buffer (a shard of a gather-copy, any buffer of a reduce-copy) is cut: chunks of C bytes, of which the last may be
// short, in units of 1 KiB that a wavefront moves with one instruction.
struct Shape {
    int64_t shard_bytes;       // bytes per source
    int64_t chunk_bytes;       // C
    uint32_t nshards;          // of a gather-copy; 1 for a reduce-copy
    uint32_t chunks;           // per shard
    uint32_t step_shards, step_chunks;   // NC chunks further: that many shards and chunks
    uint32_t full_bytes, last_bytes;  // whole 16-byte vectors of a chunk, and of a shard's last one (0: it holds none)
};
struct CommArgs {
    const char* src[LAGOM_MAX_SRCS];
    char* dst[LAGOM_MAX_DSTS];
    int32_t nsrc, ndst;
    Shape shape;
};

Shape make_shape(int64_t shard_bytes, int64_t chunk_bytes, int nshards, int nc) {
    Shape s{};
    if (chunk_bytes > shard_bytes) chunk_bytes = (shard_bytes + 15) & ~(int64_t)15;
    // Offsets in a chunk and chunk numbers are 32-bit on the device: chunks of more than 1 GiB are taken as chunks of that, and more than
    // 2^30 of them (in 16-byte chunks those of 16 GiB) as larger ones.  The result is the same.
    if (chunk_bytes > (int64_t)1 << 30) chunk_bytes = (int64_t)1 << 30;
    while ((shard_bytes + chunk_bytes - 1) / chunk_bytes * nshards > (int64_t)1 << 30) chunk_bytes *= 2;
    s.shard_bytes = shard_bytes;
    s.chunk_bytes = chunk_bytes;
    s.nshards = (uint32_t)nshards;
    s.chunks = (uint32_t)((shard_bytes + chunk_bytes - 1) / chunk_bytes);
    s.step_shards = (uint32_t)nc / s.chunks;
    s.step_chunks = (uint32_t)nc % s.chunks;
    s.full_bytes = (uint32_t)(chunk_bytes < shard_bytes ? chunk_bytes : shard_bytes) & ~15u;
    s.last_bytes = (uint32_t)(shard_bytes - (int64_t)(s.chunks - 1) * chunk_bytes) & ~15u;
    return s;
}

typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
typedef float f32x4 __attribute__((ext_vector_type(4)));

constexpr uint32_t kStreamLoadsFromNC = 128;
// Channels that have a chunk to move count: a launch of many channels over a few chunks is as latency-bound as one of few
// channels.  us, loads with the hint -> without: eight-source reduce of 248712 bf16 at (256, 128, 256 KiB), two busy channels,
// 87.6 -> 67.1; gather of two such shards at (256, 256, 512 KiB) 14.0 -> 11.0; gather of nine shards of 1092728 bf16 at
// (128, 256, 2 MiB), eighteen busy channels, 70.0 -> 46.2.
bool stream_loads(uint32_t nc, const Shape& s) {
    const uint64_t chunks = (uint64_t)s.chunks * s.nshards;
    return (chunks < nc ? chunks : nc) >= kStreamLoadsFromNC;
}

template <bool STREAM>
__device__ __forceinline__ u32x4 ld16(const char* p) {
    if (STREAM) return __builtin_nontemporal_load(reinterpret_cast<const u32x4*>(p));
    return *reinterpret_cast<const u32x4*>(p);
}
// from an element-aligned address (global loads need no more)
typedef u32x4 u32x4_element_aligned __attribute__((aligned(2)));
typedef uint32_t u32_aligned2 __attribute__((aligned(2)));
template <bool STREAM>
__device__ __forceinline__ u32x4 ld16_ragged(const char* p) {
    if (STREAM) return __builtin_nontemporal_load(reinterpret_cast<const u32x4_element_aligned*>(p));
    return *reinterpret_cast<const u32x4_element_aligned*>(p);
}
// Bytes [0, bytes) at p as a buffer: lanes beyond them store nothing and load zeros, without a branch or an access to memory.
typedef __amdgpu_buffer_rsrc_t Buffer;
__device__ __forceinline__ Buffer buffer(char* p, uint32_t bytes) { return __builtin_amdgcn_make_buffer_rsrc(p, 0, bytes, 0x00020000 /* raw, 32-bit data */); }
template <bool STREAM>
__device__ __forceinline__ u32x4 ld16(Buffer b, uint32_t at) { return __builtin_bit_cast(u32x4, __builtin_amdgcn_raw_buffer_load_b128(b, at, 0, STREAM ? 2 : 0)); }
__device__ __forceinline__ void st16(Buffer b, uint32_t at, u32x4 v) { __builtin_amdgcn_raw_buffer_store_b128(v, b, at, 0, 2 /* non-temporal */); }
__device__ __forceinline__ void st16(char* p, u32x4 v) { __builtin_nontemporal_store(v, reinterpret_cast<u32x4*>(p)); }

// bf16 is the upper half of an fp32 pattern.
__device__ __forceinline__ float bf16_lo(uint32_t w) { return __uint_as_float(w << 16); }
__device__ __forceinline__ float bf16_hi(uint32_t w) { return __uint_as_float(w & 0xffff0000u); }

// Two fp32 -> a packed pair of bf16, round to nearest, ties to even; NaN keeps a quiet payload.  v_cvt_pk_bf16_f32
// gives the bits of the integer formula (upper + round-up, NaN: upper | 0x40) on every finite sum and every bf16 NaN
// (tests/test_gpu_comm.py); it replaces 14 integer instructions per pair, which with two sources were half of a channel's VALU time.
typedef float f32x2 __attribute__((ext_vector_type(2)));
typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
__device__ __forceinline__ uint32_t bf16_round2(float lo, float hi) {
    return __builtin_bit_cast(uint32_t, __builtin_convertvector(f32x2{lo, hi}, bf16x2));
}

template <int DT>
struct Acc;

// fp32: one 16-byte vector = 4 elements
template <>
struct Acc<LAGOM_F32> {
    f32x4 a;
    __device__ __forceinline__ void init(u32x4 v) { a = __builtin_bit_cast(f32x4, v); }
    __device__ __forceinline__ void add(u32x4 v) { a = a + __builtin_bit_cast(f32x4, v); }
    __device__ __forceinline__ u32x4 result() const { return __builtin_bit_cast(u32x4, a); }
    __device__ __forceinline__ void before(uint32_t& x) const { asm volatile("" : "+v"(x) : "v"(a)); }
};

// bf16: one 16-byte vector = 8 elements, accumulated as 8 fp32
template <>
struct Acc<LAGOM_BF16> {
    float a[8];
    __device__ __forceinline__ void init(u32x4 v) {
#pragma unroll
        for (int i = 0; i < 4; ++i) { a[2 * i] = bf16_lo(v[i]); a[2 * i + 1] = bf16_hi(v[i]); }
    }
    __device__ __forceinline__ void add(u32x4 v) {
#pragma unroll
        for (int i = 0; i < 4; ++i) { a[2 * i] = a[2 * i] + bf16_lo(v[i]); a[2 * i + 1] = a[2 * i + 1] + bf16_hi(v[i]); }
    }
    __device__ __forceinline__ u32x4 result() const {
        u32x4 r;
#pragma unroll
        for (int i = 0; i < 4; ++i) r[i] = bf16_round2(a[2 * i], a[2 * i + 1]);
        return r;
    }
    __device__ __forceinline__ void before(uint32_t& x) const { asm volatile("" : "+v"(x) : "v"(a[0]), "v"(a[1]), "v"(a[2]), "v"(a[3]), "v"(a[4]), "v"(a[5]), "v"(a[6]), "v"(a[7])); }
};

// One element of a short tail (fewer than 16 bytes left at the end of the buffer).
template <int DT, class SRC, class DST>
__device__ __forceinline__ void reduce_tail_element(const SRC& src, const DST& dst, int nsrc, int ndst, int64_t byte_off) {
    if (DT == LAGOM_F32) {
        float acc = *reinterpret_cast<const float*>(src(0) + byte_off);
        for (int s = 1; s < nsrc; ++s) acc = acc + *reinterpret_cast<const float*>(src(s) + byte_off);
        for (int d = 0; d < ndst; ++d) *reinterpret_cast<float*>(dst(d) + byte_off) = acc;
    } else {
        float acc = bf16_lo(*reinterpret_cast<const uint16_t*>(src(0) + byte_off));
        for (int s = 1; s < nsrc; ++s) acc = acc + bf16_lo(*reinterpret_cast<const uint16_t*>(src(s) + byte_off));
        const uint16_t r = (uint16_t)bf16_round2(acc, acc);
        for (int d = 0; d < ndst; ++d) *reinterpret_cast<uint16_t*>(dst(d) + byte_off) = r;
    }
}

// What is left of a chunk behind whole LDS batches, moved vector by vector with the nt threads of a workgroup.
template <int DT, class SRC, class DST>
__device__ __forceinline__ void reduce_rest(const SRC& src, const DST& dst, int nsrc, int ndst, int64_t base, int64_t len, int tid, int nt) {
    const int esize = DT == LAGOM_F32 ? 4 : 2;
    const int64_t nvec = len >> 4;
    for (int64_t v = tid; v < nvec; v += nt) {
        const int64_t off = base + (v << 4);
        Acc<DT> acc;
        acc.init(ld16<false>(src(0) + off));
        for (int s = 1; s < nsrc; ++s) acc.add(ld16<false>(src(s) + off));
        const u32x4 o = acc.result();
        for (int d = 0; d < ndst; ++d) st16(dst(d) + off, o);
    }
    // fewer than 16 bytes at the very end of the buffer
    const int tail_elems = (int)(len & 15) / esize;
    if (tid < tail_elems) reduce_tail_element<DT>(src, dst, nsrc, ndst, base + (nvec << 4) + (int64_t)tid * esize);
}
template <class DST>
__device__ __forceinline__ void copy_rest(const char* src, const DST& dst, int ndst, int64_t dst_off, int64_t len, int tid, int nt) {
    const int64_t nvec = len >> 4;
    for (int64_t v = tid; v < nvec; v += nt) {
        const u32x4 x = ld16<false>(src + (v << 4));
        for (int d = 0; d < ndst; ++d) st16(dst(d) + dst_off + (v << 4), x);
    }
    const int tail = (int)(len & 15);          // only at the very end of a buffer: bytes, copied one by one
    if (tid < tail) {
        const char b = src[(nvec << 4) + tid];
        for (int d = 0; d < ndst; ++d) dst(d)[dst_off + (nvec << 4) + tid] = b;
    }
}

// ------------------------------------------------------------------ the pipelined mover
// A gather-copy of shards that are no multiple of 16 bytes: shard r starts r * shard_bytes bytes behind a 16-byte boundary of
// the destination.  Stores stay aligned: the shard's first `head` bytes and what is left behind its last whole vector are
// copied apart (at most 30 bytes a shard), and the vectors between them are read from element-aligned addresses, which on the 4-byte grid
// cost 5 - 8 % against the 16-byte grid.  (A chunk's last vector then reaches up to 14 bytes into the next chunk.)
// Of shards of an odd number of bf16 every second one starts off the 4-byte grid as well, and loads from there take 1.8 times as
// long.  GATHER_HALVES reads its vectors two bytes early and shifts them: a lane's last two bytes are the first ones of the next lane's
// vector (a DPP move), those of a unit's last vector are loaded apart, by one lane for each unit of the batch.
// Eight shards of 1000003 bf16 at (32, 256, 64 KiB): 19.1 -> 15.0 us, of 1000000 13.4.
__device__ __forceinline__ uint32_t ragged_head(uint32_t r, int64_t shard_bytes) { return (16u - ((r * (uint32_t)shard_bytes) & 15u)) & 15u; }

// A wavefront's walk over its share: chunks blockIdx, blockIdx + NC, ... of every shard in turn, and in each chunk the
// 1 KiB units wave, wave + nw, ...  All of it is wave-uniform: 32-bit arithmetic on scalar registers (gfx9 has no 64-bit
// scalar compare), and a step is straight-line code -- with loops in it the compiler's control flow holds paths on which
// a batch seems never to be waited for, and it drains the memory pipeline on each.  Which lane moves an element
// depends on the sizes, NC, NT and C only, not on how many units are in flight: the steps of one launch rely on that.
// Within a chunk a step is an addition to the offset and a subtraction from what is left; all else is done once a chunk, and stores
// go through buffers that end where the chunk does.  With the offset multiplied out for every unit, its end looked for in front of
// every load and store, and the destinations' pointers loaded behind them, a unit of eight bf16 sources took 249 instructions, 105 of them
// scalar, at five cycles each.  us, that -> this, sources of 1000000 elements at (8, NT, 32 KiB): eight bf16, NT 64 128 -> 92, 128 66.7
// -> 50.8, 256 34.4 -> 25.3, 512 20.5 -> 19.9; six fp32, 128 74.2 -> 42.5, 256 39.0 -> 29.5; sixteen bf16, 128 110 -> 81, 256 57.0 -> 43.9;
// two fp32, 64 37.1 -> 25.9; a gather of eight, 64 76.9 -> 55.3, 256 35.3 -> 32.8.  (Two destinations
// written by twenty channels of 256 threads and 2 MiB, ten shards of 1250232 bf16: 65 -> 62.)
// STEPS: the walk of a reduce-copy taken nshards times, once for each of a run of steps.
enum WalkKind { REDUCE, GATHER, GATHER_RAGGED, GATHER_HALVES, STEPS };
constexpr bool is_ragged(WalkKind k) { return k == GATHER_RAGGED || k == GATHER_HALVES; }
constexpr bool is_gather(WalkKind k) { return k == GATHER || is_ragged(k); }
template <WalkKind KIND>
struct Walk {
    static constexpr bool GATHERS = is_gather(KIND), RAGGED = is_ragged(KIND), HALVES = KIND == GATHER_HALVES;
    Shape s;
    uint32_t wave, nw;
    uint32_t c, r;                              // current chunk of the shard, shard (0 in a reduce-copy; the step of a run; behind the end s.nshards or more)
    int32_t left;                               // bytes of whole vectors from the unit to the chunk's end, none or fewer where it holds no unit
    int64_t off;                                // of the unit in the shard
    // The walk stands on something to move.  (Not a variable of its own: the compiler keeps truth values that loops hand on as masks
    // of lanes, and what depends on them in vector registers.)
    __device__ __forceinline__ bool more() const { return r < s.nshards; }
    __device__ __forceinline__ uint32_t shard() const { return more() ? r : 0; }
    __device__ __forceinline__ uint32_t room() const { return left > 0 ? left : 0; }
    __device__ __forceinline__ uint32_t last() const { return left > 0 ? left - 16 : 0; }     // from the unit to the chunk's last vector
    // GATHER_HALVES: how far the offset is off the 4-byte grid, 0 or 2
    __device__ __forceinline__ uint32_t half() const { return HALVES && left > 0 ? ragged_head(r, s.shard_bytes) & 2u : 0u; }
    __device__ __forceinline__ void open() {
        uint32_t head = 0;                      // bytes of the shard in front of its first destination vector
        if (RAGGED) {
            head = ragged_head(r, s.shard_bytes);
            const int64_t rem = s.shard_bytes - head - (int64_t)c * s.chunk_bytes;
            left = (int32_t)(rem < s.chunk_bytes ? rem > 0 ? rem : 0 : s.chunk_bytes) & ~15;
        } else {
            left = (int32_t)(c + 1 == s.chunks ? s.last_bytes : s.full_bytes);
        }
        left = more() ? left - (int32_t)(wave << 10) : 0;
        // Where there is nothing to move the walk points at the start of a shard, for loads that nobody uses.
        off = left > 0 ? (int64_t)c * s.chunk_bytes + head + (wave << 10) : 0;
    }
    __device__ __forceinline__ void first() {
        c = blockIdx.x; r = 0;
        if (is_gather(KIND)) {
            r = c / s.chunks; c -= r * s.chunks;
            if (s.full_bytes == 0) r = s.nshards;
            open();
        } else stop_at_end();
    }
    // reduce-copies: behind the last chunk (only that one can have fewer units) nothing is left
    __device__ __forceinline__ void stop_at_end() {
        if (c >= s.chunks) r = s.nshards;
        open();
        if (left <= 0) r = s.nshards;
    }
    __device__ __forceinline__ void next(uint32_t batch) {
        const uint32_t bytes = (batch * nw) << 10;
        off += bytes;
        left -= (int32_t)bytes;
        if (left > 0) return;
        if (KIND == REDUCE) {
            c += gridDim.x;                     // at most 2^30 + 65535
            stop_at_end();
            return;
        }
        if (KIND == STEPS) {
            c += gridDim.x;
            if (c >= s.chunks) { c = blockIdx.x; ++r; }
        } else {
            // a shard's short last chunk may hold no unit for this wavefront; the walk still stops there (and moves nothing)
            c += s.step_chunks; r += s.step_shards;
            if (c >= s.chunks) { c -= s.chunks; ++r; }
        }
        open();
    }
};

template <WalkKind KIND>
__device__ __forceinline__ Walk<KIND> make_walk(const Shape& s) {
    Walk<KIND> w{};
    w.s = s;
    w.wave = (uint32_t)__builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    w.nw = blockDim.x >> 6;
    return w;
}

// Where the walk reads and writes.
template <class SRC, class DST>
struct ReduceIo {                               // src(s) and dst(d) at the same offset
    const SRC& src; const DST& dst; int ndst;
    __device__ __forceinline__ const char* from(const Walk<REDUCE>& w, int s) const { return src(s) + w.off; }
    __device__ __forceinline__ int64_t to(const Walk<REDUCE>& w) const { return w.off; }
    __device__ __forceinline__ int copies(uint32_t) const { return ndst; }
    __device__ __forceinline__ char* out(uint32_t, int d) const { return dst(d); }
};
template <WalkKind KIND, class SRC, class DST>
struct GatherIo {                               // shard r goes to r * shard_bytes
    const SRC& src; const DST& dst; int ndst;
    __device__ __forceinline__ const char* from(const Walk<KIND>& w, int) const { return src(w.shard()) + w.off; }
    __device__ __forceinline__ int64_t to(const Walk<KIND>& w) const { return w.shard() * w.s.shard_bytes + w.off; }
    __device__ __forceinline__ int copies(uint32_t) const { return ndst; }
    __device__ __forceinline__ char* out(uint32_t, int d) const { return dst(d); }
};

// f(0), f(1), ... with their numbers as constants
template <class F, int... I>
__device__ __forceinline__ void for_each(const F& f, std::integer_sequence<int, I...>) { (f(std::integral_constant<int, I>{}), ...); }

// A batch: U units of one chunk, S sources each.
template <int S, int U>
struct Batch {
    u32x4 v[U][S];
    char* to;                  // the first unit in the first destination
    uint32_t r, room;          // the walk's shard or step, and bytes from there to the chunk's end
    uint32_t shift, edge;      // GATHER_HALVES: bits that the vectors are off by; in lane u, the last four bytes of unit u
};

// Copies (S = 1) and reductions of NB batches: while one is added and stored, the loads of the others are in flight.  Loads and
// stores share one in-order counter, so issuing the next loads in front of the stores also keeps the stores'
// acknowledgements off the path.  U: units per batch.
template <int DT, int S, int U, int NB, bool STREAM, bool COPY, class WALK, class IO>
__device__ __forceinline__ void move_batches(WALK w, const IO& io, uint32_t lane) {
    w.first();
    if (!w.more()) return;
    // The compiler must not see that the walks of a fused launch have their lanes' offsets in common: it would compute those of
    // every kind of step in front of the loop over the steps and hold them all, in registers that a product beside the kernel needs.
    asm volatile("" : "+v"(lane));
    uint32_t at[U];                             // a lane's offsets in a batch
#pragma unroll
    for (int u = 0; u < U; ++u) at[u] = lane * 16 + ((u * w.nw) << 10);
    // Whole shards on 128 channels and more, whose walks are short: nothing is read behind the walk's end.  us, the start of a shard read
    // there -> this, bf16 at (256, 256, 32 KiB): three chunks a channel 9.8 -> 9.7, into two destinations 13.4 -> 12.9, eight 4 MiB shards
    // into two 18.9 -> 17.6.  On few channels it costs more than it saves: eight 4 MiB shards at (8, 256, 2 MiB) 81.9 -> 87.5.
    constexpr bool BOUNDED = STREAM && WALK::GATHERS && !WALK::RAGGED;
    auto fetch = [&](Batch<S, U>& b) {          // past the chunk's end its last vector is read again (and not stored)
        b.to = io.out(w.shard(), 0) + io.to(w);
        b.r = w.r;
        b.room = w.room();
        const uint32_t last = w.last();
        const char* from[S];
#pragma unroll
        for (int s = 0; s < S; ++s) from[s] = io.from(w, s);
        if (WALK::HALVES) {
            static_assert(!WALK::HALVES || (U & (U - 1)) == 0, "lanes beyond U repeat those below it");
            const uint32_t unit_end = (((lane & (U - 1)) * w.nw) << 10) + 1024, end = unit_end < last + 16 ? unit_end : last + 16;
            b.edge = *reinterpret_cast<const u32_aligned2*>(from[0] + (end - 4));       // (as a whole register: nothing to widen, early)
            b.shift = w.half() * 8;
            from[0] -= w.half();
        }
#pragma unroll
        for (int u = 0; u < U; ++u) {
            if constexpr (BOUNDED) {
                b.v[u][0] = ld16<STREAM>(buffer(const_cast<char*>(from[0]), b.room), at[u]);
                continue;
            }
            const uint32_t o = at[u] < last ? at[u] : last;
#pragma unroll
            for (int s = 0; s < S; ++s) b.v[u][s] = WALK::RAGGED ? ld16_ragged<STREAM>(from[s] + o) : ld16<STREAM>(from[s] + o);
        }
        w.next(U);
    };
    auto finish = [&](const Batch<S, U>& b, int u) {
        if (WALK::HALVES) {
            // (No branch around it: the merged registers of a batch shifted and not would be more than a product leaves.)
            const u32x4 x = b.v[u][0];
            const uint32_t edge = (uint32_t)__builtin_amdgcn_readlane(b.edge, u) >> 16;
            uint32_t next = __builtin_amdgcn_update_dpp(edge, x[0], 0x130 /* wave_shl:1: from the lane above, the last lane keeps the first */, 0xf, 0xf, false);
            next = at[u] + 16 >= b.room ? edge : next;
            return u32x4{__builtin_amdgcn_alignbit(x[1], x[0], b.shift), __builtin_amdgcn_alignbit(x[2], x[1], b.shift),
                         __builtin_amdgcn_alignbit(x[3], x[2], b.shift), __builtin_amdgcn_alignbit(next, x[3], b.shift)};
        }
        if (COPY) return b.v[u][0];             // bytes are moved, never interpreted
        Acc<DT> acc;
        acc.init(b.v[u][0]);
#pragma unroll
        for (int s = 1; s < S; ++s) acc.add(b.v[u][s]);
        return acc.result();
    };
    auto put = [&](Batch<S, U>& b) {
        if (WALK::HALVES) asm volatile("" : "+v"(b.edge)::"memory");      // read behind the next batch's loads, and not in front of them
        const Buffer to = buffer(b.to, b.room);
        const int copies = b.r < w.s.nshards ? io.copies(b.r) : 0;
#pragma unroll
        for (int u = 0; u < U; ++u) b.v[u][0] = finish(b, u);
        // Unit by unit, from four wavefronts on.  us, destination by destination -> this: ten shards of 1250232 bf16 at (256, 256, 2 MiB) 68.6 -> 62.3,
        // eight 4 MiB ones at (16, 256, 64 KiB) 62.5 -> 60.9, but at (256, 64, 32 KiB) 19.4 -> 20.9, (16, 128, 64 KiB) 60.5 -> 61.9.
        if (WALK::GATHERS && copies == 2 && w.nw >= 4) {
            const Buffer second = buffer(io.out(b.r, 1) + (b.to - io.out(b.r, 0)), b.room);
#pragma unroll
            for (int u = 0; u < U; ++u) {
                st16(to, at[u], b.v[u][0]);
                st16(second, at[u], b.v[u][0]);
            }
            return;
        }
#pragma unroll
        for (int u = 0; u < U; ++u) st16(to, at[u], b.v[u][0]);
        for (int d = 1; d < copies; ++d) {
            const Buffer other = buffer(io.out(b.r, d) + (b.to - io.out(b.r, 0)), b.room);
#pragma unroll
            for (int u = 0; u < U; ++u) st16(other, at[u], b.v[u][0]);
        }
    };
    // NB - 1 batches are in flight while one is added and stored.  Behind the end: empty ones.  The end is looked for once for all NB: a way
    // out of the loop's middle shares a block with the way back, on which the compiler then drains the memory pipeline.
    Batch<S, U> b[NB];
#pragma unroll
    for (int i = 0; i < NB - 1; ++i) fetch(b[i]);
    while (w.more()) {
#pragma unroll
        for (int i = 0; i < NB; ++i) {
            fetch(b[(i + NB - 1) % NB]);
            put(b[i]);
        }
    }
#pragma unroll
    for (int i = 0; i < NB - 1; ++i) put(b[i]);
}

// Many sources: a unit's sources are loaded in NG groups, and while one group is added the NB - 1 behind it (of this unit, then
// of the next one) are in flight.  The registers of NB groups.
template <int DT, int S, int NG, int NB, bool STREAM, class IO>
__device__ __forceinline__ void move_groups(Walk<REDUCE> w, const IO& io, uint32_t lane) {
    static_assert(NG % NB == 0 && NB > 1, "a group's buffer is the same in every unit");
    w.first();
    if (!w.more()) return;
    const uint32_t lo = lane * 16;
    u32x4 buf[NB][(S + NG - 1) / NG];
    uint32_t o = lo < w.last() ? lo : w.last();
    auto load = [&](auto g) {
        constexpr int G = decltype(g)::value % NG, FROM = S * G / NG, N = S * (G + 1) / NG - FROM;
#pragma unroll
        for (int s = 0; s < N; ++s) buf[G % NB][s] = ld16<STREAM>(io.from(w, FROM + s) + o);
    };
    Acc<DT> acc;
    auto add = [&](auto g) {
        constexpr int G = decltype(g)::value, N = S * (G + 1) / NG - S * G / NG;
        if (G == 0) acc.init(buf[0][0]);
#pragma unroll
        for (int s = G == 0; s < N; ++s) acc.add(buf[G % NB][s]);
    };
    char* to;                                   // the unit that is added: where it goes, and its bytes
    uint32_t room;
    auto pass = [&](auto g) {
        constexpr int G = decltype(g)::value;
        if (G + NB - 1 == NG) {                     // on to the next unit (behind the end: loads that nobody uses)
            to = io.dst(0) + w.off;
            room = w.room();
            w.next(1);
            o = lo < w.last() ? lo : w.last();
        }
        load(std::integral_constant<int, G + NB - 1>{});
        add(g);
        // Left alone, the compiler loads every group in front of the additions, into registers of its own: a later group's
        // addresses are therefore made to depend on the sums so far.
        if (NG > 2) acc.before(o);
    };
    for_each(load, std::make_integer_sequence<int, NB - 1>{});
    do {
        for_each(pass, std::make_integer_sequence<int, NG>{});
        const u32x4 r = acc.result();
        st16(buffer(to, room), lo, r);
        for (int d = 1; d < io.ndst; ++d) st16(buffer(io.dst(d) + (to - io.dst(0)), room), lo, r);
    } while (w.more());
}

// Any number of sources, up to four loads in flight: the steps of more than two sources of a fused launch.  The first group
// takes what is over four, so that every later one is whole and no source is waited for by itself.
template <int DT, bool STREAM, class IO>
__device__ __forceinline__ void move_any(Walk<REDUCE> w, const IO& io, int nsrc, uint32_t lane) {
    const uint32_t lo = lane * 16;
    for (w.first(); w.more(); w.next(1)) {
        if (lo >= w.room()) continue;
        Acc<DT> acc;
        auto first = [&](auto n) {                // added in source order
            u32x4 x[decltype(n)::value];
#pragma unroll
            for (int s = 0; s < decltype(n)::value; ++s) x[s] = ld16<STREAM>(io.from(w, s) + lo);
            acc.init(x[0]);
#pragma unroll
            for (int s = 1; s < decltype(n)::value; ++s) acc.add(x[s]);
        };
        const int over = nsrc & 3;
        if (over == 1) first(std::integral_constant<int, 1>{});
        else if (over == 2) first(std::integral_constant<int, 2>{});
        else if (over == 3) first(std::integral_constant<int, 3>{});
        else first(std::integral_constant<int, 4>{});
        for (int s = over ? over : 4; s < nsrc; s += 4) {
            const u32x4 x0 = ld16<STREAM>(io.from(w, s) + lo), x1 = ld16<STREAM>(io.from(w, s + 1) + lo);
            const u32x4 x2 = ld16<STREAM>(io.from(w, s + 2) + lo), x3 = ld16<STREAM>(io.from(w, s + 3) + lo);
            acc.add(x0); acc.add(x1); acc.add(x2); acc.add(x3);
        }
        const u32x4 r = acc.result();
        for (int d = 0; d < io.ndst; ++d) st16(io.dst(d) + w.off + lo, r);
    }
}

// How much a lane keeps in flight: all that a product beside it leaves, 120 registers of a SIMD ([N,K]) or 112 ([K,N]), in
// channels of up to kDeepNT threads, one wavefront per SIMD; half of that with more threads, whose number keeps the memory
// pipeline busy instead.  us, one memory latency per batch -> loads in flight while a batch is stored -> with the walk's short
// steps:
//   64 MiB gather-copy at (8, 256, 2 MiB)                                  138.5 -> 87.8 -> 81.8
//   12 MiB two-source fp32 reduce at (4, 256, 128 KiB)                      55.1 -> 32.6 -> 32.0
//   sixteen sources of 1000003 bf16 at (32, 256, 64 KiB)                    47.6 -> 16.2 -> 13.1
//   ring share of fourteen 3 MiB steps at (32, 256, 64 KiB)                159.6 -> 61.6 -> 58.8
//   72 MiB eight-source reduce at (256, 512, 32 KiB)                        13.6 -> 13.1 -> 13.0
constexpr int kDeepNT = 256;
constexpr int units_in_batch(int S, bool deep) { return S == 1 ? (deep ? 8 : 4) : S == 2 ? (deep ? 4 : 2) : S <= 4 ? (deep ? 2 : 1) : 1; }
// Reductions of up to 256 threads: three batches, but two of seven and eight bf16 sources, of which three do not fit beside a
// product.  us, two -> three, sources of 1000000 at (8, NT, 32 KiB):
//   six fp32      NT 64 80.6 -> 76.6   128 42.9 -> 40.7   256 29.6 -> 29.3   at (128, 128, 64 KiB) 9.1 -> 7.3
//   eight fp32    NT 64 111 -> 93.4    128 59.8 -> 49.9
//   six bf16 of 4194304 at (32, 128, 32 KiB) 40.8 -> 38.3
constexpr int batches(int DT, int S, bool deep) { return deep && S <= (DT == LAGOM_F32 ? 8 : 6) ? 3 : 2; }
// A quarter of the units per batch where a wavefront has at most half a batch of them in a chunk: what a batch holds beyond
// them costs its loads' and stores' time for nothing.  us, whole batches -> this: ring shares of four 554264 at (8, 1024, 16
// KiB) fp32 95.7 -> 68.4, bf16 51.4 -> 38.5; at (16, 1024, 16 KiB) two fp32 sources of 1625440 20.4 -> 14.6, one 24 -> 11.4.
constexpr int few_units_in_batch(int S, bool deep) { return units_in_batch(S, deep) / 4 > 0 ? units_in_batch(S, deep) / 4 : 1; }
template <int S, bool DEEP>
__device__ __forceinline__ bool few_units(const Shape& s, uint32_t nw) {
    constexpr int U = units_in_batch(S, DEEP);
    return U > 1 && (s.full_bytes + 1023) >> 10 <= nw * (U / 2);
}
// The groups of move_groups (0: whole units).
// Up to 256 threads: six groups, of which five are in flight, but two whole units of up to twelve fp32 sources.  us, halves ->
// six groups | whole units, sources of 1000000 at (8, NT, 32 KiB):
//   nine bf16       NT 128 55.8 -> 51.4 | 54.7
//   twelve bf16     NT 64 128 -> 122 | 125     128 67.0 -> 63.5 | 71.1     256 36.2 -> 33.5 | 41.9
//   ten fp32        NT 64 185 -> 173 | 120     128 101 -> 90.9 | 66.4      256 55.7 -> 54.7 | 56.0
//   twelve fp32     NT 64 189 -> 175 | 127     128 104.5 -> 91.0 | 79.6    256 65.4 -> 65.3 | 66.6
//   sixteen fp32    NT 64 200 -> 185           128 105.5 -> 98.2           256 85.0 -> 83.8
// With more threads a SIMD may hold two wavefronts of a channel, which fit beside a product with up to 56 registers each: from
// nine sources on three or six groups, of which three are in flight.  Two whole halves of them do not fit, and the channel then
// keeps its compute unit from the product.  Makespan of three reduces of 2 MiB sources beside 4096^3, us, halves -> this:
//   9 fp32 at (32, 512, 64 KiB)     115 -> 93 ([N,K])    117 -> 95 ([K,N])
//   16 bf16 at (32, 512, 64 KiB)    131 -> 95            134 -> 96
//   12 fp32 at (8, 384, 256 KiB)    186 -> 146           187 -> 147
// Alone they take 0.8 to 1.0 of the time, 1.03 at worst (9 fp32 at (8, 384, 256 KiB)).
constexpr int groups(int DT, int S, bool deep) {
    if (S <= (!deep ? 4 : DT == LAGOM_F32 ? 12 : 8)) return 0;
    if (deep) return 6;
    if (S <= 8) return 2;
    return S <= (DT == LAGOM_F32 ? 11 : 9) ? 3 : 6;         // that many sources fit at a time
}
constexpr int groups_held(int DT, int S, bool deep) {
    const int ng = groups(DT, S, deep);
    return deep || ng == 2 ? ng : 3;
}

template <int DT, int S, bool STREAM, bool DEEP, class IO>
__device__ __forceinline__ void move_reduce(const Walk<REDUCE>& w, const IO& io, uint32_t lane) {
    constexpr int NG = groups(DT, S, DEEP);
    if constexpr (NG > 0) move_groups<DT, S, NG, groups_held(DT, S, DEEP), STREAM>(w, io, lane);
    else if (S <= 2 && few_units<S, DEEP>(w.s, w.nw)) move_batches<DT, S, few_units_in_batch(S, DEEP), 2, STREAM, false>(w, io, lane);
    else move_batches<DT, S, units_in_batch(S, DEEP), batches(DT, S, DEEP), STREAM, false>(w, io, lane);
}

// The channel of a buffer's last chunk moves what is left behind the last whole vector.
__device__ __forceinline__ bool owns_last(uint32_t chunks) { return (chunks - 1) % gridDim.x == blockIdx.x; }
template <int DT, class SRC, class DST>
__device__ __forceinline__ void reduce_tail(const SRC& src, const DST& dst, int nsrc, int ndst, int64_t bytes, uint32_t chunks) {
    const int esize = DT == LAGOM_F32 ? 4 : 2;
    const int left = (int)(bytes & 15) / esize, tid = threadIdx.x;
    if (tid < left && owns_last(chunks)) reduce_tail_element<DT>(src, dst, nsrc, ndst, (bytes & ~(int64_t)15) + tid * esize);
}
// E: what a lane takes.  In a fused launch it is the element, as in a reduction's tail: a step then reads what the same lane wrote.
template <class E, class DST>
__device__ __forceinline__ void copy_tail(const char* src, const DST& dst, int ndst, int64_t bytes, uint32_t chunks) {
    const int left = (int)(bytes & 15) / (int)sizeof(E), tid = threadIdx.x;
    if (tid < left && owns_last(chunks)) {
        const int64_t at = (bytes & ~(int64_t)15) + tid * (int)sizeof(E);
        const E b = *reinterpret_cast<const E*>(src + at);
        for (int d = 0; d < ndst; ++d) *reinterpret_cast<E*>(dst(d) + at) = b;
    }
}

template <int DT, int S, bool STREAM, bool DEEP>
__global__ void __launch_bounds__(DEEP ? kDeepNT : 1024) reduce_copy_kernel(const CommArgs p) {
    const auto src = [&p](int s) { return p.src[s]; };
    const auto dst = [&p](int d) { return p.dst[d]; };
    const ReduceIo<decltype(src), decltype(dst)> io{src, dst, p.ndst};
    move_reduce<DT, S, STREAM, DEEP>(make_walk<REDUCE>(p.shape), io, threadIdx.x & 63);
    reduce_tail<DT>(src, dst, S, p.ndst, p.shape.shard_bytes, p.shape.chunks);
}

// Gathers of whole shards in batches of eight units take three of them, but on 128 channels and more (streamed loads) only with up to three
// wavefronts.  us, two -> three: six layers' gathers on 8 channels beside products of 2176 x 3328 x 1408 418 -> 409, eight 4 MiB shards at (16, 128, 64
// KiB) 46.5 -> 41.4, (32, 256, 64 KiB) 24.2 -> 23.7, (256, 128, 32 KiB) 13.2 -> 12.7.  Three are walked at a time, with empty ones behind the end, and
// with four wavefronts two are as fast: (256, 256, 32 KiB) 13.6 -> 13.9; with three chunks a channel 9.8 -> 11.0, nine at (128, 256, 32 KiB) 16.7 -> 17.4.
template <WalkKind KIND, bool STREAM, int U>
__device__ __forceinline__ bool three_batches(uint32_t nw) { return KIND == GATHER && U == units_in_batch(1, true) && (!STREAM || nw < 4); }

// KIND GATHER: every shard starts 16-byte aligned in the destination (shard_bytes % 16 == 0, or a single shard).
template <WalkKind KIND, bool STREAM, int U>
__device__ __forceinline__ void gather_copy_body(const CommArgs& p) {
    const auto src = [&p](int s) { return p.src[s]; };
    const auto dst = [&p](int d) { return p.dst[d]; };
    const GatherIo<KIND, decltype(src), decltype(dst)> io{src, dst, p.ndst};
    const Walk<KIND> w = make_walk<KIND>(p.shape);
    if (three_batches<KIND, STREAM, U>(w.nw)) move_batches<LAGOM_F32, 1, U, 3, STREAM, true>(w, io, threadIdx.x & 63);
    else move_batches<LAGOM_F32, 1, U, 2, STREAM, true>(w, io, threadIdx.x & 63);
    if (KIND == GATHER) {
        if (p.nsrc == 1) copy_tail<uint8_t>(p.src[0], dst, p.ndst, p.shape.shard_bytes, p.shape.chunks);
        return;
    }
    // both ends of every shard, byte by byte: lanes 0..15 the head, lanes 16..31 the tail
    for (int r = blockIdx.x; r < p.nsrc; r += gridDim.x) {
        const int64_t n = p.shape.shard_bytes;
        const int64_t head = ragged_head(r, n) < n ? ragged_head(r, n) : n, tail = (n - head) & 15;
        const int t = threadIdx.x;
        const int64_t at = t < 16 ? t : n - tail + (t - 16);
        if (t < 16 ? t < head : t - 16 < tail) {
            const char b = p.src[r][at];
            for (int d = 0; d < p.ndst; ++d) p.dst[d][r * n + at] = b;
        }
    }
}

template <WalkKind KIND, bool STREAM, int U>
__global__ void __launch_bounds__(U == units_in_batch(1, true) ? kDeepNT : 1024) gather_copy_kernel(const CommArgs p) { gather_copy_body<KIND, STREAM, U>(p); }
// shards of an odd number of two-byte elements
template <bool STREAM, int U>
__global__ void __launch_bounds__(U == units_in_batch(1, true) ? kDeepNT : 1024) gather_halves_kernel(const CommArgs p) { gather_copy_body<GATHER_HALVES, STREAM, U>(p); }

template <int DT, bool STREAM, bool DEEP, int S>
void launch_reduce_s(const CommArgs& a, dim3 grid, dim3 block, hipStream_t st) {
    if constexpr (S > LAGOM_MAX_SRCS) return;
    else if (a.nsrc == S) hipLaunchKernelGGL((reduce_copy_kernel<DT, S, STREAM, DEEP>), grid, block, 0, st, a);
    else launch_reduce_s<DT, STREAM, DEEP, S + 1>(a, grid, block, st);
}
template <int DT>
void launch_reduce(const CommArgs& a, dim3 grid, dim3 block, hipStream_t st) {
    const bool stream = stream_loads(grid.x, a.shape), deep = block.x <= kDeepNT;
    if (stream) deep ? launch_reduce_s<DT, true, true, 1>(a, grid, block, st) : launch_reduce_s<DT, true, false, 1>(a, grid, block, st);
    else deep ? launch_reduce_s<DT, false, true, 1>(a, grid, block, st) : launch_reduce_s<DT, false, false, 1>(a, grid, block, st);
}

// Units per batch of a gather-copy: no more than a wavefront has in a chunk, rounded up to a power of two.  What a batch holds
// beyond them is loaded for nothing, three loads of four at 16 KiB and 1024 threads.  us, four or eight units whatever the chunk -> this,
// eight shards of 2097152 bf16 from HBM: (512, 1024, 16 KiB) 15.9 -> 13.6, (256, 1024, 32 KiB) 15.0 -> 14.1, (1024, 256, 16 KiB) 14.5 -> 13.8;
// in the last-level cache (512, 1024, 16 KiB) 14.6 -> 12.8; shards of 1000003 there 15.6 -> 8.1.  No shape of 16 to 1024 channels, 256 to 1024
// threads and 16 to 64 KiB got slower.  Half as many units where loads are streamed: up to 9 % slower at 64 KiB.
int gather_units(const Shape& s, uint32_t nt) {
    int units = units_in_batch(1, nt <= kDeepNT);
    const uint32_t nw = nt >> 6, full_units = (s.full_bytes + 1023) >> 10, mine = (full_units + nw - 1) / nw;
    while (units > 1 && (uint32_t)units / 2 >= mine) units /= 2;
    return units;
}

// Shards of an odd number of two-byte elements: two bytes early and shifted back, or as they lie, off the 4-byte grid.  What the shift
// costs is its instructions, which one or two wavefronts cannot hide, and a load per batch for the units' last bytes, as many lines as
// there are units: it takes four wavefronts, chunks of 32 KiB and batches of four units, and (as a chunk's units fill the last
// batch badly otherwise) a power of two of wavefronts.  us, as they lie -> shifted, eight shards of 1000003 in the last-level cache: (16, 256,
// 32 KiB) 33.5 -> 24.8, x 256 KiB 44.9 -> 26.0; (32, 256, 64 KiB) 19.1 -> 15.0; (128, 256, 64 KiB) 12.1 -> 10.2; (16, 512, 32 KiB) 31.4 -> 27.2; (16, 1024, 64 KiB) 32.5
// -> 27.2, x 256 KiB 40.7 -> 27.2; but (16, 256, 16 KiB) 33.7 -> 33.9, (16, 512, 16 KiB) 36.0 -> 38.3, (16, 1024, 16 KiB) 52.3 -> 61.9, two wavefronts (16, 128,
// 64 KiB) 37.9 -> 40.9, three (16, 192, 16 KiB) 53.4 -> 74.7, one (8, 64, 64 KiB) 184 -> 255.
bool halves_pay(const Shape& s, uint32_t nt) {
    const uint32_t nw = nt >> 6;
    return (s.shard_bytes & 2) && nw >= 4 && (nw & (nw - 1)) == 0 && s.full_bytes > ((nw > 8 ? 4 * nw : 32) - 1) << 10;
}

template <WalkKind KIND, bool STREAM, int U>
void launch_gather_u(const CommArgs& a, int units, dim3 grid, dim3 block, hipStream_t st) {
    if (units == U) {
        if constexpr (KIND == GATHER_HALVES) hipLaunchKernelGGL((gather_halves_kernel<STREAM, U>), grid, block, 0, st, a);
        else hipLaunchKernelGGL((gather_copy_kernel<KIND, STREAM, U>), grid, block, 0, st, a);
    } else if constexpr (U > (KIND == GATHER_HALVES ? 4 : 1)) launch_gather_u<KIND, STREAM, U / 2>(a, units, grid, block, st);
}
template <WalkKind KIND>
void launch_gather(const CommArgs& a, dim3 grid, dim3 block, hipStream_t st) {
    const bool stream = stream_loads(grid.x, a.shape);
    const int units = gather_units(a.shape, block.x);
    if (stream) launch_gather_u<KIND, true, units_in_batch(1, true)>(a, units, grid, block, st);
    else launch_gather_u<KIND, false, units_in_batch(1, true)>(a, units, grid, block, st);
}

// Several local steps of one collective in one launch: the channels are persistent and every channel walks the steps in
// order, taking chunks k, k+NC, ... of each (how a ring collective runs inside a collective library: one kernel whose
// channels loop over the ring steps).  Every buffer of every step holds the same number of bytes, so a given byte offset
// is always moved by the same lane of the same channel: a location that one step writes and a later step reads or
// overwrites through the same pointer is ordered by that lane's program order.  There is no synchronisation between channels.
// Consecutive steps of one kind are one walk, so that the first loads of a step are in flight while the last batch of the step
// before it is added and stored: a wavefront has one batch of loads in front of its stores and no more, and with two batches
// or more to a step that one lies at other offsets than the stores it passes.  A wavefront with a single batch
// takes the steps one by one.  Ring share of a 25 MiB bucket over eight ranks at (32, 256, 64 KiB), four to eight batches a step: 65.9 us
// with the loads drained at every step's end -> 62.2, 93 GB/s on each of the eighteen channels that have two chunks.
constexpr int kMaxSteps = LAGOM_MAX_STEPS;
constexpr int kMaxStepPtrs = LAGOM_MAX_STEP_PTRS;
struct StepsArgs {
    const char* ptr[kMaxStepPtrs];    // per step: its sources, then its destinations
    uint32_t step[kMaxSteps];         // first pointer | sources << 8 | destinations << 16 | operation << 24: one scalar load
    int32_t nsteps;
    Shape shape;                      // one shard: a buffer
    __device__ __forceinline__ const char* src(uint32_t st, int s) const { return ptr[(step[st] & 255) + s]; }
    __device__ __forceinline__ char* dst(uint32_t st, int d) const { return const_cast<char*>(ptr[(step[st] & 255) + nsrc(st) + d]); }
    __device__ __forceinline__ int nsrc(uint32_t st) const { return step[st] >> 8 & 255; }
    __device__ __forceinline__ int ndst(uint32_t st) const { return step[st] >> 16 & 255; }
    __device__ __forceinline__ int kind(uint32_t st) const { return (int)(step[st] & 0xff00ff00u); }    // operation and sources
    static __device__ __forceinline__ int kind_of(int op, int nsrc) { return op << 24 | nsrc << 8; }
};
static_assert(kMaxStepPtrs <= 256 && LAGOM_MAX_SRCS < 256 && LAGOM_MAX_DSTS < 256, "a step is packed in bytes");

struct StepsIo {                      // step r of the walk is step st + r of the launch
    const StepsArgs& p; uint32_t st;
    __device__ __forceinline__ const char* from(const Walk<STEPS>& w, int s) const { return p.src(st + w.shard(), s) + w.off; }
    __device__ __forceinline__ int64_t to(const Walk<STEPS>& w) const { return w.off; }
    __device__ __forceinline__ int copies(uint32_t r) const { return p.ndst(st + r); }
    __device__ __forceinline__ char* out(uint32_t r, int d) const { return p.dst(st + r, d); }
};

// Steps st and following of one kind, as far as they may go in one walk: their number, which w's shards become.
__device__ __forceinline__ int steps_in_walk(const StepsArgs& p, int st, uint32_t units, Walk<STEPS>& w) {
    w.s.nshards = 2;
    w.first();
    w.next(units);
    int run = 1;
    if (w.r == 0)                     // the first step holds another batch
        while (st + run < p.nsteps && p.kind(st + run) == p.kind(st)) ++run;
    w.s.nshards = run;
    return run;
}

template <int DT, bool STREAM, bool DEEP>
__global__ void __launch_bounds__(DEEP ? kDeepNT : 1024) comm_steps_kernel(const StepsArgs p) {
    const Walk<STEPS> w = make_walk<STEPS>(p.shape);
    const uint32_t lane = threadIdx.x & 63;
    auto walk = [&](int st, auto s, auto u, auto copy) {
        constexpr int S = decltype(s)::value, U = decltype(u)::value;
        // (As with the lane in move_batches: what every kind of walk needs of the wavefronts' number would be held for all of them at once.)
        Walk<STEPS> mine = w;
        asm volatile("" : "+s"(mine.nw), "+s"(mine.wave));
        const int run = steps_in_walk(p, st, U, mine);
        move_batches<DT, S, U, 2, STREAM, decltype(copy)::value>(mine, StepsIo{p, (uint32_t)st}, lane);
        return run;
    };
    constexpr std::integral_constant<int, 1> one{};
    constexpr std::integral_constant<int, 2> two{};
    constexpr std::integral_constant<int, units_in_batch(1, DEEP)> u1{};
    constexpr std::integral_constant<int, few_units_in_batch(1, DEEP)> f1{};
    constexpr std::integral_constant<int, units_in_batch(2, DEEP)> u2{};
    constexpr std::integral_constant<int, few_units_in_batch(2, DEEP)> f2{};
    for (int st = 0; st < p.nsteps;) {
        int run = 1;
        if (p.kind(st) == StepsArgs::kind_of(LAGOM_GATHER_COPY, 1)) {        // a plain copy to every destination
            run = few_units<1, DEEP>(p.shape, w.nw) ? walk(st, one, f1, std::true_type{}) : walk(st, one, u1, std::true_type{});
        } else if (DT == LAGOM_BF16 && p.kind(st) == StepsArgs::kind_of(LAGOM_REDUCE_COPY, 1)) {     // (of fp32: a copy)
            run = few_units<1, DEEP>(p.shape, w.nw) ? walk(st, one, f1, std::false_type{}) : walk(st, one, u1, std::false_type{});
        } else if (p.kind(st) == StepsArgs::kind_of(LAGOM_REDUCE_COPY, 2)) {
            run = few_units<2, DEEP>(p.shape, w.nw) ? walk(st, two, f2, std::false_type{}) : walk(st, two, u2, std::false_type{});
        } else {
            const auto src = [&p, st](int s) { return p.src(st, s); };
            const auto dst = [&p, st](int d) { return p.dst(st, d); };
            move_any<DT, STREAM>(make_walk<REDUCE>(p.shape), ReduceIo<decltype(src), decltype(dst)>{src, dst, p.ndst(st)}, p.nsrc(st), lane);
        }
        for (const int end = st + run; st < end; ++st) {       // behind the last whole vector: bytes that no walk touches
            const auto src = [&p, st](int s) { return p.src(st, s); };
            const auto dst = [&p, st](int d) { return p.dst(st, d); };
            if (p.step[st] >> 24 == LAGOM_GATHER_COPY) copy_tail<std::conditional_t<DT == LAGOM_F32, uint32_t, uint16_t>>(src(0), dst, p.ndst(st), p.shape.shard_bytes, p.shape.chunks);
            else reduce_tail<DT>(src, dst, p.nsrc(st), p.ndst(st), p.shape.shard_bytes, p.shape.chunks);
        }
    }
}

// Whether a step reads what another one reads or writes as well: a ring's steps take turns with a few wire buffers.
bool reads_again(const StepsArgs& a) {
    auto first = [&](int st) { return a.step[st] & 255; };
    auto nsrc = [&](int st) { return a.step[st] >> 8 & 255; };
    auto end = [&](int st) { return first(st) + nsrc(st) + (a.step[st] >> 16 & 255); };
    for (int st = 0; st < a.nsteps; ++st)
        for (uint32_t s = first(st); s < first(st) + nsrc(st); ++s)
            for (int other = 0; other < a.nsteps; ++other)
                for (uint32_t q = first(other); other != st && q < end(other); ++q)
                    if (a.ptr[q] == a.ptr[s]) return true;
    return false;
}

// Loads that carry the non-temporal hint leave nothing behind in the last-level cache: not for steps that read it again.  us, with the hint ->
// without, ring shares, buffers of the same share each time | of another one each time: eight ranks of 1051544 bf16 at (256, 256, 16 KiB) 22.3 -> 14.8 |
// 24.7 -> 23.1, sixteen of 1295728 fp32 at (256, 128, 32 KiB) 85.5 -> 66.2 | 87.5 -> 66.8, four of 1873712 fp32 at (128, 128, 32 KiB) 32.6 -> 24.9 | 34.3 -> 28.3, two of
// 1417128 fp32 at (128, 256, 32 KiB) 8.9 -> 7.5 | 12.0 -> 11.8; thirty shares 0.80 | 0.89 in the mean, 1.02 at worst.  (A reduce or gather of
// its own gains as much where its sources are those of the call before, but loses 4 - 9 % where they come from HBM.)
// Not so where a buffer fills that cache (256 MiB) by itself: what is read again is gone by then.  us, with the hint -> without, two ranks of bf16 and four of
// fp32 at (256, 256, 128 KiB), eight of bf16 at (256, 512, 128 KiB), four of bf16 at (128, 256, 64 KiB): buffers of 160 MiB 183 -> 149, 544 -> 539, 1275 -> 1204,
// 614 -> 619; 192 MiB 219 -> 219, 650 -> 653, 1538 -> 1476, 737 -> 748; 224 MiB 256 -> 261, 768 -> 777, 1819 -> 1753, 863 -> 875; 320 MiB 369 -> 378, 1108 -> 1133,
// 2648 -> 2653, 1235 -> 1255.
constexpr int64_t kReadAgainBelow = 224ll << 20;
template <int DT>
void launch_steps(const StepsArgs& a, dim3 grid, dim3 block, hipStream_t st) {
    const bool kept = a.shape.shard_bytes < kReadAgainBelow && reads_again(a), stream = stream_loads(grid.x, a.shape) && !kept, deep = block.x <= kDeepNT;
    if (stream) {
        if (deep) hipLaunchKernelGGL((comm_steps_kernel<DT, true, true>), grid, block, 0, st, a);
        else hipLaunchKernelGGL((comm_steps_kernel<DT, true, false>), grid, block, 0, st, a);
    } else {
        if (deep) hipLaunchKernelGGL((comm_steps_kernel<DT, false, true>), grid, block, 0, st, a);
        else hipLaunchKernelGGL((comm_steps_kernel<DT, false, false>), grid, block, 0, st, a);
    }
}

// ------------------------------------------------------------------ staged through LDS
// The same operators with every source vector staged through LDS by direct-to-LDS loads (global_load_lds, 16 bytes per
// lane).  Each wavefront owns a ring of LDS_STAGES stages of LDS_U KiB and
// treats (batch of LDS_U KiB of the chunk, source) pairs as a stream of items: the loads of the next LDS_STAGES - 1 items
// are in flight while the current one is read back (ds_read_b128) and folded into the lane's accumulators, in source
// order, so the arithmetic and its order are exactly those of the register path; after the last source the batch is
// rounded and stored.  LDS per workgroup is (NT / 64) * LDS_STAGES * LDS_U KiB whatever the number of sources.  A
// wavefront reads only what its own loads wrote and waits for them with its own vmcnt, so there are no barriers.
// What does not fill whole batches at the end of a chunk goes through the register path.
// Measured against the register path: 72 MiB eight-source reduce at 256 channels and more 15.1 us against 13.9, 64 MiB gather 13.3 against 13.8, on
// eight channels of 256 threads half the speed and less (a wavefront has 6 KiB in flight); and a workgroup that holds LDS cannot share a
// compute unit with a GEMM workgroup (which takes all 160 KiB): kept as a selectable path, not the default.
constexpr int LDS_STAGES = 4, LDS_U = 2;                  // 8 KiB per wavefront, 128 KiB for 1024 threads
constexpr int LDS_BYTES_PER_WAVE = LDS_STAGES * LDS_U * 1024;

__device__ __forceinline__ void dma16(const char* g, u32x4* lds_wave_uniform) {
    __builtin_amdgcn_global_load_lds((const __attribute__((address_space(1))) void*)g,
                                     (__attribute__((address_space(3))) void*)lds_wave_uniform, 16, 0, 0);
}

// waits until at most `younger` items issued after the wanted one are still in flight (loads complete in issue order;
// stores share the counter and can only make the wait longer)
__device__ __forceinline__ void wait_items(int younger) {
    if (younger >= 3) asm volatile("s_waitcnt vmcnt(%0)" ::"n"(3 * LDS_U) : "memory");
    else if (younger == 2) asm volatile("s_waitcnt vmcnt(%0)" ::"n"(2 * LDS_U) : "memory");
    else if (younger == 1) asm volatile("s_waitcnt vmcnt(%0)" ::"n"(LDS_U) : "memory");
    else asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
}

// GATHER: items are batches of the one source `src(0)`, copied to dst(d) + dst_off; else a reduce-copy of nsrc sources.
template <int DT, bool GATHER, class SRC, class DST>
__device__ __forceinline__ void lds_chunk(u32x4* ring, const SRC& src, const DST& dst, int nsrc, int ndst, int64_t base, int64_t dst_base,
                                          int64_t len, int lane, int wave, int nw) {
    constexpr int64_t BATCH = LDS_U * 1024;                       // bytes of one source a wavefront moves per batch
    const int64_t nbatch = len / BATCH;                           // whole batches of the chunk, dealt to the wavefronts round-robin
    const int64_t mine = nbatch > wave ? (nbatch - wave + nw - 1) / nw : 0;
    const int S = GATHER ? 1 : nsrc;
    const int64_t items = mine * S;
    auto issue = [&](int64_t i) {
        const int64_t b = i / S;
        const int s = (int)(i - b * S);
        const char* g = src(s) + base + (wave + b * nw) * BATCH + lane * 16;
        u32x4* st = ring + (i % LDS_STAGES) * (LDS_U * 64);
#pragma unroll
        for (int u = 0; u < LDS_U; ++u) dma16(g + u * 1024, st + u * 64);
    };
    int64_t issued = 0;
    for (; issued < items && issued < LDS_STAGES - 1; ++issued) issue(issued);
    Acc<DT> acc[LDS_U];
    for (int64_t i = 0; i < items; ++i) {
        if (issued < items) { issue(issued); ++issued; }
        wait_items((int)(issued - i - 1));
        const u32x4* st = ring + (i % LDS_STAGES) * (LDS_U * 64);
        const int64_t b = i / S;
        const int s = (int)(i - b * S);
        const int64_t off = (wave + b * nw) * BATCH + lane * 16;
        if (GATHER) {
#pragma unroll
            for (int u = 0; u < LDS_U; ++u) {
                const u32x4 x = st[u * 64 + lane];
                for (int d = 0; d < ndst; ++d) st16(dst(d) + dst_base + off + u * 1024, x);
            }
        } else {
#pragma unroll
            for (int u = 0; u < LDS_U; ++u) {
                const u32x4 x = st[u * 64 + lane];
                if (s == 0) acc[u].init(x); else acc[u].add(x);
            }
            if (s == S - 1) {
#pragma unroll
                for (int u = 0; u < LDS_U; ++u) {
                    const u32x4 o = acc[u].result();
                    for (int d = 0; d < ndst; ++d) st16(dst(d) + dst_base + off + u * 1024, o);
                }
            }
        }
    }
}

template <int DT, bool GATHER, int MAXNT>
__global__ void __launch_bounds__(MAXNT) comm_lds_kernel(const CommArgs p) {
    extern __shared__ u32x4 lds_ring[];
    const int tid = threadIdx.x, lane = tid & 63, nw = blockDim.x >> 6;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    u32x4* ring = lds_ring + wave * (LDS_BYTES_PER_WAVE / 16);
    const auto dst = [&p](int d) { return p.dst[d]; };
    for (int64_t g = blockIdx.x; g < (int64_t)p.shape.chunks * (GATHER ? p.nsrc : 1); g += gridDim.x) {
        const int64_t r = GATHER ? g / p.shape.chunks : 0;
        const int64_t base = (g - r * p.shape.chunks) * p.shape.chunk_bytes;
        const int64_t left = p.shape.shard_bytes - base;
        const int64_t len = left < p.shape.chunk_bytes ? left : p.shape.chunk_bytes;
        const int64_t bulk = len / (LDS_U * 1024) * (LDS_U * 1024);
        const int64_t dst_base = r * p.shape.shard_bytes + base;
        if (GATHER) {
            const char* one = p.src[r];
            const auto src = [one](int) { return one; };
            lds_chunk<DT, true>(ring, src, dst, 1, p.ndst, base, dst_base, len, lane, wave, nw);
            copy_rest(one + base + bulk, dst, p.ndst, dst_base + bulk, len - bulk, tid, blockDim.x);
        } else {
            const auto src = [&p](int s) { return p.src[s]; };
            lds_chunk<DT, false>(ring, src, dst, p.nsrc, p.ndst, base, dst_base, len, lane, wave, nw);
            reduce_rest<DT>(src, dst, p.nsrc, p.ndst, base + bulk, len - bulk, tid, blockDim.x);
        }
    }
}

template <void (*KERNEL)(const CommArgs)>
int launch_lds(const CommArgs& a, dim3 grid, dim3 block, hipStream_t st) {
    const int lds_bytes = (int)(block.x / 64) * LDS_BYTES_PER_WAVE;
    static std::atomic<uint64_t> done_on_device{0};     // once per kernel and device; a failure is not remembered
    int dev = 0;
    if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev > 63) dev = 63;
    const uint64_t bit = uint64_t{1} << dev;
    if (dev == 63 || !(done_on_device.load(std::memory_order_acquire) & bit)) {
        const hipError_t attr = hipFuncSetAttribute(reinterpret_cast<const void*>(KERNEL), hipFuncAttributeMaxDynamicSharedMemorySize, 16 * LDS_BYTES_PER_WAVE);
        if (attr != hipSuccess) return lagom::fail(LAGOM_EHIP, "cannot raise the LDS limit: %s", hipGetErrorString(attr));
        done_on_device.fetch_or(bit, std::memory_order_release);
    }
    hipLaunchKernelGGL(KERNEL, grid, block, lds_bytes, st, a);
    return LAGOM_OK;
}

}  // namespace

namespace lagom {

int check_cfg(const lagom_cfg* cfg) {
    if (!cfg) return fail(LAGOM_EINVAL, "null configuration");
    if (cfg->nc < 1 || cfg->nc > 65535) return fail(LAGOM_EINVAL, "nc=%d outside 1..65535", cfg->nc);
    if (cfg->nt < 64 || cfg->nt > 1024 || cfg->nt % 64) return fail(LAGOM_EINVAL, "nt=%d must be a multiple of 64 in 64..1024", cfg->nt);
    if (cfg->chunk_bytes < 16 || cfg->chunk_bytes % 16) return fail(LAGOM_EINVAL, "chunk_bytes=%lld must be a positive multiple of 16", (long long)cfg->chunk_bytes);
    return LAGOM_OK;
}

int check_comm_args(int op, int dtype, const void* const* srcs, int nsrc, void* const* dsts, int ndst, int64_t count) {
    if (op != LAGOM_REDUCE_COPY && op != LAGOM_GATHER_COPY) return fail(LAGOM_EINVAL, "unknown op %d", op);
    if (elem_size(dtype) == 0) return fail(LAGOM_EINVAL, "unknown dtype %d", dtype);
    if (!srcs || !dsts) return fail(LAGOM_EINVAL, "null pointer array");
    if (nsrc < 1 || nsrc > LAGOM_MAX_SRCS) return fail(LAGOM_EINVAL, "nsrc=%d outside 1..%d", nsrc, LAGOM_MAX_SRCS);
    if (ndst < 1 || ndst > LAGOM_MAX_DSTS) return fail(LAGOM_EINVAL, "ndst=%d outside 1..%d", ndst, LAGOM_MAX_DSTS);
    if (count < 0 || count > (int64_t)1 << 40) return fail(LAGOM_EINVAL, "count=%lld out of range", (long long)count);
    for (int s = 0; s < nsrc; ++s) {
        if (!srcs[s]) return fail(LAGOM_EINVAL, "source %d is null", s);
        if ((uintptr_t)srcs[s] & 15) return fail(LAGOM_EALIGN, "source %d is not 16-byte aligned", s);
    }
    for (int d = 0; d < ndst; ++d) {
        if (!dsts[d]) return fail(LAGOM_EINVAL, "destination %d is null", d);
        if ((uintptr_t)dsts[d] & 15) return fail(LAGOM_EALIGN, "destination %d is not 16-byte aligned", d);
    }
    return LAGOM_OK;
}

}  // namespace lagom

extern "C" int64_t lagom_comm_bytes(int op, int dtype, int nsrc, int ndst, int64_t count) {
    const int es = lagom::elem_size(dtype);
    if (es == 0 || nsrc < 1 || ndst < 1 || count < 0) return -1;
    if (op == LAGOM_REDUCE_COPY) return (int64_t)(nsrc + ndst) * count * es;
    if (op == LAGOM_GATHER_COPY) return (int64_t)(1 + ndst) * nsrc * count * es;
    return -1;
}

extern "C" int lagom_comm_kernel(lagom_op op, lagom_dtype dt, const void* const* srcs, int nsrc,
                                 void* const* dsts, int ndst, int64_t count, const lagom_cfg* cfg, void* hip_stream) {
    if (int rc = lagom::check_comm_args(op, dt, srcs, nsrc, dsts, ndst, count)) return rc;
    if (int rc = lagom::check_cfg(cfg)) return rc;
    if (count == 0) return LAGOM_OK;

    CommArgs a{};
    for (int s = 0; s < nsrc; ++s) a.src[s] = static_cast<const char*>(srcs[s]);
    for (int d = 0; d < ndst; ++d) a.dst[d] = static_cast<char*>(dsts[d]);
    a.nsrc = nsrc; a.ndst = ndst;
    a.shape = make_shape(count * lagom::elem_size(dt), cfg->chunk_bytes, op == LAGOM_REDUCE_COPY ? 1 : nsrc, cfg->nc);

    hipStream_t st = static_cast<hipStream_t>(hip_stream);
    const dim3 grid((unsigned)cfg->nc), block((unsigned)cfg->nt);
    if (op == LAGOM_REDUCE_COPY) dt == LAGOM_F32 ? launch_reduce<LAGOM_F32>(a, grid, block, st) : launch_reduce<LAGOM_BF16>(a, grid, block, st);
    else if (nsrc == 1 || (a.shape.shard_bytes & 15) == 0) launch_gather<GATHER>(a, grid, block, st);
    else if (halves_pay(a.shape, block.x)) launch_gather<GATHER_HALVES>(a, grid, block, st);
    else launch_gather<GATHER_RAGGED>(a, grid, block, st);
    const hipError_t e = hipGetLastError();
    if (e != hipSuccess) return lagom::fail(LAGOM_EHIP, "comm kernel launch: %s", hipGetErrorString(e));
    return LAGOM_OK;
}

namespace lagom {

// Shape rules of lagom_comm_steps; also used by the overlap runner before it fuses launches.
int check_comm_steps(int dtype, const lagom_comm_step* steps, int nsteps, int64_t count) {
    if (elem_size(dtype) == 0) return fail(LAGOM_EINVAL, "unknown dtype %d", dtype);
    if (!steps || nsteps < 1 || nsteps > LAGOM_MAX_STEPS) return fail(LAGOM_EINVAL, "nsteps=%d outside 1..%d", nsteps, LAGOM_MAX_STEPS);
    if (count < 0 || count > (int64_t)1 << 40) return fail(LAGOM_EINVAL, "count=%lld out of range", (long long)count);
    int nptr = 0;
    for (int i = 0; i < nsteps; ++i) {
        const lagom_comm_step& s = steps[i];
        if (int rc = check_comm_args(s.op, dtype, s.srcs, s.nsrc, s.dsts, s.ndst, count)) return rc;
        if (s.op == LAGOM_GATHER_COPY && s.nsrc != 1)
            return fail(LAGOM_EINVAL, "step %d: a gather-copy step of a fused launch forwards one source (every buffer of every step holds `count` elements)", i);
        nptr += s.nsrc + s.ndst;
    }
    if (nptr > LAGOM_MAX_STEP_PTRS) return fail(LAGOM_EINVAL, "%d buffers in all steps together, at most %d", nptr, LAGOM_MAX_STEP_PTRS);
    // two steps may touch the same memory only through the same pointer (then the same lane moves it in both);
    // buffers that overlap in part would be moved by different lanes with nothing ordering them
    const int64_t bytes = count * elem_size(dtype);
    for (int i = 0; i < nsteps; ++i)
        for (int j = i + 1; j < nsteps; ++j) {
            const lagom_comm_step &a = steps[i], &b = steps[j];
            for (int x = 0; x < a.nsrc + a.ndst; ++x)
                for (int y = 0; y < b.nsrc + b.ndst; ++y) {
                    if (x < a.nsrc && y < b.nsrc) continue;        // both only read
                    const uintptr_t pa = (uintptr_t)(x < a.nsrc ? a.srcs[x] : a.dsts[x - a.nsrc]);
                    const uintptr_t pb = (uintptr_t)(y < b.nsrc ? b.srcs[y] : b.dsts[y - b.nsrc]);
                    if (pa != pb && pa < pb + (uintptr_t)bytes && pb < pa + (uintptr_t)bytes)
                        return fail(LAGOM_EINVAL, "steps %d and %d touch buffers that overlap in part", i, j);
                }
        }
    return LAGOM_OK;
}

}  // namespace lagom

extern "C" int lagom_comm_steps(lagom_dtype dt, const lagom_comm_step* steps, int nsteps, int64_t count,
                                const lagom_cfg* cfg, void* hip_stream) {
    if (int rc = lagom::check_comm_steps(dt, steps, nsteps, count)) return rc;
    if (int rc = lagom::check_cfg(cfg)) return rc;
    if (count == 0) return LAGOM_OK;
    StepsArgs a{};
    int n = 0;
    for (int i = 0; i < nsteps; ++i) {
        // one source of fp32 is added to nothing: a copy, bit for bit (bf16 may hold a NaN that the reduction makes quiet)
        const int op = dt == LAGOM_F32 && steps[i].nsrc == 1 ? (int)LAGOM_GATHER_COPY : steps[i].op;
        a.step[i] = (uint32_t)n | (uint32_t)steps[i].nsrc << 8 | (uint32_t)steps[i].ndst << 16 | (uint32_t)op << 24;
        for (int s = 0; s < steps[i].nsrc; ++s) a.ptr[n++] = static_cast<const char*>(steps[i].srcs[s]);
        for (int d = 0; d < steps[i].ndst; ++d) a.ptr[n++] = static_cast<const char*>(steps[i].dsts[d]);
    }
    a.nsteps = nsteps;
    a.shape = make_shape(count * lagom::elem_size(dt), cfg->chunk_bytes, 1, cfg->nc);
    hipStream_t st = static_cast<hipStream_t>(hip_stream);
    const dim3 grid((unsigned)cfg->nc), block((unsigned)cfg->nt);
    dt == LAGOM_F32 ? launch_steps<LAGOM_F32>(a, grid, block, st) : launch_steps<LAGOM_BF16>(a, grid, block, st);
    const hipError_t e = hipGetLastError();
    if (e != hipSuccess) return lagom::fail(LAGOM_EHIP, "comm steps launch: %s", hipGetErrorString(e));
    return LAGOM_OK;
}

extern "C" int lagom_comm_kernel_lds(lagom_op op, lagom_dtype dt, const void* const* srcs, int nsrc,
                                     void* const* dsts, int ndst, int64_t count, const lagom_cfg* cfg, void* hip_stream) {
    if (int rc = lagom::check_comm_args(op, dt, srcs, nsrc, dsts, ndst, count)) return rc;
    if (int rc = lagom::check_cfg(cfg)) return rc;
    if (count == 0) return LAGOM_OK;
    const int64_t shard_bytes = count * lagom::elem_size(dt);
    if (op == LAGOM_GATHER_COPY && nsrc > 1 && (shard_bytes & 15))     // element-aligned shards: nothing to stage 16 bytes at a time
        return lagom_comm_kernel(op, dt, srcs, nsrc, dsts, ndst, count, cfg, hip_stream);
    CommArgs a{};
    for (int s = 0; s < nsrc; ++s) a.src[s] = static_cast<const char*>(srcs[s]);
    for (int d = 0; d < ndst; ++d) a.dst[d] = static_cast<char*>(dsts[d]);
    a.nsrc = nsrc; a.ndst = ndst;
    a.shape = make_shape(shard_bytes, cfg->chunk_bytes, op == LAGOM_REDUCE_COPY ? 1 : nsrc, cfg->nc);
    hipStream_t st = static_cast<hipStream_t>(hip_stream);
    const dim3 grid((unsigned)cfg->nc), block((unsigned)cfg->nt);
    const bool small = block.x <= 512;
    int rc;
    if (op == LAGOM_GATHER_COPY) rc = small ? launch_lds<comm_lds_kernel<LAGOM_F32, true, 512>>(a, grid, block, st) : launch_lds<comm_lds_kernel<LAGOM_F32, true, 1024>>(a, grid, block, st);
    else if (dt == LAGOM_F32) rc = small ? launch_lds<comm_lds_kernel<LAGOM_F32, false, 512>>(a, grid, block, st) : launch_lds<comm_lds_kernel<LAGOM_F32, false, 1024>>(a, grid, block, st);
    else rc = small ? launch_lds<comm_lds_kernel<LAGOM_BF16, false, 512>>(a, grid, block, st) : launch_lds<comm_lds_kernel<LAGOM_BF16, false, 1024>>(a, grid, block, st);
    if (rc) return rc;
    const hipError_t e = hipGetLastError();
    if (e != hipSuccess) return lagom::fail(LAGOM_EHIP, "comm kernel launch: %s", hipGetErrorString(e));
    return LAGOM_OK;
}
