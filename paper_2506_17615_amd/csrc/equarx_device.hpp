// Device code of libequarx: gfx950 (CDNA4, wave64) kernels for the block-wise
// int8 quantized reduction of EQuARX (arXiv 2506.17615, Sec. 3.1-3.4).
//
// Work decomposition shared by all kernels
//   lane   : owns 8 consecutive elements of a tile (one 16-byte bf16 load, one
//            8-byte code load/store), so it sees the same elements in both
//            streams;
//   group  : the G = B/8 consecutive lanes that cover one quantization block
//            (G = 4 .. 64, always inside one wavefront), reduced with DPP row
//            operations and the gfx950 row-swap permutes;
//   wave   : 512 consecutive elements per tile;
//   workgroup of T threads : 8*T consecutive elements per tile, K tiles per
//            thread in flight, tile k of a workgroup starting 8*T*k further.
// Every load instruction of a workgroup therefore reads one contiguous 16*T
// (bf16) or 8*T byte (codes) span.  Elements past n read as zero -- a zero never
// changes a block's max-abs, so a ragged last block needs no special
// arithmetic -- and are not stored.
//
// Parameter order of the kernels: the library is built with kernarg preload, so
// up to 14 dwords of LEADING scalar and pointer parameters are in scalar
// registers when a wave starts; a table passed by value ends the run, so tables
// come last.  Without the preload every launch begins with a scalar load from
// the argument segment that nothing can overlap: measured on MI355X, 0.25-0.35
// us per launch of the hop-by-hop chains (9 launches, 27B shape: 124.6 -> 122.5
// us; 2.75 M elements: 33.1 -> 30.7 us; 17 launches of a 1.2 M element message:
// 49.4 -> 45.4 us).
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

namespace equarx {

typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));   // one 16-byte access
typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));   // one 8-byte access

// Build-time tuning knobs (defaults are what the library ships with).
#ifndef EQUARX_NT_LOAD_BF16
#define EQUARX_NT_LOAD_BF16 1       // bf16 inputs are read once: non-temporal loads
#endif
#ifndef EQUARX_NT_STORE_BF16
#define EQUARX_NT_STORE_BF16 1      // the bf16 output is not read again by this library
#endif
#ifndef EQUARX_CHAIN_PAIRED
#define EQUARX_CHAIN_PAIRED 1       // single-launch chain, blocks >= 128: two pieces of one block per lane
#endif
#ifndef EQUARX_SCHED_BARRIER
#define EQUARX_SCHED_BARRIER 1      // keep every load of a thread ahead of its arithmetic
#endif
constexpr int kLaneElems = 8;
constexpr int kThreads = 256;       // workgroups of kernels without a shape of their own

// Shape of a launch: T threads per workgroup, K tiles per thread in flight, so
// T*K*8 consecutive elements per workgroup.
template <int T_, int K_>
struct Shape {
    static constexpr int T = T_, K = K_;
    static constexpr int64_t kElems = (int64_t)T_ * K_ * kLaneElems;
};

// Elements of one tile of a workgroup of T threads.
template <int T>
constexpr int tile_elems = T * kLaneElems;

// The most elements a launch of that shape takes: a dimension of a grid holds fewer than 2^32 threads.
template <typename S>
constexpr int64_t kMostElems = (int64_t)(0xffffffffu / S::T) * S::kElems;

// Workgroups of a launch of that shape over n elements.
template <typename S>
inline unsigned grid_for(int64_t n)
{
    return (unsigned)((n + S::kElems - 1) / S::kElems);
}

// The two shapes of the kernels that make one pass over a message: quantize, hop, dequantize, the ends-fused
// chain's head and tail, the ring steps.
//
// NarrowPass, one tile per thread: a launch is over when its slowest wave is, and with everything resident at once
// a wave's time is one memory round trip plus its own arithmetic; a second and third tile per thread only make that
// chain longer.  WidePass once the message no longer fits the chip in one round of workgroups (256 CUs x 8
// workgroups x 2048 elements = 4 Mi): from there what counts is few workgroups to dispatch and two loads per lane
// in flight.  Measured on MI355X, us per hop-by-hop chain (P = 6, block 256), against 256 threads x 3 tiles for
// every size:
//     elements      256 x 3    256 x 1    512 x 2    256 x 2
//     40 k            20.6       14.5       17.0       16.6
//     640 k           23.9       15.8       19.2       18.7
//     2.75 M          28.2       23.3       24.6       27.5
//     4.0 M           35.2       27.7       30.6       28.7
//     5.5 M           39.8       35.1       34.7       33.9
//     12 M            59.1       57.2       54.9       55.1
//     22 M            94.0      101.6       93.9       95.5
//     33.5 M         140.1      145.0      137.5      137.6
constexpr int pass_threads(int K) { return K == 1 ? 256 : 512; }
template <int K>
using PassShape = Shape<pass_threads(K), K>;
using NarrowPass = PassShape<1>;
using WidePass = PassShape<2>;
constexpr int64_t kOneRound = (int64_t)2048 * NarrowPass::kElems;

// f(shape) with the shape for a pass over n elements.
template <typename F>
inline void with_pass_shape(int64_t n, F f)
{
    if (n <= kOneRound) {
        f(NarrowPass{});
    } else {
        f(WidePass{});
    }
}

// A dequantization of what an all-gather brought runs alone on a tensor that no cache holds, where other shapes than
// WidePass stream better: 256 threads x 2 tiles while that is one round on the chip (1792 workgroups, seven per CU),
// 1024 x 1 for the longest, whose sixteen waves walk one piece together.  Measured on MI355X, us, block 256, many sets of
// buffers in turn:
//     elements     256 x 2   512 x 2   1024 x 1
//     4.2 M          3.02      3.21      4.18
//     5.2 M          3.48      3.86      4.15
//     7.3 M          4.30      5.21      5.30
//     7.9 M          5.49      5.37      5.45
//     10.5 M         6.86      6.65      6.93
//     12.6 M         8.07      7.84      7.89
//     14.7 M         9.16      8.93      8.69
//     22 M          12.74     12.30     12.04
//     88 M          43.06     42.28     41.66     (block 32: 43.65, 42.83, 41.72)
//     200 M         95.06     94.20     91.21     (block 32: 96.93, 94.67, 92.32)
//     34.4 G          --      16858     15933     (block 32: 17794, 16989)
// The other steps of a device stay with WidePass: with 256 x 2 a quantization gains up to 3 % below 22 M and loses 2 %
// above with small blocks, a batch of them loses more (seven of 16.8 M and their flat reduce together 84.9 -> 88.8), the
// hop takes 15.42 instead of 15.22 at 22 M.  In the chains, whose wire the next launch finds in a cache, all of these
// are within 0.3 us.
constexpr int64_t kOneNarrowPairRound = (int64_t)1792 * Shape<256, 2>::kElems;
constexpr int64_t kLongDequantize = (int64_t)13 << 20;

template <typename F>
inline void with_stream_dequantize_shape(int64_t n, F f)
{
    if (n <= kOneRound) {
        f(NarrowPass{});
    } else if (n <= kOneNarrowPairRound) {
        f(Shape<256, 2>{});
    } else if (n < kLongDequantize || n > kMostElems<Shape<1024, 1>>) {
        f(WidePass{});
    } else {
        f(Shape<1024, 1>{});
    }
}

// The chains that walk their wire through memory, hop by hop, rewrite ONE wire buffer in place, and from kTurnFrom
// elements of wire on every second launch takes its tiles in the opposite order.  What bounds a hop is what it moves
// beyond the L2s (8 x 4 MB, write-back, and the lines stay from one launch to the next; workgroup b runs on XCD b % 8,
// so a tile comes back to the L2 that holds it): with two buffers in turn a message of more than 16 M elements finds
// nothing of its wire there, with one it finds it up to 28 M, and beyond that a launch that begins where the last one
// ended still finds the 25 MB written last, where one that begins at the front again has always just lost what it asks
// for.  Measured on MI355X, us per hop-by-hop chain:
//     P, elements, block       two buffers    one, always forward    one, turning
//     6, 4.4 M, 256                28.6              27.7                28.0
//     8, 12.6 M, 256               72.7              69.9                70.5
//     8, 16.8 M, 64                98.4              86.9                87.1
//     8, 22 M, 256                122.5             109.1               108.3
//     8, 30 M, 256                163.0             152.1               143.3
//     8, 33.5 M, 32               190.1             189.8               166.9
//     8, 42 M, 64                 223.9             227.3               206.5
//     4, 60 M, 256                163.8             164.3               156.7
//     2, 90 M, 256                139.9             133.5               130.3
// (Turning with two buffers: no gain.  One buffer, the part past 23 M accessed with non-temporal hints: 148.5 at 30 M,
// 177.2 at 33.5 M, 165.1 at 60 M.)
constexpr int64_t kTurnFrom = (int64_t)20 << 20;

__host__ __device__ inline bool walks_back(int64_t wire_elems, int pass) { return wire_elems >= kTurnFrom && (pass & 1) != 0; }

// A launch that walks back takes its workgroups' tiles in groups of eight, the last group first, so that every tile stays
// on its XCD; what a last, partial group would take stays where it is.  `mirror` is the number of elements in whole groups
// (mirrored), 0 in a launch that walks forward.
template <typename S>
inline int64_t mirrored(int64_t n, bool backward)
{
    return backward ? (int64_t)(grid_for<S>(n) & ~7u) * S::kElems : 0;
}

// The workgroup's first element.  Launches that never walk back -- one tile per thread, so the message (or the last piece
// of a longer one) is far below kTurnFrom, and the steps of a ring between devices -- do not ask: their loads begin with
// this address (MI355X, one device's nine calls in a ring of eight, 27B shape: 38.5 -> 38.3 us).
template <int T, int K, bool kTurns = true>
__device__ __forceinline__ int64_t first_element(int64_t mirror)
{
    constexpr int64_t kSpan = T * K * kLaneElems;
    const int64_t at = blockIdx.x * kSpan;
    if (!kTurns || K == 1) return at;
    return at < mirror ? mirror - 8 * kSpan - at + 2 * (int64_t)(blockIdx.x & 7u) * kSpan : at;
}

// Smallest max-abs that still gets a non-zero scale: 127 * 2^-126, so that
// scale = absmax/127 stays a normal number and 127/absmax stays finite.
constexpr float kTinyAbsmax = 127.0f * 1.17549435e-38f;

// A device address as a kernel parameter.  The runtime looks every parameter that is declared a pointer up in its map of
// allocations, under a lock, at every launch; an integer goes through as it is.  In the kernel it is a pointer to global
// memory like any other, and arrives preloaded in scalar registers like one.  Measured on MI355X, host us per launch of a
// kernel with four of them among its seven parameters, 400 in a row: 2.33 -> 2.21 on one box, 2.72 -> 2.59 on another;
// hop-by-hop chains through the binding, P = 4 of 4096 elements 15.4 -> 14.6, P = 16 of 344 k 52.0 -> 48.3.
template <typename T>
struct Global {
    uint64_t address;
    Global() = default;
    __host__ __device__ Global(T *p) : address(reinterpret_cast<uint64_t>(p)) {}
    __device__ __forceinline__ operator T *() const { return (T *)(__attribute__((address_space(1))) T *)address; }
};

// ---------------------------------------------------------------- lane exchange

template <int kCtrl>
__device__ __forceinline__ uint32_t dpp_read(uint32_t v)
{
    return (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, kCtrl, 0xf, 0xf, false);
}

__device__ __forceinline__ uint32_t umax(uint32_t a, uint32_t b) { return a > b ? a : b; }

// Max over the G lanes of a group, result in every lane of the group.  The
// operand is the bit pattern of a non-negative float, for which unsigned
// integer order equals float order.  All 64 lanes of the wave must be active.
template <int G>
__device__ __forceinline__ uint32_t group_max_bits(uint32_t m)
{
    static_assert(G == 4 || G == 8 || G == 16 || G == 32 || G == 64, "group width");
    m = umax(m, dpp_read<0xB1>(m));                 // quad_perm:[1,0,3,2]  lane ^ 1
    m = umax(m, dpp_read<0x4E>(m));                 // quad_perm:[2,3,0,1]  lane ^ 2
    if (G >= 8) m = umax(m, dpp_read<0x141>(m));    // row_half_mirror      the other quad of 8
    if (G >= 16) m = umax(m, dpp_read<0x140>(m));   // row_mirror           the other half of 16
    if (G >= 32) {                                  // rows 0<->1 and 2<->3 trade places
        auto r = __builtin_amdgcn_permlane16_swap(m, m, false, false);
        m = umax(r[0], r[1]);
    }
    if (G >= 64) {                                  // lower and upper 32 lanes trade places
        auto r = __builtin_amdgcn_permlane32_swap(m, m, false, false);
        m = umax(r[0], r[1]);
    }
    return m;
}

// ---------------------------------------------------------------- element codecs

__device__ __forceinline__ void widen_bf16x4(const u32x2 &w, float (&f)[4])
{
    const uint32_t d[2] = {w.x, w.y};
#pragma unroll
    for (int i = 0; i < 2; ++i) {
        f[2 * i] = __uint_as_float(d[i] << 16);
        f[2 * i + 1] = __uint_as_float(d[i] & 0xFFFF0000u);
    }
}

__device__ __forceinline__ void widen_bf16x8(const u32x4 &w, float (&f)[8])
{
    const uint32_t d[4] = {w.x, w.y, w.z, w.w};
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        f[2 * i] = __uint_as_float(d[i] << 16);
        f[2 * i + 1] = __uint_as_float(d[i] & 0xFFFF0000u);
    }
}

__device__ __forceinline__ void widen_i8x8(const u32x2 &w, float (&f)[8])
{
    const uint32_t d[2] = {w.x, w.y};
#pragma unroll
    for (int i = 0; i < 2; ++i) {
#pragma unroll
        for (int b = 0; b < 4; ++b) {
            f[4 * i + b] = (float)(int)(int8_t)(d[i] >> (8 * b));
        }
    }
}

__device__ __forceinline__ uint32_t narrow_bf16x2(float lo, float hi)
{
    // gfx950 converts in hardware (round to nearest, ties to even)
    typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
    typedef float floatx2 __attribute__((ext_vector_type(2)));
    floatx2 v = {lo, hi};
    bf16x2 h = __builtin_convertvector(v, bf16x2);
    return __builtin_bit_cast(uint32_t, h);
}

// ---------------------------------------------------------------- guarded tile I/O
// A lane's 8 elements are those at [base + off, base + off + 8): `base`, the tile's first element, is the same in
// every lane, so an access is one scalar base and one 32-bit lane offset.  `full` is a compile-time constant at every call: the whole tile lies inside [0, n).
//
// Otherwise the workgroup holds the end of the tensor, and its accesses go through buffer descriptors that end there:
// the hardware drops the 32-bit words of an access that lie past the end (loads give zero), each on its own.  The
// elements of a last, partial word are accessed one by one.  Nothing is behind a condition, so the loads of all tiles
// stay in flight together; with a branch per access every load of this one workgroup waited for the one before, and a
// message of odd length waited for it (MI355X, 344,063 elements, us with branches -> without: hop-by-hop chain of six
// 16.3 -> 14.6, flat reduce of five wires 6.5 -> 3.9, eight partials in one launch 9.5 -> 3.4; 344,064, where no
// workgroup is ragged: 14.6, 3.8 and 3.4).

__device__ __forceinline__ __amdgpu_buffer_rsrc_t bounded(const void *p, int bytes)
{
    return __builtin_amdgcn_make_buffer_rsrc(const_cast<void *>(p), 0, bytes, 0x00027000);
}

// Elements from `base` to the end; a workgroup's last tiles may lie past it.
__device__ __forceinline__ int left_of(int64_t n, int64_t base) { return n > base ? (int)(n - base) : 0; }

constexpr int kNonTemporal = 2;         // cache policy bits of a buffer access
constexpr int kThroughL2 = 1 | 16;      // sc0 sc1
constexpr int kNowhere = 0x7ffffff0;    // an offset past the end of every descriptor here

// A lane's access at the end of a tensor: its whole words, and the elements of a last, partial word (0 if there are none),
// which whole_end puts in the lane they belong to.  Two steps, so that a thread with several tiles can request all of
// them before it looks at the first: with both in one the compiler waited for a tile before it asked for the next, in
// the semi-loop once per partial (MI355X: 16 partials of 4.3 M elements, blocks of 512, 30.0 us, 27.1 in two steps;
// dequantization of 4.2 M 4.0 -> 3.3, of 6.2 M 4.7 -> 4.2).
struct EndOfBf16 {
    u32x4 words;
    uint32_t last;
    int whole;      // elements in whole words, from the tile's first
};

__device__ __forceinline__ EndOfBf16 request_end(const uint16_t *p, int64_t base, int off, int64_t n)
{
    const int left = left_of(n, base);
    const int whole = left & ~1;
    constexpr int kPolicy = EQUARX_NT_LOAD_BF16 ? kNonTemporal : 0;
    EndOfBf16 e;
    e.words = __builtin_bit_cast(u32x4, __builtin_amdgcn_raw_buffer_load_b128(bounded(p + base, whole * 2), off * 2, 0, kPolicy));
    e.last = __builtin_amdgcn_raw_buffer_load_b16(bounded(p + base, left * 2), whole * 2, 0, 0);
    e.whole = whole;
    return e;
}

__device__ __forceinline__ u32x4 whole_end(const EndOfBf16 &e, int off)
{
    u32x4 w = e.words;
    if (off == e.whole) w.x = e.last;
    if (off + 2 == e.whole) w.y = e.last;
    if (off + 4 == e.whole) w.z = e.last;
    if (off + 6 == e.whole) w.w = e.last;
    return w;
}

__device__ __forceinline__ u32x4 load_bf16x8(const uint16_t *p, int64_t base, int off, int64_t n, bool full)
{
    if (full) {
        const u32x4 *v = reinterpret_cast<const u32x4 *>(p + base + off);
        return EQUARX_NT_LOAD_BF16 ? __builtin_nontemporal_load(v) : *v;
    }
    return whole_end(request_end(p, base, off, n), off);
}

struct EndOfI8 {
    u32x2 words;
    uint32_t last[3];
    int whole;
};

template <bool kStream>
__device__ __forceinline__ EndOfI8 request_end(const int8_t *p, int64_t base, int off, int64_t n)
{
    const int left = left_of(n, base);
    EndOfI8 e;
    e.whole = left & ~3;
    e.words = __builtin_bit_cast(u32x2, __builtin_amdgcn_raw_buffer_load_b64(bounded(p + base, e.whole), off, 0, kStream ? kNonTemporal : 0));
    const auto end = bounded(p + base, left);
#pragma unroll
    for (int i = 0; i < 3; ++i) e.last[i] = __builtin_amdgcn_raw_buffer_load_b8(end, e.whole + i, 0, 0);
    return e;
}

__device__ __forceinline__ u32x2 whole_end(const EndOfI8 &e, int off)
{
    u32x2 w = e.words;
    const uint32_t last = e.last[0] | (e.last[1] << 8) | (e.last[2] << 16);
    if (off == e.whole) w.x = last;
    if (off + 4 == e.whole) w.y = last;
    return w;
}

// Wire accesses come in two flavours.  kStream = false: ordinary cached accesses, for a wire that the next launch
// on this device reads back (the single-device chain: the 256 MB Infinity Cache still holds it).  kStream = true:
// non-temporal accesses, for a wire that arrives from and leaves for somewhere else, as in a ring step between
// devices: it is read once and what is written is not read here again.  Measured on MI355X at the 27B shape: with
// every wire cold, streaming accesses make a hop 15.8 us instead of 17.3 us; with a warm wire they make it 16.0 us
// instead of 14.7 us, because the next launch then misses the cache.
template <bool kStream = false>
__device__ __forceinline__ u32x2 load_i8x8(const int8_t *p, int64_t base, int off, int64_t n, bool full)
{
    if (full) {
        const u32x2 *v = reinterpret_cast<const u32x2 *>(p + base + off);
        return kStream ? __builtin_nontemporal_load(v) : *v;
    }
    return whole_end(request_end<kStream>(p, base, off, n), off);
}

// kKeepsHint: a streamed store by an access that keeps its hint.  With one tile per thread the compiler joins the two copies
// that the rare branch of the quotients makes of a store, and drops the hint of __builtin_nontemporal_store with it.
// Measured on MI355X at 2.75 M elements, 20 sets of buffers in turn, us without -> with the hint: quantize 3.04 -> 2.86,
// hop 3.52 -> 3.40, flat reduce of one wire 4.22 -> 3.90; one device's calls in a ring of eight (27B shape) 39.9 -> 38.6.
template <bool kStream = false, bool kKeepsHint = false>
__device__ __forceinline__ void store_i8x8(int8_t *p, int64_t base, int off, int64_t n, bool full, const u32x2 &w)
{
    if (full) {
        u32x2 *v = reinterpret_cast<u32x2 *>(p + base + off);
        if (kStream && kKeepsHint) {
            __builtin_amdgcn_raw_buffer_store_b64(w, bounded(p + base, 0x7fffffff), off, 0, kNonTemporal);
        } else if (kStream) {
            __builtin_nontemporal_store(w, v);
        } else {
            *v = w;
        }
        return;
    }
    const int left = left_of(n, base);
    const int whole = left & ~3;
    __builtin_amdgcn_raw_buffer_store_b64(w, bounded(p + base, whole), off, 0, kStream ? kNonTemporal : 0);
    const bool holds = off == whole || off + 4 == whole;        // the lane with the last, partial word
    const uint32_t last = off == whole ? w.x : w.y;
    const auto end = bounded(p + base, left);
#pragma unroll
    for (int i = 0; i < 3; ++i) {
        __builtin_amdgcn_raw_buffer_store_b8((uint8_t)(last >> (8 * i)), end, holds ? whole + i : kNowhere, 0, 0);
    }
}

// The output of chain_kernel and semi_kernel is, for full workgroups, either streamed (non-temporal, straight to memory)
// or cached: written through L2 (sc0 sc1) so that it stays in the 256 MB Infinity Cache, where the next kernel that reads
// it, or the next call that writes the same buffer, finds it; worth it while the output is a modest part of that cache.
// small_kernel, the strided chain (cached 1 % slower at the 27B shape) and the end of a message stream.
// Measured on MI355X, P = 8, us streamed -> cached: three output buffers in turn 23.0 -> 22.6 (7.9 M elements), 61.8 -> 60.1
// (22 M), 96.4 -> 92.3 (33.5 M), 131.4 -> 125.8 (44 M), 176.9 -> 182.4 (60 M); nine in turn, so that none is found
// again, 23.4 -> 23.0, 62.5 -> 62.5, 97.0 -> 96.2, 132.0 -> 132.3, 179.0 -> 181.4.
constexpr int64_t kCachedOutElems = (int64_t)32 << 20;      // 64 MiB of bf16, a quarter of the cache

// A call that keeps its wire writes P rows of codes, too, which the cache holds as long as they fit with everything else
// that is in use; there the rows count instead of the output.  MI355X, us, output cached -> streamed, three sets of
// buffers in turn: six partials of 14 M elements 50.5 -> 45.5, four of 20.9 M 54.0 -> 48.3, two of 28 M 40.5 -> 38.3, but
// two of 1 M 3.0 -> 3.3 and four of 8 M 21.5 -> 21.9.
__device__ __forceinline__ bool out_stays_cached(int64_t n, int rows) { return n * rows <= kCachedOutElems; }

// cached is looked at for a full tile only.  kKeepsHint: as in store_i8x8.
template <bool kKeepsHint = false>
__device__ __forceinline__ void store_bf16x8(uint16_t *p, int64_t base, int off, int64_t n, bool full, const u32x4 &w,
                                             bool cached = false)
{
    if (full) {
        if (cached) {
            __builtin_amdgcn_raw_buffer_store_b128(w, bounded(p + base, 0x7fffffff), off * 2, 0, kThroughL2);
        } else if (kKeepsHint) {
            __builtin_amdgcn_raw_buffer_store_b128(w, bounded(p + base, 0x7fffffff), off * 2, 0, kNonTemporal);
        } else {
            u32x4 *v = reinterpret_cast<u32x4 *>(p + base + off);
            if (EQUARX_NT_STORE_BF16) {
                __builtin_nontemporal_store(w, v);
            } else {
                *v = w;
            }
        }
        return;
    }
    const int left = left_of(n, base);
    const int whole = left & ~1;
    __builtin_amdgcn_raw_buffer_store_b128(w, bounded(p + base, whole * 2), off * 2, 0, EQUARX_NT_STORE_BF16 ? kNonTemporal : 0);
    const bool holds = off <= whole && whole < off + 8;         // the lane with the last element of an odd length
    const uint32_t last = off == whole ? w.x : off + 2 == whole ? w.y : off + 4 == whole ? w.z : w.w;
    __builtin_amdgcn_raw_buffer_store_b16((uint16_t)last, bounded(p + base, left * 2), holds ? whole * 2 : kNowhere, 0, 0);
}

// With all K tiles of a thread in one basic block the instruction scheduler
// would sink some loads between the arithmetic of earlier tiles to save
// registers; the kernels want every request in flight before the first wait.
__device__ __forceinline__ void loads_first()
{
    asm volatile("" ::: "memory");      // nor may a load move into a conditional block that uses it
#if EQUARX_SCHED_BARRIER
    __builtin_amdgcn_sched_barrier(0);
#endif
}

// ---------------------------------------------------------------- the two quotients of a block

// 127 / a is taken through the hardware reciprocal of a below this bound; from
// 2^126 on, 1/a is subnormal and the reciprocal is no longer accurate enough,
// so a/16 is used there.
constexpr float kRcpSafeBelow = 8.507059173e37f;    // 2^126

// scale = fl32(a / 127) and inv = fl32(127 / a), both CORRECTLY ROUNDED, for a
// block whose max-abs is a (scale = inv = 0 below the tiny threshold).
//
// The compiler's IEEE division costs about 11 instructions per quotient and
// every lane of a group computes both, which is a third of the hop's ALU work.
// These shorter sequences give the same bits:
//   a / 127 : q0 = a*c with c = fl32(1/127), then one exact-remainder
//             correction (the divisor is a constant whose reciprocal is known
//             to half an ulp);
//   127 / a : q0 = 127*rcp(a), then the same correction with the 1-ulp
//             hardware reciprocal.
// That they equal the IEEE quotient is not argued but CHECKED, exhaustively,
// over every finite fp32 a >= 127*2^-126 -- selftest_quotients_kernel below,
// run by the GPU tests.
__device__ __forceinline__ void block_quotients(float a, float &scale, float &inv)
{
    // Straight-line code (selects, no branches): the K tiles of a thread then
    // form one basic block and the compiler interleaves their dependent chains.
    const float c = 1.0f / 127.0f;                      // folded at compile time: fl32(1/127)
    const float q0 = a * c;
    const float e = __builtin_fmaf(-127.0f, q0, a);     // exact remainder a - 127*q0
    const float s = __builtin_fmaf(e, c, q0);
    // From 2^126 on, 1/a is subnormal: divide a/16 instead and scale the
    // quotient by 1/16, both exact (127/a >= 127*2^-128 is still normal).
    const float f = a < kRcpSafeBelow ? 1.0f : 0.0625f;
    const float af = a * f;
    const float y = __builtin_amdgcn_rcpf(af);
    const float p0 = 127.0f * y;
    const float r = __builtin_fmaf(-af, p0, 127.0f);    // exact remainder 127 - af*p0
    const float v = __builtin_fmaf(r, y, p0) * f;
    const bool tiny = a < kTinyAbsmax;                  // what the lanes computed above (inf, NaN) is dropped
    scale = tiny ? 0.0f : s;
    inv = tiny ? 0.0f : v;
}

// Reference form of the same two quotients: the compiler's IEEE division.
__device__ __forceinline__ void block_quotients_ieee(float a, float &scale, float &inv)
{
    if (a < kTinyAbsmax) {
        scale = 0.0f;
        inv = 0.0f;
    } else {
        scale = a / 127.0f;
        inv = 127.0f / a;
    }
}

// ---------------------------------------------------------------- Q_B on registers

// Quantize the E values a lane holds, given that the G lanes of its group hold
// one block.  r[i] receives the code of t[i] as a float (an integer in
// [-127, 127]); `scale` is the block's scale (the same in every lane of the group).
//
// kPositiveZero: a code that rounds to zero from below is -0.0 as a float,
// where the int8 code converted back would be +0.0.  Kernels that keep the
// codes as floats and multiply them again set this flag, which adds +0.0
// (turning -0.0 into +0.0 and changing nothing else); the sign of a zero
// product would otherwise leak into a sum whose other term is -0.0.
template <int G, bool kPositiveZero = false, int E>
__device__ __forceinline__ void quantize_lane_f(const float (&t)[E], float (&r)[E], float &scale)
{
    float m = 0.0f;
#pragma unroll
    for (int i = 0; i < E; ++i) m = __builtin_fmaxf(m, __builtin_fabsf(t[i]));
    const float a = __uint_as_float(group_max_bits<G>(__float_as_uint(m)));

    float inv;
    block_quotients(a, scale, inv);
#pragma unroll
    for (int i = 0; i < E; ++i) {
        // |t*inv| <= 127*(1+2^-23): rounds to at most 127, no clamp needed
        r[i] = __builtin_rintf(t[i] * inv);
        if (kPositiveZero) r[i] += 0.0f;
    }
}

// Adding 1.5 * 2^23 to a float p, |p| < 2^22, rounds p to the nearest integer
// (ties to even, the sum's ulp being 1 and the constant even) and leaves that
// integer, in two's complement, in the low mantissa bits of the sum: the int8
// code of p is the sum's low byte.  Two instructions (multiply, add) where
// round + convert + mask would be four.
constexpr float kRoundMagic = 12582912.0f;

// Byte 0 of each of four words, gathered into one word.
__device__ __forceinline__ uint32_t gather_low_bytes(uint32_t b0, uint32_t b1, uint32_t b2, uint32_t b3)
{
    // v_perm_b32: selector 0..3 = byte of the second operand, 4..7 = byte of the first, 0x0c = zero
    const uint32_t lo = __builtin_amdgcn_perm(b1, b0, 0x0c0c0400u);
    const uint32_t hi = __builtin_amdgcn_perm(b3, b2, 0x04000c0cu);
    return lo | hi;
}

// The 8 float-valued codes of a lane (integers in [-127, 127]) as packed int8.
__device__ __forceinline__ u32x2 pack_codes(const float (&r)[8])
{
    uint32_t b[8];
#pragma unroll
    for (int i = 0; i < 8; ++i) b[i] = __float_as_uint(r[i] + kRoundMagic);     // exact: r[i] is an integer
    u32x2 w;
    w.x = gather_low_bytes(b[0], b[1], b[2], b[3]);
    w.y = gather_low_bytes(b[4], b[5], b[6], b[7]);
    return w;
}

// Q_B of the 8 values of a lane, as packed int8 codes (same codes as
// quantize_lane_f followed by pack_codes).
template <int G>
__device__ __forceinline__ u32x2 quantize_lane(const float (&t)[8], float &scale)
{
    float m = 0.0f;
#pragma unroll
    for (int i = 0; i < 8; ++i) m = __builtin_fmaxf(m, __builtin_fabsf(t[i]));
    const float a = __uint_as_float(group_max_bits<G>(__float_as_uint(m)));
    float inv;
    block_quotients(a, scale, inv);
    uint32_t b[8];
#pragma unroll
    for (int i = 0; i < 8; ++i) b[i] = __float_as_uint(t[i] * inv + kRoundMagic);   // two roundings: product, then sum
    u32x2 w;
    w.x = gather_low_bytes(b[0], b[1], b[2], b[3]);
    w.y = gather_low_bytes(b[4], b[5], b[6], b[7]);
    return w;
}

// ---------------------------------------------------------------- kernels
// Each kernel body exists twice: kFull = true for workgroups whose K tiles lie
// entirely inside [0, n) (straight-line vector code), kFull = false for the one
// workgroup that holds the ragged end (every access guarded).

// The K scales a group leader holds, stored after all K tiles are computed: one
// conditional region at the end instead of one per tile, so the tiles'
// arithmetic stays in a single basic block.
template <int B, int T, int K, bool kFull>
__device__ __forceinline__ void store_group_scales(float *scales, const float (&scale)[K], int64_t wg_at, int64_t nb)
{
    constexpr int G = B / kLaneElems;
    if ((threadIdx.x % G) == 0) {
#pragma unroll
        for (int k = 0; k < K; ++k) {
            const int64_t blk = (wg_at + k * tile_elems<T>) / B + threadIdx.x / G;
            if (kFull || blk < nb) scales[blk] = scale[k];
        }
    }
}

template <int B, int T, int K, bool kFull, bool kStream = false>
__device__ __forceinline__ void quantize_body(const uint16_t *__restrict__ x, int64_t n, int8_t *__restrict__ codes,
                                              float *__restrict__ scales, int64_t nb, int64_t wg_at)
{
    constexpr int G = B / kLaneElems;
    const int lane_at = threadIdx.x * kLaneElems;

    u32x4 xv[K];
#pragma unroll
    for (int k = 0; k < K; ++k) xv[k] = load_bf16x8(x, wg_at + k * tile_elems<T>, lane_at, n, kFull);
    loads_first();

    float scale[K];
#pragma unroll
    for (int k = 0; k < K; ++k) {
        const int64_t base = wg_at + k * tile_elems<T>;
        float t[8];
        widen_bf16x8(xv[k], t);
        const u32x2 w = quantize_lane<G>(t, scale[k]);
        store_i8x8<kStream, K == 1>(codes, base, lane_at, n, kFull, w);
    }
    store_group_scales<B, T, K, kFull>(scales, scale, wg_at, nb);
}

// Pass 0 of the chain: quantize a bf16 tensor.
template <int B, int K, bool kStream = false>
__global__ __launch_bounds__(pass_threads(K)) void quantize_kernel(Global<const uint16_t> x, int64_t n,
                                                            Global<int8_t> codes, Global<float> scales,
                                                            int64_t nb)
{
    constexpr int T = pass_threads(K);
    const int64_t wg_at = (int64_t)blockIdx.x * (tile_elems<T> * K);
    if (wg_at + tile_elems<T> * K <= n) {
        quantize_body<B, T, K, true, kStream>(x, n, codes, scales, nb, wg_at);
    } else {
        quantize_body<B, T, K, false, kStream>(x, n, codes, scales, nb, wg_at);
    }
}

// Several tensors of the same length in one launch (blockIdx.y picks the
// tensor): what a device does before an all-to-all, when it quantizes one shard
// per peer.  One launch instead of one per shard spares the per-launch ramp.
constexpr int kMaxBatch = 64;

struct QuantizeBatch {
    const uint16_t *x[kMaxBatch];
    int8_t *codes[kMaxBatch];
    float *scales[kMaxBatch];
};

template <int B, int K, bool kStream = false>
__global__ __launch_bounds__(pass_threads(K)) void quantize_batch_kernel(int64_t n, int64_t nb, const QuantizeBatch tab)
{
    constexpr int T = pass_threads(K);
    const uint16_t *x = tab.x[blockIdx.y];
    int8_t *codes = tab.codes[blockIdx.y];
    float *scales = tab.scales[blockIdx.y];
    const int64_t wg_at = (int64_t)blockIdx.x * (tile_elems<T> * K);
    if (wg_at + tile_elems<T> * K <= n) {
        quantize_body<B, T, K, true, kStream>(x, n, codes, scales, nb, wg_at);
    } else {
        quantize_body<B, T, K, false, kStream>(x, n, codes, scales, nb, wg_at);
    }
}

template <int B, int T, int K, bool kFull, bool kStream = false>
__device__ __forceinline__ void hop_body(const int8_t *cin, const float *sin, const uint16_t *__restrict__ x,
                                         int64_t n, int8_t *cout, float *sout, int64_t nb, int64_t wg_at)
{
    constexpr int G = B / kLaneElems;
    const int lane_at = threadIdx.x * kLaneElems;

    u32x4 xv[K];
    u32x2 cv[K];
    float sv[K];
#pragma unroll
    for (int k = 0; k < K; ++k) {
        const int64_t base = wg_at + k * tile_elems<T>;
        xv[k] = load_bf16x8(x, base, lane_at, n, kFull);
        cv[k] = load_i8x8<kStream>(cin, base, lane_at, n, kFull);
        const int64_t blk = base / B + lane_at / B;
        sv[k] = sin[kFull || blk < nb ? blk : nb - 1];
    }
    loads_first();

    float scale[K];
#pragma unroll
    for (int k = 0; k < K; ++k) {
        const int64_t base = wg_at + k * tile_elems<T>;
        float xf[8], qf[8], t[8];
        widen_bf16x8(xv[k], xf);
        widen_i8x8(cv[k], qf);
#pragma unroll
        for (int i = 0; i < 8; ++i) t[i] = __builtin_fmaf(qf[i], sv[k], xf[i]);
        const u32x2 w = quantize_lane<G>(t, scale[k]);
        store_i8x8<kStream, K == 1>(cout, base, lane_at, n, kFull, w);
    }
    store_group_scales<B, T, K, kFull>(sout, scale, wg_at, nb);
}

// One hop: dequantize the incoming wire, add the local bf16 shard in fp32
// (one fused multiply-add per element), quantize the partial sum.  The output
// wire may be the input wire: a thread reads its own elements, and a group its
// own scale, before either is written.
template <int B, int K, bool kStream = false>
__global__ __launch_bounds__(pass_threads(K)) void hop_kernel(Global<const int8_t> cin, Global<const float> sin,
                                                       Global<const uint16_t> x, int64_t n,
                                                       Global<int8_t> cout, Global<float> sout, int64_t mirror)
{
    constexpr int T = pass_threads(K);
    const int64_t wg_at = first_element<T, K, !kStream>(mirror);
    const int64_t nb = (n + B - 1) / B;
    if (wg_at + tile_elems<T> * K <= n) {
        hop_body<B, T, K, true, kStream>(cin, sin, x, n, cout, sout, nb, wg_at);
    } else {
        hop_body<B, T, K, false, kStream>(cin, sin, x, n, cout, sout, nb, wg_at);
    }
}

template <int B, int T, int K, bool kFull, bool kStream = false>
__device__ __forceinline__ void dequantize_body(const int8_t *__restrict__ codes, const float *__restrict__ scales,
                                                int64_t n, uint16_t *__restrict__ out, int64_t nb, int64_t wg_at)
{
    const int lane_at = threadIdx.x * kLaneElems;

    u32x2 cv[K];
    EndOfI8 end[K];
    float sv[K];
#pragma unroll
    for (int k = 0; k < K; ++k) {
        const int64_t base = wg_at + k * tile_elems<T>;
        if (kFull) cv[k] = load_i8x8<kStream>(codes, base, lane_at, n, true);
        else end[k] = request_end<kStream>(codes, base, lane_at, n);
        const int64_t blk = base / B + lane_at / B;
        sv[k] = scales[kFull || blk < nb ? blk : nb - 1];
    }
    if (!kFull) {
        loads_first();
#pragma unroll
        for (int k = 0; k < K; ++k) cv[k] = whole_end(end[k], lane_at);
    }
#pragma unroll
    for (int k = 0; k < K; ++k) {
        const int64_t base = wg_at + k * tile_elems<T>;
        float qf[8];
        widen_i8x8(cv[k], qf);
        u32x4 w;
        w.x = narrow_bf16x2(qf[0] * sv[k], qf[1] * sv[k]);
        w.y = narrow_bf16x2(qf[2] * sv[k], qf[3] * sv[k]);
        w.z = narrow_bf16x2(qf[4] * sv[k], qf[5] * sv[k]);
        w.w = narrow_bf16x2(qf[6] * sv[k], qf[7] * sv[k]);
        store_bf16x8(out, base, lane_at, n, kFull, w);
    }
}

// Last pass: dequantize the wire to bf16.
template <int B, int K, bool kStream = false, int T = pass_threads(K)>
__global__ __launch_bounds__(T) void dequantize_kernel(Global<const int8_t> codes,
                                                              Global<const float> scales, int64_t n,
                                                              Global<uint16_t> out, int64_t mirror)
{
    const int64_t wg_at = first_element<T, K, !kStream>(mirror);
    const int64_t nb = (n + B - 1) / B;
    if (wg_at + tile_elems<T> * K <= n) {
        dequantize_body<B, T, K, true, kStream>(codes, scales, n, out, nb, wg_at);
    } else {
        dequantize_body<B, T, K, false, kStream>(codes, scales, n, out, nb, wg_at);
    }
}

// ---------------------------------------------------------------- the whole chain in one launch
// Blocks never interact, so a workgroup can run all hops on its own tiles with
// the running sum held in registers: the same operations in the same order as
// the hop-by-hop passes, hence the same bits.  The partials are read once each
// (the next one's loads are issued before the current hop's arithmetic); the
// wire is written only if the caller keeps it (kWire) and is never read back.
//
// Template knobs (the stage selection of Sec. 3.4):
//   kRS  what a device forwards during the reduce-scatter is quantized
//        (otherwise the running sum stays fp32 and is added with plain adds);
//   kAG  the finished sum is quantized once more for the all-gather and
//        dequantized (otherwise it is narrowed to bf16 directly).
// Ring layout: with shard_elems > 0 the tensor is cut into gridDim.y shards of
// shard_elems elements (a multiple of B) and shard k is reduced in the rotated
// order rot+0, rot+1, ... (mod P) with rot = k + rot_bias.

constexpr int kMaxPartials = 64;

struct PartialTable {
    const uint16_t *x[kMaxPartials];
};

template <int T, int K, bool kFull>
__device__ __forceinline__ void load_tiles(const uint16_t *p, int64_t wg_at, int64_t n, u32x4 (&v)[K])
{
    const int lane_at = threadIdx.x * kLaneElems;
#pragma unroll
    for (int k = 0; k < K; ++k) v[k] = load_bf16x8(p, wg_at + k * tile_elems<T>, lane_at, n, kFull);
}

// load_tiles with the end of a tensor in the two steps above, for a loop in which the compiler would not keep the tiles'
// requests together by itself (semi_body).  Not for the full loop: there it does, and in two steps it waits for the tiles
// before the quantization that could have run meanwhile (MI355X, eight partials of 4.2 M elements 13.4 -> 13.9 us).
template <int T, int K, bool kFull>
__device__ __forceinline__ void load_tiles_together(const uint16_t *p, int64_t wg_at, int64_t n, u32x4 (&v)[K])
{
    if (kFull || K == 1) {
        load_tiles<T, K, kFull>(p, wg_at, n, v);
        return;
    }
    const int lane_at = threadIdx.x * kLaneElems;
    EndOfBf16 e[K];
#pragma unroll
    for (int k = 0; k < K; ++k) e[k] = request_end(p, wg_at + k * tile_elems<T>, lane_at, n);
    loads_first();
#pragma unroll
    for (int k = 0; k < K; ++k) v[k] = whole_end(e[k], lane_at);
}

// What becomes of the wire in a single launch: it stays in registers, or the caller keeps it (cached stores, or through L2).
enum KeptWire { kNoWire, kCachedWire, kWireThroughL2 };

// From the shapes of 1024 threads or 4 tiles on, a kept wire is written through L2, as the output is (store_bf16x8): P rows of
// codes pushed out of the L2s as they fall cost the partials' reads more than stores that go straight on.  Not if its rows
// do not begin on 64-byte lines: then every wave's stores begin and end within one, and written through those are two writes.
// Non-temporal stores would be better still while no buffer is found again, and worse where the caller's are.  Measured on
// MI355X, us, cached -> through L2 -> non-temporal, with buffers in turn and with one wire for all calls:
//     P = 2, 20 M elements, block 256     28.8 -> 29.1 -> 28.4     27.9 -> 27.0 -> 28.5
//     5, 10 M, 64                         32.5 -> 31.7 -> 30.4     29.1 -> 28.4 -> 30.2
//     8, 5.8 M, 256                       28.6 -> 28.8 -> 27.7     26.0 -> 26.0 -> 27.7
//     8, 12 M, 32                         61.4 -> 58.4 -> 54.4     51.9 -> 50.4 -> 54.2
//     8, 22 M, 256                       105.1 -> 99.6 -> 97.6     91.4 -> 88.9 -> 97.5
//     8, 12,000,001, 256                  60.5 -> 66.5             51.2 -> 51.0       (rows 16 bytes off)
//     16, 16 M, 128                        161 -> 151 -> 139        125 -> 121 -> 138
// Nine sets of buffers, three and one for all calls, another time: P = 2, 20 M 29.2 -> 29.0, 28.2 -> 26.9, 27.8 -> 26.7; P = 8, 5.8 M
// 28.9 -> 29.0, 26.1 -> 25.9, 26.1 -> 25.8; 22 M 105.1 -> 99.9, 105.4 -> 99.7, 90.5 -> 87.7; and of 160 calls (P = 2 to 16, 4.8 to 33.6 M,
// blocks 64 and 256) with three sets and one none is slower by more than 0.6 %.
// Shorter messages' shapes keep cached stores: P = 12, 4.7 M 36.9 -> 40.0 -> 34.7, P = 3, 3 M 7.9 -> 8.2 -> 8.0.
constexpr bool wire_through_l2(int T, int K) { return T == 1024 || K == 4; }

// Writes what the wire carries after a quantization of one tile (8 codes per
// lane starting at element base + off): row `row` of the kept wire.
template <int B, bool kFull, KeptWire kWire>
__device__ __forceinline__ void store_wire_tile(int8_t *__restrict__ wire_codes, float *__restrict__ wire_scales,
                                                int64_t c_step, int64_t s_step, int row, int64_t base, int off,
                                                int64_t n, const float (&r)[8], float s)
{
    constexpr int G = B / kLaneElems;
    int8_t *codes = wire_codes + (int64_t)row * c_step;
    if (kWire == kWireThroughL2 && kFull) {
        __builtin_amdgcn_raw_buffer_store_b64(pack_codes(r), bounded(codes + base, 0x7fffffff), off, 0, kThroughL2);
    } else {
        store_i8x8(codes, base, off, n, kFull, pack_codes(r));
    }
    if ((threadIdx.x % G) == 0 && (kFull || base + off < n)) wire_scales[(int64_t)row * s_step + (base + off) / B] = s;
}

// out = bf16(v) for the 8 fp32 values of one lane.
template <bool kFull, bool kKeepsHint = false>
__device__ __forceinline__ void store_narrowed_tile(uint16_t *out, int64_t base, int off, int64_t n,
                                                    const float (&v)[8], bool cached = false)
{
    u32x4 w;
    w.x = narrow_bf16x2(v[0], v[1]);
    w.y = narrow_bf16x2(v[2], v[3]);
    w.z = narrow_bf16x2(v[4], v[5]);
    w.w = narrow_bf16x2(v[6], v[7]);
    store_bf16x8<kKeepsHint>(out, base, off, n, kFull, w, cached);
}

// The last step of a chain for one tile: quantize the finished fp32 sum once
// more and dequantize it (quantized all-gather, Sec. 3.4), or narrow it directly.
template <int B, bool kAG, KeptWire kWire, bool kFull>
__device__ __forceinline__ void finish_tile(const float (&t)[8], uint16_t *out,
                                            int8_t *__restrict__ wire_codes, float *__restrict__ wire_scales,
                                            int64_t c_step, int64_t s_step, int row, int64_t base, int off, int64_t n,
                                            bool cached = false)
{
    constexpr int G = B / kLaneElems;
    if (kAG) {
        float r[8], s;
        quantize_lane_f<G, true>(t, r, s);      // +0.0 codes: the product below shows the sign of a zero
        if (kWire) store_wire_tile<B, kFull, kWire>(wire_codes, wire_scales, c_step, s_step, row, base, off, n, r, s);
        float d[8];
#pragma unroll
        for (int j = 0; j < 8; ++j) d[j] = r[j] * s;
        store_narrowed_tile<kFull, kWire != kNoWire>(out, base, off, n, d, cached);
    } else {
        store_narrowed_tile<kFull, kWire != kNoWire>(out, base, off, n, t, cached);
    }
}

// ---------------------------------------------------------------- first and last launch of the end-fused schedule
//
// The hop-by-hop chain spends its first two launches on Q_B(x_0) and on hop 1,
// and its last two on hop P-1 and on the dequantization.  On one device each
// pair can share a launch: c_0 and c_(P-1) then stay in registers and 2 of the
// P+1 passes (and 2 of the P wire round trips) disappear.  Same operations in
// the same order, so the same bits.

// (c_1, s_1) = Q_B( fma(codes_0, s_0, x_1) ),  (codes_0, s_0) = Q_B(x_0) kept in registers.
template <int B, int T, int K, bool kFull>
__device__ __forceinline__ void head_body(const uint16_t *__restrict__ x0, const uint16_t *__restrict__ x1, int64_t n,
                                          int8_t *__restrict__ cout, float *__restrict__ sout, int64_t nb,
                                          int64_t wg_at)
{
    constexpr int G = B / kLaneElems;
    const int lane_at = threadIdx.x * kLaneElems;
    u32x4 av[K], bv[K];
    load_tiles<T, K, kFull>(x0, wg_at, n, av);
    load_tiles<T, K, kFull>(x1, wg_at, n, bv);
    loads_first();
    float scale[K];
#pragma unroll
    for (int k = 0; k < K; ++k) {
        const int64_t base = wg_at + k * tile_elems<T>;
        float t[8], r[8], xf[8], s0;
        widen_bf16x8(av[k], t);
        quantize_lane_f<G, false>(t, r, s0);        // a -0.0 code only flips the sign of a zero sum, which Q_B ignores
        widen_bf16x8(bv[k], xf);
#pragma unroll
        for (int j = 0; j < 8; ++j) t[j] = __builtin_fmaf(r[j], s0, xf[j]);
        const u32x2 w = quantize_lane<G>(t, scale[k]);
        store_i8x8(cout, base, lane_at, n, kFull, w);
    }
    store_group_scales<B, T, K, kFull>(sout, scale, wg_at, nb);
}

template <int B, int K>
__global__ __launch_bounds__(pass_threads(K)) void head_kernel(Global<const uint16_t> x0,
                                                        Global<const uint16_t> x1, int64_t n,
                                                        Global<int8_t> cout, Global<float> sout,
                                                        int64_t nb)
{
    constexpr int T = pass_threads(K);
    const int64_t wg_at = (int64_t)blockIdx.x * (tile_elems<T> * K);
    if (wg_at + tile_elems<T> * K <= n) {
        head_body<B, T, K, true>(x0, x1, n, cout, sout, nb, wg_at);
    } else {
        head_body<B, T, K, false>(x0, x1, n, cout, sout, nb, wg_at);
    }
}

// out = bf16( DQ( Q_B( fma(codes_in, s_in, x) ) ) ): the last hop and the quantized all-gather's pair (Sec. 3.4);
// kAG = false: out = bf16( fma(codes_in, s_in, x) ), the all-gather left unquantized.
template <int B, int T, int K, bool kAG, bool kFull>
__device__ __forceinline__ void tail_body(const int8_t *__restrict__ cin, const float *__restrict__ sin,
                                          const uint16_t *x, int64_t n, uint16_t *out,
                                          int64_t nb, int64_t wg_at)
{
    const int lane_at = threadIdx.x * kLaneElems;
    u32x4 xv[K];
    u32x2 cv[K];
    float sv[K];
#pragma unroll
    for (int k = 0; k < K; ++k) {
        const int64_t base = wg_at + k * tile_elems<T>;
        xv[k] = load_bf16x8(x, base, lane_at, n, kFull);
        cv[k] = load_i8x8(cin, base, lane_at, n, kFull);
        const int64_t blk = base / B + lane_at / B;
        sv[k] = sin[kFull || blk < nb ? blk : nb - 1];
    }
    loads_first();
#pragma unroll
    for (int k = 0; k < K; ++k) {
        float xf[8], qf[8], t[8];
        widen_bf16x8(xv[k], xf);
        widen_i8x8(cv[k], qf);
#pragma unroll
        for (int j = 0; j < 8; ++j) t[j] = __builtin_fmaf(qf[j], sv[k], xf[j]);
        finish_tile<B, kAG, kNoWire, kFull>(t, out, nullptr, nullptr, 0, 0, 0, wg_at + k * tile_elems<T>, lane_at, n);
    }
}

template <int B, int K, bool kAG>
__global__ __launch_bounds__(pass_threads(K)) void tail_kernel(Global<const int8_t> cin, Global<const float> sin,
                                                        Global<const uint16_t> x, int64_t n,      // out may be x (in place)
                                                        Global<uint16_t> out, int64_t mirror)
{
    constexpr int T = pass_threads(K);
    const int64_t wg_at = first_element<T, K>(mirror);
    const int64_t nb = (n + B - 1) / B;
    if (wg_at + tile_elems<T> * K <= n) {
        tail_body<B, T, K, kAG, true>(cin, sin, x, n, out, nb, wg_at);
    } else {
        tail_body<B, T, K, kAG, false>(cin, sin, x, n, out, nb, wg_at);
    }
}

// Position -> partial index on a ring of P devices, without a division: the
// callers only ever step by one.
__device__ __forceinline__ int ring_next(int j, int P) { return j + 1 == P ? 0 : j + 1; }
__device__ __forceinline__ int ring_prev(int j, int P) { return j == 0 ? P - 1 : j - 1; }

// One hop on the K tiles of a workgroup: (what the previous device sends) = Q_B(t),
// t = fma(codes, scale, x) -- or a plain fp32 add when the reduce-scatter is
// not quantized.  The quantization does not need x, so it runs while x arrives.
//
// kPositiveZero (see quantize_lane_f) is needed only where the sign of a zero
// sum can reach the output, i.e. when the all-gather is NOT quantized; with a
// quantized all-gather a -0.0 code can only flip the sign of zero sums along
// the chain, which no max-abs, scale or integer code sees, and the last
// quantization hands out +0.0 codes.
template <int B, int T, int K, bool kRS, KeptWire kWire, bool kPositiveZero, bool kFull>
__device__ __forceinline__ void hop_tiles(float (&t)[K][8], const u32x4 (&x)[K], int8_t *__restrict__ wire_codes,
                                          float *__restrict__ wire_scales, int64_t c_step, int64_t s_step, int row,
                                          int64_t wg_at, int64_t n)
{
    constexpr int G = B / kLaneElems;
    const int lane_at = threadIdx.x * kLaneElems;
#pragma unroll
    for (int k = 0; k < K; ++k) {
        if (kRS) {
            float r[8], s;
            quantize_lane_f<G, kPositiveZero>(t[k], r, s);
            if (kWire) {
                store_wire_tile<B, kFull, kWire>(wire_codes, wire_scales, c_step, s_step, row,
                                                 wg_at + k * tile_elems<T>, lane_at, n, r, s);
            }
            float xf[8];
            widen_bf16x8(x[k], xf);
#pragma unroll
            for (int j = 0; j < 8; ++j) t[k][j] = __builtin_fmaf(r[j], s, xf[j]);
        } else {
            float xf[8];
            widen_bf16x8(x[k], xf);
#pragma unroll
            for (int j = 0; j < 8; ++j) t[k][j] = t[k][j] + xf[j];
        }
    }
}

// Full-loop adder chain over the partials in the order rot, rot+1, ... (mod P).
// Per tile the only state carried from hop to hop is the fp32 sum t.  Each hop
// loads its partial and then computes; the quantization of the running sum
// does not need the new data and runs while it arrives.  Starting the loads a
// hop (or several) ahead was measured with four tiles per thread and is SLOWER
// on MI355X (63 -> 67..72 us at the 27B-shaped size): the memory system is
// saturated as it is, and more outstanding requests only lengthen its queues.
template <int B, int T, int K, bool kRS, bool kAG, KeptWire kWire, bool kFull>
__device__ __forceinline__ void chain_body(const PartialTable &tab, int P, int rot, int64_t n,
                                           uint16_t *out, int8_t *__restrict__ wire_codes,
                                           float *__restrict__ wire_scales, int64_t c_step, int64_t s_step,
                                           int64_t wg_at, bool cached)
{
    const int lane_at = threadIdx.x * kLaneElems;
    float t[K][8];      // running fp32 sum
    u32x4 x0[K], xv[K];     // separate registers: partial 1 may be requested before partial 0 has arrived

    int j = rot >= P ? rot - P : rot;               // rot < 2P
    load_tiles<T, K, kFull>(tab.x[j], wg_at, n, x0);
#pragma unroll
    for (int k = 0; k < K; ++k) widen_bf16x8(x0[k], t[k]);
    for (int i = 1; i < P; ++i) {
        j = ring_next(j, P);
        load_tiles<T, K, kFull>(tab.x[j], wg_at, n, xv);
        hop_tiles<B, T, K, kRS, kWire, !kAG, kFull>(t, xv, wire_codes, wire_scales, c_step, s_step, i - 1, wg_at, n);
    }

#pragma unroll
    for (int k = 0; k < K; ++k) {
        finish_tile<B, kAG, kWire, kFull>(t[k], out, wire_codes, wire_scales, c_step, s_step, P - 1,
                                          wg_at + k * tile_elems<T>, lane_at, n, cached);
    }
}

// The same chain with TWO pieces per lane taken from the same block (B >= 128):
// the B/16 lanes of a block each hold elements [8l, 8l+8) and [B/2 + 8l, B/2 +
// 8l + 8) of it, so the max-abs reduction crosses half as many lanes and the
// two quotients are computed once per 16 elements instead of once per 8 --
// a fifth less arithmetic per element-hop in the one kernel whose vector ALU
// is busy half the time (measured at the 27B shape: 4 % faster).  Every wave
// access still covers whole 128-byte lines: the lanes of a block read B/2
// consecutive elements, B bytes, per load.  Same operations per element in the
// same order: same bits.  Full tiles only; the kept-wire form stays on chain_body.
template <int B, int T, int K2, bool kRS, bool kAG>
__device__ __forceinline__ void chain_body_paired(const PartialTable &tab, int P, int rot,
                                                  uint16_t *out, int64_t wg_at, bool cached)
{
    constexpr int Gh = B / 16;                      // lanes per block
    constexpr int kPairElems = 2 * tile_elems<T>;      // the workgroup's pairs of pieces: 16 T elements
    const int lane_off = (threadIdx.x / Gh) * B + (threadIdx.x % Gh) * kLaneElems;
    float t[K2][2][8];
    u32x4 x0[K2][2], xv[K2][2];

    int j = rot >= P ? rot - P : rot;
    {
        const uint16_t *p = tab.x[j];
#pragma unroll
        for (int k = 0; k < K2; ++k) {
#pragma unroll
            for (int h = 0; h < 2; ++h) x0[k][h] = load_bf16x8(p, wg_at + k * kPairElems, lane_off + h * (B / 2), 0, true);
        }
    }
#pragma unroll
    for (int k = 0; k < K2; ++k) {
#pragma unroll
        for (int h = 0; h < 2; ++h) widen_bf16x8(x0[k][h], t[k][h]);
    }
    for (int i = 1; i < P; ++i) {
        j = ring_next(j, P);
        const uint16_t *p = tab.x[j];
#pragma unroll
        for (int k = 0; k < K2; ++k) {
#pragma unroll
            for (int h = 0; h < 2; ++h) xv[k][h] = load_bf16x8(p, wg_at + k * kPairElems, lane_off + h * (B / 2), 0, true);
        }
#pragma unroll
        for (int k = 0; k < K2; ++k) {
            float xf[2][8];
            if (kRS) {
                float m = 0.0f;
#pragma unroll
                for (int h = 0; h < 2; ++h) {
#pragma unroll
                    for (int e = 0; e < 8; ++e) m = __builtin_fmaxf(m, __builtin_fabsf(t[k][h][e]));
                }
                const float a = __uint_as_float(group_max_bits<Gh>(__float_as_uint(m)));
                float s, inv;
                block_quotients(a, s, inv);
#pragma unroll
                for (int h = 0; h < 2; ++h) {
                    widen_bf16x8(xv[k][h], xf[h]);
#pragma unroll
                    for (int e = 0; e < 8; ++e) {
                        float r = __builtin_rintf(t[k][h][e] * inv);
                        if (!kAG) r += 0.0f;        // see hop_tiles: only an unquantized all-gather shows a zero's sign
                        t[k][h][e] = __builtin_fmaf(r, s, xf[h][e]);
                    }
                }
            } else {
#pragma unroll
                for (int h = 0; h < 2; ++h) {
                    widen_bf16x8(xv[k][h], xf[h]);
#pragma unroll
                    for (int e = 0; e < 8; ++e) t[k][h][e] = t[k][h][e] + xf[h][e];
                }
            }
        }
    }

#pragma unroll
    for (int k = 0; k < K2; ++k) {
        if (kAG) {
            float m = 0.0f;
#pragma unroll
            for (int h = 0; h < 2; ++h) {
#pragma unroll
                for (int e = 0; e < 8; ++e) m = __builtin_fmaxf(m, __builtin_fabsf(t[k][h][e]));
            }
            const float a = __uint_as_float(group_max_bits<Gh>(__float_as_uint(m)));
            float s, inv;
            block_quotients(a, s, inv);
#pragma unroll
            for (int h = 0; h < 2; ++h) {
                float d[8];
#pragma unroll
                for (int e = 0; e < 8; ++e) d[e] = (__builtin_rintf(t[k][h][e] * inv) + 0.0f) * s;
                store_narrowed_tile<true>(out, wg_at + k * kPairElems, lane_off + h * (B / 2), 0, d, cached);
            }
        } else {
#pragma unroll
            for (int h = 0; h < 2; ++h) {
                store_narrowed_tile<true>(out, wg_at + k * kPairElems, lane_off + h * (B / 2), 0, t[k][h], cached);
            }
        }
    }
}

// Where a workgroup works: its shard [lo, hi) and rotation, its first element.
struct Span {
    int64_t wg_at, hi;
    int rot;
    bool any;
};

// Workgroups per shard in a launch whose shards are walked back (ring layout): whole groups of eight, so that a
// workgroup's XCD follows from its place in the row whatever the row.
template <typename S>
__host__ __device__ inline int64_t ring_groups(int64_t shard_elems) { return ((shard_elems + S::kElems - 1) / S::kElems + 7) & ~(int64_t)7; }

// kTurns, back: the number of shards if the launch walks back (ring layout only), the last shard first and each from its
// end.  Launches that never walk back do not ask, as in first_element (MI355X, ring order hop by hop, block 64, P = 5, 4.4 M
// elements: 24.11 -> 23.79 us).
template <int T, int K, bool kTurns = false>
__device__ __forceinline__ Span workgroup_span(int64_t n, int64_t shard_elems, int rot_bias, int back = 0)
{
    Span sp;
    int64_t lo = 0;
    sp.hi = n;
    sp.rot = 0;
    if (shard_elems > 0) {
        const int shard = kTurns && back ? back - 1 - (int)blockIdx.y : (int)blockIdx.y;
        lo = (int64_t)shard * shard_elems;
        sp.hi = lo + shard_elems < n ? lo + shard_elems : n;
        sp.rot = shard + rot_bias;
    }
    sp.wg_at = lo + first_element<T, K, kTurns>(kTurns && back ? ring_groups<Shape<T, K>>(shard_elems) * Shape<T, K>::kElems : 0);
    sp.any = sp.wg_at < sp.hi;
    return sp;
}

// Waves per SIMD the compiler may plan for.  The shape for the largest messages is held to two, of the five its
// registers would allow: eight tiles of one partial after the other are enough requests in flight, and the fewer
// places of memory are read at once the better they stream.  Measured on MI355X, P = 8, block 256, us with five / four /
// three / two / one: 255.9 / 258.2 / 258.8 / 247.5 / 332 at 88 M elements, 93.7 / 91.0 / 91.9 / 90.0 / 139 at 33.5 M; 6
// tiles or 512 threads under the same cap 264 at 88 M, 3 tiles 264, 8 tiles and one wave 252.  The other flavours, with
// all the registers allow -> with two (and 1024 x 1 instead):
//                                    22 M                   33.5 M                    88 M
//     block 32                62.2 -> 62.8 (60.9)     94.0 ->  91.3 (93.2)    262.9 -> 246.5 (260.6)
//     block 64, ring order    62.1 -> 62.6 (61.1)     94.1 ->  91.1 (91.8)    261.0 -> 245.2 (258.7)
//     block 64, kept wire    107.6 -> 106.1 (106.6)  164.1 -> 162.6 (165.7)   431.4 -> 422.9 (429.8)
//     block 64, RS in fp32    62.6 -> 62.5 (61.1)     93.8 ->  90.9 (91.8)    264.4 -> 252.4 (260.0)
//     block 256, AG in bf16   62.1 -> 61.1 (61.4)     93.9 ->  89.6 (91.5)    261.5 -> 244.3 (257.4)
constexpr int chain_waves(int K) { return K == 4 ? 2 : 8; }

template <int B, int T, int K, bool kRS, bool kAG, KeptWire kWire>
__global__ __launch_bounds__(T) __attribute__((amdgpu_waves_per_eu(1, chain_waves(K))))
void chain_kernel(int P, int64_t n, int64_t shard_elems, Global<uint16_t> out,
                  Global<int8_t> wire_codes,
                  Global<float> wire_scales, int64_t c_step,
                  int64_t s_step, const PartialTable tab)
{
    const Span sp = workgroup_span<T, K>(n, shard_elems, 1);     // shard k: devices k+1, k+2, ..., k
    if (!sp.any) return;                                      // uniform over the workgroup
    if (sp.wg_at + tile_elems<T> * K <= sp.hi) {
        if (EQUARX_CHAIN_PAIRED && B >= 128 && K % 2 == 0 && !kWire) {
            chain_body_paired<(B >= 128 ? B : 128), T, (K >= 2 ? K / 2 : 1), kRS, kAG>(tab, P, sp.rot, out, sp.wg_at,
                                                                                            out_stays_cached(n, kWire ? P : 1));
        } else {
            chain_body<B, T, K, kRS, kAG, kWire, true>(tab, P, sp.rot, sp.hi, out, wire_codes, wire_scales, c_step,
                                                    s_step, sp.wg_at, out_stays_cached(n, kWire ? P : 1));
        }
    } else {
        chain_body<B, T, K, kRS, kAG, kWire, false>(tab, P, sp.rot, sp.hi, out, wire_codes, wire_scales, c_step, s_step,
                                                 sp.wg_at, out_stays_cached(n, kWire ? P : 1));
    }
}

// ---------------------------------------------------------------- ring order, hop by hop
//
// What all devices of a ring do in one step, as one launch: grid row k works on
// shard k, whose chain visits devices k+1, k+2, ..., k (mod P), so in step i it
// adds device (k + 1 + i)'s partial.  Same bodies as the plain per-pass
// kernels; only the partial, and the end of the range, depend on the grid row.

template <int B, int K>
__global__ __launch_bounds__(pass_threads(K)) void quantize_ring_kernel(int P, int64_t n, int64_t shard_elems,
                                                                 Global<int8_t> codes,
                                                                 Global<float> scales, const PartialTable tab)
{
    constexpr int T = pass_threads(K);
    const Span sp = workgroup_span<T, K>(n, shard_elems, 1);
    if (!sp.any) return;
    const uint16_t *x = tab.x[sp.rot >= P ? sp.rot - P : sp.rot];
    const int64_t nb = (sp.hi + B - 1) / B;
    if (sp.wg_at + tile_elems<T> * K <= sp.hi) {
        quantize_body<B, T, K, true>(x, sp.hi, codes, scales, nb, sp.wg_at);
    } else {
        quantize_body<B, T, K, false>(x, sp.hi, codes, scales, nb, sp.wg_at);
    }
}

// kTurns: the wire is long enough that every second launch walks back (kTurnFrom).
template <int B, int K, bool kTurns>
__global__ __launch_bounds__(pass_threads(K)) void hop_ring_kernel(Global<const int8_t> cin, Global<const float> sin, int P, int step,
                                                            int64_t n, int64_t shard_elems, Global<int8_t> cout, Global<float> sout,
                                                            const PartialTable tab)
{
    constexpr int T = pass_threads(K);
    const Span sp = workgroup_span<T, K, kTurns>(n, shard_elems, 1 + step, (step & 1) != 0 ? P : 0);    // row + 1 + step < 2P
    if (!sp.any) return;
    const uint16_t *x = tab.x[sp.rot >= P ? sp.rot - P : sp.rot];
    const int64_t nb = (sp.hi + B - 1) / B;
    if (sp.wg_at + tile_elems<T> * K <= sp.hi) {
        hop_body<B, T, K, true>(cin, sin, x, sp.hi, cout, sout, nb, sp.wg_at);
    } else {
        hop_body<B, T, K, false>(cin, sin, x, sp.hi, cout, sout, nb, sp.wg_at);
    }
}

template <int B, int K, bool kAG, bool kTurns>
__global__ __launch_bounds__(pass_threads(K)) void tail_ring_kernel(Global<const int8_t> cin,
                                                             Global<const float> sin, int P, int step, int64_t n,
                                                             int64_t shard_elems, Global<uint16_t> out,
                                                             const PartialTable tab)
{
    constexpr int T = pass_threads(K);
    const Span sp = workgroup_span<T, K, kTurns>(n, shard_elems, 1 + step, (step & 1) != 0 ? P : 0);
    if (!sp.any) return;
    const uint16_t *x = tab.x[sp.rot >= P ? sp.rot - P : sp.rot];
    const int64_t nb = (sp.hi + B - 1) / B;
    if (sp.wg_at + tile_elems<T> * K <= sp.hi) {
        tail_body<B, T, K, kAG, true>(cin, sin, x, sp.hi, out, nb, sp.wg_at);
    } else {
        tail_body<B, T, K, kAG, false>(cin, sin, x, sp.hi, out, nb, sp.wg_at);
    }
}

// Small messages: the same flavours, organised for latency instead of bandwidth.
// With few tiles the bandwidth-shaped kernels leave most compute units idle
// and pay one memory round trip per hop.  Here a workgroup takes ONE tile and
// requests the tiles of N partials at once, so a chain of up to N partials
// costs one round trip (a longer one ceil(P / N)).  Every load is
// unconditional -- positions past the last one repeat it and are ignored --
// because a load behind a condition makes the compiler wait for all
// outstanding loads where the paths join.
//
// What bounds it then is the chain of quantizations: a wave or two per SIMD
// issue some 55 instructions per hop one after the other, with nothing to fill
// the waits between them.
// * A step is nested in the one before (small_steps), so that a hop costs one
//   compare and branch; leaving a loop over the positions cost eight scalar
//   instructions per hop.  And there is no loop around the steps unless kMany
//   (or 9 to 16 partials keep their wire, which are faster in one: 16 of 262 k,
//   block 256, 6.84 -> 6.23, of 524 k 8.86 -> 8.39; 12 of 262 k 5.67 -> 5.31):
//   in one, the first step asks at run time whether it is the first.  Measured
//   on MI355X, GPU us per call (captured calls one after the other, inputs
//   cold), loop over positions -> nested in a loop -> as it is, 8 elements per
//   lane: 16 partials of 344 k elements, block 128, 4.90 -> 4.90 -> 4.77, of
//   600 k 7.13 -> 7.32 -> 7.11; 8 partials, block 256, of 4 k 3.08 -> 3.07 ->
//   2.96, of 600 k 4.60 -> 4.84 -> 4.66; 4 partials of 344 k 2.93 -> 2.97 ->
//   2.83, of 600 k 3.57 -> 3.61 -> 3.48.
// * E = 4 elements per lane in workgroups of a single wave, while the chip has
//   a SIMD for each (SmallLane): half the arithmetic per hop for one more lane
//   exchange, and the requests come from more CUs.  After the step above: 16
//   partials of 4 k 3.99 -> 3.41, of 66 k 4.22 -> 3.66, of 344 k 4.77 -> 5.21
//   (not taken); 8 of 4 k 2.96 -> 2.63, of 66 k 3.14 -> 2.93.
//
// The full loop (kSemi = false) takes position i at step i.  The semi-loop
// takes the owner at step 0, positions h+1 .. P-1 at steps 1 .. na = P-1-h and
// positions h .. 1 at the steps after that: at step i > na that is P - i.

// What a lane of small_kernel holds: E elements of each tile.
template <int E>
struct SmallLane;

template <>
struct SmallLane<8> {
    typedef u32x4 Raw;
    static constexpr int T = kThreads;
    template <bool kFull>
    static __device__ __forceinline__ Raw load(const uint16_t *p, int64_t base, int off, int64_t n)
    {
        return load_bf16x8(p, base, off, n, kFull);
    }
    static __device__ __forceinline__ void widen(const Raw &w, float (&f)[8]) { widen_bf16x8(w, f); }
    template <bool kFull>
    static __device__ __forceinline__ void store_codes(int8_t *p, int64_t base, int off, int64_t n, const float (&r)[8])
    {
        store_i8x8(p, base, off, n, kFull, pack_codes(r));
    }
    template <bool kFull, bool kKeepsHint>
    static __device__ __forceinline__ void store(uint16_t *out, int64_t base, int off, int64_t n, const float (&v)[8])
    {
        store_narrowed_tile<kFull, kKeepsHint>(out, base, off, n, v);
    }
};

template <>
struct SmallLane<4> {
    typedef u32x2 Raw;
    static constexpr int T = 64;
    template <bool kFull>
    static __device__ __forceinline__ Raw load(const uint16_t *p, int64_t base, int off, int64_t n)
    {
        if (kFull) {
            const Raw *v = reinterpret_cast<const Raw *>(p + base + off);
            return EQUARX_NT_LOAD_BF16 ? __builtin_nontemporal_load(v) : *v;
        }
        // the end of a tensor, as request_end and whole_end
        const int left = left_of(n, base);
        const int whole = left & ~1;
        constexpr int kPolicy = EQUARX_NT_LOAD_BF16 ? kNonTemporal : 0;
        Raw w = __builtin_bit_cast(Raw, __builtin_amdgcn_raw_buffer_load_b64(bounded(p + base, whole * 2), off * 2, 0, kPolicy));
        const uint32_t last = __builtin_amdgcn_raw_buffer_load_b16(bounded(p + base, left * 2), whole * 2, 0, 0);
        if (off == whole) w.x = last;
        if (off + 2 == whole) w.y = last;
        return w;
    }
    static __device__ __forceinline__ void widen(const Raw &w, float (&f)[4]) { widen_bf16x4(w, f); }
    template <bool kFull>
    static __device__ __forceinline__ void store_codes(int8_t *p, int64_t base, int off, int64_t n, const float (&r)[4])
    {
        uint32_t b[4];
#pragma unroll
        for (int i = 0; i < 4; ++i) b[i] = __float_as_uint(r[i] + kRoundMagic);
        const uint32_t w = gather_low_bytes(b[0], b[1], b[2], b[3]);
        if (kFull) {
            *reinterpret_cast<uint32_t *>(p + base + off) = w;
            return;
        }
        const int left = left_of(n, base);
        const int whole = left & ~3;
        __builtin_amdgcn_raw_buffer_store_b32(w, bounded(p + base, whole), off, 0, 0);
        const auto end = bounded(p + base, left);
#pragma unroll
        for (int i = 0; i < 3; ++i) {
            __builtin_amdgcn_raw_buffer_store_b8((uint8_t)(w >> (8 * i)), end, off == whole ? whole + i : kNowhere, 0, 0);
        }
    }
    template <bool kFull, bool kKeepsHint>
    static __device__ __forceinline__ void store(uint16_t *out, int64_t base, int off, int64_t n, const float (&v)[4])
    {
        Raw w;
        w.x = narrow_bf16x2(v[0], v[1]);
        w.y = narrow_bf16x2(v[2], v[3]);
        if (kFull) {
            Raw *o = reinterpret_cast<Raw *>(out + base + off);
            if (EQUARX_NT_STORE_BF16) {
                __builtin_nontemporal_store(w, o);
            } else {
                *o = w;
            }
            return;
        }
        const int left = left_of(n, base);
        const int whole = left & ~1;
        __builtin_amdgcn_raw_buffer_store_b64(w, bounded(out + base, whole * 2), off * 2, 0, EQUARX_NT_STORE_BF16 ? kNonTemporal : 0);
        const bool holds = off == whole || off + 2 == whole;        // the lane with the last element of an odd length
        const uint32_t last = off == whole ? w.x : w.y;
        __builtin_amdgcn_raw_buffer_store_b16((uint16_t)last, bounded(out + base, left * 2), holds ? whole * 2 : kNowhere, 0, 0);
    }
};

template <int E>
struct SmallShape {
    static constexpr int T = SmallLane<E>::T;
    static constexpr int64_t kElems = (int64_t)T * E;
};

// Where a lane of a small chain is, and where its wire goes (kWire).
struct SmallPlace {
    int P, na, off;
    int64_t wg_at, n;
    int8_t *wire_codes;
    float *wire_scales;
    int64_t c_step, s_step;
};

// The wire after a quantization: row `row` of the kept wire.
template <int B, int E, bool kFull>
__device__ __forceinline__ void store_small_wire(const SmallPlace &at, int row, const float (&r)[E], float s)
{
    constexpr int G = B / E;
    SmallLane<E>::template store_codes<kFull>(at.wire_codes + (int64_t)row * at.c_step, at.wg_at, at.off, at.n, r);
    if ((threadIdx.x % G) == 0 && (kFull || at.wg_at + at.off < at.n)) {
        at.wire_scales[(int64_t)row * at.s_step + (at.wg_at + at.off) / B] = s;
    }
}

// Step i = base + U of the chain, and within it all that follow: `own` the owner's sum (semi-loop), `t` the running sum.
template <int B, int E, int N, int U, bool kSemi, bool kRS, bool kAG, bool kWire, bool kFull>
__device__ __forceinline__ void small_steps(const SmallPlace &at, int base, const typename SmallLane<E>::Raw (&x)[N],
                                            float (&own)[E], float (&t)[E])
{
    if constexpr (U < N) {
        const int i = base + U;
        if (i >= at.P) return;                                      // uniform, as every condition here
        constexpr int G = B / E;
        float xf[E];
        SmallLane<E>::widen(x[U], xf);
        if (U == 0 && i == 0) {
#pragma unroll
            for (int e = 0; e < E; ++e) (kSemi ? own : t)[e] = xf[e];
        } else {
            if (kSemi && (i == 1 || i == at.na + 1)) {              // a half chain starts
#pragma unroll
                for (int e = 0; e < E; ++e) t[e] = xf[e];
            } else if (kRS) {
                float r[E], s;
                quantize_lane_f<G, !kAG>(t, r, s);
                if (kWire) store_small_wire<B, E, kFull>(at, i - 1, r, s);
#pragma unroll
                for (int e = 0; e < E; ++e) t[e] = __builtin_fmaf(r[e], s, xf[e]);
            } else {
#pragma unroll
                for (int e = 0; e < E; ++e) t[e] = t[e] + xf[e];
            }
            if (kSemi && (i == at.na || i == at.P - 1)) {           // ... and ends at the owner
                float r[E], s;
                quantize_lane_f<G, !kAG>(t, r, s);
#pragma unroll
                for (int e = 0; e < E; ++e) own[e] = __builtin_fmaf(r[e], s, own[e]);
            }
        }
        small_steps<B, E, N, U + 1, kSemi, kRS, kAG, kWire, kFull>(at, base, x, own, t);
    }
}

template <int B, int E, int N, bool kMany, bool kSemi, bool kRS, bool kAG, bool kWire, bool kFull>
__device__ __forceinline__ void small_body(const PartialTable &tab, int P, int rot, int64_t n, uint16_t *out,
                                           int8_t *__restrict__ wire_codes, float *__restrict__ wire_scales,
                                           int64_t c_step, int64_t s_step, int64_t wg_at)
{
    typedef SmallLane<E> Lane;
    const int h = P / 2, na = kSemi ? P - 1 - h : 0;
    const SmallPlace at{P, na, (int)threadIdx.x * E, wg_at, n, wire_codes, wire_scales, c_step, s_step};
    float t[E], own[E];
    typename Lane::Raw x[N];

    for (int base = 0; base < (kMany || (kWire && N == 16) ? P : 1); base += N) {
#pragma unroll
        for (int u = 0; u < N; ++u) {
            // The table repeats after P entries, so a position may run past P (rot <= P <= N, unless kMany).
            int j = rot + base + u;
            if (kMany) {
                const int i = base + u < P ? base + u : P - 1;
                j = rot + (!kSemi || i == 0 ? i : i <= na ? h + i : P - i);
                if (j >= P) j -= P;
            } else if (kSemi && u > 0) {
                j = u <= na ? rot + h + u : rot + 2 * P - u;
                if (j < 0) j = 0;               // u past 2 P: a repeat like any other
            }
            x[u] = Lane::template load<kFull>(tab.x[j], wg_at, at.off, n);
        }
        loads_first();
        small_steps<B, E, N, 0, kSemi, kRS, kAG, kWire, kFull>(at, base, x, own, t);
    }

    const float (&sum)[E] = kSemi ? own : t;
    if (!kAG) {
        Lane::template store<kFull, kWire>(out, wg_at, at.off, n, sum);
        return;
    }
    float r[E], d[E], s;
    quantize_lane_f<B / E, true>(sum, r, s);        // +0.0 codes: the product below shows the sign of a zero
    if (kWire) store_small_wire<B, E, kFull>(at, P - 1, r, s);
#pragma unroll
    for (int e = 0; e < E; ++e) d[e] = r[e] * s;
    Lane::template store<kFull, kWire>(out, wg_at, at.off, n, d);
}

template <int B, int E, int N, bool kMany, bool kSemi, bool kRS, bool kAG, bool kWire>
__global__ __launch_bounds__(SmallShape<E>::T) void small_kernel(int P, int64_t n, int64_t shard_elems, Global<uint16_t> out,
                                                                 Global<int8_t> wire_codes, Global<float> wire_scales,
                                                                 int64_t c_step, int64_t s_step, const PartialTable tab)
{
    static_assert(B / E <= 64, "a block inside one wave");
    constexpr int64_t kElems = SmallShape<E>::kElems;
    const Span sp = workgroup_span<(int)(kElems / kLaneElems), 1>(n, shard_elems, kSemi ? 0 : 1);
    if (!sp.any) return;
    if (sp.wg_at + kElems <= sp.hi) {
        small_body<B, E, N, kMany, kSemi, kRS, kAG, kWire, true>(tab, P, sp.rot, sp.hi, out, wire_codes, wire_scales, c_step, s_step, sp.wg_at);
    } else {
        small_body<B, E, N, kMany, kSemi, kRS, kAG, kWire, false>(tab, P, sp.rot, sp.hi, out, wire_codes, wire_scales, c_step, s_step, sp.wg_at);
    }
}

// Semi-loop adder tree (Sec. 3.3).  Position 0 (device rot) owns the shard; the
// other positions follow in ring order.  With h = P/2 the counter-clockwise
// chain h+1, h+2, ..., P-1 and the clockwise chain h, h-1, ..., 1 each end in a
// quantized send to the owner, which adds them to its own fp32 shard, the
// shorter counter-clockwise chain first.
template <int B, int T, int K, bool kAG, bool kFull>
__device__ __forceinline__ void semi_body(const PartialTable &tab, int P, int rot, int64_t n,
                                          uint16_t *out, int64_t wg_at, bool cached)
{
    const int lane_at = threadIdx.x * kLaneElems;
    const int h = P / 2;
    float own[K][8], t[K][8];
    u32x4 xv[K];

    const int owner = rot >= P ? rot - P : rot;     // rot < 2P
    load_tiles<T, K, kFull>(tab.x[owner], wg_at, n, xv);
#pragma unroll
    for (int k = 0; k < K; ++k) widen_bf16x8(xv[k], own[k]);

#pragma unroll 1
    for (int dir = 0; dir < 2; ++dir) {
        // dir 0: positions h+1 .. P-1 ascending; dir 1: positions h .. 1 descending
        const int count = dir == 0 ? P - 1 - h : h;
        if (count <= 0) continue;
        int j = owner + (dir == 0 ? h + 1 : h);     // < 2P
        if (j >= P) j -= P;
        load_tiles<T, K, kFull>(tab.x[j], wg_at, n, xv);
#pragma unroll
        for (int k = 0; k < K; ++k) widen_bf16x8(xv[k], t[k]);
        for (int c = 1; c < count; ++c) {
            j = dir == 0 ? ring_next(j, P) : ring_prev(j, P);
            load_tiles_together<T, K, kFull>(tab.x[j], wg_at, n, xv);
            hop_tiles<B, T, K, true, kNoWire, !kAG, kFull>(t, xv, nullptr, nullptr, 0, 0, 0, wg_at, n);
        }
#pragma unroll
        for (int k = 0; k < K; ++k) {
            constexpr int G = B / kLaneElems;
            float r[8], s;
            quantize_lane_f<G, !kAG>(t[k], r, s);                      // the send that reaches the owner
#pragma unroll
            for (int jj = 0; jj < 8; ++jj) own[k][jj] = __builtin_fmaf(r[jj], s, own[k][jj]);
        }
    }

#pragma unroll
    for (int k = 0; k < K; ++k) {
        finish_tile<B, kAG, kNoWire, kFull>(own[k], out, nullptr, nullptr, 0, 0, 0, wg_at + k * tile_elems<T>, lane_at, n,
                                          cached);
    }
}

template <int B, int T, int K, bool kAG>
__global__ __launch_bounds__(T) void semi_kernel(int P, int64_t n, int64_t shard_elems, Global<uint16_t> out,
                                                        const PartialTable tab)
{
    const Span sp = workgroup_span<T, K>(n, shard_elems, 0);     // shard k: owner is device k
    if (!sp.any) return;
    if (sp.wg_at + tile_elems<T> * K <= sp.hi) {
        semi_body<B, T, K, kAG, true>(tab, P, sp.rot, sp.hi, out, sp.wg_at, out_stays_cached(n, 1));
    } else {
        semi_body<B, T, K, kAG, false>(tab, P, sp.rot, sp.hi, out, sp.wg_at, out_stays_cached(n, 1));
    }
}

// ---------------------------------------------------------------- flat one-shot reduce
// The reduce-scatter as an all-to-all followed by a local reduction (the
// decomposition Sec. 2 describes for ZeRO++, and the shape a full xGMI mesh
// favours over a ring): the owner of a shard holds its own bf16 shard and R
// received (codes, scales) pairs, each quantized once by its sender.  It
// dequantizes and accumulates them in fp32 in array order -- one fused
// multiply-add each -- and quantizes the sum once for the all-gather.

struct WireTable {
    const int8_t *codes[kMaxPartials];
    const float *scales[kMaxPartials];
};

// U received wires are requested at a time.  A wide launch has enough waves to cover the wait for one (U = 1: 36.1 us
// for seven wires of 22 M elements on MI355X, 42.0 with U = 2, whose requests only queue); a narrow one has a wave or
// two per SIMD, and asking for the next wire only when the last one has been added leaves it waiting R times over:
// seven wires of 50 k elements 9.4 us with 256 threads x 4 tiles and U = 1, 3.1 with 256 x 1 and U = 8; of 2.75 M
// 8.9 -> 6.1.  U = 2 for up to two wires (one wire of 50 k: 2.4 us, 2.9 with U = 4, 3.9 with U = 8), 4 for up to
// four (three of 1.5 M: 3.6 us, 5.2 with U = 8).  Requests past the last wire repeat it and are ignored, so that no
// load is behind a condition.
template <int B, int K, int U, bool kOutBf16, bool kOutWire, bool kAG, bool kFull, bool kStream = false>
__device__ __forceinline__ void flat_body(const uint16_t *local, const WireTable &tab, int R, int64_t n,
                                          uint16_t *out, int8_t *__restrict__ codes_out,
                                          float *__restrict__ scales_out, int64_t nb, int64_t wg_at)
{
    constexpr int G = B / kLaneElems, T = pass_threads(K);
    const int lane_at = threadIdx.x * kLaneElems;
    float acc[K][8];
    u32x4 xv[K];
    load_tiles<T, K, kFull>(local, wg_at, n, xv);
#pragma unroll
    for (int k = 0; k < K; ++k) widen_bf16x8(xv[k], acc[k]);

    for (int r0 = 0; r0 < R; r0 += U) {
        u32x2 cv[U][K];
        float sv[U][K];
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int r = r0 + u < R ? r0 + u : R - 1;
            const int8_t *c = tab.codes[r];
            const float *sc = tab.scales[r];
#pragma unroll
            for (int k = 0; k < K; ++k) {
                const int64_t base = wg_at + k * tile_elems<T>;
                cv[u][k] = load_i8x8<kStream>(c, base, lane_at, n, kFull);
                const int64_t blk = base / B + lane_at / B;
                sv[u][k] = sc[kFull || blk < nb ? blk : nb - 1];
            }
        }
        if (U > 1) loads_first();
#pragma unroll
        for (int u = 0; u < U; ++u) {
            if (r0 + u >= R) break;             // uniform
#pragma unroll
            for (int k = 0; k < K; ++k) {
                float qf[8];
                widen_i8x8(cv[u][k], qf);
#pragma unroll
                for (int j = 0; j < 8; ++j) acc[k][j] = __builtin_fmaf(qf[j], sv[u][k], acc[k][j]);
            }
        }
    }

#pragma unroll
    for (int k = 0; k < K; ++k) {
        const int64_t base = wg_at + k * tile_elems<T>;
        if (!kAG) {                 // all-gather left unquantized (the semi-loop's owner, Sec. 3.3/3.4): no wire out
            store_narrowed_tile<kFull>(out, base, lane_at, n, acc[k]);
            continue;
        }
        float q[8], s;
        quantize_lane_f<G, true>(acc[k], q, s);
        if (kOutWire) {
            store_i8x8<kStream, K == 1>(codes_out, base, lane_at, n, kFull, pack_codes(q));
            if ((threadIdx.x % G) == 0 && (kFull || base + lane_at < n)) scales_out[base / B + lane_at / B] = s;
        }
        if (kOutBf16) {
            float d[8];
#pragma unroll
            for (int j = 0; j < 8; ++j) d[j] = q[j] * s;
            store_narrowed_tile<kFull>(out, base, lane_at, n, d);
        }
    }
}

template <int B, int K, int U, bool kOutBf16, bool kOutWire, bool kAG = true, bool kStream = false>
__global__ __launch_bounds__(pass_threads(K)) void flat_kernel(Global<const uint16_t> local, int R, int64_t n, Global<uint16_t> out,
                                                        Global<int8_t> codes_out, Global<float> scales_out,
                                                        int64_t mirror, const WireTable tab)
{
    const int64_t wg_at = first_element<pass_threads(K), K, !kStream>(mirror);
    const int64_t nb = (n + B - 1) / B;
    if (wg_at + tile_elems<pass_threads(K)> * K <= n) {
        flat_body<B, K, U, kOutBf16, kOutWire, kAG, true, kStream>(local, tab, R, n, out, codes_out, scales_out, nb, wg_at);
    } else {
        flat_body<B, K, (U > 2 ? 2 : U), kOutBf16, kOutWire, kAG, false, kStream>(local, tab, R, n, out, codes_out, scales_out, nb, wg_at);
    }
}

// ---------------------------------------------------------------- semi-loop in ring order, hop by hop
//
// What all devices of a ring do in one iteration of the semi-loop reduce-scatter (Sec. 3.3), as one launch: grid
// row k works on shard k, which device k owns; the devices k+1, k+2, ... sit around it at positions 1, 2, ....
// With h = P/2 the counter-clockwise chain runs over positions h+1, h+2, ..., P-1 and the clockwise chain over
// positions h, h-1, ..., 1; in iteration t both advance one device (blockIdx.z picks the direction), so the whole
// reduce-scatter takes h iterations, as the paper's N/2.  Same bodies as the plain per-pass kernels.

struct WirePair {           // one wire buffer per direction
    int8_t *codes[2];
    float *scales[2];
};

template <int B, int K, bool kTurns>
__global__ __launch_bounds__(pass_threads(K)) void semi_ring_step_kernel(int P, int t, int64_t n, int64_t shard_elems,
                                                                  const WirePair wire, const PartialTable tab)
{
    constexpr int T = pass_threads(K);
    const bool backward = kTurns && (t & 1) != 0;
    const Span sp = workgroup_span<T, K, kTurns>(n, shard_elems, 0, backward ? P : 0);     // rot = the owner's device number
    if (!sp.any) return;
    const int dir = backward ? 1 - (int)blockIdx.z : (int)blockIdx.z, h = P / 2;
    const int count = dir == 0 ? P - 1 - h : h;                 // devices in this direction's chain
    if (t >= count) return;                                     // the shorter chain has already arrived
    int dev = sp.rot + (dir == 0 ? h + 1 + t : h - t);          // < 2P
    if (dev >= P) dev -= P;
    const uint16_t *x = tab.x[dev];
    const int64_t nb = (sp.hi + B - 1) / B;
    const bool full = sp.wg_at + tile_elems<T> * K <= sp.hi;
    if (t == 0) {
        if (full) {
            quantize_body<B, T, K, true>(x, sp.hi, wire.codes[dir], wire.scales[dir], nb, sp.wg_at);
        } else {
            quantize_body<B, T, K, false>(x, sp.hi, wire.codes[dir], wire.scales[dir], nb, sp.wg_at);
        }
    } else if (full) {
        hop_body<B, T, K, true>(wire.codes[dir], wire.scales[dir], x, sp.hi, wire.codes[dir], wire.scales[dir], nb, sp.wg_at);
    } else {
        hop_body<B, T, K, false>(wire.codes[dir], wire.scales[dir], x, sp.hi, wire.codes[dir], wire.scales[dir], nb, sp.wg_at);
    }
}

// The owner's last step: its own shard plus the wires that arrived (counter-clockwise first), then the all-gather's
// quantize/dequantize pair or the plain narrowing.
template <int B, int K, int U, bool kAG, bool kTurns>
__global__ __launch_bounds__(pass_threads(K)) void semi_ring_owner_kernel(int P, int64_t n, int64_t shard_elems,
                                                                   int received, Global<uint16_t> out, const WireTable wires,
                                                                   const PartialTable tab)
{
    constexpr int T = pass_threads(K);
    const Span sp = workgroup_span<T, K, kTurns>(n, shard_elems, 0, (P / 2 & 1) != 0 ? P : 0);
    if (!sp.any) return;
    const uint16_t *own = tab.x[sp.rot >= P ? sp.rot - P : sp.rot];
    const int64_t nb = (sp.hi + B - 1) / B;
    if (sp.wg_at + tile_elems<T> * K <= sp.hi) {
        flat_body<B, K, U, true, false, kAG, true>(own, wires, received, sp.hi, out, nullptr, nullptr, nb, sp.wg_at);
    } else {
        flat_body<B, K, U, true, false, kAG, false>(own, wires, received, sp.hi, out, nullptr, nullptr, nb, sp.wg_at);
    }
}

}  // namespace equarx
