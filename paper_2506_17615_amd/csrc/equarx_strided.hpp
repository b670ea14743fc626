// The paper's own block geometry on gfx950 (EQuARX, arXiv 2506.17615, Sec. 3.2).
//
// There a shard is cut into chunks of 8 x 128 = 1024 elements (the TPU's vector
// register shape, contiguous in its tiled memory layout) and a minishard of
// `chunks` consecutive chunks gets 1024 scales: scale j comes from the max-abs
// over position j of every chunk, so a quantization block is `chunks` entries
// that lie 1024 elements apart.  On the TPU this avoids any reduction inside a
// vector register.  On a GPU it means the opposite of the contiguous layout:
// no reduction over neighbouring elements (a lane keeps its own 8 positions),
// but one ACROSS the chunks of a minishard.
//
// Decomposition of the per-pass kernels (quantize, hop: codes go to memory, and
// 8-byte code pieces want 16 lanes or more side by side to fill a 128-byte
// line; the single-launch chain further down writes no codes and uses a
// layout without LDS): a workgroup of 256 threads takes one slice of 256 positions of
// one minishard.  Thread (g, l), g = 0..7, l = 0..31, owns positions 8l..8l+7
// of the slice in chunks g, g+8, g+16, ...; it keeps the raw inputs of its
// chunks/8 chunks in registers, so global memory is read once.  The 8 partial
// maxima per position meet in LDS (8 KiB), every thread derives the scales of
// its 8 positions, recomputes its values from the registers, scales, rounds
// and stores.  Loads of a half-wave cover 512 contiguous bytes.
#pragma once

#include "equarx_device.hpp"

namespace equarx {

constexpr int kChunk = 1024;                               // elements per chunk (8 x 128)
// Measured at the 27B-shaped size: 32 lanes per slice is best overall (16: within 2 % for 64 and 128 chunks, 8 %
// slower for 32; 64: 3 % slower for 32, 30 % slower for 128).  Capping the waves per SIMD at 2 or 3, or dropping
// the first of the two barriers (a kernel takes the maximum once), changes nothing beyond 2 %; the 8 x 8 in-wave
// layout of the single-launch chain makes these kernels 5-8 % slower (64-byte code pieces); workgroups of 512 or 1024
// threads with 1 or 2 KiB runs per chunk are no faster for 64 chunks and 4-100 % slower otherwise.
#ifndef EQUARX_STRIDED_SLICE_LANES
#define EQUARX_STRIDED_SLICE_LANES 32
#endif
constexpr int kSliceLanes = EQUARX_STRIDED_SLICE_LANES;    // lanes across a slice of a chunk
constexpr int kSlicePos = kSliceLanes * kLaneElems;        // 256 positions per workgroup
constexpr int kChunkGroups = kThreads / kSliceLanes;       // 8 groups of lanes, each walking every 8th chunk
constexpr int kSlicesPerChunk = kChunk / kSlicePos;        // 4 workgroups per minishard
static_assert(kThreads == 256, "the strided kernels are laid out for 256-thread workgroups");

// A launch that walks back (walks_back): workgroup b of the first `mirror`, a multiple of eight, takes the place of one
// in the opposite group of eight.  mirror == 0: it walks forward.
__device__ __forceinline__ unsigned mirrored_place(unsigned b, unsigned mirror)
{
    return b < mirror ? mirror - 8 - (b & ~7u) + (b & 7u) : b;
}

__host__ __device__ inline unsigned whole_groups(unsigned count) { return (count + 7) & ~7u; }

struct StridedSpot {
    int64_t minishard;  // which minishard the workgroup works on
    int64_t elem;       // first element of the lane in chunk `g` of its minishard
    int64_t scale;      // index of the lane's first scale
    int g;              // chunk group
};

// at: the workgroup's place in the tensor.
__device__ __forceinline__ StridedSpot strided_spot(int chunks, unsigned at)
{
    StridedSpot sp;
    const int l = threadIdx.x % kSliceLanes;
    sp.g = threadIdx.x / kSliceLanes;
    const int64_t ms = at / kSlicesPerChunk;
    const int pos = (at % kSlicesPerChunk) * kSlicePos + l * kLaneElems;
    sp.minishard = ms;
    sp.elem = ms * ((int64_t)kChunk * chunks) + (int64_t)sp.g * kChunk + pos;
    sp.scale = ms * kChunk + pos;
    return sp;
}

// The bf16 tensor a per-pass kernel reads.  Array order (per_shard == 0): partial `offset` for every workgroup.
// Ring layout (Sec. 3; per_shard > 0): the tensor is cut into shards of per_shard minishards, shard k ends on device
// k, and a launch is one ring step on every shard at once -- the workgroups of shard k read the partial of device
// (k + offset) mod P.  0 <= offset < P.
struct StridedSource {
    PartialTable tab;
    int P;
    int per_shard;
    int offset;
};

__device__ __forceinline__ const uint16_t *strided_source(const StridedSource &src, int64_t minishard)
{
    const int j = (src.per_shard > 0 ? (int)(minishard / src.per_shard) : 0) + src.offset;     // < 2P
    return src.tab.x[j >= src.P ? j - src.P : j];
}

// Max over the 8 chunk groups for each of the lane's 8 positions, through LDS.
// m: bit patterns of non-negative floats.  Every thread of the workgroup calls this.
__device__ __forceinline__ void across_chunks_max(uint32_t (&m)[8], uint32_t (*red)[kSlicePos])
{
    const int l = threadIdx.x % kSliceLanes;
    const int g = threadIdx.x / kSliceLanes;
    __syncthreads();                                        // the previous round's readers are done
    u32x4 *row = reinterpret_cast<u32x4 *>(&red[g][l * kLaneElems]);
    row[0] = u32x4{m[0], m[1], m[2], m[3]};
    row[1] = u32x4{m[4], m[5], m[6], m[7]};
    __syncthreads();
#pragma unroll
    for (int h = 0; h < kChunkGroups; ++h) {
        const u32x4 *other = reinterpret_cast<const u32x4 *>(&red[h][l * kLaneElems]);
        const u32x4 a = other[0], b = other[1];
        m[0] = umax(m[0], a.x); m[1] = umax(m[1], a.y); m[2] = umax(m[2], a.z); m[3] = umax(m[3], a.w);
        m[4] = umax(m[4], b.x); m[5] = umax(m[5], b.y); m[6] = umax(m[6], b.z); m[7] = umax(m[7], b.w);
    }
}

template <int V>
__device__ __forceinline__ void note_absmax(const float (&t)[V], uint32_t (&m)[V])
{
#pragma unroll
    for (int j = 0; j < V; ++j) m[j] = umax(m[j], __float_as_uint(t[j]) & 0x7FFFFFFFu);
}

__device__ __forceinline__ u32x2 scale_and_pack(const float (&t)[8], const float (&inv)[8])
{
    uint32_t b[8];
#pragma unroll
    for (int j = 0; j < 8; ++j) b[j] = __float_as_uint(t[j] * inv[j] + kRoundMagic);  // rounds to the integer code
    u32x2 w;
    w.x = gather_low_bytes(b[0], b[1], b[2], b[3]);
    w.y = gather_low_bytes(b[4], b[5], b[6], b[7]);
    return w;
}

// R = chunks / 8 chunks per thread.
template <int R>
__device__ __forceinline__ void quantize_strided_body(const uint16_t *__restrict__ x, int8_t *__restrict__ codes,
                                                      float *__restrict__ scales, const StridedSpot &sp,
                                                      uint32_t (*red)[kSlicePos])
{
    u32x4 xv[R];
#pragma unroll
    for (int r = 0; r < R; ++r) {
        xv[r] = __builtin_nontemporal_load(reinterpret_cast<const u32x4 *>(x + sp.elem + (int64_t)r * kChunkGroups * kChunk));
    }
    uint32_t m[8] = {0, 0, 0, 0, 0, 0, 0, 0};
#pragma unroll
    for (int r = 0; r < R; ++r) {
        float t[8];
        widen_bf16x8(xv[r], t);
        note_absmax(t, m);
    }
    across_chunks_max(m, red);

    float scale[8], inv[8];
#pragma unroll
    for (int j = 0; j < 8; ++j) block_quotients(__uint_as_float(m[j]), scale[j], inv[j]);
#pragma unroll
    for (int r = 0; r < R; ++r) {
        float t[8];
        widen_bf16x8(xv[r], t);
        *reinterpret_cast<u32x2 *>(codes + sp.elem + (int64_t)r * kChunkGroups * kChunk) = scale_and_pack(t, inv);
    }
    if (sp.g == 0) {
        float *s = scales + sp.scale;
        *reinterpret_cast<u32x4 *>(s) = u32x4{__float_as_uint(scale[0]), __float_as_uint(scale[1]),
                                              __float_as_uint(scale[2]), __float_as_uint(scale[3])};
        *reinterpret_cast<u32x4 *>(s + 4) = u32x4{__float_as_uint(scale[4]), __float_as_uint(scale[5]),
                                                  __float_as_uint(scale[6]), __float_as_uint(scale[7])};
    }
}

template <int R>
__global__ __launch_bounds__(kThreads) void quantize_strided_kernel(Global<int8_t> codes,
                                                                    Global<float> scales,
                                                                    const StridedSource src)
{
    __shared__ __align__(16) uint32_t red[kChunkGroups][kSlicePos];
    const StridedSpot sp = strided_spot(R * kChunkGroups, blockIdx.x);
    quantize_strided_body<R>(strided_source(src, sp.minishard), codes, scales, sp, red);
}

// One hop in the strided geometry.  Output wire may be the input wire: a
// workgroup holds all its inputs in registers before it stores anything.
template <int R>
__device__ __forceinline__ void hop_strided_body(const int8_t *cin, const float *sin, const uint16_t *__restrict__ x,
                                                 int8_t *cout, float *sout, const StridedSpot &sp,
                                                 uint32_t (*red)[kSlicePos])
{
    u32x4 xv[R];
    u32x2 cv[R];
#pragma unroll
    for (int r = 0; r < R; ++r) {
        const int64_t at = sp.elem + (int64_t)r * kChunkGroups * kChunk;
        xv[r] = __builtin_nontemporal_load(reinterpret_cast<const u32x4 *>(x + at));
        cv[r] = *reinterpret_cast<const u32x2 *>(cin + at);
    }
    float s_in[8];
    {
        const u32x4 a = *reinterpret_cast<const u32x4 *>(sin + sp.scale);
        const u32x4 b = *reinterpret_cast<const u32x4 *>(sin + sp.scale + 4);
        s_in[0] = __uint_as_float(a.x); s_in[1] = __uint_as_float(a.y);
        s_in[2] = __uint_as_float(a.z); s_in[3] = __uint_as_float(a.w);
        s_in[4] = __uint_as_float(b.x); s_in[5] = __uint_as_float(b.y);
        s_in[6] = __uint_as_float(b.z); s_in[7] = __uint_as_float(b.w);
    }

    uint32_t m[8] = {0, 0, 0, 0, 0, 0, 0, 0};
#pragma unroll
    for (int r = 0; r < R; ++r) {
        float xf[8], qf[8], t[8];
        widen_bf16x8(xv[r], xf);
        widen_i8x8(cv[r], qf);
#pragma unroll
        for (int j = 0; j < 8; ++j) t[j] = __builtin_fmaf(qf[j], s_in[j], xf[j]);
        note_absmax(t, m);
    }
    across_chunks_max(m, red);

    float scale[8], inv[8];
#pragma unroll
    for (int j = 0; j < 8; ++j) block_quotients(__uint_as_float(m[j]), scale[j], inv[j]);
#pragma unroll
    for (int r = 0; r < R; ++r) {
        float xf[8], qf[8], t[8];
        widen_bf16x8(xv[r], xf);
        widen_i8x8(cv[r], qf);
#pragma unroll
        for (int j = 0; j < 8; ++j) t[j] = __builtin_fmaf(qf[j], s_in[j], xf[j]);      // same operands, same bits
        *reinterpret_cast<u32x2 *>(cout + sp.elem + (int64_t)r * kChunkGroups * kChunk) = scale_and_pack(t, inv);
    }
    if (sp.g == 0) {
        float *s = sout + sp.scale;
        *reinterpret_cast<u32x4 *>(s) = u32x4{__float_as_uint(scale[0]), __float_as_uint(scale[1]),
                                              __float_as_uint(scale[2]), __float_as_uint(scale[3])};
        *reinterpret_cast<u32x4 *>(s + 4) = u32x4{__float_as_uint(scale[4]), __float_as_uint(scale[5]),
                                                  __float_as_uint(scale[6]), __float_as_uint(scale[7])};
    }
}

template <int R>
__global__ __launch_bounds__(kThreads) void hop_strided_kernel(Global<const int8_t> cin, Global<const float> sin,
                                                               Global<int8_t> cout, Global<float> sout, unsigned mirror,
                                                               const StridedSource src)
{
    __shared__ __align__(16) uint32_t red[kChunkGroups][kSlicePos];
    const StridedSpot sp = strided_spot(R * kChunkGroups, mirrored_place(blockIdx.x, mirror));
    hop_strided_body<R>(cin, sin, strided_source(src, sp.minishard), cout, sout, sp, red);
}

// One iteration of the semi-loop reduce-scatter (Sec. 3.3) on both of its chains at once: the first half of the grid
// (`count` workgroups, in whole groups of eight) advances the chain that walks up from device h+1, the second the one that
// walks down from device h, each by one device -- the first iteration quantizes the chain's first shard (no incoming wire: cin == nullptr), the later ones are hops on
// the chain's own wire buffer in place.  The two halves share nothing.
struct StridedDirection {
    int offset;             // as StridedSource::offset
    const int8_t *cin;      // nullptr: this is the chain's first device, it only quantizes its shard
    const float *sin;
    int8_t *cout;
    float *sout;
};

struct StridedDirections {
    StridedDirection d[2];
};

template <int R>
__global__ __launch_bounds__(kThreads) void semi_step_strided_kernel(int P, int per_shard, unsigned count, int backward,
                                                                     const StridedDirections dirs, const PartialTable tab)
{
    __shared__ __align__(16) uint32_t red[kChunkGroups][kSlicePos];
    const unsigned half = whole_groups(count);
    const unsigned place = mirrored_place(blockIdx.x, backward ? 2 * half : 0);
    const unsigned at = place < half ? place : place - half;
    if (at >= count) return;            // uniform over the workgroup
    const StridedSpot sp = strided_spot(R * kChunkGroups, at);
    const StridedDirection d = place < half ? dirs.d[0] : dirs.d[1];
    const int j = (per_shard > 0 ? (int)(sp.minishard / per_shard) : 0) + d.offset;     // < 2P
    const uint16_t *x = tab.x[j >= P ? j - P : j];
    if (d.cin == nullptr) {             // uniform over the workgroup
        quantize_strided_body<R>(x, d.cout, d.sout, sp, red);
    } else {
        hop_strided_body<R>(d.cin, d.sin, x, d.cout, d.sout, sp, red);
    }
}

// The last launch of a hop-by-hop flavour in the strided geometry: the device that ends up with the sum adds what
// it received to its own bf16 shard -- one wire at the end of the full loop, one or two at the owner of the
// semi-loop (Sec. 3.3: the shorter chain's wire first), none when it is alone -- each with one fused multiply-add
// per element, and hands the sum to the all-gather: quantized once more and dequantized (kAG), or narrowed to
// bf16 as it is (Sec. 3.4).  out may be `own`: a thread reads its elements before it writes them.
struct StridedWires {
    const int8_t *codes[2];
    const float *scales[2];
};

template <int R, bool kAG>
__global__ __launch_bounds__(kThreads) void owner_strided_kernel(int received, unsigned mirror, Global<uint16_t> out,
                                                                 const StridedWires wires, const StridedSource src)
{
    __shared__ __align__(16) uint32_t red[kChunkGroups][kSlicePos];
    constexpr int chunks = R * kChunkGroups;
    const StridedSpot sp = strided_spot(chunks, mirrored_place(blockIdx.x, mirror));
    const uint16_t *own = strided_source(src, sp.minishard);

    float acc[R][8];
    {
        u32x4 xv[R];
#pragma unroll
        for (int r = 0; r < R; ++r) {
            xv[r] = __builtin_nontemporal_load(
                reinterpret_cast<const u32x4 *>(own + sp.elem + (int64_t)r * kChunkGroups * kChunk));
        }
#pragma unroll
        for (int r = 0; r < R; ++r) widen_bf16x8(xv[r], acc[r]);
    }
    for (int k = 0; k < received; ++k) {
        const int8_t *codes = wires.codes[k];
        const float *scales = wires.scales[k];
        u32x2 cv[R];
#pragma unroll
        for (int r = 0; r < R; ++r) {
            cv[r] = *reinterpret_cast<const u32x2 *>(codes + sp.elem + (int64_t)r * kChunkGroups * kChunk);
        }
        const u32x4 a = *reinterpret_cast<const u32x4 *>(scales + sp.scale);
        const u32x4 b = *reinterpret_cast<const u32x4 *>(scales + sp.scale + 4);
        const float s_in[8] = {__uint_as_float(a.x), __uint_as_float(a.y), __uint_as_float(a.z), __uint_as_float(a.w),
                               __uint_as_float(b.x), __uint_as_float(b.y), __uint_as_float(b.z), __uint_as_float(b.w)};
#pragma unroll
        for (int r = 0; r < R; ++r) {
            float qf[8];
            widen_i8x8(cv[r], qf);
#pragma unroll
            for (int j = 0; j < 8; ++j) acc[r][j] = __builtin_fmaf(qf[j], s_in[j], acc[r][j]);
        }
    }

    float scale[8], inv[8];
    if (kAG) {
        uint32_t m[8] = {0, 0, 0, 0, 0, 0, 0, 0};
#pragma unroll
        for (int r = 0; r < R; ++r) note_absmax(acc[r], m);
        across_chunks_max(m, red);
#pragma unroll
        for (int j = 0; j < 8; ++j) block_quotients(__uint_as_float(m[j]), scale[j], inv[j]);
    }
#pragma unroll
    for (int r = 0; r < R; ++r) {
        float d[8];
#pragma unroll
        for (int j = 0; j < 8; ++j) {
            d[j] = kAG ? (__builtin_rintf(acc[r][j] * inv[j]) + 0.0f) * scale[j] : acc[r][j];     // +0.0: the code as an integer
        }
        u32x4 w;
        w.x = narrow_bf16x2(d[0], d[1]);
        w.y = narrow_bf16x2(d[2], d[3]);
        w.z = narrow_bf16x2(d[4], d[5]);
        w.w = narrow_bf16x2(d[6], d[7]);
        __builtin_nontemporal_store(w, reinterpret_cast<u32x4 *>(out + sp.elem + (int64_t)r * kChunkGroups * kChunk));
    }
}

// ---------------------------------------------------------------- the chain and its flavours in one launch
//
// The full-loop chain, the semi-loop reduce-scatter (Sec. 3.3) and the stage
// knob (Sec. 3.4) with the blocks of Sec. 3.2, one launch each.  The running
// fp32 sums of a thread's chunks stay in registers from the first partial to
// the output; every quantized send needs the max-abs across the chunks of a
// minishard and nothing else from other threads.
//
// Layout: lane = 8 * g + l inside a wave, so the 8 chunk groups of a position
// sit in ONE wave, 8 lanes apart, and their maximum is three lane exchanges
// per value -- no LDS, no barrier.  A wave covers 64 positions (a 128-byte
// piece of each of 8 chunks per load) and, with W = 1, the chunks g, g+8, ...
// of its group: R = chunks/8 rows of 8 running sums per thread.  For 128
// chunks that would be 16 rows (128 sums, 64 load registers: one wave per
// SIMD), so there W = 2 waves share a position piece, wave w taking the chunk
// groups 8w .. 8w+7 (R = 8), and the two maxima meet through 256 bytes of LDS
// and one barrier per send (the buffer alternates, so the barrier of the next
// send also separates this send's reads from the writes of the one after).
// Same operations in the same order as the hop-by-hop strided chain, hence
// the same bits.
//
// A message of few minishards is bound by the time one wave takes per send,
// not by memory: W = 4 waves share a piece and a lane has V = 4 positions
// instead of 8, so a wave has an eighth of the rows and quotients and a
// minishard 32 workgroups instead of 4 (one minishard of 64 chunks, P = 8:
// 10.6 -> 5.6 us on MI355X).

struct WaveSpot {
    int64_t minishard;  // which minishard the workgroup works on
    int64_t elem;       // first element of the lane in the first of its chunks
    int64_t scale;      // index of the lane's first scale
    int64_t row_step;   // elements between two consecutive chunks of the lane
    bool first_group;   // the lane stores the scales of its positions
};

// W waves per position piece, V positions per lane; a 256-thread workgroup covers (4 / W) * 8 V positions.
template <int W, int V>
constexpr int wave_layout_wgs = kChunk / ((kThreads / 64) / W * 8 * V);      // workgroups per minishard

template <int W, int V>
__device__ __forceinline__ WaveSpot wave_spot(int chunks)
{
    static_assert((W == 1 || W == 2 || W == 4) && (V == 4 || V == 8), "waves per position piece, positions per lane");
    constexpr int kPieces = (kThreads / 64) / W;                // position pieces per workgroup
    constexpr int kPerChunk = wave_layout_wgs<W, V>;
    const int lane = threadIdx.x % 64, wave = threadIdx.x / 64;
    const int g = (wave % W) * 8 + lane / 8;                    // chunk group, 0 .. 8W-1
    const int64_t ms = blockIdx.x / kPerChunk;
    const int pos = (blockIdx.x % kPerChunk) * (kPieces * 8 * V) + (wave / W) * (8 * V) + (lane % 8) * V;
    WaveSpot sp;
    sp.minishard = ms;
    sp.elem = ms * ((int64_t)kChunk * chunks) + (int64_t)g * kChunk + pos;
    sp.scale = ms * kChunk + pos;
    sp.row_step = (int64_t)8 * W * kChunk;
    sp.first_group = g == 0;
    return sp;
}


// A maximum that waves exchange: one row per wave, two buffers in turn.
template <int W, int V>
struct ChunkMaxRows {
    uint32_t row[W > 1 ? 2 : 1][kThreads / 64][8 * V];
};

template <int W, int V>
struct ChunkMaxState {
    ChunkMaxRows<W, V> &red;
    int parity;
};

// Max over all chunk groups for each of the lane's V positions.  Every thread of the workgroup calls this; the state
// matters for W > 1 only.
template <int W, int V>
__device__ __forceinline__ void across_chunks_max_wave(uint32_t (&m)[V], ChunkMaxState<W, V> &st)
{
#pragma unroll
    for (int j = 0; j < V; ++j) {
        uint32_t v = m[j];
        v = umax(v, dpp_read<0x128>(v));                                    // row_ror:8: lane ^ 8 within a row of 16
        auto a = __builtin_amdgcn_permlane16_swap(v, v, false, false);      // lane ^ 16
        v = umax(a[0], a[1]);
        auto b = __builtin_amdgcn_permlane32_swap(v, v, false, false);      // lane ^ 32
        m[j] = umax(b[0], b[1]);
    }
    if (W > 1) {
        const int lane = threadIdx.x % 64, wave = threadIdx.x / 64;
        const int at = (lane % 8) * V;
        if (lane < 8) {
            u32x4 *row = reinterpret_cast<u32x4 *>(&st.red.row[st.parity][wave][at]);
#pragma unroll
            for (int q = 0; q < V / 4; ++q) row[q] = u32x4{m[4 * q], m[4 * q + 1], m[4 * q + 2], m[4 * q + 3]};
        }
        __syncthreads();
#pragma unroll
        for (int w = 1; w < W; ++w) {
            const u32x4 *other = reinterpret_cast<const u32x4 *>(&st.red.row[st.parity][wave ^ w][at]);
#pragma unroll
            for (int q = 0; q < V / 4; ++q) {
                const u32x4 a = other[q];
                m[4 * q] = umax(m[4 * q], a.x);
                m[4 * q + 1] = umax(m[4 * q + 1], a.y);
                m[4 * q + 2] = umax(m[4 * q + 2], a.z);
                m[4 * q + 3] = umax(m[4 * q + 3], a.w);
            }
        }
        st.parity ^= 1;
    }
}

// What a lane loads of one chunk row: V bf16 values.
template <int V>
struct PieceOf;
template <>
struct PieceOf<8> {
    typedef u32x4 type;
};
template <>
struct PieceOf<4> {
    typedef u32x2 type;
};
template <int V>
using Piece = typename PieceOf<V>::type;

template <int R, int V>
__device__ __forceinline__ void load_strided(const uint16_t *x, const WaveSpot &sp, Piece<V> (&xv)[R])
{
#pragma unroll
    for (int r = 0; r < R; ++r) {
        xv[r] = __builtin_nontemporal_load(reinterpret_cast<const Piece<V> *>(x + sp.elem + r * sp.row_step));
    }
}

template <int V>
__device__ __forceinline__ void widen_piece(const Piece<V> &w, float (&f)[V])
{
#pragma unroll
    for (int i = 0; i < V / 2; ++i) {
        f[2 * i] = __uint_as_float(w[i] << 16);
        f[2 * i + 1] = __uint_as_float(w[i] & 0xFFFF0000u);
    }
}

template <int V>
__device__ __forceinline__ void store_piece(uint16_t *out, const float (&d)[V])
{
    Piece<V> w;
#pragma unroll
    for (int i = 0; i < V / 2; ++i) w[i] = narrow_bf16x2(d[2 * i], d[2 * i + 1]);
    __builtin_nontemporal_store(w, reinterpret_cast<Piece<V> *>(out));
}

template <int R, int V>
__device__ __forceinline__ void widen_strided(const Piece<V> (&xv)[R], float (&t)[R][V])
{
#pragma unroll
    for (int r = 0; r < R; ++r) widen_piece<V>(xv[r], t[r]);
}

// scale and inverse scale of the lane's V blocks for the sums t.
template <int R, int W, int V>
__device__ __forceinline__ void strided_quotients(const float (&t)[R][V], ChunkMaxState<W, V> &st, float (&scale)[V],
                                                  float (&inv)[V])
{
    uint32_t m[V] = {};
#pragma unroll
    for (int r = 0; r < R; ++r) note_absmax(t[r], m);
    across_chunks_max_wave<W, V>(m, st);
#pragma unroll
    for (int j = 0; j < V; ++j) block_quotients(__uint_as_float(m[j]), scale[j], inv[j]);
}

// The code of v as a float.  kPositiveZero: a value that rounds to zero from below gives +0.0, as the integer
// code converted back would (needed only where the sign of a zero sum can reach the output, i.e. when the
// all-gather is not quantized).
template <bool kPositiveZero>
__device__ __forceinline__ float code_of(float v, float inv)
{
    const float q = __builtin_rintf(v * inv);
    return kPositiveZero ? q + 0.0f : q;
}

// One hop: t <- fma(code(t), scale, x), what the device holding x has after it received the quantized t.
template <int R, int W, int V, bool kPositiveZero>
__device__ __forceinline__ void strided_hop(float (&t)[R][V], const Piece<V> (&xv)[R], ChunkMaxState<W, V> &st)
{
    float scale[V], inv[V];
    strided_quotients<R, W, V>(t, st, scale, inv);
#pragma unroll
    for (int r = 0; r < R; ++r) {
        float xf[V];
        widen_piece<V>(xv[r], xf);
#pragma unroll
        for (int j = 0; j < V; ++j) t[r][j] = __builtin_fmaf(code_of<kPositiveZero>(t[r][j], inv[j]), scale[j], xf[j]);
    }
}

// The send that ends a half chain of the semi-loop: acc <- fma(code(t), scale, acc).
template <int R, int W, int V, bool kPositiveZero>
__device__ __forceinline__ void strided_send_into(const float (&t)[R][V], float (&acc)[R][V], ChunkMaxState<W, V> &st)
{
    float scale[V], inv[V];
    strided_quotients<R, W, V>(t, st, scale, inv);
#pragma unroll
    for (int r = 0; r < R; ++r) {
#pragma unroll
        for (int j = 0; j < V; ++j) acc[r][j] = __builtin_fmaf(code_of<kPositiveZero>(t[r][j], inv[j]), scale[j], acc[r][j]);
    }
}

// Waves per SIMD the compiler may plan for.  The full loop with a quantized reduce-scatter runs 3-4 us faster (of
// 63-75 at the 27B-shaped size) held to two waves than at the four its ~120 registers would allow: the loads of one
// partial per wave already fill the memory queues, and more waves only lengthen them.  The semi-loop (two dependent
// half chains) and the unquantized reduce-scatter measured the other way round and keep the default.
// The small-message layout keeps the default, too.
constexpr int strided_chain_waves(bool semi, bool rs, int V) { return (!semi && rs && V == 8) ? 2 : 8; }

// chunks = 8 * W * R.  kSemi: the semi-loop with partials[0] as the owner (always a quantized reduce-scatter);
// otherwise the full loop in array order with the reduce-scatter quantized (kRS) or added in plain fp32.  kAG: the
// finished sum is quantized once more and dequantized; otherwise narrowed to bf16 directly.
// Ring layout (Sec. 3): with per_shard > 0 the tensor is cut into shards of per_shard minishards and shard k ends
// on device k: the full loop takes the partials in the order k+1, k+2, ..., k (mod P), the semi-loop has device k
// as its owner and the devices k+1, k+2, ... around it.  per_shard == 0: array order everywhere.
template <int R, int W, int V, bool kSemi, bool kRS, bool kAG>
__global__ __launch_bounds__(kThreads) __attribute__((amdgpu_waves_per_eu(1, strided_chain_waves(kSemi, kRS, V))))
void chain_strided_kernel(int P, int per_shard, Global<uint16_t> out, const PartialTable tab)
{
    static_assert(kRS || !kSemi, "the semi-loop is a quantized reduce-scatter");
    __shared__ __align__(16) ChunkMaxRows<W, V> red;
    ChunkMaxState<W, V> st{red, 0};
    constexpr int chunks = 8 * W * R;
    const WaveSpot sp = wave_spot<W, V>(chunks);
    // position i of the chain -> partial; `first` <= P and i < P, so one conditional subtraction wraps
    const int first = per_shard > 0 ? (int)(sp.minishard / per_shard) + (kSemi ? 0 : 1) : 0;
    const auto part = [&](int i) {
        const int j = first + i;
        return tab.x[j >= P ? j - P : j];
    };

    float sum[R][V];
    Piece<V> xv[R];
    load_strided<R, V>(part(0), sp, xv);
    widen_strided<R, V>(xv, sum);
    if (kSemi) {
        const int h = P / 2;
        float t[R][V];
        if (h + 1 <= P - 1) {                       // h+1 -> h+2 -> ... -> P-1 -> owner: the shorter chain arrives first
            load_strided<R, V>(part(h + 1), sp, xv);
            widen_strided<R, V>(xv, t);
            for (int i = h + 2; i <= P - 1; ++i) {
                load_strided<R, V>(part(i), sp, xv);
                strided_hop<R, W, V, !kAG>(t, xv, st);
            }
            strided_send_into<R, W, V, !kAG>(t, sum, st);
        }
        if (h >= 1) {                               // h -> h-1 -> ... -> 1 -> owner
            load_strided<R, V>(part(h), sp, xv);
            widen_strided<R, V>(xv, t);
            for (int i = h - 1; i >= 1; --i) {
                load_strided<R, V>(part(i), sp, xv);
                strided_hop<R, W, V, !kAG>(t, xv, st);
            }
            strided_send_into<R, W, V, !kAG>(t, sum, st);
        }
    } else {
        for (int i = 1; i < P; ++i) {
            // With two waves per SIMD and two waves per piece the loop's time hangs on how its instructions lie on 8-byte
            // boundaries: moved by 4 bytes by whatever stands before it, it takes up to 9 % longer (MI355X, 40 minishards of
            // 128 chunks, P = 16: 42.1 us; 38.7 like this; 154 minishards 122.8 and 119.5).
            if (kRS && W == 2 && V == 8) asm volatile(".p2align 3");
            load_strided<R, V>(part(i), sp, xv);
            if (kRS) {
                strided_hop<R, W, V, !kAG>(sum, xv, st);
            } else {
#pragma unroll
                for (int r = 0; r < R; ++r) {
                    float xf[V];
                    widen_piece<V>(xv[r], xf);
#pragma unroll
                    for (int j = 0; j < V; ++j) sum[r][j] = sum[r][j] + xf[j];
                }
            }
        }
    }

    float scale[V], inv[V];
    if (kAG) strided_quotients<R, W, V>(sum, st, scale, inv);
#pragma unroll
    for (int r = 0; r < R; ++r) {
        float d[V];
#pragma unroll
        for (int j = 0; j < V; ++j) d[j] = kAG ? code_of<true>(sum[r][j], inv[j]) * scale[j] : sum[r][j];
        store_piece<V>(out + sp.elem + r * sp.row_step, d);
    }
}

// ---------------------------------------------------------------- the per-pass kernels for few minishards
//
// The same passes in the wave layout: W = 4 waves share a piece of 64 positions, R = chunks / 32 rows per thread
// instead of chunks / 8, 16 workgroups per minishard instead of 4.  Code pieces are 64 bytes, half a line, which is
// why the per-pass kernels above have another layout; a message of few minishards is not bound by that but by the
// time one wave takes (MI355X, hop-by-hop chain of four, five passes, 8 minishards: 64 chunks 17.9 -> 15.0 us, 128
// chunks 24.4 -> 17.6).

template <int R>
struct WavePass {
    static constexpr int W = 4, V = 8, kChunks = 8 * W * R;
    WaveSpot sp;
    ChunkMaxState<W, V> st;

    __device__ __forceinline__ explicit WavePass(ChunkMaxRows<W, V> &red) : sp(wave_spot<W, V>(kChunks)), st{red, 0} {}

    __device__ __forceinline__ void load(const uint16_t *x, float (&t)[R][V]) const
    {
        Piece<V> xv[R];
        load_strided<R, V>(x, sp, xv);
        widen_strided<R, V>(xv, t);
    }

    // t += codes * scales, one fused multiply-add per element
    __device__ __forceinline__ void add_wire(const int8_t *codes, const float *scales, float (&t)[R][V]) const
    {
        u32x2 cv[R];
#pragma unroll
        for (int r = 0; r < R; ++r) cv[r] = *reinterpret_cast<const u32x2 *>(codes + sp.elem + r * sp.row_step);
        const u32x4 a = *reinterpret_cast<const u32x4 *>(scales + sp.scale);
        const u32x4 b = *reinterpret_cast<const u32x4 *>(scales + sp.scale + 4);
#pragma unroll
        for (int r = 0; r < R; ++r) {
            float qf[V];
            widen_i8x8(cv[r], qf);
#pragma unroll
            for (int j = 0; j < V; ++j) t[r][j] = __builtin_fmaf(qf[j], __uint_as_float(j < 4 ? a[j & 3] : b[j & 3]), t[r][j]);
        }
    }

    __device__ __forceinline__ void send(const float (&t)[R][V], int8_t *codes, float *scales)
    {
        float scale[V], inv[V];
        strided_quotients<R, W, V>(t, st, scale, inv);
#pragma unroll
        for (int r = 0; r < R; ++r) *reinterpret_cast<u32x2 *>(codes + sp.elem + r * sp.row_step) = scale_and_pack(t[r], inv);
        if (sp.first_group) {
            u32x4 *s = reinterpret_cast<u32x4 *>(scales + sp.scale);
            s[0] = u32x4{__float_as_uint(scale[0]), __float_as_uint(scale[1]), __float_as_uint(scale[2]), __float_as_uint(scale[3])};
            s[1] = u32x4{__float_as_uint(scale[4]), __float_as_uint(scale[5]), __float_as_uint(scale[6]), __float_as_uint(scale[7])};
        }
    }
};

// kWire: a hop; otherwise the chain's first shard is quantized.  The output wire may be the input wire: the waves of a
// piece meet at a barrier between their last load and their first store.
template <int R, bool kWire>
__global__ __launch_bounds__(kThreads) void pass_strided_small_kernel(Global<const int8_t> cin, Global<const float> sin, Global<int8_t> cout,
                                                                      Global<float> sout, const StridedSource src)
{
    __shared__ __align__(16) ChunkMaxRows<4, 8> red;
    WavePass<R> pass(red);
    float t[R][8];
    pass.load(strided_source(src, pass.sp.minishard), t);
    if (kWire) pass.add_wire(cin, sin, t);
    pass.send(t, cout, sout);
}

template <int R>
__global__ __launch_bounds__(kThreads) void semi_step_strided_small_kernel(int P, int per_shard,
                                                                           const StridedDirections dirs,
                                                                           const PartialTable tab)
{
    __shared__ __align__(16) ChunkMaxRows<4, 8> red;
    WavePass<R> pass(red);
    const StridedDirection d = blockIdx.y == 0 ? dirs.d[0] : dirs.d[1];
    const int j = (per_shard > 0 ? (int)(pass.sp.minishard / per_shard) : 0) + d.offset;     // < 2P
    float t[R][8];
    pass.load(tab.x[j >= P ? j - P : j], t);
    if (d.cin != nullptr) pass.add_wire(d.cin, d.sin, t);       // uniform over the workgroup
    pass.send(t, d.cout, d.sout);
}

template <int R, bool kAG>
__global__ __launch_bounds__(kThreads) void owner_strided_small_kernel(int received, Global<uint16_t> out,
                                                                       const StridedWires wires, const StridedSource src)
{
    __shared__ __align__(16) ChunkMaxRows<4, 8> red;
    WavePass<R> pass(red);
    float t[R][8];
    pass.load(strided_source(src, pass.sp.minishard), t);
    for (int k = 0; k < received; ++k) pass.add_wire(wires.codes[k], wires.scales[k], t);
    float scale[8], inv[8];
    if (kAG) strided_quotients<R, 4, 8>(t, pass.st, scale, inv);
#pragma unroll
    for (int r = 0; r < R; ++r) {
        float d[8];
#pragma unroll
        for (int j = 0; j < 8; ++j) d[j] = kAG ? code_of<true>(t[r][j], inv[j]) * scale[j] : t[r][j];
        store_piece<8>(out + pass.sp.elem + r * pass.sp.row_step, d);
    }
}

// Dequantize in the strided geometry: element e uses scale (e / (1024*chunks)) * 1024 + e % 1024, so the 8
// elements of a lane use 8 consecutive scales.  n is a multiple of 1024: 8 elements are inside or outside as a whole.
template <int K>
__global__ __launch_bounds__(pass_threads(K)) void dequantize_strided_kernel(Global<const int8_t> codes,
                                                                      Global<const float> scales, int64_t n,
                                                                      int chunks, Global<uint16_t> out, int64_t mirror)
{
    constexpr int T = pass_threads(K);
    const int64_t wg_at = first_element<T, K>(mirror);
    const int lane_at = threadIdx.x * kLaneElems;
    const int64_t minishard = (int64_t)kChunk * chunks;
#pragma unroll
    for (int k = 0; k < K; ++k) {
        const int64_t at = wg_at + k * tile_elems<T> + lane_at;
        if (at >= n) continue;                       // n % 8 == 0: a lane is inside or outside as a whole
        const u32x2 cv = *reinterpret_cast<const u32x2 *>(codes + at);
        const float *s = scales + (at / minishard) * kChunk + at % kChunk;
        const u32x4 a = *reinterpret_cast<const u32x4 *>(s);
        const u32x4 b = *reinterpret_cast<const u32x4 *>(s + 4);
        float qf[8];
        widen_i8x8(cv, qf);
        u32x4 w;
        w.x = narrow_bf16x2(qf[0] * __uint_as_float(a.x), qf[1] * __uint_as_float(a.y));
        w.y = narrow_bf16x2(qf[2] * __uint_as_float(a.z), qf[3] * __uint_as_float(a.w));
        w.z = narrow_bf16x2(qf[4] * __uint_as_float(b.x), qf[5] * __uint_as_float(b.y));
        w.w = narrow_bf16x2(qf[6] * __uint_as_float(b.z), qf[7] * __uint_as_float(b.w));
        __builtin_nontemporal_store(w, reinterpret_cast<u32x4 *>(out + at));
    }
}

}  // namespace equarx
