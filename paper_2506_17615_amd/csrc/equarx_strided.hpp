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
// Decomposition of the per-pass kernels (quantize, hop, owner): a workgroup of 256 threads takes one slice of 8 L
// positions of one minishard, L = 8, 16 or 32 lanes across it.  Thread (g, l) owns positions 8l..8l+7 of the slice in
// chunks g, g + 256/L, ...; its sums stay in registers, so memory is read once and nothing is computed twice.  The
// 256/L partial maxima per position meet in LDS (8 KiB), thread t turns those of position t into the two quotients, and
// every thread reads the quotients of its 8 positions back.  A row of L lanes covers 16 L contiguous bytes of bf16 and
// 8 L of codes.  (The single-launch chain further down writes no codes and uses a layout without LDS.)
//
// What bounds a pass is memory, but with all its workgroups resident at once they read together and then compute
// together, so arithmetic that memory does not cover is paid for.  Measured on MI355X, us per launch of a hop of 64 chunks,
// 22 M elements inside the hop-by-hop chain: 14.3 with each thread deriving the quotients of its 8 positions and computing
// its values twice (673 vector instructions at 8 rows), 13.7 as it is but with 64-bit addresses per row and the tensor's
// address looked up in a table (482), 13.2 as it is (430); the contiguous hop takes 12.3.
#pragma once

#include "equarx_device.hpp"

namespace equarx {

constexpr int kChunk = 1024;                               // elements per chunk (8 x 128)

// Layout of a per-pass kernel for minishards of kChunks chunks: L lanes across a slice of a chunk.
template <int kChunks_, int L_>
struct Slices {
    static constexpr int kChunks = kChunks_, L = L_;
    static constexpr int kPos = L * kLaneElems;             // positions of a slice, which is a workgroup's
    static constexpr int kGroups = kThreads / L;            // groups of lanes, each walking every kGroups'th chunk
    static constexpr int R = kChunks / kGroups;             // chunks per thread
    static constexpr int kParts = kChunk / kPos;            // workgroups per minishard
    static constexpr int kRow = kGroups * kChunk;           // elements from a lane's chunk to its next
    static_assert(R >= 1 && kPos <= kThreads, "layout");
};

// A launch that walks back (walks_back): workgroup b of the first `mirror`, a multiple of eight, takes the place of one
// in the opposite group of eight.  mirror == 0: it walks forward.
__device__ __forceinline__ unsigned mirrored_place(unsigned b, unsigned mirror)
{
    return b < mirror ? mirror - 8 - (b & ~7u) + (b & 7u) : b;
}

__host__ __device__ inline unsigned whole_groups(unsigned count) { return (count + 7) & ~7u; }

// Which minishard, and which of its kParts equal parts, the workgroup at place `at` of a launch takes.  The first places
// go to the XCDs in runs of 2^18 elements, whole minishards, the parts of each one after the other; those that follow,
// fewer than 8 runs, count the parts of one minishard after another.  `owned`: the number of the first, a multiple of 8
// kParts runs; in its low two bits the logarithm of the run's minishards, and in the three above by how many minishards the
// first run is shorter, so that runs begin where the wire's address is a multiple of 2^18 (as nearly as minishards allow).
// The places of what is missing there are for minishards below 0 (strided_spot's `outside`).
//
// So a minishard is on one XCD in every launch, also in the dequantization, which takes consecutive elements: each finds
// the wire in the L2 that holds it.  With the parts of a minishard on four XCDs the dequantization did not.  Runs, because
// what an XCD touches then differs in all the lower address bits: with minishard m on XCD m % 8 the L2s keep less of the
// wire, as if 256 KiB of address chose the place in them.  Measured on MI355X, P = 8, hop by hop, us with the parts on four
// XCDs / minishard m on XCD m % 8 / runs of 2^17 / of 2^18 elements (the four kernels otherwise the same): 64 chunks, 16.8 M
// elements 97.8 / 103.8 / 103.9 / 93.1; 22 M 127.7 / 127.4 / 125.1 / 122.8; 32 chunks, 16.8 M (after the steps above) runs of
// 2^17 101.7, of 2^18 91.1.  A contiguous eighth of the tensor to an XCD is as good in the hops and worse without any (P = 2,
// 35.7 M: 51.3, runs 50.9, four XCDs 49.2).
struct MinishardPart {
    int minishard;
    int part;
};

__host__ __device__ inline unsigned missing_minishards(unsigned owned) { return owned >> 2 & 7u; }

template <int kParts>
__device__ __forceinline__ MinishardPart minishard_part(unsigned at, unsigned owned)
{
    static_assert(kParts % 4 == 0, "five bits to spare");
    const unsigned run = owned & 3u, missing = missing_minishards(owned);
    if (at >= (owned & ~31u)) return MinishardPart{(int)(at / kParts - missing), (int)(at % kParts)};
    const unsigned in_xcd = at / 8, in_run = in_xcd & ((kParts << run) - 1), group = in_xcd / kParts >> run;
    return MinishardPart{(int)((group * 8 + at % 8 << run) + in_run / kParts - missing), (int)(in_run % kParts)};
}

template <int kChunks, int kParts>
inline unsigned owned_places(int64_t minishards, const void *wire)
{
    constexpr int kLen = kChunk * kChunks;
    int run = kChunks == 32 ? 3 : kChunks == 64 ? 2 : 1;
    while (run > 0 && minishards < (int64_t)8 << run) --run;
    const unsigned missing = (unsigned)((reinterpret_cast<uintptr_t>(wire) + kLen / 2) / kLen) & ((1u << run) - 1);
    return ((unsigned)((minishards + missing) >> (3 + run) << (3 + run)) * kParts) | missing << 2 | run;
}

struct StridedSpot {
    bool outside;       // nothing to do here
    int minishard;      // which minishard the workgroup works on
    int64_t elem;       // first element of the slice in the first chunk of its minishard
    int64_t scale;      // index of the slice's first scale
    int at, pos;        // the lane's first element, from there, in the first of its chunks; its first position
};

// at: the workgroup's place in the tensor.
template <typename S>
__device__ __forceinline__ StridedSpot strided_spot(unsigned at, unsigned owned)
{
    StridedSpot sp;
    const MinishardPart slice = minishard_part<S::kParts>(at, owned);
    sp.outside = slice.minishard < 0;
    sp.minishard = slice.minishard;
    sp.elem = (int64_t)slice.minishard * (kChunk * S::kChunks) + slice.part * S::kPos;
    sp.scale = (int64_t)slice.minishard * kChunk + slice.part * S::kPos;
    sp.pos = threadIdx.x % S::L * kLaneElems;
    sp.at = threadIdx.x / S::L * kChunk + sp.pos;
    return sp;
}

// A lane's access in row r, kRow elements further on in every row: a buffer descriptor that begins where the workgroup
// does, the lane's offset and, in a scalar register, the row's, so that no row costs vector instructions.  The 16-byte
// store has its row in the descriptor: the compiler takes an offset in a scalar register for a reason to let the next
// instruction overwrite what the store is still reading, and on MI355X it does overwrite it (words of the output held later
// values, now and then, with two workgroups on a CU).  The 8-byte store keeps it there: the architecture's manual names the hazard
// for stores of more than 64 bits, whose data the memory unit takes in a second step, and for no others.
constexpr int kMinishardEnd = kChunk * 128 * 2;     // bytes from there that no descriptor has to reach past

template <int kRow>
__device__ __forceinline__ u32x4 load_row_bf16x8(const uint16_t *base, int at, int r)
{
    return __builtin_bit_cast(u32x4, __builtin_amdgcn_raw_buffer_load_b128(bounded(base, kMinishardEnd), at * 2, r * kRow * 2, kNonTemporal));
}

template <int kRow>
__device__ __forceinline__ u32x2 load_row_i8x8(const int8_t *base, int at, int r)
{
    return __builtin_bit_cast(u32x2, __builtin_amdgcn_raw_buffer_load_b64(bounded(base, kMinishardEnd), at, r * kRow, 0));
}

template <int kRow>
__device__ __forceinline__ void store_row_i8x8(int8_t *base, int at, int r, const u32x2 &w)
{
    __builtin_amdgcn_raw_buffer_store_b64(w, bounded(base, kMinishardEnd), at, r * kRow, 0);
}

template <int kRow>
__device__ __forceinline__ void store_row_bf16x8(uint16_t *base, int at, int r, const float (&v)[8])
{
    u32x4 w;
    w.x = narrow_bf16x2(v[0], v[1]);
    w.y = narrow_bf16x2(v[2], v[3]);
    w.z = narrow_bf16x2(v[4], v[5]);
    w.w = narrow_bf16x2(v[6], v[7]);
    __builtin_amdgcn_raw_buffer_store_b128(w, bounded(base + r * kRow, kMinishardEnd), at * 2, 0, kNonTemporal);
}

// The bf16 tensor a per-pass kernel reads, as its last parameters: one tensor, in array order; or in the ring layout
// (Sec. 3), where the tensor is cut into shards of per_shard minishards, shard k ends on device k and a launch is one
// ring step on every shard at once, the partial of device (k + offset) mod P for the workgroups of shard k, 0 <= offset < P.
// One tensor's address is in scalar registers when a wave starts; a table has to be asked first, so the shard, on which that
// waits, is taken without a division: floor(m / per_shard) is the high word of 2 m * magic, shifted (ring_division).  `ring`: P,
// the offset from bit 8 on, in bits 24 to 28 the shift.  Array order out of a table: magic == 0.  Measured on MI355X, us per
// chain in ring order, P = 8, with a division -> as it is: 32 chunks, 4.2 M elements 42.2 -> 40.7, 8.4 M 53.3 -> 51.7; 64 chunks, 4.2 M
// 41.4 -> 39.5 (in array order 34.1: what is left of the difference is the table).
__device__ __forceinline__ const uint16_t *strided_source(int, Global<const uint16_t> x) { return x; }

__device__ __forceinline__ const uint16_t *strided_source(int minishard, unsigned magic, unsigned ring, const PartialTable &tab)
{
    const int P = ring & 255;
    const int j = (int)(__umulhi(2u * (unsigned)minishard, magic) >> (ring >> 24 & 31u)) + (int)(ring >> 8 & 255);     // < 2P
    return tab.x[j >= P ? j - P : j];
}

// The larger of two, a NaN if one of them is one (v_maximum3_f32, where fmaxf's v_max3_f32 drops it; two values per
// instruction either way): a NaN becomes its block's scale, so that all of the block comes out as NaN and never a finite
// value in a NaN's place.
__device__ __forceinline__ float larger(float a, float b) { return __builtin_elementwise_maximum(a, b); }

// The quotients of a slice's positions, through LDS: each group leaves its 8 maxima per lane, then thread t works on
// position t alone and hands the quotients back.
template <typename S>
struct SliceQuotients {
    float part[S::kGroups][S::kPos];
    float inv[S::kPos];
    float scale[S::kPos];
};

__device__ __forceinline__ void read_eight(const float *p, float (&v)[8])
{
    const u32x4 *w = reinterpret_cast<const u32x4 *>(p);
    const u32x4 a = w[0], b = w[1];
#pragma unroll
    for (int j = 0; j < 4; ++j) {
        v[j] = __uint_as_float(a[j]);
        v[4 + j] = __uint_as_float(b[j]);
    }
}

// m: the lane's max-abs over its chunks.  Returns the scale of position threadIdx.x; inv (and with kScales scale) are
// those of the lane's 8 positions.
template <bool kScales, typename S>
__device__ __forceinline__ float slice_quotients(const float (&m)[8], SliceQuotients<S> &q, float (&inv)[8], float (&scale)[8])
{
    const int l = threadIdx.x % S::L;
    const int g = threadIdx.x / S::L;
    u32x4 *row = reinterpret_cast<u32x4 *>(&q.part[g][l * kLaneElems]);
    row[0] = u32x4{__float_as_uint(m[0]), __float_as_uint(m[1]), __float_as_uint(m[2]), __float_as_uint(m[3])};
    row[1] = u32x4{__float_as_uint(m[4]), __float_as_uint(m[5]), __float_as_uint(m[6]), __float_as_uint(m[7])};
    __syncthreads();
    const int mine = threadIdx.x % S::kPos;
    float a = q.part[0][mine];
#pragma unroll
    for (int h = 1; h < S::kGroups; ++h) a = larger(a, q.part[h][mine]);
    float own, own_inv;
    block_quotients(a, own, own_inv);
    q.inv[mine] = own_inv;
    if (kScales) q.scale[mine] = own;
    __syncthreads();
    read_eight(&q.inv[l * kLaneElems], inv);
    if (kScales) read_eight(&q.scale[l * kLaneElems], scale);
    return own;
}

// m[j]: the largest |t[r][j]|.  All positions of a row at once, because the compiler makes a tree of two-operand maxima out of
// the rows of a single position: half as many instructions again, and the loads before them in another order (reduce-scatter
// in fp32, 96 minishards of 64 chunks, P = 8: 24.9 us instead of 19.4).
template <int R, int V>
__device__ __forceinline__ void absmax_of_rows(const float (&t)[R][V], float (&m)[V])
{
    typedef float Row __attribute__((ext_vector_type(V)));
    Row a;
#pragma unroll
    for (int r = 0; r < R; ++r) {
        Row b;
#pragma unroll
        for (int j = 0; j < V; ++j) b[j] = __builtin_fabsf(t[r][j]);
        a = r == 0 ? b : __builtin_elementwise_maximum(a, b);
    }
#pragma unroll
    for (int j = 0; j < V; ++j) m[j] = a[j];
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

// The slice's values t to the wire.
template <typename S>
__device__ __forceinline__ void send_slice(const float (&t)[S::R][8], int8_t *codes, float *scales, const StridedSpot &sp, SliceQuotients<S> &q)
{
    float m[8];
    absmax_of_rows(t, m);
    float inv[8];
    const float own = slice_quotients<false>(m, q, inv, inv);
    if (threadIdx.x < S::kPos) scales[sp.scale + threadIdx.x] = own;
#pragma unroll
    for (int r = 0; r < S::R; ++r) {
        store_row_i8x8<S::kRow>(codes + sp.elem, sp.at, r, scale_and_pack(t[r], inv));
    }
}

template <typename S>
__device__ __forceinline__ void quantize_strided_body(const uint16_t *__restrict__ x, int8_t *__restrict__ codes,
                                                      float *__restrict__ scales, const StridedSpot &sp, SliceQuotients<S> &q)
{
    u32x4 xv[S::R];
#pragma unroll
    for (int r = 0; r < S::R; ++r) xv[r] = load_row_bf16x8<S::kRow>(x + sp.elem, sp.at, r);
    float t[S::R][8];
#pragma unroll
    for (int r = 0; r < S::R; ++r) widen_bf16x8(xv[r], t[r]);
    send_slice<S>(t, codes, scales, sp, q);
}

template <typename S, typename... Source>
__global__ __launch_bounds__(kThreads) void quantize_strided_kernel(Global<int8_t> codes, Global<float> scales, unsigned owned,
                                                                    const Source... src)
{
    __shared__ __align__(16) SliceQuotients<S> q;
    const StridedSpot sp = strided_spot<S>(blockIdx.x, owned);
    if (sp.outside) return;             // uniform over the workgroup
    quantize_strided_body<S>(strided_source(sp.minishard, src...), codes, scales, sp, q);
}

// One hop in the strided geometry.  Output wire may be the input wire: a
// workgroup holds all its inputs in registers before it stores anything.
template <typename S>
__device__ __forceinline__ void hop_strided_body(const int8_t *cin, const float *sin, const uint16_t *__restrict__ x,
                                                 int8_t *cout, float *sout, const StridedSpot &sp, SliceQuotients<S> &q)
{
    u32x4 xv[S::R];
    u32x2 cv[S::R];
    float s_in[8];
    read_eight(sin + sp.scale + sp.pos, s_in);
#pragma unroll
    for (int r = 0; r < S::R; ++r) {        // in turn: all codes first is 6 % slower (64 chunks, 16.8 M elements, 86.3 -> 91.2 us)
        xv[r] = load_row_bf16x8<S::kRow>(x + sp.elem, sp.at, r);
        cv[r] = load_row_i8x8<S::kRow>(cin + sp.elem, sp.at, r);
    }
    loads_first();
    float t[S::R][8];
#pragma unroll
    for (int r = 0; r < S::R; ++r) {
        float xf[8], qf[8];
        widen_bf16x8(xv[r], xf);
        widen_i8x8(cv[r], qf);
#pragma unroll
        for (int j = 0; j < 8; ++j) t[r][j] = __builtin_fmaf(qf[j], s_in[j], xf[j]);
    }
    send_slice<S>(t, cout, sout, sp, q);
}

template <typename S, typename... Source>
__global__ __launch_bounds__(kThreads) void hop_strided_kernel(Global<const int8_t> cin, Global<const float> sin, Global<int8_t> cout,
                                                               Global<float> sout, unsigned mirror, unsigned owned, const Source... src)
{
    __shared__ __align__(16) SliceQuotients<S> q;
    const StridedSpot sp = strided_spot<S>(mirrored_place(blockIdx.x, mirror), owned);
    if (sp.outside) return;             // uniform over the workgroup
    hop_strided_body<S>(cin, sin, strided_source(sp.minishard, src...), cout, sout, sp, q);
}

// One iteration of the semi-loop reduce-scatter (Sec. 3.3) on both of its chains at once: the first half of the grid
// (`count` workgroups and those of missing minishards, in whole groups of eight) advances the chain that walks up from device h+1, the second the one that
// walks down from device h, each by one device -- the first iteration quantizes the chain's first shard, the later ones are
// hops on the chain's own wire buffer in place.  The two halves share nothing.  `ring`: as in strided_source, the second
// direction's offset from bit 16 on.
template <typename S>
__host__ __device__ inline unsigned semi_step_half(unsigned count, unsigned owned0, unsigned owned1)
{
    const unsigned a = missing_minishards(owned0), b = missing_minishards(owned1);
    return whole_groups(count + (a > b ? a : b) * S::kParts);
}

// backward_first: bit 0, the launch walks back; bit 1, it is the first iteration.
template <typename S>
__global__ __launch_bounds__(kThreads) void semi_step_strided_kernel(Global<int8_t> codes0, Global<float> scales0, Global<int8_t> codes1,
                                                                     Global<float> scales1, unsigned magic, unsigned ring, unsigned count,
                                                                     unsigned owned0, unsigned owned1, int backward_first, const PartialTable tab)
{
    __shared__ __align__(16) SliceQuotients<S> q;
    const unsigned half = semi_step_half<S>(count, owned0, owned1);
    const unsigned place = mirrored_place(blockIdx.x, backward_first & 1 ? 2 * half : 0);
    const bool second = place >= half;
    const unsigned at = second ? place - half : place, owned = second ? owned1 : owned0;
    const StridedSpot sp = strided_spot<S>(at, owned);
    if (sp.outside || at >= count + missing_minishards(owned) * S::kParts) return;      // uniform over the workgroup
    int8_t *codes = second ? codes1 : codes0;
    float *scales = second ? scales1 : scales0;
    const uint16_t *x = strided_source(sp.minishard, magic, second ? (ring & 0xff0000ffu) | (ring >> 8 & 0xff00u) : ring, tab);
    if (backward_first & 2) {           // uniform over the workgroup
        quantize_strided_body<S>(x, codes, scales, sp, q);
    } else {
        hop_strided_body<S>(codes, scales, x, codes, scales, sp, q);
    }
}

// The last launch of a hop-by-hop flavour in the strided geometry: the device that ends up with the sum adds what
// it received to its own bf16 shard -- one wire at the end of the full loop, one or two at the owner of the
// semi-loop (Sec. 3.3: the shorter chain's wire first), none when it is alone (nullptr) -- each with one fused multiply-add
// per element, and hands the sum to the all-gather: quantized once more and dequantized (kAG), or narrowed to
// bf16 as it is (Sec. 3.4).  out may be `own`: a thread reads its elements before it writes them.
template <typename S, bool kAG, typename... Source>
__global__ __launch_bounds__(kThreads) void owner_strided_kernel(Global<uint16_t> out, Global<const int8_t> codes0, Global<const float> scales0,
                                                                 Global<const int8_t> codes1, Global<const float> scales1,
                                                                 unsigned mirror, unsigned owned, const Source... src)
{
    __shared__ __align__(16) SliceQuotients<S> q;
    const StridedSpot sp = strided_spot<S>(mirrored_place(blockIdx.x, mirror), owned);
    if (sp.outside) return;             // uniform over the workgroup
    const uint16_t *own = strided_source(sp.minishard, src...);

    float acc[S::R][8];
    {
        u32x4 xv[S::R];
#pragma unroll
        for (int r = 0; r < S::R; ++r) xv[r] = load_row_bf16x8<S::kRow>(own + sp.elem, sp.at, r);
#pragma unroll
        for (int r = 0; r < S::R; ++r) widen_bf16x8(xv[r], acc[r]);
    }
#pragma unroll 1
    for (int k = 0; k < 2; ++k) {
        const int8_t *codes = k ? codes1 : codes0;
        const float *scales = k ? scales1 : scales0;
        if (!codes) break;              // uniform
        u32x2 cv[S::R];
        float s_in[8];
#pragma unroll
        for (int r = 0; r < S::R; ++r) cv[r] = load_row_i8x8<S::kRow>(codes + sp.elem, sp.at, r);
        read_eight(scales + sp.scale + sp.pos, s_in);
#pragma unroll
        for (int r = 0; r < S::R; ++r) {
            float qf[8];
            widen_i8x8(cv[r], qf);
#pragma unroll
            for (int j = 0; j < 8; ++j) acc[r][j] = __builtin_fmaf(qf[j], s_in[j], acc[r][j]);
        }
    }

    float scale[8], inv[8];
    if (kAG) {
        float m[8];
        absmax_of_rows(acc, m);
        slice_quotients<true>(m, q, inv, scale);
    }
#pragma unroll
    for (int r = 0; r < S::R; ++r) {
        float d[8];
#pragma unroll
        for (int j = 0; j < 8; ++j) {
            d[j] = kAG ? (__builtin_rintf(acc[r][j] * inv[j]) + 0.0f) * scale[j] : acc[r][j];     // +0.0: the code as an integer
        }
        store_row_bf16x8<S::kRow>(out + sp.elem, sp.at, r, d);
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
// groups 8w .. 8w+7 (R = 8), and the two maxima meet through LDS, 256 bytes a
// wave and 2 KiB in all, and one barrier per send (the buffer alternates, so the
// barrier of the next send also separates this send's reads from the writes of
// the one after).
// Same operations in the same order as the hop-by-hop strided chain, hence
// the same bits.
//
// A send does not compute anything twice either: the 8 lanes of a position end their exchange with one of its 8 positions'
// maxima each (scatter_max), work out that one pair of quotients and hand it round (gather_lanes).  With every lane deriving
// all 8 pairs, and 64-bit addresses per row, the full loop had 773, 1197 and 1290 vector instructions at 32, 64 and 128 chunks,
// now 497, 857 and 881.  Measured on MI355X, us of GPU time, P = 8, before -> after: 22 M elements of 32 chunks 66.9 -> 60.8, of 64
// 61.7 -> 60.5, of 128 69.9 -> 68.5; 17 minishards of 32 chunks 10.3 -> 8.5, one 5.4 -> 4.2.  (Calls among others, with the
// launch: of 64 chunks 61.4..61.6, and up to 66 by where the partials lie in memory.)
//
// A message of few minishards is bound by the time one wave takes per send,
// not by memory: W = 4 waves share a piece and a lane has V = 4 positions
// instead of 8, so a wave has a quarter of the rows at half of the positions,
// an eighth of the work, and a minishard 32 workgroups instead of 4.  In
// between, at 64 and 128 chunks, 4 waves share a piece and a lane has its 8
// positions: a quarter of the work, and 16 workgroups.

struct WaveSpot {
    unsigned minishard; // which minishard the workgroup works on
    int64_t elem;       // first element of the workgroup's positions in the first chunk of its minishard
    int at;             // the lane's first element, from there, in the first of its chunks
};

// W waves per position piece, V positions per lane; a 256-thread workgroup covers (4 / W) * 8 V positions.
template <int W, int V>
constexpr int wave_layout_wgs = kChunk / ((kThreads / 64) / W * 8 * V);      // workgroups per minishard

template <int W, int V>
__device__ __forceinline__ WaveSpot wave_spot(int chunks, unsigned owned)
{
    static_assert((W == 1 || W == 2 || W == 4) && (V == 4 || V == 8), "waves per position piece, positions per lane");
    constexpr int kPieces = (kThreads / 64) / W;                // position pieces per workgroup
    constexpr int kPerChunk = wave_layout_wgs<W, V>;
    const int lane = threadIdx.x % 64, wave = threadIdx.x / 64;
    const int g = (wave % W) * 8 + lane / 8;                    // chunk group, 0 .. 8W-1
    const MinishardPart place = minishard_part<kPerChunk>(blockIdx.x, owned);
    const int part = place.part;
    constexpr int kPositions = kPieces * 8 * V;
    WaveSpot sp;
    sp.minishard = place.minishard;
    sp.elem = (int64_t)sp.minishard * (kChunk * chunks) + part * kPositions;
    sp.at = g * kChunk + (wave / W) * (8 * V) + (lane % 8) * V;
    return sp;
}

// Maxima that waves exchange: one row per wave, two buffers in turn.
template <int W, int V>
struct ChunkMaxRows {
    float row[W > 1 ? 2 : 1][kThreads / 64][8 * V];
};

template <int W, int V>
struct ChunkMaxState {
    ChunkMaxRows<W, V> &red;
    int parity;
};

// m: the lane's max-abs at each of its V positions.  Returns the max over the 8 chunk groups of the wave at ONE of them,
// position g = lane / 8 for V = 8 and g / 2 for V = 4: at every step a lane hands on half of what it has and takes the other
// half of what its partner has (a permlane swap does both for two values).
template <int V>
__device__ __forceinline__ float scatter_max(const float (&m)[V])
{
    uint32_t a[V / 2], b[V / 4];
#pragma unroll
    for (int j = 0; j < V / 2; ++j) {
        auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(m[j]), __float_as_uint(m[j + V / 2]), false, false);
        a[j] = umax(r[0], r[1]);
    }
#pragma unroll
    for (int j = 0; j < V / 4; ++j) {
        auto r = __builtin_amdgcn_permlane16_swap(a[j], a[j + V / 4], false, false);
        b[j] = umax(r[0], r[1]);
    }
    if constexpr (V == 4) return __uint_as_float(umax(b[0], dpp_read<0x128>(b[0])));      // row_ror:8: lane ^ 8
    const bool odd = (threadIdx.x & 8) != 0;
    const uint32_t keep = odd ? b[V / 4 - 1] : b[0], give = odd ? b[0] : b[V / 4 - 1];
    return __uint_as_float(umax(keep, dpp_read<0x128>(give)));
}

// The way back: every lane gets the values of its V positions from the lanes that have them.
template <int V>
__device__ __forceinline__ void gather_lanes(float v, float (&all)[V])
{
    const uint32_t own = __float_as_uint(v), other = dpp_read<0x128>(own);
    const bool odd = (threadIdx.x & 8) != 0;
    const uint32_t two[2] = {odd ? other : own, odd ? own : other};
    constexpr int kEach = V / 4;        // 2, or 1: both lanes of a pair have the same position
#pragma unroll
    for (int i = 0; i < kEach; ++i) {
        const uint32_t x = kEach == 2 ? two[i] : own;
        auto r = __builtin_amdgcn_permlane16_swap(x, x, false, false);
#pragma unroll
        for (int k = 0; k < 2; ++k) {
            auto q = __builtin_amdgcn_permlane32_swap(r[k], r[k], false, false);
            all[kEach * k + i] = __uint_as_float(q[0]);
            all[kEach * k + i + V / 2] = __uint_as_float(q[1]);
        }
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

// Elements from a lane's chunk to its next.
template <int W>
constexpr int kWaveRow = 8 * W * kChunk;

template <int R, int W, int V>
__device__ __forceinline__ void load_strided(const uint16_t *x, const WaveSpot &sp, Piece<V> (&xv)[R])
{
#pragma unroll
    for (int r = 0; r < R; ++r) {
        if constexpr (V == 8) {
            xv[r] = load_row_bf16x8<kWaveRow<W>>(x + sp.elem, sp.at, r);
        } else {
            xv[r] = __builtin_bit_cast(Piece<V>, __builtin_amdgcn_raw_buffer_load_b64(bounded(x + sp.elem, kMinishardEnd), sp.at * 2,
                                                                                      r * kWaveRow<W> * 2, kNonTemporal));
        }
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

// scale and inverse scale of the lane's V blocks for the sums t.  A lane works one pair out and gets the others.  Every
// thread of the workgroup calls this; the state matters for W > 1 only.
template <int R, int W, int V>
__device__ __forceinline__ void strided_quotients(const float (&t)[R][V], ChunkMaxState<W, V> &st, float (&scale)[V],
                                                  float (&inv)[V])
{
    float m[V];
    absmax_of_rows(t, m);
    float a = scatter_max(m);
    if (W > 1) {
        const int wave = threadIdx.x / 64, at = threadIdx.x % 8 * V + threadIdx.x % 64 / 8 * V / 8;
        st.red.row[st.parity][wave][at] = a;
        __syncthreads();
#pragma unroll
        for (int w = 1; w < W; ++w) a = larger(a, st.red.row[st.parity][wave ^ w][at]);
        st.parity ^= 1;
    }
    float own_scale, own_inv;
    block_quotients(a, own_scale, own_inv);
    gather_lanes(own_scale, scale);
    gather_lanes(own_inv, inv);
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

// kWaves: waves per SIMD the compiler may plan for.  Two, where the registers would allow three to five: the loads of one
// partial per wave fill the memory queues as it is, and the fewer places of memory are read at once the better they stream.
// Eight, no cap, where two waves per SIMD, 512 workgroups at a time, would leave a last round to a few: at 32 chunks one of up
// to half of the chip's workgroups, from two rounds on and with more than four partials one of up to a quarter, because there
// the others gain more; at 64 chunks the half round after the first, unless it is nearly empty (the semi-loop's registers
// allow two waves either way).  Eight for the semi-loop of 32 chunks of up to four partials too, whose chains are one or two
// sends long and do not fill the queues.  The layouts of one row have eight and no use for a cap; of 64 chunks, 2 x 4 x 8 has
// registers for as many as its workgroups need under either; 4 x 4 x 8 has four: 128 chunks, P = 8, 16 and 32 minishards
// 9.3 and 13.8 us, with two the same but 40 minishards 20.2 instead of 18.9, without one 10.8 and 14.5.  Measured on MI355X, us,
// capped / not, P = 2, 4, 8, 16:
//     32 chunks, minishards (rounds)   full loop                                   semi-loop
//         144 (1.1)      6.8/6.0  10.8/8.9   18.4/15.1  33.3/26.9     7.4/6.0  11.7/9.4   19.3/16.2  34.3/28.9
//         192 (1.5)      7.8/6.7  11.9/10.7  20.1/18.7  36.5/34.0     7.9/7.2  12.7/11.1  21.5/19.6  38.2/35.5
//         200 (1.6)      8.4/7.7  12.6/12.5  21.0/21.9  37.4/38.0     9.1/7.7  14.2/13.2  22.2/22.9  38.2/42.2
//         256 (2)        9.9/9.4  15.2/14.5  24.4/24.9  42.8/45.9    10.6/9.3  16.1/14.8  25.0/26.3  43.5/46.9
//         288 (2.25)    11.0/11.0 17.4/17.2  29.5/29.9  53.8/56.1    11.7/11.2 18.5/17.5  30.6/30.0  54.8/57.0
//         336 (2.6)     12.4/12.2 19.3/19.6  32.3/34.0  57.8/63.5    13.4/12.8 20.9/19.7  33.9/34.1  59.1/64.2
//         400 (3.1)     14.7/14.2 23.1/22.0  39.4/37.6  72.4/69.4    15.6/15.0 24.9/22.2  41.0/38.6  73.4/70.6
//         448 (3.5)     15.9/15.9 24.8/25.3  42.1/45.0  76.4/85.9    16.7/16.2 26.4/25.6  43.6/43.2  77.3/87.1
//         512 (4)       17.6/17.4 28.0/26.8  46.5/46.0  84.3/86.0    18.8/17.6 29.4/27.1  47.9/50.0  85.0/88.8
//         1000 (7.8)    31.7/31.7 51.5/51.7  89.1/92.3   166/175     33.8/32.3 54.5/51.8  91.5/93.3   165/176
//     64 chunks                        full loop                                   reduce-scatter in fp32
//         144 (1.1)     10.6/11.1 17.4/18.6  30.8/32.3  59.3/62.0    10.5/11.2 16.9/17.4  30.4/30.9  57.6/58.2
//         176 (1.4)     12.8/12.8 20.1/19.9  35.5/35.4  65.9/67.8    12.9/12.6 20.3/19.1  34.6/34.2  62.7/60.0
//         184 (1.44)    13.4/13.1 21.3/20.4  37.3/36.8  68.4/67.8
//         192 (1.5)     14.3/13.6 22.5/20.8  37.3/36.2  67.3/67.3    14.2/13.4 22.6/20.6  39.0/36.5  73.6/69.5
//         220 (1.7)     15.9/15.8 24.8/24.9  42.9/44.1  80.4/84.2    15.6/15.5 24.8/24.0  42.8/43.2  79.8/81.1
//         336 (2.6)     23.1/23.2 36.9/38.0  66.5/69.2   113/125     23.3/23.6 37.1/38.0  64.8/65.3   125/130
// chunks = 8 * W * R.  kSemi: the semi-loop with partials[0] as the owner (always a quantized reduce-scatter);
// otherwise the full loop in array order with the reduce-scatter quantized (kRS) or added in plain fp32.  kAG: the
// finished sum is quantized once more and dequantized; otherwise narrowed to bf16 directly.
// Ring layout (Sec. 3): with per_shard > 0 the tensor is cut into shards of per_shard minishards and shard k ends
// on device k: the full loop takes the partials in the order k+1, k+2, ..., k (mod P), the semi-loop has device k
// as its owner and the devices k+1, k+2, ... around it.  per_shard == 0: array order everywhere.
template <int R, int W, int V, bool kSemi, bool kRS, bool kAG, int kWaves>
__global__ __launch_bounds__(kThreads) __attribute__((amdgpu_waves_per_eu(1, kWaves)))
void chain_strided_kernel(int P, int per_shard, Global<uint16_t> out, unsigned owned, const PartialTable tab)
{
    static_assert(kRS || !kSemi, "the semi-loop is a quantized reduce-scatter");
    __shared__ __align__(16) ChunkMaxRows<W, V> red;
    ChunkMaxState<W, V> st{red, 0};
    constexpr int chunks = 8 * W * R;
    const WaveSpot sp = wave_spot<W, V>(chunks, owned);
    // position i of the chain -> partial; `first` <= P and i < P, so one conditional subtraction wraps
    const int first = per_shard > 0 ? (int)(sp.minishard / (unsigned)per_shard) + (kSemi ? 0 : 1) : 0;
    const auto part = [&](int i) {
        const int j = first + i;
        return tab.x[j >= P ? j - P : j];
    };

    float sum[R][V];
    Piece<V> xv[R];
    load_strided<R, W, V>(part(0), sp, xv);
    widen_strided<R, V>(xv, sum);
    if (kSemi) {
        const int h = P / 2;
        float t[R][V];
        if (h + 1 <= P - 1) {                       // h+1 -> h+2 -> ... -> P-1 -> owner: the shorter chain arrives first
            load_strided<R, W, V>(part(h + 1), sp, xv);
            widen_strided<R, V>(xv, t);
            for (int i = h + 2; i <= P - 1; ++i) {
                load_strided<R, W, V>(part(i), sp, xv);
                strided_hop<R, W, V, !kAG>(t, xv, st);
            }
            strided_send_into<R, W, V, !kAG>(t, sum, st);
        }
        if (h >= 1) {                               // h -> h-1 -> ... -> 1 -> owner
            load_strided<R, W, V>(part(h), sp, xv);
            widen_strided<R, V>(xv, t);
            for (int i = h - 1; i >= 1; --i) {
                load_strided<R, W, V>(part(i), sp, xv);
                strided_hop<R, W, V, !kAG>(t, xv, st);
            }
            strided_send_into<R, W, V, !kAG>(t, sum, st);
        }
    } else {
        for (int i = 1; i < P; ++i) {
            // With two waves per piece the partial is requested before anything else of the hop: left to the compiler, 160
            // minishards of 128 chunks take 66.3 us instead of 64.7, P = 16 120.4 instead of 117.4 (176: 71.6 and 72.2, 128.6 and
            // 129.2).  An earlier body of this loop took up to 9 % longer off 8-byte boundaries; this one takes the same time on
            // either, and stays on them (tests/test_build_flags.py).
            constexpr bool kRequestFirst = W == 2 && V == 8;
            if (kRS && kRequestFirst) asm volatile(".p2align 3");
            load_strided<R, W, V>(part(i), sp, xv);
            if (kRequestFirst) loads_first();
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
        store_piece<V>(out + sp.elem + r * kWaveRow<W> + sp.at, d);
    }
}

// The quotients of the lane's V blocks with every lane working out all of them, in exchanges that do not wait for one another:
// more instructions than strided_quotients and, for one send in all, less time.
template <int R, int W, int V>
__device__ __forceinline__ void quotients_in_every_lane(const float (&t)[R][V], ChunkMaxRows<W, V> &red, float (&scale)[V], float (&inv)[V])
{
    float m[V];
    absmax_of_rows(t, m);
#pragma unroll
    for (int j = 0; j < V; ++j) {
        uint32_t v = __float_as_uint(m[j]);
        v = umax(v, dpp_read<0x128>(v));                                    // row_ror:8: lane ^ 8
        auto a = __builtin_amdgcn_permlane16_swap(v, v, false, false);
        v = umax(a[0], a[1]);
        auto b = __builtin_amdgcn_permlane32_swap(v, v, false, false);
        m[j] = __uint_as_float(umax(b[0], b[1]));
    }
    if (W > 1) {
        const int wave = threadIdx.x / 64, at = threadIdx.x % 8 * V;
        if (threadIdx.x % 64 < 8) {
#pragma unroll
            for (int j = 0; j < V; ++j) red.row[0][wave][at + j] = m[j];
        }
        __syncthreads();
#pragma unroll
        for (int w = 1; w < W; ++w) {
#pragma unroll
            for (int j = 0; j < V; ++j) m[j] = larger(m[j], red.row[0][wave ^ w][at + j]);
        }
    }
#pragma unroll
    for (int j = 0; j < V; ++j) block_quotients(m[j], scale[j], inv[j]);
}

// chain_strided_kernel's reduce-scatter in fp32 for the sizes at which that kernel is slower (sums_apart): the partials are
// added and the sum is quantized once.  What bounds it is how the partials stream.  With eight rows a wave asks for two,
// waits for the first and then asks for the other six, so that less of a partial is requested at once; addresses are 64 bits
// per row, which spreads the requests; nothing limits the waves per SIMD.  Measured on MI355X, us, chain_strided_kernel -> this,
// P = 2, 8 and 16: 64 chunks, 192 minishards 13.3, 36.1, 64.0 -> 12.4, 35.6, 61.6; 128 chunks, 96 14.6, 38.0, 68.6 -> 13.0, 35.8,
// 67.7; P = 8 and 16, 64 chunks, 132 29.9, 52.9 -> 27.6, 49.3; P = 2, 32 chunks, 256 9.9 -> 8.7, 128 chunks, 64 9.2 -> 8.5.  With buffer
// loads, all rows at once or the quotients handed round, at most half of that.
template <int R, int W>
__global__ __launch_bounds__(kThreads) void sum_strided_kernel(int P, int per_shard, Global<uint16_t> out, const PartialTable tab)
{
    constexpr int V = 8;
    __shared__ __align__(16) ChunkMaxRows<W, V> red;
    const WaveSpot sp = wave_spot<W, V>(8 * W * R, 0u);
    const int first = per_shard > 0 ? (int)(sp.minishard / (unsigned)per_shard) + 1 : 0;       // as in chain_strided_kernel
    const auto part = [&](int i) {
        const int j = first + i;
        return tab.x[j >= P ? j - P : j];
    };
    const int64_t at = sp.elem + sp.at;

    float sum[R][V];
    Piece<V> xv[R];
    const auto request = [&](const uint16_t *x, int r) {
        xv[r] = __builtin_nontemporal_load(reinterpret_cast<const Piece<V> *>(x + at + r * kWaveRow<W>));
    };
    const auto add = [&](int r) {
        float xf[V];
        widen_piece<V>(xv[r], xf);
#pragma unroll
        for (int j = 0; j < V; ++j) sum[r][j] = sum[r][j] + xf[j];
    };
    {
        const uint16_t *x = part(0);
#pragma unroll
        for (int r = 0; r < R; ++r) request(x, r);
        widen_strided<R, V>(xv, sum);
    }
    for (int i = 1; i < P; ++i) {
        constexpr int kAhead = R == 8 ? 2 : R;
        const uint16_t *x = part(i);
#pragma unroll
        for (int r = 0; r < kAhead; ++r) request(x, r);
        if (kAhead < R) {
            __builtin_amdgcn_sched_barrier(0);
            add(0);
            __builtin_amdgcn_sched_barrier(0);
        }
#pragma unroll
        for (int r = kAhead; r < R; ++r) request(x, r);
        if (kAhead < R) loads_first();
#pragma unroll
        for (int r = kAhead < R ? 1 : 0; r < R; ++r) add(r);
    }

    float scale[V], inv[V];
    quotients_in_every_lane<R, W, V>(sum, red, scale, inv);
#pragma unroll
    for (int r = 0; r < R; ++r) {
        float d[V];
#pragma unroll
        for (int j = 0; j < V; ++j) d[j] = code_of<true>(sum[r][j], inv[j]) * scale[j];
        store_piece<V>(out + at + r * kWaveRow<W>, d);
    }
}

// Dequantize in the strided geometry: element e uses scale (e / (1024*chunks)) * 1024 + e % 1024, so the 8 elements of a
// lane use 8 consecutive scales, the same ones in each of its K tiles.  A workgroup takes T*K*8 consecutive elements of a
// minishard, on the XCD that has it in the passes.
template <int kChunks, int T, int K>
__global__ __launch_bounds__(T) void dequantize_strided_kernel(Global<const int8_t> codes, Global<const float> scales,
                                                               Global<uint16_t> out, unsigned mirror, unsigned owned)
{
    static_assert(tile_elems<T> % kChunk == 0 && kChunk * kChunks % (tile_elems<T> * K) == 0, "whole chunks");
    constexpr int kParts = kChunk * kChunks / (tile_elems<T> * K);
    const MinishardPart place = minishard_part<kParts>(mirrored_place(blockIdx.x, mirror), owned);
    if (place.minishard < 0) return;    // uniform over the workgroup
    const int lane_at = threadIdx.x * kLaneElems;
    const int64_t at = (int64_t)place.minishard * (kChunk * kChunks) + place.part * (tile_elems<T> * K);
    u32x2 cv[K];
#pragma unroll
    for (int k = 0; k < K; ++k) cv[k] = *reinterpret_cast<const u32x2 *>(codes + at + k * tile_elems<T> + lane_at);
    const float *s = scales + (int64_t)place.minishard * kChunk + lane_at % kChunk;
    const u32x4 a = *reinterpret_cast<const u32x4 *>(s);
    const u32x4 b = *reinterpret_cast<const u32x4 *>(s + 4);
    loads_first();
#pragma unroll
    for (int k = 0; k < K; ++k) {
        float qf[8];
        widen_i8x8(cv[k], qf);
        u32x4 w;
        w.x = narrow_bf16x2(qf[0] * __uint_as_float(a.x), qf[1] * __uint_as_float(a.y));
        w.y = narrow_bf16x2(qf[2] * __uint_as_float(a.z), qf[3] * __uint_as_float(a.w));
        w.z = narrow_bf16x2(qf[4] * __uint_as_float(b.x), qf[5] * __uint_as_float(b.y));
        w.w = narrow_bf16x2(qf[6] * __uint_as_float(b.z), qf[7] * __uint_as_float(b.w));
        __builtin_nontemporal_store(w, reinterpret_cast<u32x4 *>(out + at + k * tile_elems<T> + lane_at));
    }
}

}  // namespace equarx
