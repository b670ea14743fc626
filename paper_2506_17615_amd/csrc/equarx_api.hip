// Host side of libequarx: argument validation, kernel selection and launch.
// The C ABI is declared and documented in include/equarx.h.
#include "equarx.h"

#include <atomic>
#include <type_traits>

#include "equarx_device.hpp"
#include "equarx_launch.hpp"
#include "equarx_passes.hpp"
#include "equarx_strided.hpp"

// Wire buffers of equarx_reduce_quantized_static, for callers that cannot allocate: one array per GPU, created
// when the library's code object is loaded on that GPU and held until the process ends.  In host code this name
// is only a handle for hipGetSymbolAddress -- never a device address.
static __device__ __align__(256) unsigned char scratch[EQUARX_STATIC_WORKSPACE_BYTES];

namespace {

using namespace equarx;
using namespace equarx::host;

// The device address of `scratch` on each GPU, resolved on the first call made with that GPU current.
constexpr int kMaxDevices = 64;
std::atomic<unsigned char *> g_scratch_on_device[kMaxDevices];

// EQUARX_OK and the current device's copy of `scratch`, or EQUARX_DEVICE_ERROR.
int static_scratch(unsigned char **ptr)
{
    int device = -1;
    if (hipGetDevice(&device) != hipSuccess || device < 0 || device >= kMaxDevices) return EQUARX_DEVICE_ERROR;
    unsigned char *p = g_scratch_on_device[device].load(std::memory_order_acquire);
    if (!p) {
        void *resolved = nullptr;
        if (hipGetSymbolAddress(&resolved, HIP_SYMBOL(scratch)) != hipSuccess || !resolved) {
            (void)hipGetLastError();
            return EQUARX_DEVICE_ERROR;
        }
        p = static_cast<unsigned char *>(resolved);     // two threads racing here resolve the same address
        g_scratch_on_device[device].store(p, std::memory_order_release);
    }
    *ptr = p;
    return EQUARX_OK;
}

template <int B>
void launch_head(const uint16_t *x0, const uint16_t *x1, int64_t n, int8_t *cout, float *sout, LaunchCtx &ctx)
{
    in_pieces(n, [&](int64_t at, int64_t m) {
        with_pass_shape(m, [&](auto shape) {
            using S = decltype(shape);
            ctx.launch(head_kernel<B, S::K>, grid_for<S>(m), S::T, x0 + at, x1 + at, m, cout + at, sout + at / B,
                       blocks_of(m, B));
        });
    });
}

template <int B>
void launch_tail(const int8_t *cin, const float *sin, const uint16_t *x, int64_t n, uint16_t *out, LaunchCtx &ctx,
                 bool ag, bool backward)
{
    in_pieces(n, [&](int64_t at, int64_t m) {
        with_pass_shape(m, [&](auto shape) {
            using S = decltype(shape);
            ctx.launch(ag ? tail_kernel<B, S::K, true> : tail_kernel<B, S::K, false>, grid_for<S>(m), S::T, cin + at,
                       sin + at / B, x + at, m, out + at, mirrored<S>(m, backward));
        });
    });
}

// P >= 3: [Q_B(x_0) + hop 1], hops 2 .. P-2, [hop P-1 + quantize/dequantize pair]
template <int B>
void launch_fused_ends(const PartialTable &tab, int P, int64_t n, int8_t *c, float *s, uint16_t *out, LaunchCtx &ctx)
{
    launch_head<B>(tab.x[0], tab.x[1], n, c, s, ctx);
    for (int i = 2; i + 1 < P; ++i) launch_hop<B>(c, s, tab.x[i], n, c, s, ctx, false, walks_back(n, i - 1));
    launch_tail<B>(c, s, tab.x[P - 1], n, out, ctx, true, walks_back(n, P - 2));
}

// f(shape, whether every second launch walks back) for the launches over `work_elems` elements in the ring layout, one
// grid row per shard, whose wires are of `wire_elems` (see walks_back).
template <typename F>
void with_ring_shape(int64_t work_elems, int64_t wire_elems, F f)
{
    if (wire_elems >= kTurnFrom) {
        f(WidePass{}, std::true_type{});
    } else {
        with_pass_shape(work_elems, [&](auto shape) { f(shape, std::false_type{}); });
    }
}

// Workgroups per row.
template <typename S, bool kTurns>
inline unsigned ring_grid(int64_t shard_elems)
{
    return kTurns ? (unsigned)ring_groups<S>(shard_elems) : grid_for<S>(shard_elems);
}

// The two wire buffers at the front of a workspace: codes, then scales, each part rounded up to the workspace alignment.
// A chain rewrites one of them in place, but a short one in ring order takes them in turn; the two chains of a semi-loop take
// one each.
struct WireBuffers {
    int8_t *c[2];
    float *s[2];
};

inline WireBuffers carve_workspace(void *workspace, int64_t n, int64_t scales_count)
{
    const size_t codes = round_up((size_t)n, kWorkspaceAlign);
    const size_t scales = round_up((size_t)scales_count * sizeof(float), kWorkspaceAlign);
    char *w = static_cast<char *>(workspace);
    WireBuffers b;
    for (int i = 0; i < 2; ++i) {
        b.c[i] = reinterpret_cast<int8_t *>(w + (size_t)i * (codes + scales));
        b.s[i] = reinterpret_cast<float *>(w + (size_t)i * (codes + scales) + codes);
    }
    return b;
}

// Full loop in ring order, hop by hop: P launches, each over all P shards (one grid row per shard).  Up to kOneRound
// elements two wire buffers take turns, which in this layout is a little faster there than one that is rewritten in place
// (MI355X, us per call, P = 3, 4, 5 and 8, in place -> in turn: 2 M elements of block 256 10.26 -> 9.91, 13.37 -> 13.25,
// 17.11 -> 17.00, 26.87 -> 26.84; 4 M of block 64 13.36 -> 12.98, 17.92 -> 17.59, 22.17 -> 21.72, 36.45 -> 36.00; 4.4 M
// 14.51 -> 14.44, 19.25 -> 19.33, 23.98 -> 23.98, 38.65 -> 38.46; 8 M 20.02 -> 20.10, 26.54 -> 26.82, 32.77 -> 34.01,
// 53.70 -> 54.35).
template <int B>
void launch_ring_hops(const PartialTable &tab, int P, int64_t n, bool ag, const WireBuffers &w, uint16_t *out, LaunchCtx &ctx)
{
    const int other = n <= kOneRound ? 1 : 0;
    const int64_t nb = blocks_of(n, B);
    const int64_t shard_elems = (nb + P - 1) / P * B;       // ceil(nb / P) blocks per shard, as the single launch
    const unsigned gy = (unsigned)P;
    with_ring_shape(n, n, [&](auto shape, auto turns) {
        using S = decltype(shape);
        constexpr bool kTurns = decltype(turns)::value;
        const unsigned gx = ring_grid<S, kTurns>(shard_elems);
        ctx.launch2d(quantize_ring_kernel<B, S::K>, gx, gy, S::T, P, n, shard_elems, w.c[0], w.s[0], tab);
        for (int i = 1; i + 1 < P; ++i) {
            const int from = (i - 1) & other, to = i & other;
            ctx.launch2d(hop_ring_kernel<B, S::K, kTurns>, gx, gy, S::T, w.c[from], w.s[from], P, i, n, shard_elems, w.c[to],
                         w.s[to], tab);
        }
        const int last = (P - 2) & other;
        ctx.launch2d(ag ? tail_ring_kernel<B, S::K, true, kTurns> : tail_ring_kernel<B, S::K, false, kTurns>, gx, gy, S::T,
                     w.c[last], w.s[last], P, P - 1, n, shard_elems, out, tab);
    });
}

static_assert(kMostElems<Shape<1024, 1>> / 8192 * 1024 <= kGridThreads && kMostElems<WidePass> >= kPieceElems, "grid limits");
static_assert(kMaxPartials == EQUARX_MAX_PARTIALS && kMaxBatch == EQUARX_MAX_PARTIALS, "header and device limits differ");

// Shape of a chain launch: the whole tensor in array order, or (ring layout) one grid row per shard.
struct ChainGrid {
    unsigned x, y;
    int64_t shard_elems;
};

template <typename S>
inline ChainGrid chain_grid(int64_t n, int32_t block, int32_t P, bool ring)
{
    ChainGrid g;
    if (ring) {
        const int64_t nb = blocks_of(n, block);
        g.shard_elems = (nb + P - 1) / P * block;           // ceil(nb / P) blocks per shard
        g.x = grid_for<S>(g.shard_elems);
        g.y = (unsigned)P;
    } else {
        g.shard_elems = 0;
        g.x = grid_for<S>(n);
        g.y = 1;
    }
    return g;
}

// Which single-launch calls the latency-shaped small_kernel takes: messages of up to three workgroups per CU, with
// enough partials that requesting them together pays.  The semi-loop, whose code is twice as long, needs enough tiles to
// repay fetching it if its chain is long (or its blocks of 512, which keep it to 8 elements per lane).  Measured on MI355X,
// GPU us per call (captured calls one after the other, inputs cold, block 256), bandwidth kernel (256 x 1) / small_kernel with
// 8 / with 4 elements per lane, full loop:
//                        P = 2                 4                 8                12                16                24                32
//     4,099     1.86/1.99/2.00    2.16/2.13/2.01    2.86/2.66/2.43    3.63/3.51/2.99    4.36/4.08/3.42    5.90/6.36/5.55    7.46/7.49/6.54
//     66 k      2.11/2.11/2.12    2.60/2.39/2.39    4.05/3.04/2.89    6.62/3.84/3.37    8.89/4.38/3.82   12.96/7.12/6.28   17.01/8.23/7.20
//     262 k     2.74/2.46/2.57    3.86/2.70/2.76    5.94/3.34/3.43    8.00/4.06/4.18    9.95/4.66/4.80   14.05/7.72/7.20   18.20/9.11/8.68
//     344 k     2.81/2.45/2.64    4.01/2.76/2.95    6.16/3.52/3.76    8.06/4.30/4.67   10.14/4.85/5.59   14.31/8.20/8.72   18.23/9.55/9.66
//     524 k     3.01/2.61/2.94    4.22/3.01/3.25    6.49/4.09/4.36    8.70/4.96/5.44   11.01/5.74/6.64   15.38/9.06/9.40  20.05/11.14/10.65
//     600 k     3.22/3.04/3.02    4.40/3.45/3.37    6.75/4.60/4.54    8.98/6.24/5.76   11.20/7.35/7.02  15.60/10.91/10.48  20.12/12.18/12.31
//     786 k     3.24/3.20/3.41    4.50/3.58/3.74    6.78/4.87/5.01    9.13/6.78/6.67   11.39/7.64/7.88  16.11/11.26/11.49  20.69/12.66/13.56
//     800 k     3.27/3.23/3.27    4.56/3.58/3.75    6.89/4.89/5.07    9.11/6.73/6.93   11.48/7.65/8.20  16.24/11.39/12.38  20.75/12.65/15.15
//     1.05 M    3.35/3.49/3.70    4.71/3.85/4.12    7.13/5.54/5.95    9.61/7.45/7.80   11.91/8.28/9.39  16.74/13.11/13.90  21.47/15.81/16.86
//     1.07 M    3.41/3.77/3.85    4.78/4.17/4.24    7.23/5.98/6.02    9.62/8.61/8.16   12.06/9.89/9.71  16.93/15.84/14.57  21.93/19.53/17.78
//     1.31 M    3.56/4.10/4.18    5.06/4.50/4.70    7.74/6.36/6.49   10.26/9.39/8.90  12.78/10.33/10.68  18.27/16.64/16.14  23.21/20.17/19.16
//     1.34 M    3.67/4.02/4.33    5.15/4.53/4.76    7.76/6.33/6.59   10.28/9.18/9.22  12.74/10.24/11.15  18.00/16.45/17.00  23.35/20.32/20.19
//     1.57 M    3.79/4.21/4.62    5.27/4.82/5.05    8.10/7.08/7.28  10.85/11.08/10.34  13.54/12.49/12.54  19.00/18.56/18.95  24.46/23.62/23.27
// semi-loop:
//                        P = 4                 5                 8                12                16                17                24
//     4,099     2.45/2.45/2.31    2.69/2.68/2.49    3.31/3.37/3.03    4.20/4.62/4.08    5.16/5.51/4.83    5.38/7.71/6.67    7.02/8.73/7.81
//     66 k      2.89/2.70/2.70    3.13/2.98/2.90    4.46/3.76/3.48    7.13/4.99/4.48    9.45/5.92/5.26   10.07/7.52/6.77   13.74/8.87/7.96
//     262 k     4.10/3.12/3.38    4.63/3.25/3.32    6.21/4.12/4.01    8.37/5.27/5.03   10.50/6.26/5.73   11.00/7.35/6.90   14.78/8.60/8.01
//     344 k     4.20/3.10/3.30    4.72/3.32/3.51    6.36/4.24/4.29    8.50/5.48/5.80   10.70/6.38/6.81   11.21/7.37/7.85   15.12/8.87/9.31
//     524 k     4.42/3.32/3.61    5.02/3.68/3.86    6.84/4.77/4.87    9.10/6.20/6.25   11.62/7.55/7.46   12.20/8.16/8.69   16.19/9.53/9.83
//     600 k     4.41/3.90/3.77    5.02/4.11/3.99    6.85/5.34/5.09    9.11/7.32/6.87   11.65/8.71/8.33  12.19/10.20/9.91  16.32/11.61/11.42
//     786 k     4.56/4.00/4.10    5.20/4.38/4.37    7.02/5.58/5.50    9.57/7.79/7.44   11.97/8.87/8.62  12.59/10.39/10.19  16.93/11.85/11.75
//     800 k     4.59/3.91/4.14    5.22/4.35/4.43    7.06/5.62/5.58    9.54/7.72/7.90   11.92/8.88/9.31  12.49/10.37/11.06  16.84/11.89/12.98
//     1.05 M    4.81/4.22/4.52    5.42/4.56/4.77    7.43/6.24/6.36    9.89/8.40/8.43  12.37/9.79/10.11  12.96/11.16/12.18  17.43/12.84/14.58
//     1.07 M    4.84/4.49/4.59    5.46/4.94/4.89    7.55/6.65/6.49    9.95/9.56/9.07  12.50/10.92/10.79  13.12/13.04/13.28  17.68/15.16/16.03
//     1.31 M    5.15/4.90/5.00    5.71/5.22/5.24    7.96/7.05/6.90  10.52/10.19/9.59  13.20/11.73/11.45  13.86/13.87/13.99  18.80/16.65/16.76
//     1.34 M    5.25/4.93/5.14    5.91/5.21/5.32    8.02/7.12/7.04  10.57/10.05/10.18  13.20/11.63/12.13  13.88/13.88/15.05  18.60/16.61/17.89
//     1.57 M    5.38/5.06/5.35    6.01/5.55/5.65    8.30/7.78/7.61  11.06/11.92/10.94  13.92/13.77/13.35  14.58/15.52/15.98  19.51/19.43/18.90
constexpr int64_t kSmallElems = (int64_t)768 * NarrowPass::kElems;
constexpr int64_t kSmallSemiFrom = (int64_t)32 * NarrowPass::kElems;

inline bool small_chain(int64_t n, int P) { return n <= kSmallElems && P >= 4; }
inline bool small_semi(int64_t n, int P, int32_t block)
{
    return n <= kSmallElems && P >= 5 && (n > kSmallSemiFrom || (P <= 8 && block <= 256));
}

// Do all partials begin on a 128-byte line?
inline bool on_lines(const PartialTable &tab, int P)
{
    uintptr_t bits = 0;
    for (int i = 0; i < P; ++i) bits |= reinterpret_cast<uintptr_t>(tab.x[i]);
    return bits % 128 == 0;
}

// 4 elements per lane instead of 8 (blocks of up to 256): half the arithmetic per hop, twice the waves.  What a message takes
// goes by how many waves its fullest SIMD has (MI355X has 1024), and 8 per lane come in workgroups of four, one per SIMD of
// a CU, so that a SIMD has half of the next even number of the waves that it would have with 4: an odd number of those is
// where 4 wins, an even one where 8 does, as the table shows at 524 k | 600 k, 786 k | 800 k and 1.05 | 1.07 M.  Chains of up
// to 8, which wait for memory more than for arithmetic, gain too little from 4 beyond the first wave.  The semi-loop of up
// to 16, whose steps are longer, does not mind an even number; with more, whose partials come in two requests, three waves are
// the most that pays.  (Full loops of more than 24 in three waves, and of up to 14 in six, are as measured.)  In ring order a
// shard's last workgroup is one of each shard's, so both layouts' workgroups are counted (us, semi-loop of 524 k, block 256, 8
// against 4: P = 17 9.88/8.70, P = 24 11.68/10.10, where 8 per lane have 272 and 264 workgroups and not 256).
//
// The partials begin on 128-byte lines (on_lines).  Those of one tensor that was cut into pieces may not, and then the 512
// bytes that a workgroup of one wave reads of each are five lines for four, the 4 KB of one of four waves 33 for 32.  us, 8 /
// 4 elements per lane, on lines and 16 bytes off them: full loop, P = 12, block 256, 655 k 6.41/5.89 and 6.58/6.33, 1.31 M
// 9.21/8.83 and 9.35/9.88; P = 16, block 64, 786 k 7.29/7.14 and 7.51/7.79, 1.18 M 9.65/9.31 and 9.85/10.68; P = 24, block 256,
// 786 k 11.41/11.50 and 11.54/12.80; semi-loop, P = 8, block 64, 786 k 5.53/5.18 and 5.61/5.64, 1.05 M 6.05/5.92 and 6.11/6.75;
// P = 16, block 256, 786 k 8.93/8.66 and 9.07/9.33, 1.57 M 12.62/13.07 and 12.88/14.49.
constexpr int64_t kOneWaveEach = (int64_t)1024 * SmallShape<4>::kElems;
inline bool small_lanes_of_4(const PartialTable &tab, int64_t n, int32_t block, int P, bool ring, bool semi, bool keeps_wire)
{
    if (n <= kOneWaveEach) return true;
    if (!semi && P <= 8) return false;
    const bool lines = on_lines(tab, P);
    if (semi && P <= 16 && lines) return true;
    const ChainGrid g4 = chain_grid<SmallShape<4>>(n, block, P, ring), g8 = chain_grid<SmallShape<8>>(n, block, P, ring);
    const unsigned wgs = g4.x * g4.y, waves = (wgs + 1023) / 1024;      // 2 .. 6, or a little more
    const bool fewer = waves < (g8.x * g8.y + 255) / 256 * 2;           // in array order: an odd number
    if (semi) return fewer && waves == 3 && (P <= 16 || lines || wgs <= 2560);       // off lines: half a wave at most
    if (!lines) return fewer && waves == 3 && P <= 12;
    return (fewer && (waves == 5 || (waves == 3 && P <= 24))) || (waves == 6 && P <= 14 && !keeps_wire);
}

// Launch shapes of the bandwidth kernels of the single-launch calls.  What a message of a few million elements pays
// for is the last round of workgroups, so each shape is used where its rounds come out even:
//   256 x 1   while that is one round on the chip (2048 workgroups, 4.2 M elements);
//   256 x 2   while that gives no CU more than five (1280 workgroups, 5.2 M elements), where 512 x 2 gives some CUs three
//             of its workgroups and others two: with many partials, whose every hop waits for the slower CUs, it costs
//             up to 8 % (table below);
//   512 x 2   while that is one round (768 workgroups, 6.3 M elements; their registers allow three per CU).  A chain
//             that writes its wire out stores at every hop, and with more than six partials 1024 x 1 does that better,
//             before the one round ends (512 x 2 -> 1024 x 1, P = 2, 4, 8, 12 and 16: 10.0 -> 11.0, 15.0 -> 16.5, 26.2
//             -> 26.1, 39.0 -> 38.8 and 61.5 -> 58.3 us at 6 M elements; 10.3 -> 11.5, 15.4 -> 17.6, 27.1 -> 27.2, 39.7 ->
//             39.6 and 62.0 -> 60.6 at 6.2 M);
//   1024 x 1  above: sixteen waves walk one 16 KiB piece of every partial together, each with a single load in flight;
//   256 x 4   for the chain from 21 M elements on, two waves per SIMD (chain_waves) with all tiles of one partial after the
//             other; blocks of 128 and more hold two pieces of a block per lane (chain_body_paired).  Not for few partials
//             (few_partials): there a workgroup ends soon, and 1024 x 1 overlaps the ends of more of them.  The semi-loop,
//             with its two sums per element, stays at 1024 x 1 (22 M elements: 61.3 us, 78.5 with 256 x 4 and two waves).
// Measured on MI355X, us, P = 8, block 256 (semi-loop: P = 7, block 64):
//     elements      256 x 4   512 x 2   1024 x 1     semi-loop: 256 x 2   512 x 2   1024 x 1
//     5.0 M           18.1      15.5      17.9                     14.3      14.2      16.1
//     6.0 M           18.6      17.1      18.8                     16.5      15.9      17.2
//     6.7 M           21.8      22.0      20.3                     18.7      19.3      18.7
//     7.9 M           22.8      23.9      22.1                     21.7      20.8      20.2
//     8.4 M           31.9      28.2      26.8                     24.4      24.8      23.9
//     12.5 M          36.4      36.4      35.2                     33.2      32.5      31.6
//     16 M            45.4      45.1      44.1                     42.3      40.4      39.9
//     20 M            58.4      56.7      54.9                     52.0      50.1      49.3
//     22 M            60.8      61.4      61.2                     58.0      54.8      55.3
//     33.5 M          90.0      93.9      92.2                     85.2      83.1      81.9
//     88 M           247.5       264       262
// and around the line between 256 x 2 and 512 x 2, 512 x 2 -> 256 x 2:
//     elements      chain, P = 8, B = 256    P = 16, B = 32    semi-loop, P = 8, B = 64    P = 16, B = 512
//     4.25 M             13.9 -> 12.9         25.4 -> 23.7            14.3 -> 13.2           26.5 -> 24.6
//     4.6 M              15.0 -> 13.9         26.8 -> 25.1            15.2 -> 14.1           27.5 -> 25.8
//     5.1 M              15.6 -> 14.9         28.4 -> 27.1            16.0 -> 15.3           28.9 -> 27.6
//     5.6 M              16.8 -> 16.8         30.1 -> 30.7            16.9 -> 17.3           30.7 -> 31.3
constexpr int64_t kFivePerCU = (int64_t)5 * 256 * Shape<256, 2>::kElems;
constexpr int64_t kOneWideRound = (int64_t)768 * Shape<512, 2>::kElems;
constexpr int64_t kPairedFrom = (int64_t)2560 * Shape<1024, 1>::kElems;

// Two or three partials, or up to seven of less than 168 M elements in all (not with a kept wire: four of 33.5 M 84.0 us
// with 256 x 4, 86.4 with 1024 x 1).  Measured on MI355X, us, 256 x 4 -> 1024 x 1, block 32:
//     elements       P = 2            3               4               5               6                7
//     21.5 M      23.1 -> 21.3   30.2 -> 27.8    36.4 -> 34.0    42.7 -> 40.6    49.0 -> 47.0     55.6 -> 53.5
//     33.5 M      33.4 -> 31.3   43.1 -> 40.4    54.0 -> 51.0    63.6 -> 61.6    73.5 -> 73.4     83.3 -> 83.4
//     60 M        59.7 -> 56.7   77.4 -> 75.6
inline bool few_partials(int64_t n, int P, bool keeps_wire)
{
    return P < 4 || (P < 8 && !keeps_wire && P * n <= 8 * kPairedFrom);
}

template <typename F>
void with_chain_shape(int64_t n, int P, bool keeps_wire, F f)
{
    if (n <= kOneRound) {
        f(Shape<256, 1>{});
    } else if (n <= kFivePerCU) {
        f(Shape<256, 2>{});
    } else if (n <= kOneWideRound && (!keeps_wire || P <= 6)) {
        f(Shape<512, 2>{});
    } else if (n <= kPairedFrom || (n <= kMostElems<Shape<1024, 1>> && few_partials(n, P, keeps_wire))) {
        f(Shape<1024, 1>{});
    } else {
        f(Shape<256, 4>{});
    }
}

template <typename F>
void with_semi_shape(int64_t n, F f)
{
    if (n <= kOneRound) {
        f(Shape<256, 1>{});
    } else if (n <= kFivePerCU) {
        f(Shape<256, 2>{});
    } else if (n <= kOneWideRound || n > kMostElems<Shape<1024, 1>>) {
        f(Shape<512, 2>{});
    } else {
        f(Shape<1024, 1>{});
    }
}

template <int B, typename S>
void launch_chain_as(const PartialTable &tab, int P, int64_t n, bool rs, bool ag, bool ring, uint16_t *out,
                    int8_t *wire_codes, float *wire_scales, int64_t c_step, int64_t s_step, LaunchCtx &ctx)
{
    const ChainGrid g = chain_grid<S>(n, B, P, ring);
#define EQUARX_CHAIN(RS, AG, WIRE)                                                                        \
    ctx.launch2d(chain_kernel<B, S::T, S::K, RS, AG, WIRE>, g.x, g.y, S::T, P, n, g.shard_elems, out, wire_codes,        \
                 wire_scales, c_step, s_step, tab)
    if (rs && ag) {
        constexpr KeptWire kLong = wire_through_l2(S::T, S::K) ? kWireThroughL2 : kCachedWire;
        if (!wire_codes) {
            EQUARX_CHAIN(true, true, kNoWire);
        } else if ((reinterpret_cast<uintptr_t>(wire_codes) | (uintptr_t)c_step) % 64 == 0) {
            EQUARX_CHAIN(true, true, kLong);
        } else {
            EQUARX_CHAIN(true, true, kCachedWire);
        }
    } else if (rs) {
        EQUARX_CHAIN(true, false, kNoWire);
    } else {
        EQUARX_CHAIN(false, true, kNoWire);
    }
#undef EQUARX_CHAIN
}

template <int B, int E, bool kSemi, bool kRS, bool kAG, bool kWire>
void launch_small_as(const PartialTable &tab, int P, int64_t n, bool ring, uint16_t *out, int8_t *wire_codes,
                     float *wire_scales, int64_t c_step, int64_t s_step, LaunchCtx &ctx)
{
    const ChainGrid g = chain_grid<SmallShape<E>>(n, B, P, ring);
    ctx.launch2d(P <= 8    ? small_kernel<B, E, 8, false, kSemi, kRS, kAG, kWire>
                 : P <= 16 ? small_kernel<B, E, 16, false, kSemi, kRS, kAG, kWire>
                           : small_kernel<B, E, 16, true, kSemi, kRS, kAG, kWire>,
                 g.x, g.y, SmallShape<E>::T, P, n, g.shard_elems, out, wire_codes, wire_scales, c_step, s_step, tab);
}

template <int B, bool kSemi, bool kRS, bool kAG, bool kWire>
void launch_small(const PartialTable &tab, int P, int64_t n, bool ring, uint16_t *out, int8_t *wire_codes,
                  float *wire_scales, int64_t c_step, int64_t s_step, LaunchCtx &ctx)
{
    if constexpr (B > 256) {            // 4 elements per lane would spread a block over two waves
        launch_small_as<B, 8, kSemi, kRS, kAG, kWire>(tab, P, n, ring, out, wire_codes, wire_scales, c_step, s_step, ctx);
    } else if (small_lanes_of_4(tab, n, B, P, ring, kSemi, kWire)) {
        launch_small_as<B, 4, kSemi, kRS, kAG, kWire>(tab, P, n, ring, out, wire_codes, wire_scales, c_step, s_step, ctx);
    } else {
        launch_small_as<B, 8, kSemi, kRS, kAG, kWire>(tab, P, n, ring, out, wire_codes, wire_scales, c_step, s_step, ctx);
    }
}

template <int B>
void launch_chain(const PartialTable &tab, int P, int64_t n, bool rs, bool ag, bool ring, uint16_t *out,
                  int8_t *wire_codes, float *wire_scales, int64_t c_step, int64_t s_step, LaunchCtx &ctx)
{
    if (small_chain(n, P)) {
        if (rs && ag && wire_codes) {
            launch_small<B, false, true, true, true>(tab, P, n, ring, out, wire_codes, wire_scales, c_step, s_step, ctx);
        } else if (rs && ag) {
            launch_small<B, false, true, true, false>(tab, P, n, ring, out, nullptr, nullptr, 0, 0, ctx);
        } else if (rs) {
            launch_small<B, false, true, false, false>(tab, P, n, ring, out, nullptr, nullptr, 0, 0, ctx);
        } else {
            launch_small<B, false, false, true, false>(tab, P, n, ring, out, nullptr, nullptr, 0, 0, ctx);
        }
    } else {
        with_chain_shape(n, P, wire_codes != nullptr, [&](auto shape) {
            launch_chain_as<B, decltype(shape)>(tab, P, n, rs, ag, ring, out, wire_codes, wire_scales, c_step, s_step, ctx);
        });
    }
}

template <int B>
void launch_semi(const PartialTable &tab, int P, int64_t n, bool ag, bool ring, uint16_t *out, LaunchCtx &ctx)
{
    if (small_semi(n, P, B)) {
        if (ag) {
            launch_small<B, true, true, true, false>(tab, P, n, ring, out, nullptr, nullptr, 0, 0, ctx);
        } else {
            launch_small<B, true, true, false, false>(tab, P, n, ring, out, nullptr, nullptr, 0, 0, ctx);
        }
        return;
    }
    with_semi_shape(n, [&](auto shape) {
        using S = decltype(shape);
        const ChainGrid g = chain_grid<S>(n, B, P, ring);
        if (ag) {
            ctx.launch2d(semi_kernel<B, S::T, S::K, true>, g.x, g.y, S::T, P, n, g.shard_elems, out, tab);
        } else {
            ctx.launch2d(semi_kernel<B, S::T, S::K, false>, g.x, g.y, S::T, P, n, g.shard_elems, out, tab);
        }
    });
}

// f(shape, how many received wires to request at a time) for a flat reduce of R wires over n elements: see flat_body.
template <typename F>
void with_flat_shape(int64_t n, int R, F f)
{
    using std::integral_constant;
    if (n > kOneRound) {
        f(WidePass{}, integral_constant<int, 1>{});
    } else if (R <= 2) {
        f(NarrowPass{}, integral_constant<int, 2>{});
    } else if (R <= 4) {
        f(NarrowPass{}, integral_constant<int, 4>{});
    } else {
        f(NarrowPass{}, integral_constant<int, 8>{});
    }
}

// The owner's launch of a semi-loop: at most two wires, from this device, kept cacheable.
template <int B>
void launch_flat_owner(const uint16_t *local, const WireTable &tab, int R, int64_t n, uint16_t *out, LaunchCtx &ctx, bool ag,
                       bool backward)
{
    with_flat_shape(n, 2, [&](auto shape, auto batch) {
        using S = decltype(shape);
        constexpr int U = decltype(batch)::value;
        if constexpr (U <= 2) {
            if (ag) {
                ctx.launch(flat_kernel<B, S::K, U, true, false, true, false>, grid_for<S>(n), S::T, local, R, n, out,
                           nullptr, nullptr, mirrored<S>(n, backward), tab);
            } else {
                ctx.launch(flat_kernel<B, S::K, U, true, false, false, false>, grid_for<S>(n), S::T, local, R, n, out,
                           nullptr, nullptr, mirrored<S>(n, backward), tab);
            }
        }
    });
}

// The per-step entry points are what a device calls once per step of a collective: equarx_quantize,
// equarx_reduce_stage and equarx_dequantize in a ring, equarx_quantize_batch and equarx_reduce_flat around an
// all-to-all.  The wire they read came from another device and the wire they write goes to one, so they access it
// with non-temporal hints.  The chain entry points, which run every step on this device, know that the next launch
// reads what this one wrote and keep the wire cacheable.
constexpr bool kWireLeavesTheDevice = true;

template <int B>
void launch_flat(const uint16_t *local, const WireTable &tab, int R, int64_t n, uint16_t *out, int8_t *codes_out,
                 float *scales_out, LaunchCtx &ctx)
{
    in_pieces(n, [&](int64_t at, int64_t m) {
        WireTable part = tab;
        for (int r = 0; at > 0 && r < R; ++r) {
            part.codes[r] += at;
            part.scales[r] += at / B;
        }
        uint16_t *o = out ? out + at : nullptr;
        int8_t *co = codes_out ? codes_out + at : nullptr;
        float *so = codes_out ? scales_out + at / B : nullptr;
        with_flat_shape(m, R, [&](auto shape, auto batch) {
            using S = decltype(shape);
            constexpr int U = decltype(batch)::value;
            constexpr bool kStream = kWireLeavesTheDevice;
            ctx.launch(o && co ? flat_kernel<B, S::K, U, true, true, true, kStream>
                       : o     ? flat_kernel<B, S::K, U, true, false, true, kStream>
                               : flat_kernel<B, S::K, U, false, true, true, kStream>,
                       grid_for<S>(m), S::T, local + at, R, m, o, co, so, 0, part);
        });
    });
}

// The output of a chain may BE one of the partials (in-place reduction: every
// kernel reads an element of every partial before the thread that owns the
// element writes it, and in the hop-by-hop schedules the output is written by
// the last launch only): partials and output carry this tag, so the output may
// coincide with a partial exactly and may not overlap one in any other way.
constexpr int kInPlace = 1;

// Validates the P device pointers of a chain call and lists them as read.
inline int check_partials(const void *const *partials_bf16, int32_t P, int64_t n, Aliasing &mem)
{
    for (int32_t i = 0; i < P; ++i) {
        if (!partials_bf16[i]) return EQUARX_NULL_POINTER;
        if (misaligned(partials_bf16[i], kAlign)) return EQUARX_MISALIGNED;
        mem.reads(partials_bf16[i], (size_t)n * sizeof(uint16_t), kInPlace);
    }
    return EQUARX_OK;
}

// ... and copies them into the kernel's table.
inline int fill_table(const void *const *partials_bf16, int32_t P, int64_t n, Aliasing &mem, PartialTable &tab)
{
    if (int st = check_partials(partials_bf16, P, n, mem)) return st;
    for (int32_t i = 0; i < P; ++i) tab.x[i] = static_cast<const uint16_t *>(partials_bf16[i]);
    for (int32_t i = P; i < kMaxPartials; ++i) tab.x[i] = tab.x[i - P];     // small_kernel reads on around the ring
    return EQUARX_OK;
}

// Semi-loop in ring order, hop by hop: h = P/2 launches in which both chains of every shard advance one device
// (grid row = shard, grid layer = direction), then the owners' launch.  Direction d rewrites wire buffer d in place.
//
// The owners' launch takes the steps' shape, and a layer's workgroups are a multiple of eight, so that a tile is on the
// same XCD in either direction and in every launch: that XCD's L2 may hold the wire, and another one has to wait for it.
// Measured on MI355X, us per call, block 64, with the owners' own shape and rows without padding -> as it is:
//     elements     P = 2             3               4               5               8
//     1 M       6.71 ->  6.17    6.83 ->  6.54  10.31 ->  9.63  10.44 -> 10.10  16.58 -> 16.52
//     2 M       7.89 ->  7.37    8.38 ->  8.20  12.42 -> 11.83  13.22 -> 12.72  20.91 -> 20.84
//     3 M       9.97 ->  8.21   11.87 ->  9.97  16.11 -> 14.26  17.60 -> 16.15  26.97 -> 25.12
//     4 M      11.14 ->  9.06   14.25 -> 11.47  19.50 -> 15.97  21.49 -> 19.30  33.08 -> 29.72
//     6 M      14.01 -> 11.24   17.02 -> 14.90  20.47 -> 20.29  27.13 -> 24.19  38.45 -> 38.08
//     8 M      17.32 -> 13.60   21.99 -> 18.53  29.66 -> 25.56  33.13 -> 29.31  47.27 -> 47.02
// Rows of a single workgroup are padded for an odd P only: 4096 elements, P = 5 6.33 -> 5.59, but P = 4 5.82 -> 6.22.
template <int B>
void launch_semi_ring_hops(const PartialTable &tab, int P, int64_t n, bool ag, const WireBuffers &w, uint16_t *out,
                           LaunchCtx &ctx)
{
    const int64_t nb = blocks_of(n, B);
    const int64_t shard_elems = (nb + P - 1) / P * B;       // ceil(nb / P) blocks per shard, as the single launch
    const unsigned gy = (unsigned)P;
    const int h = P / 2, count[2] = {P - 1 - h, h};
    const WirePair wire = {{w.c[0], w.c[1]}, {w.s[0], w.s[1]}};
    WireTable wires;
    for (int r = 0; r < kMaxPartials; ++r) {
        wires.codes[r] = nullptr;
        wires.scales[r] = nullptr;
    }
    int received = 0;
    for (int d = 0; d < 2; ++d) {       // counter-clockwise first, as the single launch adds them
        if (count[d] == 0) continue;
        wires.codes[received] = w.c[d];
        wires.scales[received] = w.s[d];
        ++received;
    }
    // two shards' worth of work per shard: one per direction.  With one step no wire is rewritten, and nothing turns (P = 2,
    // 21 M elements 32.9 -> 32.6 us, 42 M 61.1 -> 60.3).
    with_ring_shape(2 * n, h > 1 ? 2 * n : 0, [&](auto shape, auto turns) {
        using S = decltype(shape);
        constexpr bool kTurns = decltype(turns)::value;
        constexpr int U = S::K == 1 ? 2 : 1;            // received wires to request at a time, as with_flat_shape
        unsigned gx = ring_grid<S, kTurns>(shard_elems);
        const unsigned unit = P & 1 ? 8 : P & 2 ? 4 : P & 4 ? 2 : 1;        // P rows of a multiple of this are one of eight
        if (gx > 1 || (P & 1) != 0) gx = (gx + unit - 1) & ~(unit - 1);
        for (int t = 0; t < h; ++t) {
            ctx.launch3d(semi_ring_step_kernel<B, S::K, kTurns>, gx, gy, 2u, S::T, P, t, n, shard_elems, wire, tab);
        }
        if (ag) {
            ctx.launch2d(semi_ring_owner_kernel<B, S::K, U, true, kTurns>, gx, gy, S::T, P, n, shard_elems, received, out, wires, tab);
        } else {
            ctx.launch2d(semi_ring_owner_kernel<B, S::K, U, false, kTurns>, gx, gy, S::T, P, n, shard_elems, received, out, wires, tab);
        }
    });
}

// ---- strided (Sec. 3.2) geometry ----

inline int check_strided(int64_t n, int32_t chunks)
{
    if (chunks != 32 && chunks != 64 && chunks != 128) return EQUARX_BAD_BLOCK;
    if (n < 0 || too_long(n) || n % ((int64_t)kChunk * chunks) != 0) return EQUARX_BAD_SHAPE;
    return EQUARX_OK;
}

#define EQUARX_DISPATCH_CHUNKS(chunks, CALL) \
    switch (chunks) {                        \
        case 32: CALL(32); break;            \
        case 64: CALL(64); break;            \
        case 128: CALL(128); break;          \
        default: break;                      \
    }

inline int64_t minishards_of(int64_t n, int32_t chunks) { return n / ((int64_t)kChunk * chunks); }

// f(layout) with the layout of the per-pass kernels: 16 lanes across a slice, where a code piece is a whole line and a thread
// has 2, 4 or 8 rows.  8 lanes for few minishards of 64 and 128 chunks, which otherwise leave CUs idle.  32 for many of 32
// chunks, and of 64 if the workgroups that gives are a whole number per CU (256), or over half of the next: every workgroup
// is resident, so the slowest CU counts.  Measured on MI355X, us (GPU time of captured calls), hop-by-hop chain of P = 8 and
// semi-loop in ring order of P = 8, 8 / 16 / 32 lanes:
//     minishards       32 chunks                                   64                                          128
//     1        19.4/18.0/20.4   12.3/11.1/13.1     20.5/20.3/27.2   13.3/13.4/17.1     26.6/29.3/39.4   16.7/18.4/24.4
//     8        21.8/22.0/23.3   13.8/14.0/14.8     23.1/24.4/29.7   15.0/15.8/18.8     27.9/31.2/41.5   18.5/20.5/26.8
//     16       22.2/22.8/24.0   14.8/14.7/15.6     24.3/25.1/30.5   17.2/17.3/20.2     30.5/33.0/43.6   22.3/22.9/29.2
//     24       24.8/23.4/24.6   16.9/15.7/16.3     29.2/26.8/32.0   20.4/19.5/21.3     38.8/36.3/46.5   28.2/26.9/31.1
//     64       29.2/27.9/27.8   22.0/20.4/20.5     37.7/36.4/37.4   32.3/29.0/29.5     62.6/52.8/59.5   53.5/45.0/47.4
//     128      38.9/35.3/36.1   33.7/28.8/27.8     61.6/52.7/52.2   53.5/45.4/43.8      111/92.9/97.0   98.0/87.1/87.6
//     160           40.1/41.7        33.2/32.4          62.9/64.2        55.1/53.5           112/122          107/111
//     192           44.0/43.9        37.8/35.8          73.1/70.7        64.9/62.6           133/140          129/129
//     256           53.5/52.0        46.6/44.1          93.2/90.0        87.6/84.3           170/176          169/168
//     272           57.0/57.1        50.3/48.8          99.0/99.9        92.6/92.4           178/193          180/182
//     320           63.5/61.7        58.2/54.0         112.3/108.8      107.8/106.2
//     400           77.4/76.8        71.0/69.0         135.5/138.4      133.9/135.1
//     544           97.3/97.2        91.7/93.7         176.7/177.8      178.3/176.6
// What they replace (32 lanes, every value computed twice, and up to 16 minishards the chain's layout, which is 8 lanes) took
// 22.8, 27.5, 30.6 | 37.5, 44.7, 65.3 | 81.7, 98.2, 117.7 us for 1, 8, 16 | 24, 64, 128 | 192, 256, 320 minishards of 64 chunks.
// From 2^35 elements on a minishard of 64 chunks takes 32 lanes whatever the rounds: half as many workgroups, because a launch
// holds fewer than 2^32 threads, and with 16 lanes a step of the semi-loop had that many at 2^36 elements, which the card's
// memory holds if the partials are one tensor.  (128 chunks reach it at 2^37, where the wires alone take 2^38 bytes and a
// partial as much again: no card of 288 GiB holds them.)
template <typename F>
inline void with_slices(int64_t n, int32_t chunks, F f)
{
    const int64_t ms = minishards_of(n, chunks);
    switch (chunks) {
        case 32:
            if (ms < 192) f(Slices<32, 16>{});
            else f(Slices<32, 32>{});
            break;
        case 64:
            if (ms <= 16) f(Slices<64, 8>{});
            else if (ms < 128 || ((4 * ms - 1) % 256 < 128 && n < (int64_t)1 << 35)) f(Slices<64, 16>{});
            else f(Slices<64, 32>{});
            break;
        case 128:
            if (ms <= 16) f(Slices<128, 8>{});
            else f(Slices<128, 16>{});
            break;
        default: break;
    }
}

// f(layout) with the layout of the owner's kernel: that of the other passes, but of 128 chunks 32 lanes where 16 would give more
// than three and at most four workgroups per CU.  A workgroup there reads its own values first and then the wires, and the
// fourth of a CU does so after the others.  Measured on MI355X, us per call, 16 -> 32 lanes in this launch, semi-loop and full loop in
// ring order, P = 2 and 3: 96 minishards 18.7 -> 19.7, 18.5 -> 19.5, 27.5 -> 28.1, 26.5 -> 28.9; 97 21.7 -> 20.2, 21.2 -> 20.0, 30.2 -> 28.0, 30.6 ->
// 30.7; 112 23.5 -> 21.6, 23.2 -> 21.7, 33.2 -> 30.7, 32.7 -> 32.9; 128 25.1 -> 24.1, 24.9 -> 23.9, 35.7 -> 34.7, 35.3 -> 35.6; 140 28.7 -> 28.9, 28.4 ->
// 28.9, 40.3 -> 41.3, 40.5 -> 42.3.  An owner that is `alone`, with no wire to wait for, has 32 lanes from 96 minishards of 64 chunks and
// 80 of 128 on: 64 chunks, 64 minishards 4.13 -> 4.14, 96 5.27 -> 4.72, 120 5.87 -> 5.47, 160 8.5 -> 7.4, 128 chunks, 64 6.04 -> 5.87, 80 8.68 ->
// 8.18, 112 12.2 -> 9.2, 170 18.0 -> 16.8, 192 19.4 -> 19.0, 256 25.1 -> 24.7.
template <typename F>
inline void with_owner_slices(int64_t n, int32_t chunks, bool alone, F f)
{
    const int64_t ms = minishards_of(n, chunks);
    if (chunks == 128 && ((ms > 96 && ms <= 128) || (alone && ms >= 80))) f(Slices<128, 32>{});
    else if (chunks == 64 && alone && ms >= 96) f(Slices<64, 32>{});
    else with_slices(n, chunks, f);
}

// The places of a launch that go to the XCDs by whole minishards (minishard_part), for the wire that it writes or reads.  `spread`
// (short_and_long): none.
template <typename S>
inline unsigned strided_owned(int64_t n, const void *wire, bool spread)
{
    return spread ? 0u : owned_places<S::kChunks, S::kParts>(minishards_of(n, S::kChunks), wire);
}

// The flavours hop by hop of few partials, where the wire is rewritten twice at most and runs gain the least, keep the parts of
// a minishard on all XCDs from 10 Mi elements on: two partials of 64 and up to four of 128 chunks, but three and four not where
// the owner has 32 lanes (with_owner_slices; semi-loop, 104 minishards, 29.6 -> 28.7 and 40.3 -> 38.4 with runs).  Measured on MI355X, us, runs
// -> all XCDs, semi-loop and full loop in ring order, means over four places in memory:
//     chunks, elements     P = 2                          3                              4
//     128, 10.5 M      17.8 -> 16.5, 16.4 -> 16.2     25.2 -> 24.4, 24.6 -> 24.2     32.0 -> 31.3, 32.6 -> 32.2
//          12.6 M      20.0 -> 18.6, 18.9 -> 18.5     29.1 -> 27.5, 27.7 -> 26.6     37.1 -> 35.7, 36.5 -> 35.5
//          14.7 M      21.9 -> 21.6, 22.2 -> 21.7     30.4 -> 30.7, 32.2 -> 32.9     40.6 -> 41.8, 42.6 -> 42.5
//          16.8 M      24.8 -> 24.1, 24.5 -> 23.9     34.5 -> 34.7, 34.7 -> 35.6     45.7 -> 46.3, 45.3 -> 46.0
//          25.2 M      38.1 -> 37.4, 38.0 -> 37.3     53.3 -> 52.0, 54.1 -> 53.4     69.5 -> 68.6, 69.2 -> 69.2
//          33.6 M      48.3 -> 47.7, 48.0 -> 47.2     68.0 -> 65.8, 69.0 -> 69.0     89.7 -> 88.3, 89.4 -> 90.7
//     64,  10.5 M      17.1 -> 15.6, 15.9 -> 15.4     24.9 -> 24.6, 23.5 -> 23.0     32.0 -> 31.3, 31.4 -> 30.5
//          13.1 M      21.5 -> 20.9, 21.1 -> 20.6     29.8 -> 30.5, 30.3 -> 29.6     38.6 -> 39.0, 39.7 -> 38.9
//          16.8 M      25.4 -> 25.3, 25.1 -> 25.1     35.9 -> 36.3, 35.2 -> 34.7     45.9 -> 46.5, 45.5 -> 45.6
//          19.7 M      29.9 -> 29.5, 29.6 -> 29.3     41.9 -> 43.1, 42.0 -> 41.8     54.8 -> 55.7, 54.3 -> 54.0
// (32 chunks, P = 2, 8.4 M 12.2 -> 12.8, 12.2 -> 12.7; 64 chunks, P = 2, 4.2 and 8.4 M 8.0 -> 9.3, 12.5 -> 12.7.)  One partial has no wire
// that an XCD could keep: spread from 7 Mi elements on, 32 chunks, 5.2 M 4.3 -> 4.7, 6.3 M 4.9 -> 4.9, 8.4 M 6.0 -> 5.7, 10.5 M 7.8 -> 7.5, 13.1 M
// 10.3 -> 10.0, 64 chunks, 16.8 M 12.8 -> 12.0, 128 chunks, 21 M 16.3 -> 16.1.
inline bool short_and_long(int32_t chunks, int64_t n, int P)
{
    if (P == 1) return n >= (int64_t)7 << 20;
    const int64_t ms = minishards_of(n, chunks);
    return n >= (int64_t)10 << 20 && ((chunks == 64 && P == 2) || (chunks == 128 && (P == 2 || (P <= 4 && (ms <= 96 || ms > 128)))));
}

template <typename S>
inline unsigned strided_count(int64_t n) { return (unsigned)(minishards_of(n, S::kChunks) * S::kParts); }

template <typename S>
inline unsigned strided_grid(int64_t n, unsigned owned) { return strided_count<S>(n) + missing_minishards(owned) * S::kParts; }

// The first workgroups of a grid, in whole groups of eight, that a launch takes in the opposite order (mirrored_place).
inline unsigned strided_mirror(unsigned grid, bool backward) { return backward ? grid & ~7u : 0; }

// A strided chain rewrites one wire in place to its end: the dequantization takes every tile on the XCD that wrote it, and
// finds it in that L2.  A last hop that writes beside the wire it reads costs (MI355X, us, P = 2, 3, 4 and 8, in place ->
// beside) 8.8 -> 8.8, 12.0 -> 11.9, 15.1 -> 15.3, 28.0 -> 28.3 at 2.1 M elements of 32 chunks, 21.4 -> 22.6, 29.6 -> 30.9, 36.9 -> 38.2,
// 68.7 -> 70.6 at 12.6 M of 64, 34.2 -> 38.7, 46.7 -> 52.0, 59.5 -> 64.5, 111.3 -> 116.5 at 22 M.  Which of the workspace's buffers it is
// makes no difference to the time, and the header promises nothing about it: up to 3 Mi elements and from 9 to 28 Mi the second,
// where such a chain has always left its last wire and where tests/test_launch_shapes_gpu.py looks for it.
inline int strided_chain_buffer(int64_t n, int P)
{
    return P > 1 && (n <= (int64_t)3 << 20 || (n >= (int64_t)9 << 20 && n <= (int64_t)28 << 20)) ? 1 : 0;
}

// What a per-pass strided kernel reads of bf16: partial `offset` of a table, or in the ring layout (per_shard minishards
// per shard) the partial of device (k + offset) mod P for every shard k at once.
struct StridedSource {
    const PartialTable &tab;
    int P, per_shard, offset;
};

inline Global<const uint16_t> one_tensor(const void *x) { return static_cast<const uint16_t *>(x); }

// floor(m / d) = umulhi(2 m, magic) >> shift for all m < 2^30: magic = ceil(2^(32 + shift) / (2 d)) with 2^shift <= 2 d <
// 2^(shift + 1) is off by less than a part in 2^31.  (2 d a power of two would need 2^32: half of that, and one bit less.)
struct RingDivision {
    unsigned magic, shift;
};

inline RingDivision ring_division(int d)
{
    if (d <= 0) return {0, 0};      // array order: every minishard in shard 0
    const uint64_t twice = 2 * (uint64_t)d;
    unsigned shift = 0;
    while (twice >> (shift + 1)) ++shift;
    if ((twice & (twice - 1)) == 0) return {1u << 31, shift - 1};
    return {(unsigned)(((((uint64_t)1 << (32 + shift)) + twice - 1)) / twice), shift};
}

inline unsigned ring_word(int P, unsigned shift, int offset, int second = 0)
{
    return (unsigned)P | (unsigned)offset << 8 | (unsigned)second << 16 | shift << 24;
}

// f(the source as a kernel takes it): see strided_source.
template <typename F>
inline void with_source(const StridedSource &src, F f)
{
    if (src.per_shard == 0) {
        f(Global<const uint16_t>(src.tab.x[src.offset]));
    } else {
        const RingDivision by = ring_division(src.per_shard);
        f(by.magic, ring_word(src.P, by.shift, src.offset), src.tab);
    }
}

template <typename... Source>
void do_quantize_strided(int64_t n, int32_t chunks, int8_t *codes, float *scales, LaunchCtx &ctx, bool spread, Source... src)
{
    with_slices(n, chunks, [&](auto slices) {
        using S = decltype(slices);
        const unsigned owned = strided_owned<S>(n, codes, spread);
        ctx.launch(quantize_strided_kernel<S, Source...>, strided_grid<S>(n, owned), kThreads, codes, scales, owned, src...);
    });
}

template <typename... Source>
void do_hop_strided(const int8_t *cin, const float *sin, int64_t n, int32_t chunks, int8_t *cout, float *sout, LaunchCtx &ctx,
                    bool backward, bool spread, Source... src)
{
    with_slices(n, chunks, [&](auto slices) {
        using S = decltype(slices);
        const unsigned owned = strided_owned<S>(n, cout, spread), grid = strided_grid<S>(n, owned);
        ctx.launch(hop_strided_kernel<S, Source...>, grid, kThreads, cin, sin, cout, sout, strided_mirror(grid, backward), owned, src...);
    });
}

// Step t of the semi-loop's two chains, the first device of one at `up` and of the other at `down` from the owner.
void do_semi_step_strided(const WireBuffers &w, const PartialTable &tab, int P, int per_shard, int up, int down, bool first, int64_t n,
                          int32_t chunks, LaunchCtx &ctx, bool backward, bool spread)
{
    const RingDivision by = ring_division(per_shard);
    with_slices(n, chunks, [&](auto slices) {
        using S = decltype(slices);
        const unsigned count = strided_count<S>(n);
        const unsigned owned0 = strided_owned<S>(n, w.c[0], spread), owned1 = strided_owned<S>(n, w.c[1], spread);
        ctx.launch(semi_step_strided_kernel<S>, 2 * semi_step_half<S>(count, owned0, owned1), kThreads, w.c[0], w.s[0], w.c[1], w.s[1],
                   by.magic, ring_word(P, by.shift, up, down), count, owned0, owned1, (backward ? 1 : 0) | (first ? 2 : 0), tab);
    });
}

// The wires that the owner received; nullptr: none.
struct StridedWires {
    const int8_t *codes[2];
    const float *scales[2];
};

template <bool kAG, typename... Source>
void do_owner_strided(const StridedWires &in, int64_t n, int32_t chunks, uint16_t *out, LaunchCtx &ctx, bool backward, bool spread,
                      Source... src)
{
    with_owner_slices(n, chunks, !in.codes[0], [&](auto slices) {
        using S = decltype(slices);
        const unsigned owned = strided_owned<S>(n, in.codes[1] ? in.codes[1] : in.codes[0], spread), grid = strided_grid<S>(n, owned);
        ctx.launch(owner_strided_kernel<S, kAG, Source...>, grid, kThreads, out, in.codes[0], in.scales[0], in.codes[1],
                   in.scales[1], strided_mirror(grid, backward), owned, src...);
    });
}

// The single-launch chain and its flavours: chunks = 8 * W * R (see chain_strided_kernel).
template <int R, int W, int V, int kWaves>
void launch_chain_strided_as(const PartialTable &tab, int P, int64_t minishards, int per_shard, bool semi, bool rs, bool ag,
                             uint16_t *out, LaunchCtx &ctx)
{
    const unsigned grid = (unsigned)(minishards * wave_layout_wgs<W, V>);
    // Runs of minishards to an XCD (minishard_part), though nothing is read twice here, where the partials stream better so: at
    // 32 chunks with the cap beyond the first round, and for sums in fp32 in the middle of its second half; at 128 chunks from 96
    // minishards on, except that where they are just two rounds more than four partials, and sums in fp32, do not.  MI355X, us, parts
    // of a minishard on all XCDs -> runs; P = 8 and 16: 64 chunks, 128 minishards 23.1 -> 24.4, 41.0 -> 44.1, 336 61.0 -> 62.9, 111.5 ->
    // 117.9; 32 chunks, 672 62.6 -> 60.8, 113.7 -> 112.9, 1000 90.1 -> 88.9 (400, without the cap, 37.3 -> 38.0, 68.4 -> 70.7).
    // 32 chunks, P = 2, 3, 4 and 8:
    //     minishards   full loop                                               sums in fp32
    //     64       3.31 -> 3.62, 4.25 -> 4.66, 5.34 -> 5.51, 9.16 -> 9.12     3.36 -> 3.32, 4.10 -> 4.41, 5.21 -> 5.58, 8.57 -> 8.73
    //     96       5.04 -> 4.80, 5.76 -> 5.79, 6.92 -> 7.00, 10.9 -> 10.7     4.72 -> 4.29, 5.33 -> 5.20, 6.74 -> 6.65, 10.4 -> 10.2
    //     128      5.25 -> 5.75, 6.44 -> 6.85, 7.70 -> 7.97, 12.7 -> 12.7     4.79 -> 5.53, 6.29 -> 6.82, 7.51 -> 7.92, 12.5 -> 12.4
    // 128 chunks, means over four places in memory, P = 2, 4, 8 and 16 (semi-loop and sums: P = 8):
    //     minishards   full loop                                               semi-loop        sums in fp32
    //     64                                   25.2 -> 25.8, 45.5 -> 47.3
    //     97       15.7 -> 15.1, 24.5 -> 23.5, 41.8 -> 40.1, 77.0 -> 74.3     43.0 -> 40.8     42.2 -> 38.8
    //     104      16.8 -> 16.6, 25.9 -> 25.7, 44.0 -> 43.9, 81.4 -> 79.3     44.6 -> 45.4     43.8 -> 44.2
    //     112      17.5 -> 17.2, 27.0 -> 26.8, 45.9 -> 46.0, 84.9 -> 84.7     46.3 -> 47.4     45.7 -> 46.3
    //     128      18.8 -> 19.0, 29.0 -> 29.2, 49.8 -> 51.2, 93.6 -> 95.5     50.0 -> 51.9     49.3 -> 50.9
    //     136      20.9 -> 20.4, 33.2 -> 33.0, 59.3 -> 59.5,  113 -> 114      59.1 -> 59.9     56.5 -> 57.1
    //     160      23.0 -> 23.0, 36.2 -> 36.0, 63.6 -> 63.9,  124 -> 122      64.5 -> 65.2     64.6 -> 62.9
    //     256      35.5 -> 34.5, 58.1 -> 55.4,  103 -> 101,   195 -> 186       103 -> 101       103 -> 100
    constexpr int kChunks = 8 * W * R;
    const bool two_rounds = minishards >= 112 && minishards <= 128;
    const bool between = !rs && minishards > 72 && minishards < 120;
    const bool own = V == 8 && ((kChunks == 32 && kWaves == 2 && (minishards > 128 || between)) ||
                                (kChunks == 128 && minishards >= 96 && !(two_rounds && (P > 4 || !rs))));
    const unsigned owned = own ? owned_places<kChunks, wave_layout_wgs<W, V>>(minishards, nullptr) : 0u;
#define EQUARX_CHAIN(SEMI, RS, AG) \
    ctx.launch(chain_strided_kernel<R, W, V, SEMI, RS, AG, kWaves>, grid, kThreads, P, per_shard, out, owned, tab)
    constexpr bool kSemi = kChunks != 64 || V != 8 || W != 1 || kWaves == 2;        // the semi-loop comes here too
    if (kSemi && semi && ag) EQUARX_CHAIN(kSemi, true, true);
    else if (kSemi && semi) EQUARX_CHAIN(kSemi, true, false);
    else if (rs && ag) EQUARX_CHAIN(false, true, true);
    else if (rs) EQUARX_CHAIN(false, true, false);
    else EQUARX_CHAIN(false, false, true);
#undef EQUARX_CHAIN
}

// Which reduce-scatters in fp32 of `wgs` workgroups are sum_strided_kernel's: between one and one and a half rounds of the chip
// at two workgroups per CU, where the chain's kernel is left with a round that is half empty, and for two partials, where there
// is one addition in all, up to two.  Measured on MI355X, us, chain's kernel / this one:
//     chunks, minishards (rounds)   P = 2          3             4             6             8             16
//     32, 128 (1)                 5.50/4.46
//         160 (1.25)              5.90/5.68    7.88/7.89    9.47/9.97    13.0/13.3      16.6/16.7     28.9/29.1
//         192 (1.5)               6.68/7.05
//         200 (1.6)               8.30/7.28   10.32/9.83   12.30/12.35   16.25/16.21     20.1/20.7     35.5/36.7
//         224 (1.75)              9.03/8.95                13.03/13.98
//         256 (2)                 9.94/8.70   12.33/11.45  14.75/14.45   19.31/18.67     24.0/24.6     42.5/42.2
//         336 (2.6)               12.5/12.2    15.7/15.8    19.0/19.3     25.4/26.5      31.6/32.5     56.7/63.7
//     64, 112 (0.9)               8.18/8.02    10.3/10.2    12.8/12.7     17.1/16.9      21.1/21.5     39.2/37.7
//         132 (1.03)              10.4/10.2                              23.5/21.7      29.9/27.6     52.9/49.3
//         144 (1.1)               10.5/11.0    13.9/13.9    17.0/17.0     23.6/22.8      30.2/28.6     57.7/53.3
//         160 (1.25)              11.4/11.3    14.6/15.1    17.9/18.1     24.4/24.1      31.6/30.5     60.2/55.1
//         176 (1.4)               12.6/11.9    15.7/16.1    19.1/19.6     26.4/26.7      32.8/32.6     64.0/61.6
//         192 (1.5)               13.3/12.4    16.7/15.8    20.5/21.0     28.3/28.0      36.1/35.6     64.0/61.6
//         200 (1.6)               14.5/14.7    19.3/19.9    23.6/24.9     30.8/31.9      40.8/42.8     76.1/79.0
//     128, 56 (0.9)               8.41/7.90                                                            41.4/39.4
//         64 (1)                  9.24/8.48    11.6/11.6    14.0/14.8     18.9/19.7      24.0/24.4     43.3/43.3
//         72 (1.1)                11.4/11.4    15.0/14.8    18.1/18.0     24.9/24.5      32.0/31.1     59.4/56.9
//         96 (1.5)                14.6/13.0    18.0/17.4    22.0/21.7     30.6/29.2      38.0/35.8     68.6/67.7
//         112 (1.75)              17.2/16.9    21.6/22.2    26.5/27.6     36.8/36.6      46.3/47.8     84.9/88.9
//         128 (2)                 19.1/18.2    23.4/24.2    29.5/28.9     40.1/40.6      50.5/49.5     93.2/89.8
inline bool sums_apart(int32_t chunks, int64_t wgs, int P)
{
    switch (chunks) {
        case 32: return wgs <= 1024 && ((P <= 3 && wgs > 768) || (P == 2 && wgs >= 512 && wgs <= 640));
        case 64: return wgs <= 768 && (P == 2 ? wgs > 640 : P >= 6 ? wgs > 512 : P >= 4 && wgs > 512 && wgs <= 544);
        case 128: return wgs > (P == 2 || P > 8 ? 384 : 512) && wgs <= (P == 2 ? 1024 : 768);
        default: return false;
    }
}

// Few minishards take layouts whose waves have an eighth, a quarter or half of the work, so that every CU has some; where
// those are a round of the chip, the largest, which does least in all, is faster.  Measured on MI355X, us (GPU time of
// captured calls), full loop of P = 8, chunks = 8 W R as R x W x V:
//     minishards of 32    1x4x4 / 4x1x8     of 64    2x4x4 / 2x4x8 / 8x1x8     of 128    4x4x4 / 4x4x8 / 8x2x8
//     5                       6.6/                       7.6/7.5/                            8.6/8.7/
//     8                       6.8/8.3                    7.9/7.9/                            9.9/9.1/
//     12                      7.3/8.4                    9.0/8.1/                           13.2/9.4/12.8
//     20                      8.2/8.6                   10.6/9.0/10.3                       20.8/13.0/14.4
//     24                      8.8/8.7                   11.5/9.4/                           21.9/13.6/14.9
//     32                      9.5/8.9                   15.5/10.5/                          29.6/15.1/16.0
//     40                     10.1/9.0                   19.3/15.7/12.6                           19.4/20.0
//     48                                                     16.8/14.1                           21.6/21.8
//     64                                                     18.0/14.6                           28.8/25.0
// 128 chunks by the partials (P = 2, 3, 4, 8, 16): 8 minishards, 4x4x4 / 4x4x8 2.6/2.9, 4.0/4.5, 4.7/5.3, 8.0/8.5, 14.6/15.1 (and
// 15.7/15.1 another time), reduce-scatter in fp32 3.2/3.5, 3.9/4.3, 4.7/5.1, 8.7/8.0, 14.9/13.7, 9 full loop 3.1/3.3, 4.9/4.6, 6.3/5.4,
// 10.6/8.6, 19.5/15.2.  Up to 32 minishards 8x2x8, a workgroup per CU at most, is the faster for the
// reduce-scatter in fp32, where one send is all, and for two partials from 25: 4x4x8 / 8x2x8, fp32, 18 minishards 4.5/4.2, 5.9/5.1,
// 6.7/6.1, 11.6/9.8, 20.0/17.0, 32 5.9/4.9, 7.6/6.2, 8.9/7.3, 13.7/12.9, 24.1/22.4 (16: P = 4 5.5/6.3); full loop, 24 4.9/5.0, 6.2/6.4,
// 7.6/8.0, 32 6.1/5.7, 7.5/7.1, 8.7/8.7, 13.4/15.8; semi-loop, 32 5.8/5.4, 7.3/7.7.
// ring: shards of ceil(minishards / P) whole minishards, shard k in the order a ring gives it.
void launch_chain_strided(const PartialTable &tab, int P, int64_t n, int32_t chunks, bool semi, bool rs, bool ag,
                          bool ring, uint16_t *out, LaunchCtx &ctx)
{
    const int64_t ms = minishards_of(n, chunks);
    const int per_shard = ring ? (int)((ms + P - 1) / P) : 0;
    const int64_t wgs = ms * wave_layout_wgs<1, 8>;
    // see chain_strided_kernel's kWaves
    const int64_t last = (wgs - 1) % 512 + 1;       // workgroups of the last round
    const bool short_round = wgs > 512 && wgs < 2048 && last <= (wgs < 1024 || !rs || P <= 4 ? 256 : 128);
    const bool half_round = !semi && wgs > (rs ? 720 : 640) && wgs <= 768;
    if (!rs && sums_apart(chunks, chunks == 128 ? 2 * wgs : wgs, P)) {
#define EQUARX_SUM(R, W) ctx.launch(sum_strided_kernel<R, W>, (unsigned)(ms * wave_layout_wgs<W, 8>), kThreads, P, per_shard, out, tab)
        if (chunks == 32) EQUARX_SUM(4, 1);
        else if (chunks == 64) EQUARX_SUM(8, 1);
        else EQUARX_SUM(8, 2);
#undef EQUARX_SUM
        return;
    }
#define EQUARX_LAYOUT(...) launch_chain_strided_as<__VA_ARGS__>(tab, P, ms, per_shard, semi, rs, ag, out, ctx)
    switch (chunks) {
        case 32:
            if (ms <= 20) EQUARX_LAYOUT(1, 4, 4, 8);
            else if (short_round || (semi && P <= 4 && wgs > 512)) EQUARX_LAYOUT(4, 1, 8, 8);
            else EQUARX_LAYOUT(4, 1, 8, 2);
            break;
        case 64:
            if (ms <= 8) EQUARX_LAYOUT(2, 4, 4, 8);
            else if (ms <= 32) EQUARX_LAYOUT(2, 4, 8, 2);
            else if (half_round) EQUARX_LAYOUT(8, 1, 8, 8);
            else EQUARX_LAYOUT(8, 1, 8, 2);
            break;
        case 128:
            if (ms <= 6 || (ms <= 8 && P <= (rs ? 8 : 4))) EQUARX_LAYOUT(4, 4, 4, 8);
            else if (ms <= 32 && (rs ? P == 2 && ms > 24 : ms > 16)) EQUARX_LAYOUT(8, 2, 8, 2);
            else if (ms <= 48) EQUARX_LAYOUT(4, 4, 8, 4);
            else EQUARX_LAYOUT(8, 2, 8, 2);
            break;
        default: break;
    }
#undef EQUARX_LAYOUT
}

template <int kChunks, int T, int K>
void launch_dequantize_strided(const int8_t *codes, const float *scales, int64_t minishards, uint16_t *out,
                               LaunchCtx &ctx, bool backward)
{
    constexpr int kParts = kChunk * kChunks / (tile_elems<T> * K);
    const unsigned owned = owned_places<kChunks, kParts>(minishards, codes);
    const unsigned grid = (unsigned)(minishards * kParts) + missing_minishards(owned) * kParts;
    ctx.launch(dequantize_strided_kernel<kChunks, T, K>, grid, T, codes, scales, out, strided_mirror(grid, backward), owned);
}

// 256 threads x 4 tiles, where a lane reads its scales once for 32 elements; 2 while that leaves CUs without work.  Measured on
// MI355X, us, 256 x 1 / 256 x 2 / 256 x 4, three wires and outputs in turn, and one:
//     elements, chunks
//     0.5 M, 64       1.97/1.98/1.99     1.98/1.96/1.98
//     1.0 M, 64       2.04/2.08/2.04     2.05/2.08/2.07
//     2.1 M, 64       2.20/2.14/2.31     2.31/2.26/2.34
//     3.1 M, 64       2.44/2.37/2.44     2.55/2.44/2.46
//     4.2 M, 32       2.62/2.46/2.69     2.69/2.51/2.70
//     5.2 M, 64       3.00/2.70/2.96     2.93/2.73/2.99
//     5.8 M, 32       3.14/2.84/3.02     3.07/2.80/3.08
//     6.3 M, 32       3.24/3.01/3.24     3.18/2.99/3.31
//     6.3 M, 128      3.21/3.03/3.27     3.21/2.99/3.31
//     7.3 M, 32       4.06/3.84/3.50     3.53/3.34/3.53
//     8.4 M, 64       3.83/3.70/3.82     3.62/3.59/3.73
//     14.7 M, 64      11.0/9.77/9.32
//     22 M, 64        14.7/13.5/13.0
//     62.9 M, 32      36.9/32.6/32.3
// (512 x 2 is between the last two, and 256 x 1 or 512 x 2 took 3.1, 3.6 and 4.8 us at 5.2, 6.3 and 7.3 M with one instance for
// every number of chunks, which divided by it per lane, and each load behind a condition.)
constexpr int64_t kTwoTileDequantize = (int64_t)6 << 20;

void do_dequantize_strided(const int8_t *codes, const float *scales, int64_t n, int32_t chunks, void *out,
                           LaunchCtx &ctx, bool backward = false)
{
    in_pieces(n, [&](int64_t at, int64_t m) {
        uint16_t *o = static_cast<uint16_t *>(out) + at;
        const int64_t minishards = m / ((int64_t)kChunk * chunks);
#define CALL(CC)                                                                                                            \
    do {                                                                                                                    \
        const float *sc = scales + at / CC;                                                                                 \
        if (m <= kTwoTileDequantize) launch_dequantize_strided<CC, 256, 2>(codes + at, sc, minishards, o, ctx, backward);     \
        else launch_dequantize_strided<CC, 256, 4>(codes + at, sc, minishards, o, ctx, backward);                            \
    } while (0)
        EQUARX_DISPATCH_CHUNKS(chunks, CALL)
#undef CALL
    });
}

}  // namespace

extern "C" {

int64_t equarx_num_blocks(int64_t n, int32_t block)
{
    if (check_shape(n, block) != EQUARX_OK) return 0;
    return blocks_of(n, block);
}

int64_t equarx_wire_row_codes(int64_t n)
{
    return n < 0 ? 0 : (int64_t)round_up((size_t)n, kAlign);
}

int64_t equarx_wire_row_scales(int64_t n, int32_t block)
{
    if (check_shape(n, block) != EQUARX_OK) return 0;
    return (int64_t)round_up((size_t)blocks_of(n, block), kAlign / sizeof(float));
}

size_t equarx_workspace_bytes(int32_t P, int64_t n, int32_t block)
{
    if (P < 1 || P > EQUARX_MAX_PARTIALS || check_shape(n, block) != EQUARX_OK) return 0;
    const size_t codes = round_up((size_t)n, kWorkspaceAlign);
    const size_t scales = round_up((size_t)blocks_of(n, block) * sizeof(float), kWorkspaceAlign);
    return 2 * (codes + scales);
}

const char *equarx_status_string(int status)
{
    switch (status) {
        case EQUARX_OK: return "ok";
        case EQUARX_NULL_POINTER: return "a required pointer is NULL";
        case EQUARX_BAD_SHAPE: return "bad shape: n < 0, P out of range, or forbidden overlap of buffers";
        case EQUARX_BAD_BLOCK: return "block size must be 32, 64, 128, 256 or 512";
        case EQUARX_MISALIGNED: return "a data pointer is not 16-byte aligned";
        case EQUARX_WORKSPACE_TOO_SMALL:
            return "workspace (the caller's, or the static array of equarx_reduce_quantized_static) is smaller than the "
                   "call needs: see equarx_workspace_bytes() / equarx_variant_workspace_bytes()";
        case EQUARX_DEVICE_ERROR: return "the HIP runtime reported an error at kernel launch";
        default: return "unknown status";
    }
}

int equarx_quantize(const void *x_bf16, int64_t n, int32_t block, int8_t *codes, float *scales, void *stream)
{
    LaunchCtx ctx(stream);
    if (int st = check_shape(n, block)) return st;
    if (n == 0) return EQUARX_OK;
    if (!x_bf16 || !codes || !scales) return EQUARX_NULL_POINTER;
    if (misaligned(x_bf16, kAlign) || misaligned(codes, kAlign) || misaligned(scales, kAlign)) return EQUARX_MISALIGNED;
    Aliasing mem;
    mem.reads(x_bf16, (size_t)n * 2);
    mem.writes(codes, (size_t)n);
    mem.writes(scales, (size_t)blocks_of(n, block) * sizeof(float));
    if (int st = mem.check()) return st;
    do_quantize(x_bf16, n, block, codes, scales, ctx, kWireLeavesTheDevice);
    return ctx.status();
}

int equarx_quantize_batch(const void *const *x_bf16, int8_t *const *codes, float *const *scales, int32_t count,
                          int64_t n, int32_t block, void *stream)
{
    LaunchCtx ctx(stream);
    if (int st = check_shape(n, block)) return st;
    if (count < 0 || count > kMaxBatch) return EQUARX_BAD_SHAPE;
    if (count == 0 || n == 0) return EQUARX_OK;
    if (!x_bf16 || !codes || !scales) return EQUARX_NULL_POINTER;
    QuantizeBatch tab;
    for (int32_t i = 0; i < kMaxBatch; ++i) {
        tab.x[i] = nullptr;
        tab.codes[i] = nullptr;
        tab.scales[i] = nullptr;
    }
    Aliasing mem;
    const size_t scale_bytes = (size_t)blocks_of(n, block) * sizeof(float);
    for (int32_t i = 0; i < count; ++i) {
        if (!x_bf16[i] || !codes[i] || !scales[i]) return EQUARX_NULL_POINTER;
        if (misaligned(x_bf16[i], kAlign) || misaligned(codes[i], kAlign) || misaligned(scales[i], kAlign))
            return EQUARX_MISALIGNED;
        mem.reads(x_bf16[i], (size_t)n * 2);
        mem.writes(codes[i], (size_t)n);
        mem.writes(scales[i], scale_bytes);
        tab.x[i] = static_cast<const uint16_t *>(x_bf16[i]);
        tab.codes[i] = codes[i];
        tab.scales[i] = scales[i];
    }
    if (int st = mem.check()) return st;      // two tensors sharing an output, or an output inside an input
    in_pieces(n, [&](int64_t at, int64_t m) {
        for (int32_t i = 0; at > 0 && i < count; ++i) {
            tab.x[i] += kPieceElems;
            tab.codes[i] += kPieceElems;
            tab.scales[i] += kPieceElems / block;
        }
#define CALL(BB)                                                                                                  \
    with_pass_shape(count * m, [&](auto shape) {                                                                  \
        using S = decltype(shape);                                                                                \
        ctx.launch2d(quantize_batch_kernel<BB, S::K, kWireLeavesTheDevice>, grid_for<S>(m), (unsigned)count,    \
                     S::T, m, blocks_of(m, BB), tab);                                                             \
    })
        EQUARX_DISPATCH_BLOCK(block, CALL)
#undef CALL
    });
    return ctx.status();
}

int equarx_dequantize(const int8_t *codes, const float *scales, int64_t n, int32_t block, void *out_bf16,
                      void *stream)
{
    LaunchCtx ctx(stream);
    if (int st = check_shape(n, block)) return st;
    if (n == 0) return EQUARX_OK;
    if (!codes || !scales || !out_bf16) return EQUARX_NULL_POINTER;
    if (misaligned(codes, kAlign) || misaligned(scales, kAlign) || misaligned(out_bf16, kAlign)) return EQUARX_MISALIGNED;
    Aliasing mem;
    mem.reads(codes, (size_t)n);
    mem.reads(scales, (size_t)blocks_of(n, block) * sizeof(float));
    mem.writes(out_bf16, (size_t)n * 2);
    if (int st = mem.check()) return st;
    do_dequantize(codes, scales, n, block, out_bf16, ctx, kWireLeavesTheDevice);
    return ctx.status();
}

// What a hop reads and writes: the wire may be updated in place (codes over codes, scales over scales, each
// coinciding exactly); nothing else may share memory with what is written.
static int check_hop_memory(const int8_t *codes_in, const float *scales_in, const void *local_bf16, int64_t n,
                            int64_t scales_count, const int8_t *codes_out, const float *scales_out)
{
    Aliasing mem;
    mem.reads(codes_in, (size_t)n, 1);
    mem.reads(scales_in, (size_t)scales_count * sizeof(float), 2);
    mem.reads(local_bf16, (size_t)n * 2);
    mem.writes(codes_out, (size_t)n, 1);
    mem.writes(scales_out, (size_t)scales_count * sizeof(float), 2);
    return mem.check();
}

int equarx_reduce_stage(const int8_t *codes_in, const float *scales_in, const void *local_bf16, int64_t n,
                        int32_t block, int8_t *codes_out, float *scales_out, void *stream)
{
    LaunchCtx ctx(stream);
    if (int st = check_shape(n, block)) return st;
    if (n == 0) return EQUARX_OK;
    if (!codes_in || !scales_in || !local_bf16 || !codes_out || !scales_out) return EQUARX_NULL_POINTER;
    if (misaligned(codes_in, kAlign) || misaligned(scales_in, kAlign) || misaligned(local_bf16, kAlign) ||
        misaligned(codes_out, kAlign) || misaligned(scales_out, kAlign))
        return EQUARX_MISALIGNED;
    if (int st = check_hop_memory(codes_in, scales_in, local_bf16, n, blocks_of(n, block), codes_out, scales_out)) return st;
    do_hop(codes_in, scales_in, local_bf16, n, block, codes_out, scales_out, ctx, kWireLeavesTheDevice);
    return ctx.status();
}

int equarx_reduce_quantized(const void *const *partials_bf16, int32_t P, int64_t n, int32_t block, void *out_bf16,
                            void *workspace, size_t workspace_bytes, int8_t *wire_codes, float *wire_scales,
                            void *stream)
{
    LaunchCtx ctx(stream);
    if (int st = check_shape(n, block)) return st;
    if (P < 1 || P > EQUARX_MAX_PARTIALS) return EQUARX_BAD_SHAPE;
    if (!partials_bf16) return EQUARX_NULL_POINTER;
    if (n == 0) return EQUARX_OK;
    if (!out_bf16) return EQUARX_NULL_POINTER;
    if ((wire_codes == nullptr) != (wire_scales == nullptr)) return EQUARX_NULL_POINTER;
    const bool keep_wire = wire_codes != nullptr;
    if (!keep_wire && !workspace) return EQUARX_NULL_POINTER;
    if (misaligned(out_bf16, kAlign)) return EQUARX_MISALIGNED;
    Aliasing mem;
    if (int st = check_partials(partials_bf16, P, n, mem)) return st;
    mem.writes(out_bf16, (size_t)n * 2, kInPlace);
    const int64_t nb = blocks_of(n, block);
    WireBuffers w{};
    int64_t c_step = 0, s_step = 0;     // from one wire to the next: rows when they are kept, in place otherwise
    if (keep_wire) {
        if (misaligned(wire_codes, kAlign) || misaligned(wire_scales, kAlign)) return EQUARX_MISALIGNED;
        c_step = equarx_wire_row_codes(n);
        s_step = equarx_wire_row_scales(n, block);
        mem.writes(wire_codes, (size_t)P * c_step);
        mem.writes(wire_scales, (size_t)P * s_step * sizeof(float));
    } else {
        if (misaligned(workspace, kWorkspaceAlign)) return EQUARX_MISALIGNED;
        const size_t need = equarx_workspace_bytes(P, n, block);
        if (workspace_bytes < need) return EQUARX_WORKSPACE_TOO_SMALL;
        mem.writes(workspace, need);
        w = carve_workspace(workspace, n, nb);
    }
    if (int st = mem.check()) return st;

    int8_t *c = keep_wire ? wire_codes : w.c[0];
    float *sc = keep_wire ? wire_scales : w.s[0];
    do_quantize(partials_bf16[0], n, block, c, sc, ctx);
    for (int32_t i = 1; i < P; ++i) {
        int8_t *c_next = c + c_step;
        float *s_next = sc + s_step;
        do_hop(c, sc, partials_bf16[i], n, block, c_next, s_next, ctx, false, !keep_wire && walks_back(n, i));
        c = c_next;
        sc = s_next;
    }
    do_dequantize(c, sc, n, block, out_bf16, ctx, false, !keep_wire && walks_back(n, P));
    return ctx.status();
}

int equarx_reduce_quantized_static(const void *const *partials_bf16, int32_t P, int64_t n, int32_t block,
                                   void *out_bf16, void *stream)
{
    LaunchCtx ctx(stream);
    if (int st = check_shape(n, block)) return st;
    if (P < 1 || P > EQUARX_MAX_PARTIALS) return EQUARX_BAD_SHAPE;
    if (!partials_bf16) return EQUARX_NULL_POINTER;
    if (n == 0) return EQUARX_OK;
    if (!out_bf16) return EQUARX_NULL_POINTER;
    if (misaligned(out_bf16, kAlign)) return EQUARX_MISALIGNED;
    if (equarx_workspace_bytes(P, n, block) > (size_t)EQUARX_STATIC_WORKSPACE_BYTES) return EQUARX_WORKSPACE_TOO_SMALL;
    Aliasing mem;
    if (int st = check_partials(partials_bf16, P, n, mem)) return st;
    mem.writes(out_bf16, (size_t)n * 2, kInPlace);
    if (int st = mem.check()) return st;
    unsigned char *wire = nullptr;
    if (int st = static_scratch(&wire)) return st;
    // Nothing in the array has to start at zero: pass 0 writes the wire buffer completely before hop 1 reads it,
    // and every later hop reads only what the launch before it wrote.
    const WireBuffers w = carve_workspace(wire, n, blocks_of(n, block));
    do_quantize(partials_bf16[0], n, block, w.c[0], w.s[0], ctx);
    for (int32_t i = 1; i < P; ++i) {
        do_hop(w.c[0], w.s[0], partials_bf16[i], n, block, w.c[0], w.s[0], ctx, false, walks_back(n, i));
    }
    do_dequantize(w.c[0], w.s[0], n, block, out_bf16, ctx, false, walks_back(n, P));
    return ctx.status();
}

int equarx_reduce_quantized_fused_ends(const void *const *partials_bf16, int32_t P, int64_t n, int32_t block,
                                       void *out_bf16, void *workspace, size_t workspace_bytes, void *stream)
{
    LaunchCtx ctx(stream);
    if (int st = check_shape(n, block)) return st;
    if (P < 1 || P > EQUARX_MAX_PARTIALS) return EQUARX_BAD_SHAPE;
    if (!partials_bf16) return EQUARX_NULL_POINTER;
    if (n == 0) return EQUARX_OK;
    if (!out_bf16) return EQUARX_NULL_POINTER;
    if (misaligned(out_bf16, kAlign)) return EQUARX_MISALIGNED;
    PartialTable tab;
    Aliasing mem;
    if (int st = fill_table(partials_bf16, P, n, mem, tab)) return st;
    mem.writes(out_bf16, (size_t)n * 2, kInPlace);
    uint16_t *out = static_cast<uint16_t *>(out_bf16);
    if (P <= 2) {       // both ends meet: the chain is one launch and needs no wire
        if (int st = mem.check()) return st;
#define CALL(BB) launch_chain<BB>(tab, P, n, true, true, false, out, nullptr, nullptr, 0, 0, ctx)
        EQUARX_DISPATCH_BLOCK(block, CALL)
#undef CALL
        return ctx.status();
    }
    if (!workspace) return EQUARX_NULL_POINTER;
    if (misaligned(workspace, kWorkspaceAlign)) return EQUARX_MISALIGNED;
    const size_t need = equarx_workspace_bytes(P, n, block);
    if (workspace_bytes < need) return EQUARX_WORKSPACE_TOO_SMALL;
    mem.writes(workspace, need);
    if (int st = mem.check()) return st;
    const WireBuffers w = carve_workspace(workspace, n, blocks_of(n, block));
#define CALL(BB) launch_fused_ends<BB>(tab, P, n, w.c[0], w.s[0], out, ctx)
    EQUARX_DISPATCH_BLOCK(block, CALL)
#undef CALL
    return ctx.status();
}

int equarx_reduce_fused(const void *const *partials_bf16, int32_t P, int64_t n, int32_t block, void *out_bf16,
                        int8_t *wire_codes, float *wire_scales, void *stream)
{
    LaunchCtx ctx(stream);
    if (int st = check_shape(n, block)) return st;
    if (P < 1 || P > EQUARX_MAX_PARTIALS) return EQUARX_BAD_SHAPE;
    if (!partials_bf16) return EQUARX_NULL_POINTER;
    if (n == 0) return EQUARX_OK;
    if (!out_bf16) return EQUARX_NULL_POINTER;
    if ((wire_codes == nullptr) != (wire_scales == nullptr)) return EQUARX_NULL_POINTER;
    if (misaligned(out_bf16, kAlign)) return EQUARX_MISALIGNED;
    if (wire_codes && (misaligned(wire_codes, kAlign) || misaligned(wire_scales, kAlign))) return EQUARX_MISALIGNED;
    PartialTable tab;
    Aliasing mem;
    if (int st = fill_table(partials_bf16, P, n, mem, tab)) return st;
    const int64_t c_step = equarx_wire_row_codes(n);
    const int64_t s_step = equarx_wire_row_scales(n, block);
    mem.writes(out_bf16, (size_t)n * 2, kInPlace);
    mem.writes(wire_codes, (size_t)P * c_step);
    mem.writes(wire_scales, (size_t)P * s_step * sizeof(float));
    if (int st = mem.check()) return st;
#define CALL(BB)                                                                                               \
    launch_chain<BB>(tab, P, n, true, true, false, static_cast<uint16_t *>(out_bf16), wire_codes, wire_scales, \
                     c_step, s_step, ctx)
    EQUARX_DISPATCH_BLOCK(block, CALL)
#undef CALL
    return ctx.status();
}

int equarx_reduce_variant(const void *const *partials_bf16, int32_t P, int64_t n, int32_t block, uint32_t flags,
                          void *out_bf16, void *stream)
{
    LaunchCtx ctx(stream);
    if (int st = check_shape(n, block)) return st;
    if (P < 1 || P > EQUARX_MAX_PARTIALS) return EQUARX_BAD_SHAPE;
    const uint32_t known = EQUARX_SEMI_LOOP | EQUARX_RS_UNQUANTIZED | EQUARX_AG_UNQUANTIZED | EQUARX_RING_ORDER;
    if (flags & ~known) return EQUARX_BAD_SHAPE;
    const bool semi = flags & EQUARX_SEMI_LOOP, rs = !(flags & EQUARX_RS_UNQUANTIZED);
    const bool ag = !(flags & EQUARX_AG_UNQUANTIZED), ring = flags & EQUARX_RING_ORDER;
    if (!rs && !ag) return EQUARX_BAD_SHAPE;        // nothing quantized: not this library's business
    if (semi && !rs) return EQUARX_BAD_SHAPE;       // the semi-loop is a reduce-scatter schedule
    if (!partials_bf16) return EQUARX_NULL_POINTER;
    if (n == 0) return EQUARX_OK;
    if (!out_bf16) return EQUARX_NULL_POINTER;
    if (misaligned(out_bf16, kAlign)) return EQUARX_MISALIGNED;
    PartialTable tab;
    Aliasing mem;
    if (int st = fill_table(partials_bf16, P, n, mem, tab)) return st;
    mem.writes(out_bf16, (size_t)n * 2, kInPlace);
    if (int st = mem.check()) return st;
    uint16_t *out = static_cast<uint16_t *>(out_bf16);
    if (semi) {
#define CALL(BB) launch_semi<BB>(tab, P, n, ag, ring, out, ctx)
        EQUARX_DISPATCH_BLOCK(block, CALL)
#undef CALL
    } else {
#define CALL(BB) launch_chain<BB>(tab, P, n, rs, ag, ring, out, nullptr, nullptr, 0, 0, ctx)
        EQUARX_DISPATCH_BLOCK(block, CALL)
#undef CALL
    }
    return ctx.status();
}

size_t equarx_variant_workspace_bytes(uint32_t flags, int32_t P, int64_t n, int32_t block)
{
    const size_t two = equarx_workspace_bytes(P, n, block);
    if (!(flags & EQUARX_SEMI_LOOP)) return two;
    // sized for two buffers per chain that is under way, and one for a wire that waits: three, in ring order four.  The
    // chains rewrite one buffer each in place (kTurnFrom), so the launches use the first two.
    return (flags & EQUARX_RING_ORDER) ? two * 2 : two / 2 * 3;
}

int equarx_reduce_variant_hops(const void *const *partials_bf16, int32_t P, int64_t n, int32_t block, uint32_t flags,
                               void *out_bf16, void *workspace, size_t workspace_bytes, void *stream)
{
    LaunchCtx ctx(stream);
    if (int st = check_shape(n, block)) return st;
    if (P < 1 || P > EQUARX_MAX_PARTIALS) return EQUARX_BAD_SHAPE;
    if (flags & ~(uint32_t)(EQUARX_SEMI_LOOP | EQUARX_AG_UNQUANTIZED | EQUARX_RING_ORDER)) return EQUARX_BAD_SHAPE;
    const bool semi = flags & EQUARX_SEMI_LOOP, ag = !(flags & EQUARX_AG_UNQUANTIZED);
    const bool ring = flags & EQUARX_RING_ORDER;
    if (!partials_bf16) return EQUARX_NULL_POINTER;
    if (n == 0) return EQUARX_OK;
    if (!out_bf16 || !workspace) return EQUARX_NULL_POINTER;
    if (misaligned(out_bf16, kAlign) || misaligned(workspace, kWorkspaceAlign)) return EQUARX_MISALIGNED;
    const size_t need = equarx_variant_workspace_bytes(flags, P, n, block);
    if (workspace_bytes < need) return EQUARX_WORKSPACE_TOO_SMALL;
    PartialTable tab;
    Aliasing mem;
    if (int st = fill_table(partials_bf16, P, n, mem, tab)) return st;
    mem.writes(out_bf16, (size_t)n * 2, kInPlace);
    mem.writes(workspace, need);
    if (int st = mem.check()) return st;

    const WireBuffers w = carve_workspace(workspace, n, blocks_of(n, block));
    int8_t *const c = w.c[0];
    float *const s = w.s[0];
    uint16_t *out = static_cast<uint16_t *>(out_bf16);

    if (semi && ring) {     // every launch is one semi-loop iteration of the ring on all P shards, both directions
#define CALL(BB) launch_semi_ring_hops<BB>(tab, P, n, ag, w, out, ctx)
        EQUARX_DISPATCH_BLOCK(block, CALL)
#undef CALL
        return ctx.status();
    }
    if (!semi) {
        if (P == 1) {       // no hop: one launch quantizes/dequantizes (or copies) partial 0
#define CALL(BB) launch_chain<BB>(tab, P, n, true, ag, ring, out, nullptr, nullptr, 0, 0, ctx)
            EQUARX_DISPATCH_BLOCK(block, CALL)
#undef CALL
            return ctx.status();
        }
        if (ring) {         // every launch is one ring step on all P shards: grid row k takes device k+1+step's partial
#define CALL(BB) launch_ring_hops<BB>(tab, P, n, ag, w, out, ctx)
            EQUARX_DISPATCH_BLOCK(block, CALL)
#undef CALL
            return ctx.status();
        }
        // Q_B(x_0), hops 1 .. P-2, then the last hop with or without the all-gather's quantize/dequantize pair
        do_quantize(tab.x[0], n, block, c, s, ctx);
        for (int32_t i = 1; i + 1 < P; ++i) do_hop(c, s, tab.x[i], n, block, c, s, ctx, false, walks_back(n, i));
#define CALL(BB) launch_tail<BB>(c, s, tab.x[P - 1], n, out, ctx, ag, walks_back(n, P - 1))
        EQUARX_DISPATCH_BLOCK(block, CALL)
#undef CALL
        return ctx.status();
    }

    // Semi-loop (Sec. 3.3): partial 0 owns the result; the counter-clockwise chain h+1, ..., P-1 and the clockwise
    // chain h, h-1, ..., 1 each run hop by hop and end in a wire the owner receives; the owner adds them to its
    // own shard, counter-clockwise first.
    const int32_t h = P / 2, count[2] = {P - 1 - h, h};
    WireTable wires;
    for (int32_t r = 0; r < kMaxPartials; ++r) {
        wires.codes[r] = nullptr;
        wires.scales[r] = nullptr;
    }
    int32_t received = 0;
    for (int32_t d = 0; d < 2; ++d) {
        if (count[d] == 0) continue;
        const int32_t first = d == 0 ? h + 1 : h, step = d == 0 ? 1 : -1;
        do_quantize(tab.x[first], n, block, w.c[d], w.s[d], ctx);
        for (int32_t k = 1; k < count[d]; ++k) {
            do_hop(w.c[d], w.s[d], tab.x[first + k * step], n, block, w.c[d], w.s[d], ctx, false, walks_back(n, k));
        }
        wires.codes[received] = w.c[d];
        wires.scales[received] = w.s[d];
        ++received;
    }
#define CALL(BB) launch_flat_owner<BB>(tab.x[0], wires, received, n, out, ctx, ag, walks_back(n, h))
    EQUARX_DISPATCH_BLOCK(block, CALL)
#undef CALL
    return ctx.status();
}

int equarx_reduce_flat(const void *local_bf16, const int8_t *const *codes, const float *const *scales, int32_t R,
                       int64_t n, int32_t block, void *out_bf16, int8_t *codes_out, float *scales_out, void *stream)
{
    LaunchCtx ctx(stream);
    if (int st = check_shape(n, block)) return st;
    if (R < 0 || R >= EQUARX_MAX_PARTIALS) return EQUARX_BAD_SHAPE;
    if (R > 0 && (!codes || !scales)) return EQUARX_NULL_POINTER;
    if (n == 0) return EQUARX_OK;
    if (!local_bf16) return EQUARX_NULL_POINTER;
    if ((codes_out == nullptr) != (scales_out == nullptr)) return EQUARX_NULL_POINTER;
    if (!out_bf16 && !codes_out) return EQUARX_NULL_POINTER;                    // nothing to write
    if (misaligned(local_bf16, kAlign) || (out_bf16 && misaligned(out_bf16, kAlign))) return EQUARX_MISALIGNED;
    if (codes_out && (misaligned(codes_out, kAlign) || misaligned(scales_out, kAlign))) return EQUARX_MISALIGNED;
    const size_t scale_bytes = (size_t)blocks_of(n, block) * sizeof(float);
    Aliasing mem;
    mem.reads(local_bf16, (size_t)n * 2);
    mem.writes(out_bf16, (size_t)n * 2);
    mem.writes(codes_out, (size_t)n);
    mem.writes(scales_out, scale_bytes);
    WireTable tab;
    for (int32_t r = 0; r < kMaxPartials; ++r) {
        tab.codes[r] = nullptr;
        tab.scales[r] = nullptr;
    }
    for (int32_t r = 0; r < R; ++r) {
        if (!codes[r] || !scales[r]) return EQUARX_NULL_POINTER;
        if (misaligned(codes[r], kAlign) || misaligned(scales[r], kAlign)) return EQUARX_MISALIGNED;
        mem.reads(codes[r], (size_t)n);
        mem.reads(scales[r], scale_bytes);
        tab.codes[r] = codes[r];
        tab.scales[r] = scales[r];
    }
    if (int st = mem.check()) return st;          // outputs must not share memory with inputs or one another
#define CALL(BB)                                                                                                  \
    launch_flat<BB>(static_cast<const uint16_t *>(local_bf16), tab, R, n, static_cast<uint16_t *>(out_bf16), codes_out, \
                    scales_out, ctx)
    EQUARX_DISPATCH_BLOCK(block, CALL)
#undef CALL
    return ctx.status();
}

int equarx_quantize_strided(const void *x_bf16, int64_t n, int32_t chunks, int8_t *codes, float *scales, void *stream)
{
    LaunchCtx ctx(stream);
    if (int st = check_strided(n, chunks)) return st;
    if (n == 0) return EQUARX_OK;
    if (!x_bf16 || !codes || !scales) return EQUARX_NULL_POINTER;
    if (misaligned(x_bf16, kAlign) || misaligned(codes, kAlign) || misaligned(scales, kAlign)) return EQUARX_MISALIGNED;
    Aliasing mem;
    mem.reads(x_bf16, (size_t)n * 2);
    mem.writes(codes, (size_t)n);
    mem.writes(scales, (size_t)(n / chunks) * sizeof(float));
    if (int st = mem.check()) return st;
    do_quantize_strided(n, chunks, codes, scales, ctx, false, one_tensor(x_bf16));
    return ctx.status();
}

int equarx_dequantize_strided(const int8_t *codes, const float *scales, int64_t n, int32_t chunks, void *out_bf16,
                              void *stream)
{
    LaunchCtx ctx(stream);
    if (int st = check_strided(n, chunks)) return st;
    if (n == 0) return EQUARX_OK;
    if (!codes || !scales || !out_bf16) return EQUARX_NULL_POINTER;
    if (misaligned(codes, kAlign) || misaligned(scales, kAlign) || misaligned(out_bf16, kAlign)) return EQUARX_MISALIGNED;
    Aliasing mem;
    mem.reads(codes, (size_t)n);
    mem.reads(scales, (size_t)(n / chunks) * sizeof(float));
    mem.writes(out_bf16, (size_t)n * 2);
    if (int st = mem.check()) return st;
    do_dequantize_strided(codes, scales, n, chunks, out_bf16, ctx);
    return ctx.status();
}

int equarx_reduce_stage_strided(const int8_t *codes_in, const float *scales_in, const void *local_bf16, int64_t n,
                                int32_t chunks, int8_t *codes_out, float *scales_out, void *stream)
{
    LaunchCtx ctx(stream);
    if (int st = check_strided(n, chunks)) return st;
    if (n == 0) return EQUARX_OK;
    if (!codes_in || !scales_in || !local_bf16 || !codes_out || !scales_out) return EQUARX_NULL_POINTER;
    if (misaligned(codes_in, kAlign) || misaligned(scales_in, kAlign) || misaligned(local_bf16, kAlign) ||
        misaligned(codes_out, kAlign) || misaligned(scales_out, kAlign))
        return EQUARX_MISALIGNED;
    if (int st = check_hop_memory(codes_in, scales_in, local_bf16, n, n / chunks, codes_out, scales_out)) return st;
    do_hop_strided(codes_in, scales_in, n, chunks, codes_out, scales_out, ctx, false, false, one_tensor(local_bf16));
    return ctx.status();
}

int equarx_reduce_quantized_strided(const void *const *partials_bf16, int32_t P, int64_t n, int32_t chunks,
                                    void *out_bf16, void *workspace, size_t workspace_bytes, void *stream)
{
    LaunchCtx ctx(stream);
    if (int st = check_strided(n, chunks)) return st;
    if (P < 1 || P > EQUARX_MAX_PARTIALS) return EQUARX_BAD_SHAPE;
    if (!partials_bf16) return EQUARX_NULL_POINTER;
    if (n == 0) return EQUARX_OK;
    if (!out_bf16 || !workspace) return EQUARX_NULL_POINTER;
    if (misaligned(out_bf16, kAlign) || misaligned(workspace, kWorkspaceAlign)) return EQUARX_MISALIGNED;
    Aliasing mem;
    if (int st = check_partials(partials_bf16, P, n, mem)) return st;
    // one scale per `chunks` elements: the same workspace as the contiguous chain with block = chunks
    const size_t need = equarx_workspace_bytes(P, n, chunks);
    if (workspace_bytes < need) return EQUARX_WORKSPACE_TOO_SMALL;
    mem.writes(out_bf16, (size_t)n * 2, kInPlace);
    mem.writes(workspace, need);
    if (int st = mem.check()) return st;
    const WireBuffers w = carve_workspace(workspace, n, n / chunks);
    const int at = strided_chain_buffer(n, P);
    int8_t *const c = w.c[at];
    float *const sc = w.s[at];
    do_quantize_strided(n, chunks, c, sc, ctx, false, one_tensor(partials_bf16[0]));
    for (int32_t i = 1; i < P; ++i) {
        do_hop_strided(c, sc, n, chunks, c, sc, ctx, walks_back(n, i), false, one_tensor(partials_bf16[i]));
    }
    do_dequantize_strided(c, sc, n, chunks, out_bf16, ctx, walks_back(n, P));
    return ctx.status();
}

int equarx_reduce_fused_strided(const void *const *partials_bf16, int32_t P, int64_t n, int32_t chunks, void *out_bf16,
                                void *stream)
{
    LaunchCtx ctx(stream);
    if (int st = check_strided(n, chunks)) return st;
    if (P < 1 || P > EQUARX_MAX_PARTIALS) return EQUARX_BAD_SHAPE;
    if (!partials_bf16) return EQUARX_NULL_POINTER;
    if (n == 0) return EQUARX_OK;
    if (!out_bf16) return EQUARX_NULL_POINTER;
    if (misaligned(out_bf16, kAlign)) return EQUARX_MISALIGNED;
    PartialTable tab;
    Aliasing mem;
    if (int st = fill_table(partials_bf16, P, n, mem, tab)) return st;
    mem.writes(out_bf16, (size_t)n * 2, kInPlace);
    if (int st = mem.check()) return st;
    launch_chain_strided(tab, P, n, chunks, false, true, true, false, static_cast<uint16_t *>(out_bf16), ctx);
    return ctx.status();
}

int equarx_reduce_variant_strided(const void *const *partials_bf16, int32_t P, int64_t n, int32_t chunks,
                                  uint32_t flags, void *out_bf16, void *stream)
{
    LaunchCtx ctx(stream);
    if (int st = check_strided(n, chunks)) return st;
    if (P < 1 || P > EQUARX_MAX_PARTIALS) return EQUARX_BAD_SHAPE;
    if (flags & ~(uint32_t)(EQUARX_SEMI_LOOP | EQUARX_RS_UNQUANTIZED | EQUARX_AG_UNQUANTIZED | EQUARX_RING_ORDER))
        return EQUARX_BAD_SHAPE;
    const bool semi = flags & EQUARX_SEMI_LOOP, rs = !(flags & EQUARX_RS_UNQUANTIZED);
    const bool ag = !(flags & EQUARX_AG_UNQUANTIZED), ring = flags & EQUARX_RING_ORDER;
    if (!rs && !ag) return EQUARX_BAD_SHAPE;        // nothing quantized
    if (semi && !rs) return EQUARX_BAD_SHAPE;       // the semi-loop is a reduce-scatter schedule
    if (!partials_bf16) return EQUARX_NULL_POINTER;
    if (n == 0) return EQUARX_OK;
    if (!out_bf16) return EQUARX_NULL_POINTER;
    if (misaligned(out_bf16, kAlign)) return EQUARX_MISALIGNED;
    PartialTable tab;
    Aliasing mem;
    if (int st = fill_table(partials_bf16, P, n, mem, tab)) return st;
    mem.writes(out_bf16, (size_t)n * 2, kInPlace);
    if (int st = mem.check()) return st;
    launch_chain_strided(tab, P, n, chunks, semi, rs, ag, ring, static_cast<uint16_t *>(out_bf16), ctx);
    return ctx.status();
}

int equarx_reduce_variant_hops_strided(const void *const *partials_bf16, int32_t P, int64_t n, int32_t chunks,
                                       uint32_t flags, void *out_bf16, void *workspace, size_t workspace_bytes,
                                       void *stream)
{
    LaunchCtx ctx(stream);
    if (int st = check_strided(n, chunks)) return st;
    if (P < 1 || P > EQUARX_MAX_PARTIALS) return EQUARX_BAD_SHAPE;
    if (flags & ~(uint32_t)(EQUARX_SEMI_LOOP | EQUARX_AG_UNQUANTIZED | EQUARX_RING_ORDER)) return EQUARX_BAD_SHAPE;
    const bool semi = flags & EQUARX_SEMI_LOOP, ag = !(flags & EQUARX_AG_UNQUANTIZED), ring = flags & EQUARX_RING_ORDER;
    if (!partials_bf16) return EQUARX_NULL_POINTER;
    if (n == 0) return EQUARX_OK;
    if (!out_bf16 || !workspace) return EQUARX_NULL_POINTER;
    if (misaligned(out_bf16, kAlign) || misaligned(workspace, kWorkspaceAlign)) return EQUARX_MISALIGNED;
    // one scale per `chunks` elements: the contiguous variants' workspace with block = chunks
    const size_t need = equarx_variant_workspace_bytes(flags & ~(uint32_t)EQUARX_RING_ORDER, P, n, chunks);
    if (workspace_bytes < need) return EQUARX_WORKSPACE_TOO_SMALL;
    PartialTable tab;
    Aliasing mem;
    if (int st = fill_table(partials_bf16, P, n, mem, tab)) return st;
    mem.writes(out_bf16, (size_t)n * 2, kInPlace);
    mem.writes(workspace, need);
    if (int st = mem.check()) return st;

    const WireBuffers w = carve_workspace(workspace, n, n / chunks);
    uint16_t *out = static_cast<uint16_t *>(out_bf16);
    StridedWires wires = {{nullptr, nullptr}, {nullptr, nullptr}};
    const bool spread = short_and_long(chunks, n, P);
    // Ring layout: shards of ceil(M / P) whole minishards; every launch is one ring step on all P shards at once,
    // the workgroups of shard k reading the partial of device (k + offset) mod P.  Array order: offset = partial.
    const int64_t minishards = n / ((int64_t)kChunk * chunks);
    const int per_shard = ring ? (int)((minishards + P - 1) / P) : 0;
    // position i of the full loop: a ring starts shard k's chain at device k+1 and ends it on device k
    const auto at = [&](int i) { return StridedSource{tab, P, per_shard, ring ? (i + 1) % P : i}; };
    // position i of the semi-loop counts from its owner: device k in a ring, partial 0 otherwise
    const auto around = [&](int i) { return StridedSource{tab, P, per_shard, i}; };
    const auto quantize = [&](const StridedSource &from, int to) {
        with_source(from, [&](auto... src) { do_quantize_strided(n, chunks, w.c[to], w.s[to], ctx, spread, src...); });
    };
    const auto hop = [&](const StridedSource &from, int on, bool backward) {
        with_source(from, [&](auto... src) { do_hop_strided(w.c[on], w.s[on], n, chunks, w.c[on], w.s[on], ctx, backward, spread, src...); });
    };
    const auto finish = [&](const StridedSource &own, bool backward) {
        with_source(own, [&](auto... src) {
            if (ag) do_owner_strided<true>(wires, n, chunks, out, ctx, backward, spread, src...);
            else do_owner_strided<false>(wires, n, chunks, out, ctx, backward, spread, src...);
        });
    };

    if (!semi) {
        // Q_B(x_0), hops 1 .. P-2, then the device holding x_(P-1) adds the last wire and feeds the all-gather
        if (P > 1) {
            quantize(at(0), 0);
            for (int32_t i = 1; i + 1 < P; ++i) hop(at(i), 0, walks_back(n, i));
            wires = {{w.c[0], nullptr}, {w.s[0], nullptr}};
        }
        finish(at(P - 1), walks_back(n, P - 1));
        return ctx.status();
    }

    // Semi-loop (Sec. 3.3): the owner is position 0; the chain h+1, h+2, ..., P-1 (na sends) and the chain h, h-1,
    // ..., 1 (nb >= na sends) each advance one device per launch, both in the same launch while both are under way
    // (half a grid per chain), each on a wire buffer of its own that its hops rewrite in place; the owner receives the
    // shorter chain's wire first.
    const int32_t h = P / 2, na = P - 1 - h, nb = h;
    for (int32_t t = 0; t < nb; ++t) {
        const bool backward = walks_back(2 * n, t);
        if (t < na) {
            do_semi_step_strided(w, tab, P, per_shard, h + 1 + t, h - t, t == 0, n, chunks, ctx, backward, spread);
        } else if (t == 0) {
            quantize(around(h), 1);
        } else {
            hop(around(h - t), 1, backward);
        }
    }
    if (na > 0) {
        wires = {{w.c[0], w.c[1]}, {w.s[0], w.s[1]}};
    } else if (nb > 0) {
        wires = {{w.c[1], nullptr}, {w.s[1], nullptr}};
    }
    finish(around(0), walks_back(2 * n, nb));
    return ctx.status();
}

}  // extern "C"
