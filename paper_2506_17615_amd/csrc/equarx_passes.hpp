// The three per-pass launches of the hop-by-hop chain -- quantize, hop, dequantize -- chosen by block size.
// Shared by the translation units of libequarx that launch them (the entry points and the calibration aids).
#pragma once

#include "equarx_device.hpp"
#include "equarx_launch.hpp"

namespace equarx {
namespace host {

// `streaming`: the wire these passes write or read is not read back soon through this device's caches (a ring
// step between devices, as opposed to the single-device chain, whose next launch reads what this one wrote).
// `backward`: this launch takes its tiles in the opposite order (walks_back).
template <int B>
void launch_quantize(const uint16_t *x, int64_t n, int8_t *codes, float *scales, LaunchCtx &ctx, bool streaming = false)
{
    in_pieces(n, [&](int64_t at, int64_t m) {
        with_pass_shape(m, [&](auto shape) {
            using S = decltype(shape);
            ctx.launch(streaming ? quantize_kernel<B, S::K, true> : quantize_kernel<B, S::K, false>, grid_for<S>(m), S::T,
                       x + at, m, codes + at, scales + at / B, blocks_of(m, B));
        });
    });
}

template <int B>
void launch_hop(const int8_t *cin, const float *sin, const uint16_t *x, int64_t n, int8_t *cout, float *sout,
                LaunchCtx &ctx, bool streaming = false, bool backward = false)
{
    in_pieces(n, [&](int64_t at, int64_t m) {
        with_pass_shape(m, [&](auto shape) {
            using S = decltype(shape);
            ctx.launch(streaming ? hop_kernel<B, S::K, true> : hop_kernel<B, S::K, false>, grid_for<S>(m), S::T, cin + at,
                       sin + at / B, x + at, m, cout + at, sout + at / B, mirrored<S>(m, backward));
        });
    });
}

template <int B>
void launch_dequantize(const int8_t *codes, const float *scales, int64_t n, uint16_t *out, LaunchCtx &ctx,
                       bool streaming = false, bool backward = false)
{
    in_pieces(n, [&](int64_t at, int64_t m) {
        if (streaming) {
            with_stream_dequantize_shape(m, [&](auto shape) {
                using S = decltype(shape);
                ctx.launch(dequantize_kernel<B, S::K, true, S::T>, grid_for<S>(m), S::T, codes + at, scales + at / B, m,
                           out + at, 0);
            });
            return;
        }
        with_pass_shape(m, [&](auto shape) {
            using S = decltype(shape);
            ctx.launch(dequantize_kernel<B, S::K, false>, grid_for<S>(m), S::T, codes + at, scales + at / B, m, out + at,
                       mirrored<S>(m, backward));
        });
    });
}

#define EQUARX_DISPATCH_BLOCK(block, CALL)      \
    switch (block) {                            \
        case 32: CALL(32); break;               \
        case 64: CALL(64); break;               \
        case 128: CALL(128); break;             \
        case 256: CALL(256); break;             \
        case 512: CALL(512); break;             \
        default: break;                         \
    }

inline void do_quantize(const void *x, int64_t n, int32_t block, int8_t *codes, float *scales, LaunchCtx &ctx,
                        bool streaming = false)
{
#define CALL(BB) launch_quantize<BB>(static_cast<const uint16_t *>(x), n, codes, scales, ctx, streaming)
    EQUARX_DISPATCH_BLOCK(block, CALL)
#undef CALL
}

inline void do_hop(const int8_t *cin, const float *sin, const void *x, int64_t n, int32_t block, int8_t *cout,
                   float *sout, LaunchCtx &ctx, bool streaming = false, bool backward = false)
{
#define CALL(BB) launch_hop<BB>(cin, sin, static_cast<const uint16_t *>(x), n, cout, sout, ctx, streaming, backward)
    EQUARX_DISPATCH_BLOCK(block, CALL)
#undef CALL
}

inline void do_dequantize(const int8_t *codes, const float *scales, int64_t n, int32_t block, void *out,
                          LaunchCtx &ctx, bool streaming = false, bool backward = false)
{
#define CALL(BB) launch_dequantize<BB>(codes, scales, n, static_cast<uint16_t *>(out), ctx, streaming, backward)
    EQUARX_DISPATCH_BLOCK(block, CALL)
#undef CALL
}

}  // namespace host
}  // namespace equarx
