"""GPU parity: every entry point of libequarx against the CPU oracle, element by element, on the same seeded inputs.

Bar: int8 codes and fp32 scales bit-exact at every hop; the bf16 output bit-exact as well (the stated tolerance
of one bf16 ulp, 2^-7 relative, is therefore met with room to spare and is asserted separately).
"""
import ctypes

import numpy as np
import pytest
import torch

from paper_2506_17615_amd import binding as eq
from paper_2506_17615_amd import workloads as wl

pytestmark = pytest.mark.gpu

BLOCKS = (32, 64, 128, 256, 512)
# lengths chosen against the kernel's geometry: 8 elements per lane, 512 per wave, 2048 per workgroup tile,
# several tiles per workgroup -- whole tiles, a ragged last workgroup, a ragged last lane, a ragged last block
LENGTHS = (4096, 1, 7, 8, 500, 2048 * 5, 2048 * 4 + 512 + 8 * 5 + 3, 2048 * 9 + 1024, 1 << 20, (1 << 20) + 136 + 5)


def _rng(seed):
    return np.random.default_rng(seed)


def _values(kind, n, seed):
    rng = _rng(seed)
    if kind == "normal":
        v = rng.standard_normal(n)
    elif kind == "lognormal":
        v = rng.standard_normal(n) * np.exp(2 * rng.standard_normal(n))
    elif kind == "student":
        v = rng.standard_t(3, n)
    elif kind == "tiny":          # straddles the zero-scale threshold and the subnormal range
        v = rng.standard_normal(n) * 2.0 ** rng.integers(-136, -112, n)
    elif kind == "huge":
        v = rng.standard_normal(n) * 2.0 ** rng.integers(100, 124, n)
    elif kind == "sparse":        # whole blocks of zeros, isolated spikes
        v = rng.standard_normal(n) * (rng.random(n) < 0.02)
        v[: min(n, 1024)] = 0
    else:
        raise ValueError(kind)
    return v.astype(np.float32)


KINDS = ("normal", "lognormal", "student", "tiny", "huge", "sparse")


@pytest.fixture(scope="module")
def gpu():
    import gpu_util
    assert torch.cuda.is_available()
    from paper_2506_17615_amd import build
    build.ensure_built()        # builds only if no library is there; a missing library is otherwise an error
    eq.load()
    return gpu_util


@pytest.mark.parametrize("B", BLOCKS)
def test_quantize_parity(gpu, oracle, B):
    for i, n in enumerate(LENGTHS):
        for kind in KINDS if n <= 2048 * 9 + 1024 else ("normal", "tiny"):
            x = gpu.bf16_of(_values(kind, n, 100 + i))
            c, s = gpu.gpu_quantize(x, B)
            co, so = oracle.quantize_bf16(x, B)
            assert (c == co).all(), (B, n, kind, int((c != co).sum()))
            assert (s.view(np.uint32) == so.view(np.uint32)).all(), (B, n, kind)


@pytest.mark.parametrize("B", BLOCKS)
def test_dequantize_parity(gpu, oracle, B):
    for i, n in enumerate(LENGTHS):
        rng = _rng(200 + i)
        nb = oracle.num_blocks(n, B)
        c = rng.integers(-127, 128, n).astype(np.int8)
        s = (np.abs(rng.standard_normal(nb)) * 2.0 ** rng.integers(-130, 120, nb)).astype(np.float32)
        out = gpu.gpu_dequantize(c, s, B)
        assert (out == oracle.dequantize_bf16(c, s, B)).all(), (B, n)


def test_dequantize_rounds_ties_to_even(gpu, oracle):
    """code * scale values that sit exactly between two bf16 numbers."""
    B = 32
    c = np.tile(np.array([1, 3, 5, 7, -1, -3, -5, -7, 127, -127, 0, 2], np.int8), 64)[: 24 * B]
    s = np.repeat(np.array([1.0 + 2.0 ** -8, 1.0 + 3 * 2.0 ** -8, 2.0 ** -8, 255 / 256, 3.0 ** -40, 2.0 ** 100 * 1.00390625],
                           np.float32), 4)
    out = gpu.gpu_dequantize(c, s, B)
    assert (out == oracle.dequantize_bf16(c, s, B)).all()


@pytest.mark.parametrize("B", BLOCKS)
def test_hop_parity(gpu, oracle, B):
    for i, n in enumerate(LENGTHS):
        for kind in ("normal", "lognormal", "tiny", "sparse") if n <= 2048 * 9 + 1024 else ("normal",):
            rng = _rng(300 + i)
            nb = oracle.num_blocks(n, B)
            x = gpu.bf16_of(_values(kind, n, 400 + i))
            cin = rng.integers(-127, 128, n).astype(np.int8)
            mag = np.abs(oracle.bf16_to_f32(x)).max() + 1e-30
            sin = (np.abs(rng.standard_normal(nb)) * mag / 100).astype(np.float32)
            c, s = gpu.gpu_hop(cin, sin, x, B)
            co, so = oracle.hop(cin, sin, x, B)
            assert (c == co).all(), (B, n, kind, int((c != co).sum()))
            assert (s.view(np.uint32) == so.view(np.uint32)).all(), (B, n, kind)


@pytest.mark.parametrize("B", eq.BLOCK_SIZES)
def test_quantize_and_hop_parity_near_the_largest_finite_values(gpu, oracle, B):
    """Blocks whose max-abs lies in [2^126, 2^128): 1/absmax is subnormal there and the kernels take their
    scaled-reciprocal route; codes and scales must still be the oracle's."""
    n = 2048 * 4 + 5 * B + 24
    rng = _rng(900 + B)
    v = (rng.standard_normal(n) * 2.0 ** 100).astype(np.float32)
    big = rng.random(n) < 0.02
    v[big] = (rng.choice([-1.0, 1.0], big.sum()) * 2.0 ** (126 + 1.99 * rng.random(big.sum()))).astype(np.float32)
    v[:B] = np.float32(2.0 ** 126)                     # exactly the boundary
    v[B:2 * B] = np.float32(3.3895313892515355e38)     # the largest bf16
    x = gpu.bf16_of(v)
    c, s = gpu.gpu_quantize(x, B)
    co, so = oracle.quantize_bf16(x, B)
    assert (c == co).all() and (s.view(np.uint32) == so.view(np.uint32)).all()
    assert np.isfinite(so).all() and (np.abs(co[:2 * B]) == 127).all()
    zc = np.zeros(n, np.int8)
    zs = np.ones(oracle.num_blocks(n, B), np.float32)
    c2, s2 = gpu.gpu_hop(zc, zs, x, B)                 # 0 * 1 + x: the same values through the hop kernel
    assert (c2 == co).all() and (s2.view(np.uint32) == so.view(np.uint32)).all()


def test_random_shapes_and_values(gpu, oracle):
    """Three hundred seeded draws of (P, n, block, value kind): ragged lengths at every alignment, through every
    schedule of the chain (hop by hop with and without kept wire, ends fused, one launch) and one variant each."""
    rng = _rng(20250611)
    variants = (eq.SEMI_LOOP, eq.AG_UNQUANTIZED, eq.RS_UNQUANTIZED, eq.RING_ORDER, eq.SEMI_LOOP | eq.AG_UNQUANTIZED)
    for case in range(300):
        P = int(rng.integers(1, 9))
        B = int(rng.choice(eq.BLOCK_SIZES))
        n = int(rng.integers(1, 3 * 2048 * 4 + 1)) if case % 4 else int(rng.integers(1, 600))
        kind = KINDS[int(rng.integers(0, len(KINDS)))]
        if kind == "huge":
            kind = "student"       # sums of several huge values overflow; non-finite results are unspecified
        parts = [gpu.bf16_of(_values(kind, n, 31000 + 10 * case + p)) for p in range(P)]
        flags = int(variants[case % len(variants)])
        try:
            _check_chain(gpu, oracle, parts, B)
            assert (gpu.gpu_variant(parts, B, flags) == _oracle_variant(oracle, parts, B, flags)).all(), flags
        except AssertionError as e:
            raise AssertionError(f"case {case}: P={P} n={n} B={B} kind={kind}: {e}") from e


def test_hop_in_place(gpu, oracle):
    for B in (32, 256, 512):
        n = 2048 * 7 + 640
        rng = _rng(7)
        x = gpu.bf16_of(_values("normal", n, 8))
        cin = rng.integers(-127, 128, n).astype(np.int8)
        sin = (np.abs(rng.standard_normal(oracle.num_blocks(n, B))) / 50).astype(np.float32)
        c, s = gpu.gpu_hop(cin, sin, x, B, in_place=True)
        co, so = oracle.hop(cin, sin, x, B)
        assert (c == co).all() and (s == so).all()


def _check_chain(gpu, oracle, parts, B):
    out, wc, ws, _ = gpu.gpu_chain(parts, B)
    oo, owc, ows = oracle.reduce_chain(parts, B, keep_wire=True)
    for i in range(len(parts)):
        assert (wc[i] == owc[i]).all(), ("codes differ at hop", i, int((wc[i] != owc[i]).sum()))
        assert (ws[i].view(np.uint32) == ows[i].view(np.uint32)).all(), ("scales differ at hop", i)
    assert (out == oo).all()
    # the stated tolerance, 2^-7 relative (one bf16 ulp), holds a fortiori
    a, b = oracle.bf16_to_f32(out).astype(np.float64), oracle.bf16_to_f32(oo).astype(np.float64)
    assert (np.abs(a - b) <= 2.0 ** -7 * np.abs(b)).all()
    # the same call without kept wire (ping-pong workspace) gives the same output
    assert (gpu.gpu_chain(parts, B, keep_wire=False) == oo).all()
    # the single-launch chain: same bits, with and without the wire kept
    fout, fwc, fws = gpu.gpu_chain_fused(parts, B)
    assert (fout == oo).all() and (fwc == owc).all() and (fws.view(np.uint32) == ows.view(np.uint32)).all()
    assert (gpu.gpu_chain_fused(parts, B, keep_wire=False) == oo).all()
    # hop by hop with both ends fused (P-1 launches)
    assert (gpu.gpu_chain_fused_ends(parts, B) == oo).all()
    # the per-step entry points composed by hand (non-temporal wire accesses): same wire at every hop, same output
    sout, swc, sws = gpu.gpu_chain_per_step(parts, B)
    assert (sout == oo).all() and (swc == owc).all() and (sws.view(np.uint32) == ows.view(np.uint32)).all()
    # the chain whose wire buffers live in the library's static array
    assert (gpu.gpu_chain_static(parts, B) == oo).all()


CHAIN_CASES = {
    "c1": wl.WORKLOADS["c1_small"],
    "c2_rows24": wl.WORKLOADS["c2_gemma3_12b"].with_rows(24),
    "c3_rows24": wl.WORKLOADS["c3_gemma3_27b"].with_rows(24),
    "c4": wl.WORKLOADS["c4_decode"],
}


@pytest.mark.parametrize("case", sorted(CHAIN_CASES))
def test_chain_parity_workloads(gpu, oracle, case):
    w = CHAIN_CASES[case]
    parts = [wl.as_u16(p) for p in wl.make_partials(w)]
    _check_chain(gpu, oracle, parts, w.block)


@pytest.mark.parametrize("B", (32, 128, 512))
def test_chain_parity_heavy_tails(gpu, oracle, B):
    import dataclasses
    w = dataclasses.replace(wl.WORKLOADS["c5_large"], hidden=(1 << 18) + 2048 + 40, block=B)
    parts = [wl.as_u16(p) for p in wl.make_partials(w)]
    _check_chain(gpu, oracle, parts, B)


@pytest.mark.parametrize("tiles", (513, 600, 2048, 2049, 2300))
def test_chain_parity_kernel_shapes(gpu, oracle, tiles):
    """The single-launch chain picks its kernel by message size: lengths below and above one round of workgroups
    (one tile per thread, two), ragged, with the wire kept."""
    n, B = 2048 * tiles - 2048 + 1500 + 3, 128
    parts = [gpu.bf16_of(_values("lognormal", n, 700 + p)) for p in range(3)]
    oracle.set_threads(8)
    try:
        _check_chain(gpu, oracle, parts, B)
    finally:
        oracle.set_threads(1)


@pytest.mark.parametrize("P", (1, 2, 3, 64))
def test_chain_lengths_of_chain(gpu, oracle, P):
    n, B = 2048 * 3 + 300, 64
    parts = [gpu.bf16_of(_values("lognormal", n, 500 + p)) for p in range(P)]
    _check_chain(gpu, oracle, parts, B)


def test_chain_degenerate_inputs(gpu, oracle):
    n, B = 2048 * 2 + 77, 128
    x = gpu.bf16_of(_values("normal", n, 1))
    z = np.zeros(n, np.uint16)
    _check_chain(gpu, oracle, [z, z, z], B)                       # all zero: scales 0, codes 0, output 0
    _check_chain(gpu, oracle, [x, z, z, z], B)                    # requantizing the grid is idempotent
    _check_chain(gpu, oracle, [x, x ^ np.uint16(0x8000)], B)      # cancellation down to the residual
    _check_chain(gpu, oracle, [gpu.bf16_of(_values("tiny", n, 2)) for _ in range(4)], B)


def test_empty_input_is_a_no_op(gpu):
    e8 = torch.empty(0, dtype=torch.int8, device="cuda")
    e32 = torch.empty(0, dtype=torch.float32, device="cuda")
    e16 = torch.empty(0, dtype=torch.bfloat16, device="cuda")
    eq.equarx_quantize(e16, 256, e8, e32)
    eq.equarx_dequantize(e8, e32, 256, e16)
    eq.equarx_reduce_stage(e8, e32, e16, 256, e8, e32)
    eq.equarx_reduce_quantized([e16, e16], 256, e16, None)
    eq.equarx_reduce_fused([e16, e16], 256, e16)
    eq.equarx_reduce_quantized_fused_ends([e16, e16, e16], 256, e16, None)
    torch.cuda.synchronize()


def test_non_finite_inputs_do_not_fault_and_stay_in_their_block(gpu, oracle):
    """NaN/Inf results are unspecified, but blocks are independent: every block without one still matches."""
    n, B = 2048 * 4, 256
    v = _values("normal", n, 3)
    v[5] = np.inf
    v[B * 3 + 1] = np.nan
    v[B * 9 + 200] = -np.inf
    x = gpu.bf16_of(v)
    y = gpu.bf16_of(_values("normal", n, 4))
    out, wc, ws, _ = gpu.gpu_chain([x, y], B)
    oo, owc, ows = oracle.reduce_chain([x, y], B, keep_wire=True)
    clean = np.ones(n // B, bool)
    clean[[0, 3, 9]] = False
    keep = np.repeat(clean, B)
    assert (out[keep] == oo[keep]).all() and (wc[:, keep] == owc[:, keep]).all() and (ws[:, clean] == ows[:, clean]).all()


@pytest.mark.parametrize("chunks,minishards", ((32, 9), (32, 24), (32, 192), (64, 8), (64, 20), (64, 128), (128, 6), (128, 18),
                                               (128, 49)))
def test_a_nan_fills_its_block_of_the_strided_geometry(gpu, oracle, chunks, minishards):
    """In every layout, hop by hop and in one launch: no element of the block is finite, every other block matches."""
    n, P = 1024 * chunks * minishards, 3
    rng = np.random.default_rng(chunks + minishards)
    x = [gpu.bf16_of(rng.standard_normal(n, dtype=np.float32)) for _ in range(P)]
    filled = np.zeros((P, minishards, 1024), bool)
    for k, e in enumerate(rng.choice(n, 48 * P, replace=False)):
        x[k % P][e] = (0x7FC0, 0xFFC0, 0x7F81)[k % 7 % 3]
        filled[k % P, e // (1024 * chunks), e % 1024] = True
    dev = [gpu.dev_bf16(p) for p in x]

    def holds(got, want, blocks):
        """got, want: an element, or a scale, per position of a minishard."""
        blocks = np.broadcast_to(blocks[:, None], (minishards, got.size // blocks.size, 1024)).reshape(-1)
        assert np.isnan(got[blocks]).all() and (got[~blocks].view(np.uint32) == want[~blocks].view(np.uint32)).all()

    c, s = torch.empty(n, dtype=torch.int8, device="cuda"), torch.empty(n // chunks, device="cuda")
    eq.equarx_quantize_strided(dev[0], chunks, c, s)
    wc, ws = oracle.quantize_bf16_strided(x[0], chunks)
    holds(s.cpu().numpy(), ws, filled[0])
    eq.equarx_reduce_stage_strided(c, s, dev[1], chunks, c, s)
    wc, ws = oracle.hop_strided(wc, ws, x[1], chunks)
    holds(s.cpu().numpy(), ws, filled[0] | filled[1])

    def widened(u16):
        return (u16.astype(np.uint32) << 16).view(np.float32)

    out = torch.empty(n, dtype=torch.bfloat16, device="cuda")
    for flags in (0, eq.RING_ORDER, eq.SEMI_LOOP, eq.SEMI_LOOP | eq.RING_ORDER, eq.RS_UNQUANTIZED):
        want = widened(_oracle_variant_strided(oracle, x, chunks, flags))
        eq.equarx_reduce_variant_strided(dev, chunks, flags, out.fill_(5.0))
        holds(widened(gpu.host_u16(out)), want, filled.any(axis=0))
        if flags != eq.RS_UNQUANTIZED:
            work = eq.alloc_variant_workspace(flags & ~eq.RING_ORDER, P, n, chunks)
            eq.equarx_reduce_variant_hops_strided(dev, chunks, flags, out.fill_(5.0), work)
            holds(widened(gpu.host_u16(out)), want, filled.any(axis=0))
    eq.equarx_reduce_quantized_strided(dev, chunks, out.fill_(5.0), eq.alloc_workspace(P, n, chunks))
    holds(widened(gpu.host_u16(out)), widened(_oracle_variant_strided(oracle, x, chunks, 0)), filled.any(axis=0))


def test_bad_arguments_raise(gpu):
    x = torch.zeros(4096, dtype=torch.bfloat16, device="cuda")
    c = torch.zeros(4096, dtype=torch.int8, device="cuda")
    s = torch.zeros(16, dtype=torch.float32, device="cuda")
    with pytest.raises(eq.EquarxError) as e:
        eq.equarx_quantize(x, 100, c, s)
    assert e.value.status == eq.STATUS_BAD_BLOCK
    with pytest.raises(eq.EquarxError) as e:
        eq.equarx_quantize(x[1:], 256, c, s)
    assert e.value.status == eq.STATUS_MISALIGNED
    big = torch.zeros(4096 + 8, dtype=torch.bfloat16, device="cuda")
    shifted = big[8:]           # overlaps big[:4096] without being it (the output may BE a partial, see below)
    with pytest.raises(eq.EquarxError) as e:
        eq.equarx_reduce_quantized([x, big[:4096]], 256, shifted, eq.alloc_workspace(2, 4096, 256))
    assert e.value.status == eq.STATUS_BAD_SHAPE
    with pytest.raises(eq.EquarxError) as e:
        eq.equarx_reduce_fused([big[:4096], x], 256, shifted)
    assert e.value.status == eq.STATUS_BAD_SHAPE
    small = torch.empty(256, dtype=torch.uint8, device="cuda")
    with pytest.raises(eq.EquarxError) as e:
        eq.equarx_reduce_quantized([x, x], 256, torch.empty_like(x), small)
    assert e.value.status == eq.STATUS_WORKSPACE_TOO_SMALL


def test_calibration_copy(gpu):
    src = torch.randint(-128, 127, ((1 << 20) + 4096 + 16,), dtype=torch.int8, device="cuda")
    dst = torch.zeros_like(src)
    eq.equarx_calib_copy(src, dst)
    torch.cuda.synchronize()
    assert torch.equal(src, dst)


@pytest.mark.parametrize("B", (32, 256, 512))
def test_calibration_hop_traffic(gpu, B):
    """The memory-only stand-in for the chain's hops writes the documented XOR of what it read (so it really
    reads all of it), launch after launch, ping-pong between the two wires or in place, in turn for a long wire."""
    n = B * 4 * 53 + 2048 * 6          # several workgroups and a ragged last one
    _hop_traffic(B, n - n % B, False)
    _hop_traffic(B, n - n % B, True)
    _hop_traffic(B, (20 << 20) + 8192 * 3 + B, True)


def _hop_traffic(B, n, in_place):
    rng = _rng(B)
    P = 4
    xs = [torch.from_numpy(rng.integers(0, 1 << 16, n, dtype=np.int64).astype(np.uint16).view(np.int16)).cuda()
          .view(torch.bfloat16) for _ in range(P)]
    c0 = torch.from_numpy(rng.integers(-128, 128, n, dtype=np.int64).astype(np.int8)).cuda()
    s0 = torch.from_numpy(rng.standard_normal(n // B).astype(np.float32)).cuda()
    c1, s1 = (c0, s0) if in_place else (torch.zeros_like(c0), torch.zeros_like(s0))
    cw = c0.cpu().numpy().view(np.uint32).reshape(-1, 2)
    s_first = s0.clone()
    eq.equarx_calib_hop_traffic(xs, B, c0, s0, c1, s1)
    torch.cuda.synchronize()
    for i in range(1, P):
        xw = xs[i].view(torch.int16).cpu().numpy().view(np.uint32).reshape(-1, 4)
        cw = np.stack([xw[:, 0] ^ xw[:, 2] ^ cw[:, 0], xw[:, 1] ^ xw[:, 3] ^ cw[:, 1]], axis=1)
    last_c, last_s = (c1, s1) if (P - 1) & 1 else (c0, s0)
    assert (last_c.cpu().numpy().view(np.uint32).reshape(-1, 2) == cw).all()
    assert torch.equal(last_s, s_first)


def test_time_launch_span_brackets_the_hops(gpu, oracle):
    """Events recorded around launches 1..P-1 of a chain call give a plausible time, leave the result untouched,
    and the setting is consumed by that call."""
    w = wl.WORKLOADS["c1_small"]
    parts = [p.reshape(-1).cuda() for p in wl.make_partials(w)]
    out = torch.empty(w.n, dtype=torch.bfloat16, device="cuda")
    work = eq.alloc_workspace(w.P, w.n, w.block)
    want = oracle.reduce_chain([wl.as_u16(p) for p in wl.make_partials(w)], w.block)
    a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
    a.record()
    b.record()
    torch.cuda.synchronize()
    eq.equarx_time_launch_span(1, w.P - 1, a.cuda_event, b.cuda_event)
    eq.equarx_reduce_quantized(parts, w.block, out, work)
    torch.cuda.synchronize()
    first = a.elapsed_time(b)
    assert 0.0 < first < 2.0                                 # P-1 small kernels, in ms
    assert (gpu.host_u16(out) == want).all()
    eq.equarx_reduce_quantized(parts, w.block, out, work)    # nothing pending any more: the events stay as they are
    torch.cuda.synchronize()
    assert a.elapsed_time(b) == first
    assert (gpu.host_u16(out) == want).all()


@pytest.mark.parametrize("streaming", (False, True))
def test_interleaved_chains_are_the_chain(gpu, oracle, streaming):
    """The benchmark's cold-wire arrangement (several independent chains, launches interleaved pass by pass), with
    cacheable and with non-temporal wire accesses, gives every chain the oracle's result."""
    M, P, n, B = 3, 5, 2048 * 7 + 300, 128
    sets_u16 = [[gpu.bf16_of(_values("lognormal", n, 8800 + 17 * m + p)) for p in range(P)] for m in range(M)]
    sets = [[gpu.dev_bf16(p) for p in ps] for ps in sets_u16]
    outs = [torch.full((n,), 7.0, dtype=torch.bfloat16, device="cuda") for _ in range(M)]
    works = [eq.alloc_workspace(P, n, B) for _ in range(M)]
    eq.equarx_calib_interleaved_chains(sets, B, outs, works, streaming)
    torch.cuda.synchronize()
    for m in range(M):
        assert (gpu.host_u16(outs[m]) == oracle.reduce_chain(sets_u16[m], B)).all(), m


def test_per_step_calls_compose_the_chain(gpu, oracle):
    """The per-step entry points (non-temporal wire accesses) composed by hand give the chain entry point's bits,
    wire for wire, including a hop in place."""
    P, n, B = 6, 2048 * 3 * 5 + 2048 + 77, 64
    parts_u16 = [gpu.bf16_of(_values("student", n, 9100 + p)) for p in range(P)]
    want, wc, ws = oracle.reduce_chain(parts_u16, B, keep_wire=True)
    parts = [gpu.dev_bf16(p) for p in parts_u16]
    nb = eq.num_blocks(n, B)
    c = torch.full((n,), 99, dtype=torch.int8, device="cuda")
    s = torch.full((nb,), -7.0, dtype=torch.float32, device="cuda")
    eq.equarx_quantize(parts[0], B, c, s)
    for i in range(1, P):
        eq.equarx_reduce_stage(c, s, parts[i], B, c, s)         # in place: the wire buffer is reused every step
        torch.cuda.synchronize()
        assert (c.cpu().numpy() == wc[i]).all() and (s.cpu().numpy().view(np.uint32) == ws[i].view(np.uint32)).all(), i
    out = torch.full((n,), 7.0, dtype=torch.bfloat16, device="cuda")
    eq.equarx_dequantize(c, s, B, out)
    torch.cuda.synchronize()
    assert (gpu.host_u16(out) == want).all()


def test_timing_hooks_die_with_a_rejected_call(gpu, oracle):
    """Hooks armed before a call that fails validation are dropped by that call: the next, valid call neither
    records nor attaches them (the events keep the times of their own earlier records)."""
    w = wl.WORKLOADS["c1_small"]
    parts = [p.reshape(-1).cuda() for p in wl.make_partials(w)]
    out = torch.empty(w.n, dtype=torch.bfloat16, device="cuda")
    work = eq.alloc_workspace(w.P, w.n, w.block)
    a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
    a.record()
    b.record()
    torch.cuda.synchronize()
    before = a.elapsed_time(b)
    for arm in (lambda: eq.equarx_time_launch_span(0, w.P, a.cuda_event, b.cuda_event),
                lambda: eq.equarx_time_next_launch(a.cuda_event, b.cuda_event)):
        arm()
        with pytest.raises(eq.EquarxError) as err:
            eq.equarx_reduce_quantized(parts, 48, out, work)         # unsupported block size: rejected on the host
        assert err.value.status == eq.STATUS_BAD_BLOCK
        eq.equarx_reduce_quantized(parts, w.block, out, work)
        eq.equarx_reduce_fused(parts, w.block, out)
        torch.cuda.synchronize()
        assert a.elapsed_time(b) == before
    assert (gpu.host_u16(out) == oracle.reduce_chain([wl.as_u16(p) for p in wl.make_partials(w)], w.block)).all()


def test_stale_hip_error_is_not_reported_as_ours(gpu):
    """An error an unrelated HIP call left pending on the thread does not turn a good launch into
    EQUARX_DEVICE_ERROR: the status comes from the launch call's own return value."""
    import ctypes
    hip = ctypes.CDLL("libamdhip64.so")
    hip.hipGetLastError.restype = ctypes.c_int
    hip.hipFree.restype = ctypes.c_int
    hip.hipFree.argtypes = [ctypes.c_void_p]
    hip.hipGetLastError()                                   # start clean
    x = torch.randn(4096, device="cuda").to(torch.bfloat16)
    codes = torch.empty(4096, dtype=torch.int8, device="cuda")
    scales = torch.empty(16, dtype=torch.float32, device="cuda")
    assert hip.hipFree(ctypes.c_void_p(0x10)) != 0          # an invalid free: returns an error and leaves it pending
    eq.equarx_quantize(x, 256, codes, scales)               # would raise on EQUARX_DEVICE_ERROR
    torch.cuda.synchronize()
    hip.hipGetLastError()                                   # leave the thread clean for the tests that follow
    assert hip.hipGetLastError() == 0
    assert int(codes.abs().max()) == 127


@pytest.mark.parametrize("P,n,B", ((4, 2048 * 5 + 300, 64), (8, 24 * 5376, 256)))
def test_plain_c_client_drives_the_path(gpu, oracle, tmp_path, P, n, B):
    """The C ABI without Python in between: a C99 program (tests/abi_client.c) allocates with the HIP runtime,
    calls three schedules, checks they agree, and writes the result, which must be the oracle's bit for bit."""
    import subprocess
    from tests import build_abi_client
    exe = build_abi_client.ensure_built()
    parts = [gpu.bf16_of(_values("lognormal", n, 4100 + p)) for p in range(P)]
    fin, fout = tmp_path / "in.bin", tmp_path / "out.bin"
    np.concatenate(parts).astype("<u2").tofile(fin)
    run = subprocess.run([exe, str(fin), str(fout), str(P), str(n), str(B)], capture_output=True, text=True, timeout=120)
    assert run.returncode == 0, run.stdout + run.stderr
    got = np.fromfile(fout, dtype="<u2")
    assert (got == oracle.reduce_chain(parts, B)).all()


# ----------------------------------------------------------------------------- full benchmark sizes

def _sampled_blocks_check(gpu, oracle, w, n_sample=3000, seed=0):
    """At full size, in the launch configuration bench.py times (workspace path), compare sampled blocks.

    Blocks are independent of each other, so the oracle run on a gathered subset of blocks must reproduce the
    GPU's values at exactly those blocks, bit for bit: output, and the codes and scales of every hop."""
    host = wl.make_partials(w)
    u16 = [wl.as_u16(p) for p in host]
    n, B, P = w.n, w.block, w.P
    nb = eq.num_blocks(n, B)
    dev = [p.reshape(-1).cuda() for p in host]
    out = torch.empty(n, dtype=torch.bfloat16, device="cuda")
    eq.equarx_reduce_quantized(dev, B, out, eq.alloc_workspace(P, n, B))
    torch.cuda.synchronize()
    out_h = gpu.host_u16(out)
    out_f = torch.empty_like(out)
    eq.equarx_reduce_fused(dev, B, out_f)
    torch.cuda.synchronize()
    assert torch.equal(out.view(torch.int16), out_f.view(torch.int16))      # single-launch chain, every element
    eq.equarx_reduce_quantized_fused_ends(dev, B, out_f, eq.alloc_workspace(P, n, B))
    torch.cuda.synchronize()
    assert torch.equal(out.view(torch.int16), out_f.view(torch.int16))      # ends fused, every element
    rc, rs = eq.wire_row_codes(n), eq.wire_row_scales(n, B)
    wc = torch.empty((P, rc), dtype=torch.int8, device="cuda")
    ws = torch.empty((P, rs), dtype=torch.float32, device="cuda")
    out2 = torch.empty_like(out)
    eq.equarx_reduce_quantized(dev, B, out2, None, wc, ws)
    torch.cuda.synchronize()
    assert torch.equal(out.view(torch.int16), out2.view(torch.int16))
    wcf = torch.empty_like(wc)
    wsf = torch.empty_like(ws)
    eq.equarx_reduce_fused(dev, B, out_f, wcf, wsf)                             # single launch, wire kept
    torch.cuda.synchronize()
    assert torch.equal(out.view(torch.int16), out_f.view(torch.int16))
    assert torch.equal(wcf[:, :n], wc[:, :n]) and torch.equal(wsf[:, :nb], ws[:, :nb])
    del wcf, wsf

    rng = _rng(seed)
    blocks = np.unique(np.concatenate([[0, 1, nb - 2, nb - 1], rng.integers(0, nb, n_sample)]))
    idx = (blocks[:, None] * B + np.arange(B)[None, :]).reshape(-1)
    idx = idx[idx < n]
    sub = [p[idx] for p in u16]
    oo, owc, ows = oracle.reduce_chain(sub, B, keep_wire=True)
    assert (out_h[idx] == oo).all()
    idx_t = torch.from_numpy(idx).cuda()
    blk_t = torch.from_numpy(blocks).cuda()
    assert (wc[:, :n].index_select(1, idx_t).cpu().numpy() == owc).all()
    assert (ws[:, :nb].index_select(1, blk_t).cpu().numpy().view(np.uint32) == ows.view(np.uint32)).all()

    # properties that hold at any size, over the whole tensor: the codes use their range, every block's largest
    # code is +-127 unless the block is all zero, and the output stays within the method's error bound
    last = wc[-1, :n]
    assert int(last.min()) >= -127
    full = (n // B) * B
    peak = last[:full].view(-1, B).abs().amax(dim=1)
    zero_scale = ws[-1, : n // B] == 0
    assert bool(((peak == 127) | zero_scale).all())
    ref = torch.zeros(n, dtype=torch.float64, device="cuda")
    for p in dev:
        ref += p.double()
    bound = ws[:, :nb].double().sum(dim=0).repeat_interleave(B)[:n] * 0.5 * (1 + 2.0 ** -10)
    err = (out.double() - ref).abs()
    # + the final bf16 rounding of the output (half an ulp: 2^-9 relative)
    assert bool((err <= bound + ref.abs() * 2.0 ** -8 + 1e-30).all())


def test_full_size_gemma3_27b_sampled(gpu, oracle):
    _sampled_blocks_check(gpu, oracle, wl.WORKLOADS["c3_gemma3_27b"])


def test_full_size_gemma3_12b_every_element(gpu, oracle):
    w = wl.WORKLOADS["c2_gemma3_12b"]
    u16 = [wl.as_u16(p) for p in wl.make_partials(w)]
    oracle.set_threads(16)
    try:
        oo = oracle.reduce_chain(u16, w.block)
    finally:
        oracle.set_threads(1)
    assert (gpu.gpu_chain(u16, w.block, keep_wire=False) == oo).all()


@pytest.mark.parametrize("B", (32, 128, 512))
def test_full_size_large_message_sampled(gpu, oracle, B):
    _sampled_blocks_check(gpu, oracle, wl.WORKLOADS["c5_large"].with_block(B), n_sample=2000, seed=B)


def test_full_size_fig7_tensor_sampled(gpu, oracle):
    """The paper's own setting (Sec. 4.1 / Fig. 7: (4096, 4096), N(0,1), 8 devices, block 64) at full size: the
    chain with every hop's wire on sampled blocks, and every flavour the figure compares -- both forms of each,
    single launch and hop by hop -- on the same sampled blocks."""
    w = wl.FIG7
    assert (w.P, w.n, w.block) == (8, 4096 * 4096, 64)
    _sampled_blocks_check(gpu, oracle, w, n_sample=3000, seed=64)
    u16 = [wl.as_u16(p) for p in wl.make_partials(w)]
    dev = [gpu.dev_bf16(p) for p in u16]
    n, B, P = w.n, w.block, w.P
    nb = n // B
    blocks = np.unique(np.concatenate([[0, 1, nb - 2, nb - 1], _rng(65).integers(0, nb, 3000)]))
    idx = (blocks[:, None] * B + np.arange(B)[None, :]).reshape(-1)
    sub = [p[idx] for p in u16]
    out = torch.empty(n, dtype=torch.bfloat16, device="cuda")
    for name in ("rs_only", "ag_only", "semi", "semi_rs_only"):
        flags = VARIANT_FLAGS[name]
        want = _oracle_variant(oracle, sub, B, flags)
        out.fill_(3.0)
        eq.equarx_reduce_variant(dev, B, flags, out)
        torch.cuda.synchronize()
        assert (gpu.host_u16(out)[idx] == want).all(), name
        if name != "ag_only":           # without a quantized reduce-scatter there is no hop-by-hop form
            out.fill_(3.0)
            eq.equarx_reduce_variant_hops(dev, B, flags, out, eq.alloc_variant_workspace(flags, P, n, B))
            torch.cuda.synchronize()
            assert (gpu.host_u16(out)[idx] == want).all(), name + " hop by hop"
    # ring order: the sampled blocks of each shard against the pinned chain in that shard's own rotation
    per = -(-nb // P)
    for name in ("ring", "ring_rs_only", "ring_semi", "ring_semi_rs_only"):
        flags = VARIANT_FLAGS[name]
        ag = not (flags & eq.AG_UNQUANTIZED)
        semi = bool(flags & eq.SEMI_LOOP)
        for hops in (False, True):
            out.fill_(3.0)
            if hops:
                eq.equarx_reduce_variant_hops(dev, B, flags, out, eq.alloc_variant_workspace(flags, P, n, B))
            else:
                eq.equarx_reduce_variant(dev, B, flags, out)
            torch.cuda.synchronize()
            got = gpu.host_u16(out)
            for k in range(P):
                mine = blocks[(blocks >= k * per) & (blocks < (k + 1) * per)]
                ix = (mine[:, None] * B + np.arange(B)[None, :]).reshape(-1)
                if semi:            # device k owns the shard, the devices k+1, k+2, ... sit around it
                    want = oracle.reduce_semi_loop([u16[(k + i) % P][ix] for i in range(P)], B, ag)
                else:               # the chain starts at device k+1 and ends on device k
                    want = oracle.reduce_stages([u16[(k + 1 + i) % P][ix] for i in range(P)], B, True, ag)
                assert (got[ix] == want).all(), (name, hops, k)


# ----------------------------------------------------------------------------- the kernels' own arithmetic

def test_block_quotients_equal_ieee_division_for_every_fp32(gpu):
    """The short reciprocal sequences the kernels use for absmax/127 and 127/absmax give the IEEE quotient for
    EVERY fp32 absmax from the tiny threshold 127*2^-126 up to the largest finite value."""
    bad = torch.zeros(2, dtype=torch.int64, device="cuda")
    lo, hi = 0x03FE0000, 0x7F800000
    step = 1 << 28
    for first in range(lo, hi, step):
        eq.equarx_selftest_quotients(first, min(step, hi - first), bad)
    # below the threshold both forms give (0, 0)
    eq.equarx_selftest_quotients(0, lo, bad)
    torch.cuda.synchronize()
    assert bad.tolist() == [0, 0]


def test_codes_from_the_magic_number_add_equal_rint_for_every_fp32(gpu):
    """The low byte of fl32(p + 1.5 * 2^23) is the int8 code (int8) rint(p) for EVERY fp32 p with |p| < 128,
    both signs (the quantizer's scaled values lie in [-127, 127] up to rounding)."""
    bad = torch.zeros(1, dtype=torch.int64, device="cuda")
    hi = 0x43000000                    # 128.0f
    step = 1 << 28
    for first in range(0, hi, step):
        eq.equarx_selftest_rounding(first, min(step, hi - first), bad)
    torch.cuda.synchronize()
    assert bad.tolist() == [0]
    with pytest.raises(eq.EquarxError):
        eq.equarx_selftest_rounding(hi - 1, 2, bad)       # beyond |p| < 128


def test_block_quotients_equal_host_division(gpu):
    """... and the host's IEEE division (numpy fp32) on random patterns, every bf16 value and the range edges."""
    rng = _rng(77)
    bits = rng.integers(0x03FE0000, 0x7F800000, 4_000_000, dtype=np.int64).astype(np.uint32)
    bf = (np.arange(0x03FE, 0x7F80, dtype=np.uint32) << 16)
    edges = np.array([0x03FE0000, 0x03FE0001, 0x7E7FFFFF, 0x7E800000, 0x7E800001, 0x7F7FFFFF, 0x3F800000, 0x42FE0000],
                     np.uint32)
    a = np.concatenate([bits, bf, edges]).view(np.float32)
    d = torch.from_numpy(a).cuda()
    s = torch.empty_like(d)
    v = torch.empty_like(d)
    eq.equarx_eval_quotients(d, s, v)
    torch.cuda.synchronize()
    with np.errstate(all="ignore"):
        want_s = a / np.float32(127.0)
        want_v = np.float32(127.0) / a
    assert (s.cpu().numpy().view(np.uint32) == want_s.view(np.uint32)).all()
    assert (v.cpu().numpy().view(np.uint32) == want_v.view(np.uint32)).all()
    # below the threshold: zeros
    tiny = torch.tensor([0.0, 1e-45, 1.17549435e-38, 1.4928e-36], device="cuda")
    s2, v2 = torch.empty_like(tiny), torch.empty_like(tiny)
    eq.equarx_eval_quotients(tiny, s2, v2)
    torch.cuda.synchronize()
    assert s2.tolist() == [0, 0, 0, 0] and v2.tolist() == [0, 0, 0, 0]


# ----------------------------------------------------------------------------- variants of the chain

def _oracle_variant(oracle, parts, B, flags):
    semi, rs = bool(flags & eq.SEMI_LOOP), not (flags & eq.RS_UNQUANTIZED)
    ag, ring = not (flags & eq.AG_UNQUANTIZED), bool(flags & eq.RING_ORDER)
    if ring:
        return oracle.reduce_ring(parts, B, semi=semi, quantize_rs=rs, quantize_ag=ag)
    if semi:
        return oracle.reduce_semi_loop(parts, B, ag)
    return oracle.reduce_stages(parts, B, rs, ag)


VARIANT_FLAGS = {
    "full": 0,
    "rs_only": eq.AG_UNQUANTIZED,
    "ag_only": eq.RS_UNQUANTIZED,
    "semi": eq.SEMI_LOOP,
    "semi_rs_only": eq.SEMI_LOOP | eq.AG_UNQUANTIZED,
    "ring": eq.RING_ORDER,
    "ring_rs_only": eq.RING_ORDER | eq.AG_UNQUANTIZED,
    "ring_ag_only": eq.RING_ORDER | eq.RS_UNQUANTIZED,
    "ring_semi": eq.RING_ORDER | eq.SEMI_LOOP,
    "ring_semi_rs_only": eq.RING_ORDER | eq.SEMI_LOOP | eq.AG_UNQUANTIZED,
}


@pytest.mark.parametrize("name", sorted(VARIANT_FLAGS))
def test_variant_parity(gpu, oracle, name):
    flags = VARIANT_FLAGS[name]
    cases = [(4, 4096, 256, "normal"), (8, 2048 * 9 + 1024 + 40, 64, "lognormal"), (1, 3000, 32, "normal"),
             (2, 8192 * 2 + 7, 128, "student"), (3, 5000, 512, "normal"), (7, 8192 * 3 + 2048 + 8, 32, "tiny"),
             (16, 64 * 5376 // 4, 128, "normal"), (5, 300, 256, "sparse"), (64, 2048 + 100, 64, "normal")]
    for P, n, B, kind in cases:
        parts = [gpu.bf16_of(_values(kind, n, 900 + 7 * p + P)) for p in range(P)]
        got = gpu.gpu_variant(parts, B, flags)
        want = _oracle_variant(oracle, parts, B, flags)
        assert (got == want).all(), (name, P, n, B, kind, int((got != want).sum()))


def test_variant_parity_large_message(gpu, oracle):
    """Above one round of workgroups, where the chain kernels take two tiles per thread."""
    P, n, B = 3, 2048 * 2100 + 2048 * 2 + 24, 256
    parts = [gpu.bf16_of(_values("normal", n, 1300 + p)) for p in range(P)]
    oracle.set_threads(8)
    try:
        for name, flags in VARIANT_FLAGS.items():
            assert (gpu.gpu_variant(parts, B, flags) == _oracle_variant(oracle, parts, B, flags)).all(), name
    finally:
        oracle.set_threads(1)


def test_variant_workloads(gpu, oracle):
    for case in ("c2_rows24", "c3_rows24", "c4"):
        w = CHAIN_CASES[case]
        parts = [wl.as_u16(p) for p in wl.make_partials(w)]
        for name, flags in VARIANT_FLAGS.items():
            assert (gpu.gpu_variant(parts, w.block, flags) == _oracle_variant(oracle, parts, w.block, flags)).all(), (case, name)


@pytest.mark.parametrize("name", ("full", "rs_only", "semi", "semi_rs_only", "ring", "ring_rs_only", "ring_semi",
                                  "ring_semi_rs_only"))
@pytest.mark.parametrize("P", (1, 2, 3, 4, 5, 8, 9))
@pytest.mark.parametrize("B", (32, 64, 256, 512))
def test_variant_hop_by_hop_parity(gpu, oracle, name, P, B):
    """The variants in the ring-imposed schedule (one launch per hop, wires in memory): the oracle's bits, which are
    also the single-launch form's; output in place for odd P; every lane-group width of the kernels."""
    flags = VARIANT_FLAGS[name]
    n = 2048 * 7 + 5 * B + 24
    parts = [gpu.bf16_of(_values("lognormal", n, 9300 + p)) for p in range(P)]
    want = _oracle_variant(oracle, parts, B, flags)
    dev = [gpu.dev_bf16(p) for p in parts]
    out = dev[P // 2] if P % 2 else torch.full((n,), 5.0, dtype=torch.bfloat16, device="cuda")
    eq.equarx_reduce_variant_hops(dev, B, flags, out, eq.alloc_variant_workspace(flags, P, n, B))
    torch.cuda.synchronize()
    assert (gpu.host_u16(out) == want).all()
    assert (gpu.gpu_variant(parts, B, flags) == want).all()


def test_variant_hop_by_hop_workload_shape(gpu, oracle):
    w = wl.WORKLOADS["c3_gemma3_27b"].with_rows(40)
    parts = [wl.as_u16(p) for p in wl.make_partials(w)]
    oracle.set_threads(8)
    try:
        for name in ("rs_only", "semi", "semi_rs_only", "ring", "ring_rs_only", "ring_semi", "ring_semi_rs_only"):
            flags = VARIANT_FLAGS[name]
            dev = [gpu.dev_bf16(p) for p in parts]
            out = torch.empty(w.n, dtype=torch.bfloat16, device="cuda")
            eq.equarx_reduce_variant_hops(dev, w.block, flags, out, eq.alloc_variant_workspace(flags, w.P, w.n, w.block))
            torch.cuda.synchronize()
            assert (gpu.host_u16(out) == _oracle_variant(oracle, parts, w.block, flags)).all(), name
    finally:
        oracle.set_threads(1)


def test_variant_bad_flags(gpu):
    x = torch.zeros(4096, dtype=torch.bfloat16, device="cuda")
    out = torch.empty_like(x)
    for flags in (eq.RS_UNQUANTIZED | eq.AG_UNQUANTIZED, eq.SEMI_LOOP | eq.RS_UNQUANTIZED, 16, 1 << 31):
        with pytest.raises(eq.EquarxError) as e:
            eq.equarx_reduce_variant([x, x], 256, flags, out)
        assert e.value.status == eq.STATUS_BAD_SHAPE


def test_variant_error_ordering_as_in_the_paper(gpu, oracle):
    """Sec. 4.1 / Fig. 7 on the GPU path: AG-only < semi-loop < full-loop in MSE (8 devices, block 64, N(0,1))."""
    P, n, B = 8, 1 << 20, 64
    parts = [gpu.bf16_of(_values("normal", n, 4242 + p)) for p in range(P)]
    ref = sum(oracle.bf16_to_f32(p).astype(np.float64) for p in parts)

    def mse(flags):
        return float(np.mean((oracle.bf16_to_f32(gpu.gpu_variant(parts, B, flags)).astype(np.float64) - ref) ** 2))

    full, semi, ag_only = mse(0), mse(eq.SEMI_LOOP), mse(eq.RS_UNQUANTIZED)
    assert ag_only < semi < full
    assert 0.0014 / 1.5 < full < 0.0014 * 1.5 and 0.001 / 1.5 < semi < 0.001 * 1.5 and 0.0003 / 1.5 < ag_only < 0.0003 * 1.5


# ----------------------------------------------------------------------------- flat one-shot reduce

def _flat_case(gpu, oracle, R, n, B, kind, seed):
    local = gpu.bf16_of(_values(kind, n, seed))
    remote = [gpu.bf16_of(_values(kind, n, seed + 1 + r)) for r in range(R)]
    q = [oracle.quantize_bf16(x, B) for x in remote]
    want_out, want_c, want_s = oracle.reduce_flat(local, [c for c, _ in q], [s for _, s in q], B)
    # the senders' quantization runs on the GPU too (equarx_quantize), as in the real pipeline
    dl = gpu.dev_bf16(local)
    dc, ds = [], []
    nb = eq.num_blocks(n, B)
    for x in remote:
        c = torch.empty(n, dtype=torch.int8, device="cuda")
        s_ = torch.empty(max(nb, 1), dtype=torch.float32, device="cuda")
        eq.equarx_quantize(gpu.dev_bf16(x), B, c, s_)
        dc.append(c)
        ds.append(s_)
    out = torch.full((n,), 7.0, dtype=torch.bfloat16, device="cuda")
    co = torch.full((n,), 99, dtype=torch.int8, device="cuda")
    so = torch.full((max(nb, 1),), -7.0, dtype=torch.float32, device="cuda")
    eq.equarx_reduce_flat(dl, dc, ds, B, out, co, so)
    torch.cuda.synchronize()
    assert (gpu.host_u16(out) == want_out).all(), (R, n, B, kind)
    assert (co.cpu().numpy() == want_c).all() and (so.cpu().numpy()[:nb].view(np.uint32) == want_s.view(np.uint32)).all()
    # each output alone
    out2 = torch.full_like(out, 3.0)
    eq.equarx_reduce_flat(dl, dc, ds, B, out2)
    co2, so2 = torch.full_like(co, 98), torch.full_like(so, -3.0)
    eq.equarx_reduce_flat(dl, dc, ds, B, None, co2, so2)
    torch.cuda.synchronize()
    assert torch.equal(out2.view(torch.int16), out.view(torch.int16)) and torch.equal(co2, co) and torch.equal(so2[:nb], so[:nb])


@pytest.mark.parametrize("B", BLOCKS)
def test_flat_parity(gpu, oracle, B):
    for i, (R, n, kind) in enumerate([(7, 4096, "normal"), (0, 3000, "normal"), (1, 8192 * 2 + 2048 + 13, "lognormal"),
                                      (3, 8192 * 3 + 512, "student"), (15, 64 * 5376 // 2, "normal"), (7, 100, "tiny"),
                                      (63, 2048 + 9, "normal"), (5, 8192 + 1, "sparse")]):
        _flat_case(gpu, oracle, R, n, B, kind, 5000 + 100 * i)


def test_flat_workload_shape(gpu, oracle):
    w = wl.WORKLOADS["c3_gemma3_27b"].with_rows(48)
    parts = [wl.as_u16(p) for p in wl.make_partials(w)]
    q = [oracle.quantize_bf16(x, w.block) for x in parts[1:]]
    want, _, _ = oracle.reduce_flat(parts[0], [c for c, _ in q], [s for _, s in q], w.block)
    dc = [torch.from_numpy(c).cuda() for c, _ in q]
    ds = [torch.from_numpy(s).cuda() for _, s in q]
    out = torch.empty(w.n, dtype=torch.bfloat16, device="cuda")
    eq.equarx_reduce_flat(gpu.dev_bf16(parts[0]), dc, ds, w.block, out)
    torch.cuda.synchronize()
    assert (gpu.host_u16(out) == want).all()
    # two quantizations per value instead of eight: lower error than the ring's chain on the same data
    ref = sum(oracle.bf16_to_f32(p).astype(np.float64) for p in parts)
    err_flat = np.mean((oracle.bf16_to_f32(want).astype(np.float64) - ref) ** 2)
    err_ring = np.mean((oracle.bf16_to_f32(oracle.reduce_chain(parts, w.block)).astype(np.float64) - ref) ** 2)
    assert err_flat < err_ring


def test_flat_bad_arguments(gpu):
    x = torch.zeros(4096, dtype=torch.bfloat16, device="cuda")
    c = torch.zeros(4096, dtype=torch.int8, device="cuda")
    s = torch.zeros(16, dtype=torch.float32, device="cuda")
    with pytest.raises(eq.EquarxError) as e:
        eq.equarx_reduce_flat(x, [c], [s], 256)                       # no output at all
    assert e.value.status == eq.STATUS_NULL_POINTER
    with pytest.raises(eq.EquarxError) as e:
        eq.equarx_reduce_flat(x, [c], [s], 256, x)                    # out aliases the local shard
    assert e.value.status == eq.STATUS_BAD_SHAPE
    with pytest.raises(eq.EquarxError) as e:
        eq.equarx_reduce_flat(x, [c], [s], 256, None, c, torch.zeros_like(s))   # codes_out aliases an input
    assert e.value.status == eq.STATUS_BAD_SHAPE
    with pytest.raises(eq.EquarxError) as e:
        eq.equarx_reduce_flat(x, [c] * 64, [s] * 64, 256, torch.empty_like(x))
    assert e.value.status == eq.STATUS_BAD_SHAPE


@pytest.mark.parametrize("B", (32, 256))
def test_quantize_batch_parity(gpu, oracle, B):
    for count, n in ((7, 2048 * 7 + 300), (1, 4096), (64, 777), (3, 1 << 20)):
        xs = [gpu.bf16_of(_values("lognormal", n, 8000 + i)) for i in range(count)]
        nb = eq.num_blocks(n, B)
        dx = [gpu.dev_bf16(x) for x in xs]
        dc = [torch.full((n,), 99, dtype=torch.int8, device="cuda") for _ in range(count)]
        ds = [torch.full((nb,), -7.0, dtype=torch.float32, device="cuda") for _ in range(count)]
        eq.equarx_quantize_batch(dx, B, dc, ds)
        torch.cuda.synchronize()
        for i in range(count if n < (1 << 20) else 2):
            c, s_ = oracle.quantize_bf16(xs[i], B)
            assert (dc[i].cpu().numpy() == c).all() and (ds[i].cpu().numpy().view(np.uint32) == s_.view(np.uint32)).all()
    eq.equarx_quantize_batch([], B, [], [])
    x = torch.zeros(4096, dtype=torch.bfloat16, device="cuda")
    c = torch.zeros(4096, dtype=torch.int8, device="cuda")
    s_ = torch.zeros(4096 // B, dtype=torch.float32, device="cuda")
    with pytest.raises(eq.EquarxError) as e:
        eq.equarx_quantize_batch([x, x], B, [c, c], [s_, torch.zeros_like(s_)])
    assert e.value.status == eq.STATUS_BAD_SHAPE


# ----------------------------------------------------------------------------- streams, repetition, graphs

def test_side_stream_and_repetition(gpu, oracle):
    """Work is enqueued on the caller's stream, in order with what the caller put there; repeated calls give
    the same bits."""
    w = CHAIN_CASES["c4"]
    host = wl.make_partials(w)
    want = oracle.reduce_chain([wl.as_u16(p) for p in host], w.block)
    side = torch.cuda.Stream()
    outs = []
    with torch.cuda.stream(side):
        dev = [torch.empty(w.n, dtype=torch.bfloat16, device="cuda") for _ in host]
        for d, p in zip(dev, host):
            d.copy_(p.reshape(-1), non_blocking=True)          # the inputs arrive on the same stream
        work = eq.alloc_workspace(w.P, w.n, w.block)
        for rep in range(3):
            out = torch.empty(w.n, dtype=torch.bfloat16, device="cuda")
            if rep == 1:
                eq.equarx_reduce_fused(dev, w.block, out)
            else:
                eq.equarx_reduce_quantized(dev, w.block, out, work)
            outs.append(out)
    side.synchronize()
    for out in outs:
        assert (gpu.host_u16(out) == want).all()


@pytest.mark.parametrize("tiles", (3, 700, 2100))
def test_in_place_output(gpu, oracle, tiles):
    """The output may be one of the partials (an AllReduce is usually called in place): every schedule, each of
    them at small_kernel's sizes and with two tiles per thread, output = first, middle and last partial."""
    n, B, P = 2048 * tiles - 700, 128, 4
    host = [gpu.bf16_of(_values("lognormal", n, 8100 + p)) for p in range(P)]
    oracle.set_threads(8)
    try:
        want = oracle.reduce_chain(host, B)
        want_semi = oracle.reduce_semi_loop(host, B, True)
        want_ring = oracle.reduce_ring(host, B)
    finally:
        oracle.set_threads(1)
    work = eq.alloc_workspace(P, n, B)
    calls = {
        "hop by hop": (lambda d, o: eq.equarx_reduce_quantized(d, B, o, work), want),
        "ends fused": (lambda d, o: eq.equarx_reduce_quantized_fused_ends(d, B, o, work), want),
        "one launch": (lambda d, o: eq.equarx_reduce_fused(d, B, o), want),
        "semi-loop": (lambda d, o: eq.equarx_reduce_variant(d, B, eq.SEMI_LOOP, o), want_semi),
        "ring order": (lambda d, o: eq.equarx_reduce_variant(d, B, eq.RING_ORDER, o), want_ring),
    }
    for name, (call, expect) in calls.items():
        for j in (0, 1, P - 1):
            dev = [gpu.dev_bf16(h) for h in host]
            call(dev, dev[j])
            torch.cuda.synchronize()
            assert (gpu.host_u16(dev[j]) == expect).all(), (name, j)
            for i in range(P):
                if i != j:
                    assert (gpu.host_u16(dev[i]) == host[i]).all(), (name, j, i)      # the others are untouched


def test_in_place_output_strided(gpu, oracle):
    chunks, P = 64, 3
    n = 3 * 1024 * chunks
    host = [gpu.bf16_of(_values("student", n, 8200 + p)) for p in range(P)]
    want = oracle.reduce_chain_strided(host, chunks)
    for fused in (False, True):
        for j in range(P):
            dev = [gpu.dev_bf16(h) for h in host]
            if fused:
                eq.equarx_reduce_fused_strided(dev, chunks, dev[j])
            else:
                eq.equarx_reduce_quantized_strided(dev, chunks, dev[j], eq.alloc_workspace(P, n, chunks))
            torch.cuda.synchronize()
            assert (gpu.host_u16(dev[j]) == want).all(), (fused, j)


def test_two_host_threads_on_two_streams(gpu, oracle):
    """The library keeps no shared state: two host threads, each with its own stream, inputs and workspace, call
    it at the same time (ctypes releases the interpreter lock during a call) and both get the oracle's bits."""
    import threading
    cases = [CHAIN_CASES["c4"], CHAIN_CASES["c2_rows24"]]
    hosts = [wl.make_partials(w) for w in cases]
    wants = [oracle.reduce_chain([wl.as_u16(p) for p in h], w.block) for w, h in zip(cases, hosts)]
    devs = [[p.reshape(-1).cuda() for p in h] for h in hosts]
    works = [eq.alloc_workspace(w.P, w.n, w.block) for w in cases]
    outs = [[torch.empty(w.n, dtype=torch.bfloat16, device="cuda") for _ in range(3)] for w in cases]
    torch.cuda.synchronize()
    errors = []

    def worker(i):
        try:
            w = cases[i]
            stream = torch.cuda.Stream()
            with torch.cuda.stream(stream):
                for rep in range(30):
                    eq.equarx_reduce_quantized(devs[i], w.block, outs[i][0], works[i])
                    eq.equarx_reduce_fused(devs[i], w.block, outs[i][1])
                    eq.equarx_reduce_quantized_fused_ends(devs[i], w.block, outs[i][2], works[i])
            stream.synchronize()
        except Exception as e:      # surfaced in the main thread below
            errors.append(e)

    threads = [threading.Thread(target=worker, args=(i,)) for i in range(2)]
    for t in threads:
        t.start()
    for t in threads:
        t.join(timeout=100)
    assert not errors, errors
    assert not any(t.is_alive() for t in threads)
    torch.cuda.synchronize()
    for i in range(2):
        for o in outs[i]:
            assert (gpu.host_u16(o) == wants[i]).all()


def test_graph_capture_and_replay(gpu, oracle):
    """The entry points only enqueue kernels, so a caller may capture them in a HIP graph.  Replays are checked
    against the oracle after the inputs changed between replays."""
    w = CHAIN_CASES["c2_rows24"]
    n, B, P = w.n, w.block, w.P
    dev = [torch.zeros(n, dtype=torch.bfloat16, device="cuda") for _ in range(P)]
    out_a = torch.zeros(n, dtype=torch.bfloat16, device="cuda")
    out_b = torch.zeros(n, dtype=torch.bfloat16, device="cuda")
    out_c = torch.zeros(n, dtype=torch.bfloat16, device="cuda")
    out_d = torch.zeros(n, dtype=torch.bfloat16, device="cuda")
    work = eq.alloc_workspace(P, n, B)
    work_c = eq.alloc_workspace(P, n, B)
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        eq.equarx_reduce_quantized(dev, B, out_a, work)
        eq.equarx_reduce_fused(dev, B, out_b)
        eq.equarx_reduce_quantized_fused_ends(dev, B, out_c, work_c)
        eq.equarx_reduce_variant(dev, B, eq.SEMI_LOOP, out_d)
    for rep in range(3):
        host = [gpu.bf16_of(_values("lognormal", n, 6000 + 10 * rep + p)) for p in range(P)]
        for d, h in zip(dev, host):
            d.copy_(gpu.dev_bf16(h))
        torch.cuda.synchronize()
        graph.replay()
        torch.cuda.synchronize()
        want = oracle.reduce_chain(host, B)
        assert (gpu.host_u16(out_a) == want).all(), rep
        assert (gpu.host_u16(out_b) == want).all(), rep
        assert (gpu.host_u16(out_c) == want).all(), rep
        assert (gpu.host_u16(out_d) == oracle.reduce_semi_loop(host, B, True)).all(), rep


# ----------------------------------------------------------------------------- the paper's strided block geometry

@pytest.mark.parametrize("chunks", (32, 64, 128))
def test_strided_parity(gpu, oracle, chunks):
    ms = 1024 * chunks
    for i, (n, kind) in enumerate([(ms, "normal"), (3 * ms, "lognormal"), (5 * ms, "student"), (2 * ms, "tiny"),
                                   (2 * ms, "sparse"), (2 * ms, "huge")]):
        x = gpu.bf16_of(_values(kind, n, 9000 + i))
        y = gpu.bf16_of(_values(kind, n, 9100 + i))
        ns = n // chunks
        dx, dy = gpu.dev_bf16(x), gpu.dev_bf16(y)
        c = torch.full((n,), 99, dtype=torch.int8, device="cuda")
        s_ = torch.full((ns,), -7.0, dtype=torch.float32, device="cuda")
        eq.equarx_quantize_strided(dx, chunks, c, s_)
        c2, s2 = torch.full_like(c, 98), torch.full_like(s_, -3.0)
        eq.equarx_reduce_stage_strided(c, s_, dy, chunks, c2, s2)
        out = torch.full((n,), 7.0, dtype=torch.bfloat16, device="cuda")
        eq.equarx_dequantize_strided(c2, s2, chunks, out)
        torch.cuda.synchronize()
        oc, os_ = oracle.quantize_bf16_strided(x, chunks)
        assert (c.cpu().numpy() == oc).all() and (s_.cpu().numpy().view(np.uint32) == os_.view(np.uint32)).all(), (n, kind)
        oc2, os2 = oracle.hop_strided(oc, os_, y, chunks)
        assert (c2.cpu().numpy() == oc2).all() and (s2.cpu().numpy().view(np.uint32) == os2.view(np.uint32)).all(), (n, kind)
        assert (gpu.host_u16(out) == oracle.dequantize_bf16_strided(oc2, os2, chunks)).all()
        # in place
        eq.equarx_reduce_stage_strided(c, s_, dy, chunks, c, s_)
        torch.cuda.synchronize()
        assert torch.equal(c, c2) and torch.equal(s_, s2)


@pytest.mark.parametrize("chunks,P", ((64, 8), (32, 3), (128, 1), (64, 16)))
def test_strided_chain_parity(gpu, oracle, chunks, P):
    n = 3 * 1024 * chunks
    parts = [gpu.bf16_of(_values("lognormal", n, 9500 + p)) for p in range(P)]
    dev = [gpu.dev_bf16(p) for p in parts]
    out = torch.full((n,), 7.0, dtype=torch.bfloat16, device="cuda")
    eq.equarx_reduce_quantized_strided(dev, chunks, out, eq.alloc_workspace(P, n, chunks))
    out_f = torch.full((n,), 3.0, dtype=torch.bfloat16, device="cuda")
    eq.equarx_reduce_fused_strided(dev, chunks, out_f)
    torch.cuda.synchronize()
    want = oracle.reduce_chain_strided(parts, chunks)
    assert (gpu.host_u16(out) == want).all()
    assert (gpu.host_u16(out_f) == want).all()


@pytest.mark.parametrize("chunks", (32, 64, 128))
def test_strided_fused_value_kinds(gpu, oracle, chunks):
    n = 2 * 1024 * chunks
    for kind in ("tiny", "sparse", "huge", "student"):
        parts = [gpu.bf16_of(_values(kind, n, 9700 + p)) for p in range(4)]
        out = torch.full((n,), 3.0, dtype=torch.bfloat16, device="cuda")
        eq.equarx_reduce_fused_strided([gpu.dev_bf16(p) for p in parts], chunks, out)
        torch.cuda.synchronize()
        assert (gpu.host_u16(out) == oracle.reduce_chain_strided(parts, chunks)).all(), kind


def test_strided_full_size_sampled(gpu, oracle):
    """27B-shaped size, block 64 as in the paper's Fig. 7: minishards are independent, so the oracle on a sample
    of minishards must reproduce the GPU's output there bit for bit."""
    w = wl.WORKLOADS["c3_gemma3_27b"]
    chunks = 64
    host = wl.make_partials(w)
    dev = [p.reshape(-1).cuda() for p in host]
    out = torch.empty(w.n, dtype=torch.bfloat16, device="cuda")
    eq.equarx_reduce_quantized_strided(dev, chunks, out, eq.alloc_workspace(w.P, w.n, chunks))
    out_f = torch.empty_like(out)
    eq.equarx_reduce_fused_strided(dev, chunks, out_f)
    torch.cuda.synchronize()
    assert torch.equal(out.view(torch.int16), out_f.view(torch.int16))
    got = gpu.host_u16(out)
    ms = 1024 * chunks
    total = w.n // ms
    pick = np.unique(np.concatenate([[0, total - 1], _rng(5).integers(0, total, 24)]))
    idx = (pick[:, None] * ms + np.arange(ms)[None, :]).reshape(-1)
    want = oracle.reduce_chain_strided([wl.as_u16(p)[idx] for p in host], chunks)
    assert (got[idx] == want).all()


def test_strided_bad_arguments(gpu):
    x = torch.zeros(1024 * 64, dtype=torch.bfloat16, device="cuda")
    c = torch.zeros(1024 * 64, dtype=torch.int8, device="cuda")
    s_ = torch.zeros(1024, dtype=torch.float32, device="cuda")
    with pytest.raises(eq.EquarxError) as e:
        eq.equarx_quantize_strided(x, 48, c, s_)
    assert e.value.status == eq.STATUS_BAD_BLOCK
    with pytest.raises(eq.EquarxError) as e:
        eq.equarx_quantize_strided(x[:1024 * 32], 64, c, s_)
    assert e.value.status == eq.STATUS_BAD_SHAPE
    with pytest.raises(eq.EquarxError) as e:
        eq.equarx_reduce_quantized_strided([x, x], 64, torch.empty_like(x), torch.empty(256, dtype=torch.uint8, device="cuda"))
    assert e.value.status == eq.STATUS_WORKSPACE_TOO_SMALL


STRIDED_VARIANTS = ("full", "rs_only", "ag_only", "semi", "semi_rs_only")


def _oracle_variant_strided(oracle, parts, chunks, flags):
    ag = not (flags & eq.AG_UNQUANTIZED)
    if flags & eq.RING_ORDER:
        return oracle.reduce_ring_strided(parts, chunks, semi=bool(flags & eq.SEMI_LOOP),
                                          quantize_rs=not (flags & eq.RS_UNQUANTIZED), quantize_ag=ag)
    if flags & eq.SEMI_LOOP:
        return oracle.reduce_semi_loop_strided(parts, chunks, ag)
    return oracle.reduce_stages_strided(parts, chunks, not (flags & eq.RS_UNQUANTIZED), ag)


@pytest.mark.parametrize("name", STRIDED_VARIANTS)
@pytest.mark.parametrize("chunks", (32, 64, 128))
def test_strided_variant_parity(gpu, oracle, name, chunks):
    """Semi-loop and stage knob in the strided geometry: the oracle's bits for every device count's chain lengths
    (P = 1, 2, 3: a chain of the semi-loop is missing or a single send), for values whose zeros carry a sign
    ("sparse": products with -0.0) and for the extreme ranges; output in place for some."""
    flags = VARIANT_FLAGS[name]
    ms = 1024 * chunks
    cases = [(1, 1, "normal"), (2, 2, "sparse"), (3, 3, "lognormal"), (4, 2, "tiny"), (5, 2, "sparse"), (8, 3, "student"),
             (9, 1, "huge"), (16, 1, "normal")]
    for k, (P, count, kind) in enumerate(cases):
        n = count * ms
        parts = [gpu.bf16_of(_values(kind, n, 9800 + 11 * p + P)) for p in range(P)]
        want = _oracle_variant_strided(oracle, parts, chunks, flags)
        dev = [gpu.dev_bf16(p) for p in parts]
        out = dev[P // 2] if k % 2 else torch.full((n,), 5.0, dtype=torch.bfloat16, device="cuda")
        eq.equarx_reduce_variant_strided(dev, chunks, flags, out)
        torch.cuda.synchronize()
        got = gpu.host_u16(out)
        assert (got == want).all(), (name, chunks, P, kind, int((got != want).sum()))
        if name == "full":
            assert (want == oracle.reduce_chain_strided(parts, chunks)).all()


@pytest.mark.parametrize("name", ("full", "rs_only", "semi", "semi_rs_only", "ring", "ring_rs_only", "ring_semi",
                                  "ring_semi_rs_only"))
@pytest.mark.parametrize("chunks", (32, 64, 128))
def test_strided_variant_hop_by_hop_parity(gpu, oracle, name, chunks):
    """The strided flavours in the ring-imposed schedule (one launch per send, wires in memory): the oracle's bits,
    which are also the single launch's; every chain length of the semi-loop; output in place for some."""
    flags = VARIANT_FLAGS[name]
    ms = 1024 * chunks
    for k, (P, count, kind) in enumerate([(1, 1, "normal"), (2, 2, "sparse"), (3, 1, "lognormal"), (4, 2, "tiny"),
                                          (5, 3, "sparse"), (6, 1, "student"), (8, 2, "lognormal"), (9, 1, "huge")]):
        n = count * ms
        parts = [gpu.bf16_of(_values(kind, n, 9900 + 11 * p + P)) for p in range(P)]
        want = _oracle_variant_strided(oracle, parts, chunks, flags)
        dev = [gpu.dev_bf16(p) for p in parts]
        out = dev[(P - 1) // 2] if k % 2 else torch.full((n,), 5.0, dtype=torch.bfloat16, device="cuda")
        ws = eq.alloc_variant_workspace(flags & ~eq.RING_ORDER, P, n, chunks)
        eq.equarx_reduce_variant_hops_strided(dev, chunks, flags, out, ws)
        torch.cuda.synchronize()
        got = gpu.host_u16(out)
        assert (got == want).all(), (name, chunks, P, kind, int((got != want).sum()))
        for i, d in enumerate(dev):
            if d is not out:
                assert (gpu.host_u16(d) == parts[i]).all(), (name, P, i)          # the other partials are untouched


@pytest.mark.parametrize("name", ("ring", "ring_rs_only", "ring_ag_only", "ring_semi", "ring_semi_rs_only"))
@pytest.mark.parametrize("chunks", (32, 64, 128))
def test_strided_variant_ring_order_parity(gpu, oracle, name, chunks):
    """The ring layout in the strided geometry (shards of whole minishards, shard k ending on device k): rings
    shorter than, as long as and longer than the tensor has minishards (short and empty shards)."""
    flags = VARIANT_FLAGS[name]
    ms = 1024 * chunks
    for k, (P, count, kind) in enumerate([(1, 2, "normal"), (2, 3, "sparse"), (3, 4, "lognormal"), (4, 4, "student"),
                                          (5, 2, "sparse"), (8, 11, "normal"), (9, 3, "tiny")]):
        n = count * ms
        parts = [gpu.bf16_of(_values(kind, n, 9950 + 11 * p + P)) for p in range(P)]
        want = _oracle_variant_strided(oracle, parts, chunks, flags)
        dev = [gpu.dev_bf16(p) for p in parts]
        out = dev[P // 2] if k % 2 else torch.full((n,), 5.0, dtype=torch.bfloat16, device="cuda")
        eq.equarx_reduce_variant_strided(dev, chunks, flags, out)
        torch.cuda.synchronize()
        got = gpu.host_u16(out)
        assert (got == want).all(), (name, chunks, P, count, kind, int((got != want).sum()))


def test_strided_variant_full_size_sampled(gpu, oracle):
    """The Fig. 7 tensor ((4096, 4096), N(0,1), 8 devices, block 64 = 64 chunks) in the paper's own geometry, every
    flavour the figure compares: sampled minishards against the oracle, and the figure's error figures and their
    order on the whole output."""
    w = wl.FIG7
    chunks = w.block
    u16 = [wl.as_u16(p) for p in wl.make_partials(w)]
    dev = [gpu.dev_bf16(p) for p in u16]
    ms = 1024 * chunks
    total = w.n // ms
    pick = np.unique(np.concatenate([[0, total - 1], _rng(66).integers(0, total, 20)]))
    idx = (pick[:, None] * ms + np.arange(ms)[None, :]).reshape(-1)
    sub = [p[idx] for p in u16]
    ref = torch.zeros(w.n, dtype=torch.float64, device="cuda")
    for d in dev:
        ref += d.double()
    base = ref.float().to(torch.bfloat16).double()
    out = torch.empty(w.n, dtype=torch.bfloat16, device="cuda")
    mse = {}
    oracle.set_threads(8)
    try:
        for name in STRIDED_VARIANTS:
            flags = VARIANT_FLAGS[name]
            out.fill_(3.0)
            eq.equarx_reduce_variant_strided(dev, chunks, flags, out)
            torch.cuda.synchronize()
            assert (gpu.host_u16(out)[idx] == _oracle_variant_strided(oracle, sub, chunks, flags)).all(), name
            mse[name] = float(((out.double() - base) ** 2).mean())
            if name != "ag_only":       # without a quantized reduce-scatter there is no hop-by-hop form
                hops = torch.full_like(out, 3.0)
                eq.equarx_reduce_variant_hops_strided(dev, chunks, flags, hops,
                                                      eq.alloc_variant_workspace(flags, w.P, w.n, chunks))
                torch.cuda.synchronize()
                assert torch.equal(hops.view(torch.int16), out.view(torch.int16)), name + " hop by hop"
        # the ring layout at full size: 256 minishards, 32 per shard, every element against the oracle
        for name in ("ring", "ring_semi"):
            flags = VARIANT_FLAGS[name]
            out.fill_(3.0)
            eq.equarx_reduce_variant_strided(dev, chunks, flags, out)
            torch.cuda.synchronize()
            assert (gpu.host_u16(out) == _oracle_variant_strided(oracle, u16, chunks, flags)).all(), name
            hops = torch.full_like(out, 3.0)
            eq.equarx_reduce_variant_hops_strided(dev, chunks, flags, hops,
                                                  eq.alloc_variant_workspace(flags & ~eq.RING_ORDER, w.P, w.n, chunks))
            torch.cuda.synchronize()
            assert torch.equal(hops.view(torch.int16), out.view(torch.int16)), name + " hop by hop"
    finally:
        oracle.set_threads(1)
    assert mse["ag_only"] < mse["semi"] < mse["full"] and mse["rs_only"] < mse["full"]
    assert 0.0014 / 1.5 < mse["full"] < 0.0014 * 1.5 and 0.001 / 1.5 < mse["semi"] < 0.001 * 1.5
    assert 0.0003 / 1.5 < mse["ag_only"] < 0.0003 * 1.5
    fused = torch.empty_like(out)
    eq.equarx_reduce_fused_strided(dev, chunks, fused)
    eq.equarx_reduce_variant_strided(dev, chunks, 0, out)
    torch.cuda.synchronize()
    assert torch.equal(out.view(torch.int16), fused.view(torch.int16))


def test_strided_variant_bad_arguments(gpu):
    x = torch.zeros(1024 * 64, dtype=torch.bfloat16, device="cuda")
    out = torch.empty_like(x)
    for flags in (eq.RS_UNQUANTIZED | eq.AG_UNQUANTIZED, eq.SEMI_LOOP | eq.RS_UNQUANTIZED,
                  eq.RING_ORDER | eq.SEMI_LOOP | eq.RS_UNQUANTIZED, 16, 1 << 31):
        with pytest.raises(eq.EquarxError) as e:
            eq.equarx_reduce_variant_strided([x, x], 64, flags, out)
        assert e.value.status == eq.STATUS_BAD_SHAPE
    ws = eq.alloc_variant_workspace(eq.SEMI_LOOP, 2, x.numel(), 64)
    for flags in (eq.RS_UNQUANTIZED, eq.RING_ORDER | eq.RS_UNQUANTIZED, 16):
        with pytest.raises(eq.EquarxError) as e:
            eq.equarx_reduce_variant_hops_strided([x, x], 64, flags, out, ws)
        assert e.value.status == eq.STATUS_BAD_SHAPE
    with pytest.raises(eq.EquarxError) as e:
        eq.equarx_reduce_variant_hops_strided([x, x], 64, eq.SEMI_LOOP, out, ws[:256])
    assert e.value.status == eq.STATUS_WORKSPACE_TOO_SMALL
    with pytest.raises(eq.EquarxError) as e:
        eq.equarx_reduce_variant_strided([x, x], 48, 0, out)
    assert e.value.status == eq.STATUS_BAD_BLOCK
    with pytest.raises(eq.EquarxError) as e:
        eq.equarx_reduce_variant_strided([x[:1024 * 32], x[:1024 * 32]], 64, 0, out[:1024 * 32])
    assert e.value.status == eq.STATUS_BAD_SHAPE


# ----------------------------------------------------------------------------- lengths beyond 32-bit indices

def test_length_beyond_two_to_the_31(gpu, oracle):
    """A tensor of more than 2^31 elements (4.3 GB of bf16): element indices need 64 bits in every kernel.
    Blocks are independent, so blocks sampled at the start, on both sides of the 2^31 boundary and at the ragged
    end are checked against the oracle bit for bit, for quantize, hop, dequantize and the single-launch chain."""
    n, B = (1 << 31) + 2048 * 5 + 24, 256
    g = torch.Generator(device="cuda")
    g.manual_seed(77)
    x = torch.randn(n, generator=g, device="cuda", dtype=torch.bfloat16)
    y = torch.randn(n, generator=g, device="cuda", dtype=torch.bfloat16)
    nb = eq.num_blocks(n, B)
    c = torch.empty(n, dtype=torch.int8, device="cuda")
    s_ = torch.empty(nb, dtype=torch.float32, device="cuda")
    c2 = torch.empty(n, dtype=torch.int8, device="cuda")
    s2 = torch.empty(nb, dtype=torch.float32, device="cuda")
    out = torch.empty(n, dtype=torch.bfloat16, device="cuda")
    eq.equarx_quantize(x, B, c, s_)
    eq.equarx_reduce_stage(c, s_, y, B, c2, s2)
    eq.equarx_dequantize(c2, s2, B, out)
    out_f = torch.empty(n, dtype=torch.bfloat16, device="cuda")
    eq.equarx_reduce_fused([x, y], B, out_f)
    torch.cuda.synchronize()
    assert torch.equal(out.view(torch.int16), out_f.view(torch.int16))

    edge = (1 << 31) // B
    blocks = np.unique(np.concatenate([np.arange(0, 4), np.arange(edge - 4, edge + 4), np.arange(nb - 6, nb),
                                       _rng(3).integers(0, nb, 200)]))
    for b in blocks:
        lo, hi = int(b) * B, min(n, (int(b) + 1) * B)
        xs = x[lo:hi].view(torch.int16).cpu().numpy().view(np.uint16)
        ys = y[lo:hi].view(torch.int16).cpu().numpy().view(np.uint16)
        oc, os_ = oracle.quantize_bf16(xs, B)
        assert (c[lo:hi].cpu().numpy() == oc).all() and s_[b].item() == os_[0], b
        oc2, os2 = oracle.hop(oc, os_, ys, B)
        assert (c2[lo:hi].cpu().numpy() == oc2).all() and s2[b].item() == os2[0], b
        assert (out[lo:hi].view(torch.int16).cpu().numpy().view(np.uint16) == oracle.dequantize_bf16(oc2, os2, B)).all(), b


# ----------------------------------------------------------------------------- the benchmark's output line

def test_bench_prints_one_json_line_with_the_contract_keys(gpu):
    """bench.py on the small config: exactly one line on stdout, JSON, with the keys the driver and the judge read."""
    import json
    import os
    import subprocess
    import sys
    root = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
    run = subprocess.run([sys.executable, os.path.join(root, "bench.py"), "--workload", "c2_gemma3_12b", "--rows", "64",
                          "--steps", "6", "--warmup", "2", "--cpu-seconds", "1"],
                         capture_output=True, text=True, timeout=170)
    assert run.returncode == 0, run.stderr[-2000:]
    lines = [l for l in run.stdout.splitlines() if l.strip()]
    assert len(lines) == 1, lines
    d = json.loads(lines[0])
    for key in ("metric", "value", "unit", "n_gpus", "steps", "warmup", "ms_per_step", "higher_is_better", "scaling",
                "vs_baseline", "dtype", "data", "config", "roofline", "cpu_baseline"):
        assert key in d, key
    assert d["n_gpus"] == 1 and d["steps"] == 6 and d["warmup"] == 2 and d["unit"] == "GB/s" and d["value"] > 0
    assert d["vs_baseline"] is None and d["data"] == "synthetic" and "workload" in d["config"]
    r = d["roofline"]
    assert r["bound"] == "hbm" and r["peak"] == 8000.0 and r["unit"] == "GB/s"
    assert abs(r["frac"] - r["achieved"] / r["peak"]) < 1e-3 and "traffic" in r
    c = d["cpu_baseline"]
    assert c["kind"] == "oracle" and c["cores"] >= 1 and c["value"] > 0 and c["sample"] and c["cpu_model"]
    assert r["cold_wire"] is None           # a message this small is never cold: the figure is not reported
    # a message large enough for the cold-wire arrangement: both fractions are on the line, each labelled
    run = subprocess.run([sys.executable, os.path.join(root, "bench.py"), "--rows", "2048", "--steps", "8", "--warmup", "2",
                          "--cpu-seconds", "0"], capture_output=True, text=True, timeout=170)
    assert run.returncode == 0, run.stderr[-2000:]
    d = json.loads(run.stdout.strip())
    r = d["roofline"]
    assert 0.2 < r["frac"] < 1.0 and 0.2 < r["cold_wire"]["frac"] < 1.0 and "warm" in r["measured"]
    assert r["traffic_level"].startswith("bytes between L2") and d["chain"]["cold_wire"]["chains_interleaved"] >= 3
    assert {"ms_per_step", "frac_of_hbm_peak", "cacheable_wire_ms_per_step"} <= set(d["chain"]["cold_wire"])
