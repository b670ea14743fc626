"""Sizes on both sides of every line at which a call changes its launch shape, against the oracle, bit for bit."""
import numpy as np
import pytest
import torch

from paper_2506_17615_amd import binding as eq
from test_parity_gpu import _oracle_variant, _oracle_variant_strided, _values, gpu  # noqa: F401  (the fixture that loads the library)

pytestmark = pytest.mark.gpu

FIVE_PER_CU = 5 * 256 * 4096    # single-launch calls: up to here 256 threads x 2 tiles
WIDE_ROUND = 768 * 8192         # single-launch calls: up to here 512 threads x 2 tiles, above 1024 x 1
PAIRED_FROM = 2560 * 8192       # single-launch chain: above, 256 threads x 4 tiles
CACHED_OUT = 32 << 20           # single-launch calls: up to here the output stays in the Infinity Cache
TURN_FROM = 20 << 20            # elements of wire: from here every second launch of a hop-by-hop chain walks back
ONE_WAVE_EACH = 1024 * 256      # small single-launch calls: up to here 4 elements per lane, and above by waves per SIMD
PAIR_ROUND = 1792 * 4096        # a dequantization of a wire that arrived: up to here 256 threads x 2 tiles
LONG_DEQUANTIZE = 13 << 20      # ... and from here 1024 x 1
ONE_ROUND = 2048 * 2048         # elements: up to here one tile of 256 threads per workgroup, above 512 threads x 2 tiles


@pytest.fixture(scope="module")
def values(gpu):  # noqa: F811
    """Partials of the longest length used here; shorter ones are slices of them."""
    rng = np.random.default_rng(77)
    n = ONE_ROUND + (1 << 17)
    return [gpu.bf16_of(rng.standard_normal(n, dtype=np.float32) * np.exp2(rng.integers(-3, 4, n)).astype(np.float32))
            for _ in range(4)]


@pytest.fixture(autouse=True)
def threads(oracle):
    oracle.set_threads(8)
    yield
    oracle.set_threads(1)


def _bits(t):
    return t.cpu().numpy().view(np.uint32)


@pytest.mark.parametrize("n", (ONE_ROUND - 5, ONE_ROUND, ONE_ROUND + 1, ONE_ROUND + 8192 + 4096 + 24))
@pytest.mark.parametrize("B", (32, 512))
def test_passes_around_one_round_of_workgroups(gpu, oracle, values, n, B):  # noqa: F811
    x = [v[:n] for v in values[:3]]
    want, wc, ws = oracle.reduce_chain(x, B, keep_wire=True)
    got, c, s = gpu.gpu_chain_per_step(x, B)
    assert (got == want).all() and (c == wc).all() and (s.view(np.uint32) == ws.view(np.uint32)).all()
    assert (gpu.gpu_chain(x, B, keep_wire=False) == want).all()
    assert (gpu.gpu_chain_fused_ends(x, B) == want).all()
    for flags in (eq.AG_UNQUANTIZED, eq.RING_ORDER, eq.SEMI_LOOP, eq.SEMI_LOOP | eq.RING_ORDER):
        out = torch.empty(n, dtype=torch.bfloat16, device="cuda")
        eq.equarx_reduce_variant_hops([gpu.dev_bf16(p) for p in x], B, flags, out,
                                      eq.alloc_variant_workspace(flags, 3, n, B))
        assert (gpu.host_u16(out) == _oracle_variant(oracle, x, B, flags)).all(), flags


@pytest.mark.parametrize("n", (ONE_ROUND // 2 - 3, ONE_ROUND // 2 + 1))
def test_two_directions_around_one_round_of_workgroups(gpu, oracle, values, n):  # noqa: F811
    x, flags = [v[:n] for v in values], eq.SEMI_LOOP | eq.RING_ORDER
    out = torch.empty(n, dtype=torch.bfloat16, device="cuda")
    eq.equarx_reduce_variant_hops([gpu.dev_bf16(p) for p in x], 64, flags, out,
                                  eq.alloc_variant_workspace(flags, 4, n, 64))
    assert (gpu.host_u16(out) == _oracle_variant(oracle, x, 64, flags)).all()


@pytest.mark.parametrize("n,P,B", ((TURN_FROM - 1, 4, 256), (TURN_FROM, 3, 32), (TURN_FROM + 5 * 8192 + 3, 4, 512),
                                   (TURN_FROM + 8 * 8192, 5, 64), (TURN_FROM // 2, 5, 128), (TURN_FROM // 2 + 4099, 4, 64),
                                   (TURN_FROM - 3, 2, 64), (TURN_FROM + 4097, 2, 128)))
def test_chains_that_turn(gpu, oracle, long_values, n, P, B):  # noqa: F811
    x = [np.resize(long_values[i % 3], n + i)[i:].copy() for i in range(P)]
    dev = [gpu.dev_bf16(p) for p in x]
    out = torch.empty(n, dtype=torch.bfloat16, device="cuda")
    flavours = (eq.SEMI_LOOP | eq.RING_ORDER,)
    if n >= TURN_FROM - 3:
        want = oracle.reduce_chain(x, B)
        eq.equarx_reduce_quantized(dev, B, out.fill_(5.0), eq.alloc_workspace(P, n, B))
        assert (gpu.host_u16(out) == want).all()
        eq.equarx_reduce_quantized_static(dev, B, out.fill_(5.0))
        assert (gpu.host_u16(out) == want).all()
        eq.equarx_reduce_quantized_fused_ends(dev, B, out.fill_(5.0), eq.alloc_workspace(P, n, B))
        assert (gpu.host_u16(out) == want).all()
        flavours += (0, eq.AG_UNQUANTIZED, eq.RING_ORDER, eq.RING_ORDER | eq.AG_UNQUANTIZED, eq.SEMI_LOOP)
    for flags in flavours:
        eq.equarx_reduce_variant_hops(dev, B, flags, out.fill_(5.0), eq.alloc_variant_workspace(flags, P, n, B))
        assert (gpu.host_u16(out) == _oracle_variant(oracle, x, B, flags)).all(), flags


@pytest.mark.parametrize("n,B", ((TURN_FROM + 8 * 8192, 32), (TURN_FROM + 4097, 128)))
def test_a_kept_wire_does_not_turn(gpu, oracle, long_values, n, B):  # noqa: F811
    x = [np.resize(long_values[i], n + i)[i:].copy() for i in range(3)]
    want, wc, ws = oracle.reduce_chain(x, B, keep_wire=True)
    got, c, s, _ = gpu.gpu_chain(x, B)
    assert (got == want).all() and (c == wc).all() and (s.view(np.uint32) == ws.view(np.uint32)).all()


@pytest.mark.parametrize("n,P", ((4099, 2), (4099, 5), (ONE_ROUND - 3, 4), (ONE_ROUND, 3), (ONE_ROUND + 1, 4)))
@pytest.mark.parametrize("flags", (eq.RING_ORDER, eq.RING_ORDER | eq.AG_UNQUANTIZED))
def test_short_chains_in_ring_order_take_their_buffers_in_turn(gpu, oracle, values, n, P, flags):  # noqa: F811
    x = [np.resize(values[i % 4], n + i)[i:].copy() for i in range(P)]
    work, out = eq.alloc_variant_workspace(flags, P, n, 64).fill_(0x55), torch.empty(n, dtype=torch.bfloat16, device="cuda")
    eq.equarx_reduce_variant_hops([gpu.dev_bf16(p) for p in x], 64, flags, out, work)
    assert (gpu.host_u16(out) == _oracle_variant(oracle, x, 64, flags)).all()
    second = work[work.numel() // 2:]
    assert bool((second[:n] != 0x55).any()) == (P > 2 and n <= ONE_ROUND)


@pytest.mark.parametrize("n", (4099, ONE_ROUND // 2 - 5, ONE_ROUND // 2 + 1, ONE_ROUND + 9, TURN_FROM // 2 + 4099))
@pytest.mark.parametrize("P", (1, 2, 3, 4, 6, 8))
def test_a_tile_of_the_two_directions_stays_on_its_xcd(gpu, oracle, values, n, P):  # noqa: F811
    """Workgroup b runs on XCD b % 8: every launch has the same rows of the same workgroups, and a direction's are a
    multiple of eight (unless a row is a single one, and P even)."""
    flags = eq.SEMI_LOOP | eq.RING_ORDER
    x = [np.resize(values[i % 4], n + i)[i:].copy() for i in range(P)]
    dev, work = [gpu.dev_bf16(p) for p in x], eq.alloc_variant_workspace(flags, P, n, 64)
    out = torch.empty(n, dtype=torch.bfloat16, device="cuda")
    call = lambda: eq.equarx_reduce_variant_hops(dev, 64, flags, out, work)       # noqa: E731
    call()
    assert (gpu.host_u16(out) == _oracle_variant(oracle, x, 64, flags)).all()
    made = gpu.launches(call)
    assert len(made) == P // 2 + 1 and [g[2] for g, _ in made] == [2] * (P // 2) + [1]
    (x, y), = {g[:2] for g, _ in made}
    assert len({b for _, b in made}) == 1 and (x * y % 8 == 0 or (x == 1 and P % 2 == 0))


@pytest.mark.parametrize("n", (ONE_ROUND // 2, ONE_ROUND // 2 + 3))
def test_batch_around_one_round_of_workgroups(gpu, oracle, values, n):  # noqa: F811
    x, nb = [v[:n] for v in values[:2]], eq.num_blocks(n, 128)
    codes = [torch.empty(n, dtype=torch.int8, device="cuda") for _ in x]
    scales = [torch.empty(nb, dtype=torch.float32, device="cuda") for _ in x]
    eq.equarx_quantize_batch([gpu.dev_bf16(p) for p in x], 128, codes, scales)
    for p, c, s in zip(x, codes, scales):
        wc, ws = oracle.quantize_bf16(p, 128)
        assert (c.cpu().numpy() == wc).all() and (_bits(s) == ws.view(np.uint32)).all()


@pytest.mark.parametrize("n", (PAIR_ROUND, PAIR_ROUND + 1, PAIR_ROUND + 4099, LONG_DEQUANTIZE - 1, LONG_DEQUANTIZE,
                               LONG_DEQUANTIZE + 8192 * 3 + 7))
@pytest.mark.parametrize("B", (32, 256, 512))
def test_steps_of_a_ring_around_their_shapes(gpu, oracle, long_values, n, B):  # noqa: F811
    x, nb = long_values[0][:n], eq.num_blocks(n, B)
    codes = torch.full((n + 16,), 77, dtype=torch.int8, device="cuda")
    scales = torch.full((nb + 4,), 7.0, dtype=torch.float32, device="cuda")
    out = torch.full((n + 8,), 3.0, dtype=torch.bfloat16, device="cuda")
    eq.equarx_quantize(gpu.dev_bf16(x), B, codes[:n], scales[:nb])
    wc, ws = oracle.quantize_bf16(x, B)
    assert (codes[:n].cpu().numpy() == wc).all() and (_bits(scales[:nb]) == ws.view(np.uint32)).all()
    eq.equarx_dequantize(codes[:n], scales[:nb], B, out[:n])
    assert (gpu.host_u16(out[:n]) == oracle.dequantize_bf16(wc, ws, B)).all()
    assert (codes[n:] == 77).all() and (scales[nb:] == 7.0).all() and (out[n:] == 3.0).all()


SINGLE = (0, eq.RING_ORDER, eq.AG_UNQUANTIZED, eq.RS_UNQUANTIZED | eq.RING_ORDER, eq.SEMI_LOOP,
          eq.SEMI_LOOP | eq.RING_ORDER | eq.AG_UNQUANTIZED)


@pytest.mark.parametrize("n,flags", [(n, f) for n in (ONE_ROUND - 11, ONE_ROUND + 3, WIDE_ROUND, WIDE_ROUND + 8 * 1024 + 17)
                                     for f in SINGLE] + [(PAIRED_FROM, 0), (PAIRED_FROM + 5, 0)])
def test_single_launch_around_its_shapes(gpu, oracle, n, flags):  # noqa: F811
    rng = np.random.default_rng(n % 1000 + flags)
    x = [gpu.bf16_of(rng.standard_normal(n, dtype=np.float32)) for _ in range(3)]
    B = 64 if flags & eq.RING_ORDER else 256
    assert (gpu.gpu_variant(x, B, flags) == _oracle_variant(oracle, x, B, flags)).all()


@pytest.mark.parametrize("flags,P,lanes", ((0, 4, "488888"), (0, 8, "488888"), (0, 9, "484844"), (0, 14, "484844"), (0, 15, "484848"),
                                           (0, 24, "484848"), (0, 25, "488848"), (eq.AG_UNQUANTIZED, 12, "484844"),
                                           (eq.SEMI_LOOP, 5, "444444"), (eq.SEMI_LOOP, 16, "444444"),
                                           (eq.SEMI_LOOP, 17, "484888"), (eq.SEMI_LOOP, 25, "484888")))
def test_elements_per_lane_by_waves_per_simd(gpu, flags, P, lanes):  # noqa: F811
    """Of small single launches of 1 to 6 waves of 4 elements per lane for each SIMD, at both ends of each; the last partial on
    a 128-byte line and 16 bytes off one."""
    x, out = (torch.zeros(6 * ONE_WAVE_EACH + 8, dtype=torch.bfloat16, device="cuda") for _ in range(2))
    off_lines = "484888" if flags & eq.SEMI_LOOP or 8 < P <= 12 else "488888"
    for at, by_waves in ((0, lanes), (8, off_lines)):
        for waves, lane in enumerate(by_waves, 1):
            half = waves == 3 and at and P > 16         # of the third wave, at most
            for n in ((waves - 1) * ONE_WAVE_EACH + 1 if waves > 1 else 70000, waves * ONE_WAVE_EACH - half * ONE_WAVE_EACH // 2):
                parts = [x[:n]] * (P - 1) + [x[at:at + n]]
                made, = gpu.launches(lambda: eq.equarx_reduce_variant(parts, 256, flags, out[:n]))
                assert made[1] == ((64, 1, 1) if lane == "4" else (256, 1, 1)), (at, n, made)


@pytest.mark.parametrize("flags,P,n,lane", ((eq.SEMI_LOOP, 24, 2 * ONE_WAVE_EACH, 8),
                                            (eq.SEMI_LOOP | eq.RING_ORDER, 24, 2 * ONE_WAVE_EACH, 4),
                                            (eq.SEMI_LOOP | eq.RING_ORDER, 17, 2 * ONE_WAVE_EACH, 4),
                                            (eq.SEMI_LOOP | eq.RING_ORDER, 16, 2 * ONE_WAVE_EACH, 4),
                                            (eq.RING_ORDER, 12, 2 * ONE_WAVE_EACH, 4), (0, 12, 2 * ONE_WAVE_EACH, 8),
                                            (eq.RING_ORDER, 17, 3 * ONE_WAVE_EACH, 8), (0, 17, 3 * ONE_WAVE_EACH, 4)))
def test_elements_per_lane_of_shards(gpu, oracle, values, flags, P, n, lane):  # noqa: F811
    """Twelve and more shards whose last workgroups make the layouts' rounds different ones from the whole message's."""
    x = [values[i % 4][:n] for i in range(P)]
    dev, out = [gpu.dev_bf16(p) for p in x], torch.full((n,), 7.0, dtype=torch.bfloat16, device="cuda")
    made, = gpu.launches(lambda: eq.equarx_reduce_variant(dev, 256, flags, out))
    assert made[1] == ((64, 1, 1) if lane == 4 else (256, 1, 1)), made
    eq.equarx_reduce_variant(dev, 256, flags, out)
    assert (gpu.host_u16(out) == _oracle_variant(oracle, x, 256, flags)).all()


@pytest.mark.parametrize("n", (1, 2, 3, 255, 257, 4097, 65 * 1024 + 2, ONE_WAVE_EACH - 1, ONE_WAVE_EACH, ONE_WAVE_EACH + 1,
                               2 * ONE_WAVE_EACH, 2 * ONE_WAVE_EACH + 5))
@pytest.mark.parametrize("P", (4, 8, 9, 16, 17, 33))
def test_small_single_launches_by_elements_per_lane(gpu, oracle, values, n, P):  # noqa: F811
    """Every flavour around the ends of a lane's words, a wave's tile and the lines between the layouts, kept wire included."""
    x = [values[i % 4][i:i + n] for i in range(P)]
    one = gpu.dev_bf16(np.concatenate([np.concatenate([v, np.zeros(-n % 8 + 8, v.dtype)]) for v in x]))
    off_lines = [one[i * (n + -n % 8 + 8):][:n] for i in range(P)]
    for k, flags in enumerate(SINGLE):
        B = (32, 64, 128, 256, 512)[(n + P + k) % 5]
        want = _oracle_variant(oracle, x, B, flags)
        assert (gpu.gpu_variant(x, B, flags) == want).all(), (B, flags)
        out = torch.full((n,), 7.0, dtype=torch.bfloat16, device="cuda")
        eq.equarx_reduce_variant(off_lines, B, flags, out)
        assert (gpu.host_u16(out) == want).all(), (B, flags)
    B = (32, 64, 128, 256, 512)[(n + 2 * P) % 5]
    want, wc, ws = oracle.reduce_chain(x, B, keep_wire=True)
    got, c, s = gpu.gpu_chain_fused(x, B)
    assert (got == want).all() and (c == wc).all() and (s.view(np.uint32) == ws.view(np.uint32)).all()


@pytest.fixture(scope="module")
def long_values(gpu):  # noqa: F811
    rng = np.random.default_rng(78)
    return [gpu.bf16_of(rng.standard_normal(PAIRED_FROM + 5, dtype=np.float32)) for _ in range(3)]


@pytest.mark.parametrize("P,cut", ((3, 0), (7, 0), (8, 0), (8, 5), (8, 5 + 2048 * 3)))
@pytest.mark.parametrize("B,flags", ((128, 0), (64, eq.RING_ORDER), (128, eq.RING_ORDER | eq.AG_UNQUANTIZED),
                                     (256, eq.RS_UNQUANTIZED), (32, eq.AG_UNQUANTIZED), (512, eq.RS_UNQUANTIZED | eq.RING_ORDER)))
def test_longest_messages_by_partials(gpu, oracle, long_values, P, cut, B, flags):  # noqa: F811
    """256 threads x 4 tiles, with and without two pieces of a block per lane, and what stays below: every flavour."""
    x = [long_values[i % 3][:PAIRED_FROM + 5 - cut] for i in range(P)]
    assert (gpu.gpu_variant(x, B, flags) == _oracle_variant(oracle, x, B, flags)).all()


@pytest.mark.parametrize("B", (64, 256))
def test_longest_messages_in_place_and_with_their_wire(gpu, oracle, long_values, B):  # noqa: F811
    x = [long_values[i % 3] for i in range(8)]
    want = oracle.reduce_chain(x, B)
    dev = [gpu.dev_bf16(v) for v in long_values]
    out = dev[1].clone()
    eq.equarx_reduce_fused([dev[0], out] + [dev[i % 3] for i in range(2, 8)], B, out)
    assert (gpu.host_u16(out) == want).all()
    x = x[:4]
    want, wc, ws = oracle.reduce_chain(x, B, keep_wire=True)
    got, c, s = gpu.gpu_chain_fused(x, B)
    assert (got == want).all() and (c == wc).all() and (s.view(np.uint32) == ws.view(np.uint32)).all()


@pytest.mark.parametrize("n", (FIVE_PER_CU, FIVE_PER_CU - 4096 + 37, FIVE_PER_CU + 1))
@pytest.mark.parametrize("flags", SINGLE)
def test_single_launch_around_five_workgroups_per_cu(gpu, oracle, n, flags):  # noqa: F811
    rng = np.random.default_rng(n % 1000 + flags)
    x = [gpu.bf16_of(rng.standard_normal(n, dtype=np.float32)) for _ in range(3)]
    B = 512 if flags & eq.RING_ORDER else 32
    assert (gpu.gpu_variant(x, B, flags) == _oracle_variant(oracle, x, B, flags)).all()


@pytest.mark.parametrize("n", (ONE_ROUND + 24, WIDE_ROUND + 3))
def test_kept_wire_above_one_round(gpu, oracle, n):  # noqa: F811
    rng = np.random.default_rng(n % 1000)
    x = [gpu.bf16_of(rng.standard_normal(n, dtype=np.float32)) for _ in range(2)]
    want, wc, ws = oracle.reduce_chain(x, 128, keep_wire=True)
    got, c, s = gpu.gpu_chain_fused(x, 128)
    assert (got == want).all() and (c == wc).all() and (s.view(np.uint32) == ws.view(np.uint32)).all()


@pytest.mark.parametrize("n,P", ((FIVE_PER_CU - 5, 2), (FIVE_PER_CU + 19, 6), (FIVE_PER_CU + 19, 7), (WIDE_ROUND, 2),
                                 (CACHED_OUT // 4, 4), (CACHED_OUT // 4 + 1, 4)))
def test_kept_wire_around_its_shapes(gpu, oracle, values, n, P):  # noqa: F811
    x = [np.concatenate([values[i % 4], values[(i + 1) % 4]])[:n] for i in range(P)]
    want, wc, ws = oracle.reduce_chain(x, 32, keep_wire=True)
    got, c, s = gpu.gpu_chain_fused(x, 32)
    assert (got == want).all() and (c == wc).all() and (s.view(np.uint32) == ws.view(np.uint32)).all()


@pytest.mark.parametrize("n", (CACHED_OUT, CACHED_OUT + 1))
@pytest.mark.parametrize("flags", (0, eq.SEMI_LOOP))
def test_output_around_the_cache_rule(gpu, oracle, n, flags):  # noqa: F811
    rng = np.random.default_rng(n % 1000)
    one = gpu.bf16_of(rng.standard_normal(n, dtype=np.float32))
    assert (gpu.gpu_variant([one, one], 32, flags) == _oracle_variant(oracle, [one, one], 32, flags)).all()


@pytest.mark.parametrize("R", (0, 1, 2, 3, 4, 5, 8, 9, 16, 17))
@pytest.mark.parametrize("n", (2048 * 3 + 40, ONE_ROUND + 8192 + 11))
def test_flat_batches_of_received_wires(gpu, oracle, values, n, R):  # noqa: F811
    if n > ONE_ROUND and R > 3:
        n = ONE_ROUND + 3
    B, local = 64, values[0][:n]
    q = [oracle.quantize_bf16(values[1 + r % 3][:n], B) for r in range(min(R, 3))]
    codes, scales = [q[r % 3][0] for r in range(R)], [q[r % 3][1] * np.float32(1 + r // 3) for r in range(R)]
    out, wc, ws = oracle.reduce_flat(local, codes, scales, B)
    dev = [torch.from_numpy(np.ascontiguousarray(a)).cuda() for a in codes + scales]
    got = torch.empty(n, dtype=torch.bfloat16, device="cuda")
    c, s = torch.empty(n, dtype=torch.int8, device="cuda"), torch.empty(eq.num_blocks(n, B), device="cuda")
    eq.equarx_reduce_flat(gpu.dev_bf16(local), dev[:R], dev[R:], B, got, c, s)
    assert (gpu.host_u16(got) == out).all() and (c.cpu().numpy() == wc).all() and (_bits(s) == ws.view(np.uint32)).all()


STRIDED_FLAGS = (0, eq.AG_UNQUANTIZED, eq.RS_UNQUANTIZED, eq.SEMI_LOOP, eq.RING_ORDER, eq.SEMI_LOOP | eq.RING_ORDER,
                 eq.SEMI_LOOP | eq.RING_ORDER | eq.AG_UNQUANTIZED)


@pytest.mark.parametrize("chunks,minishards", ((32, 1), (32, 16), (32, 17), (64, 3), (64, 16), (64, 17), (64, 32), (64, 33),
                                               (128, 2), (128, 16), (128, 17)))
@pytest.mark.parametrize("P", (1, 2, 5))
def test_strided_layouts(gpu, oracle, chunks, minishards, P):  # noqa: F811
    """Small, medium and large layouts of every strided call, on both sides of the lines between them."""
    n = 1024 * chunks * minishards
    rng = np.random.default_rng(n % 1000 + P)
    x = [gpu.bf16_of(rng.standard_normal(n, dtype=np.float32) * np.exp2(rng.integers(-3, 4, n)).astype(np.float32))
         for _ in range(P)]
    dev = [gpu.dev_bf16(p) for p in x]
    c, s = torch.empty(n, dtype=torch.int8, device="cuda"), torch.empty(n // chunks, device="cuda")
    eq.equarx_quantize_strided(dev[0], chunks, c, s)
    wc, ws = oracle.quantize_bf16_strided(x[0], chunks)
    assert (c.cpu().numpy() == wc).all() and (_bits(s) == ws.view(np.uint32)).all()
    if P > 1:                                               # a hop in place
        eq.equarx_reduce_stage_strided(c, s, dev[1], chunks, c, s)
        wc, ws = oracle.hop_strided(wc, ws, x[1], chunks)
        assert (c.cpu().numpy() == wc).all() and (_bits(s) == ws.view(np.uint32)).all()
    out = torch.empty(n, dtype=torch.bfloat16, device="cuda")
    eq.equarx_reduce_quantized_strided(dev, chunks, out, eq.alloc_workspace(P, n, chunks))
    assert (gpu.host_u16(out) == oracle.reduce_chain_strided(x, chunks)).all()
    for flags in STRIDED_FLAGS:
        want = _oracle_variant_strided(oracle, x, chunks, flags)
        eq.equarx_reduce_variant_strided(dev, chunks, flags, out.fill_(5.0))
        assert (gpu.host_u16(out) == want).all(), flags
        if not flags & eq.RS_UNQUANTIZED:
            work = eq.alloc_variant_workspace(flags & ~eq.RING_ORDER, P, n, chunks)
            eq.equarx_reduce_variant_hops_strided(dev, chunks, flags, out.fill_(5.0), work)
            assert (gpu.host_u16(out) == want).all(), flags


@pytest.mark.parametrize("chunks,minishards,P", ((64, 319, 3), (64, 320, 4), (64, 321, 3), (128, 161, 4), (32, 641, 3),
                                                 (64, 159, 5), (64, 161, 4), (128, 81, 5)))
def test_strided_chains_that_turn(gpu, oracle, long_values, chunks, minishards, P):  # noqa: F811
    n = 1024 * chunks * minishards
    x = [np.resize(long_values[i % 3], n + i)[i:].copy() for i in range(P)]
    dev = [gpu.dev_bf16(p) for p in x]
    out = torch.empty(n, dtype=torch.bfloat16, device="cuda")
    if n > TURN_FROM // 2 * 3:
        eq.equarx_reduce_quantized_strided(dev, chunks, out, eq.alloc_workspace(P, n, chunks))
        assert (gpu.host_u16(out) == oracle.reduce_chain_strided(x, chunks)).all()
    for flags in (0, eq.RING_ORDER) if n > TURN_FROM // 2 * 3 else (eq.SEMI_LOOP, eq.SEMI_LOOP | eq.RING_ORDER | eq.AG_UNQUANTIZED):
        work = eq.alloc_variant_workspace(flags & ~eq.RING_ORDER, P, n, chunks)
        eq.equarx_reduce_variant_hops_strided(dev, chunks, flags, out.fill_(5.0), work)
        assert (gpu.host_u16(out) == _oracle_variant_strided(oracle, x, chunks, flags)).all(), flags


@pytest.mark.parametrize("chunks,minishards,P,beside", ((32, 3, 2, True), (32, 96, 3, True), (32, 97, 2, False),
                                                        (64, 143, 3, False), (64, 144, 2, True), (64, 448, 3, True),
                                                        (64, 449, 2, False), (128, 20, 1, False)))
def test_where_the_last_wire_of_a_strided_chain_is(gpu, oracle, long_values, chunks, minishards, P, beside):  # noqa: F811
    """In the workspace's second buffer, up to 3 Mi elements and from 9 to 28 Mi."""
    n = 1024 * chunks * minishards
    x = [np.resize(long_values[i], n) for i in range(P)]
    work, out = eq.alloc_workspace(P, n, chunks).fill_(0x55), torch.empty(n, dtype=torch.bfloat16, device="cuda")
    eq.equarx_reduce_quantized_strided([gpu.dev_bf16(p) for p in x], chunks, out, work)
    assert (gpu.host_u16(out) == oracle.reduce_chain_strided(x, chunks)).all()
    codes, scales = work[work.numel() // 2 if beside else 0:][:n].view(torch.int8), n // chunks
    scales = work[(work.numel() // 2 if beside else 0) + n:][:4 * scales].view(torch.float32)
    got = torch.empty_like(out)
    eq.equarx_dequantize_strided(codes, scales, chunks, got)
    assert torch.equal(got, out)
    if not beside:
        assert (work[work.numel() // 2:] == 0x55).all()


@pytest.mark.parametrize("chunks,minishards", ((32, 17), (64, 17), (64, 33), (128, 17)))
@pytest.mark.parametrize("kind", ("sparse", "tiny", "huge"))
def test_strided_layouts_above_the_small_ones_with_extreme_values(gpu, oracle, chunks, minishards, kind):  # noqa: F811
    """Signed zeros, scales at the ends of the range, and an output that is one of the partials."""
    n, P = 1024 * chunks * minishards, 4
    x = [gpu.bf16_of(_values(kind, n, 60 + p)) for p in range(P)]
    for flags in (0, eq.AG_UNQUANTIZED, eq.SEMI_LOOP, eq.SEMI_LOOP | eq.RING_ORDER | eq.AG_UNQUANTIZED):
        want = _oracle_variant_strided(oracle, x, chunks, flags)
        dev = [gpu.dev_bf16(p) for p in x]
        eq.equarx_reduce_variant_strided(dev, chunks, flags, dev[1])
        assert (gpu.host_u16(dev[1]) == want).all(), flags
        dev[1] = gpu.dev_bf16(x[1])
        work = eq.alloc_variant_workspace(flags & ~eq.RING_ORDER, P, n, chunks)
        eq.equarx_reduce_variant_hops_strided(dev, chunks, flags, dev[2], work)
        assert (gpu.host_u16(dev[2]) == want).all(), flags


@pytest.mark.parametrize("chunks,minishards", ((32, 8), (32, 65), (32, 191), (32, 192), (32, 203), (64, 9), (64, 47), (64, 127),
                                               (64, 128), (64, 161), (128, 16), (128, 18), (128, 39)))
def test_strided_passes_by_lanes_and_owners(gpu, oracle, long_values, chunks, minishards):  # noqa: F811
    """Both sides of the lines between the layouts, with minishards left over behind whole runs on every XCD."""
    n, P = 1024 * chunks * minishards, 3
    x = [np.resize(long_values[i], n + i)[i:].copy() for i in range(P)]
    dev = [gpu.dev_bf16(p) for p in x]
    c, s = torch.empty(n, dtype=torch.int8, device="cuda"), torch.empty(n // chunks, device="cuda")
    eq.equarx_quantize_strided(dev[0], chunks, c, s)
    wc, ws = oracle.quantize_bf16_strided(x[0], chunks)
    assert (c.cpu().numpy() == wc).all() and (_bits(s) == ws.view(np.uint32)).all()
    eq.equarx_reduce_stage_strided(c, s, dev[1], chunks, c, s)
    wc, ws = oracle.hop_strided(wc, ws, x[1], chunks)
    assert (c.cpu().numpy() == wc).all() and (_bits(s) == ws.view(np.uint32)).all()
    out = torch.empty(n, dtype=torch.bfloat16, device="cuda")
    for flags, moved in ((0, 0), (0, 5 << 16), (eq.SEMI_LOOP, 3 << 16 | 256), (eq.SEMI_LOOP | eq.RING_ORDER, 0),
                         (eq.RING_ORDER | eq.AG_UNQUANTIZED, 7 << 15)):      # where in memory the wires begin
        work = torch.empty(2 ** 20 + 4 * n, dtype=torch.uint8, device="cuda")
        work = work[-work.data_ptr() % 2 ** 18 + moved:][:eq.alloc_variant_workspace(flags & ~eq.RING_ORDER, P, n, chunks).numel()]
        eq.equarx_reduce_variant_hops_strided(dev, chunks, flags, out.fill_(5.0), work)
        assert (gpu.host_u16(out) == _oracle_variant_strided(oracle, x, chunks, flags)).all(), flags
    eq.equarx_reduce_quantized_strided(dev, chunks, out.fill_(5.0), eq.alloc_workspace(P, n, chunks))
    assert (gpu.host_u16(out) == _oracle_variant_strided(oracle, x, chunks, 0)).all()


@pytest.mark.parametrize("chunks,minishards", ((32, 20), (32, 21), (32, 128), (32, 129), (32, 192), (32, 193), (64, 8), (64, 9),
                                               (64, 41), (128, 6), (128, 7), (128, 48), (128, 49)))
def test_strided_single_launch_layouts(gpu, oracle, long_values, chunks, minishards):  # noqa: F811
    """Both sides of the lines between the layouts of the strided chain and its flavours."""
    n, P = 1024 * chunks * minishards, 4
    x = [np.resize(long_values[i % 3], n + i)[i:].copy() for i in range(P)]
    dev = [gpu.dev_bf16(p) for p in x]
    out = torch.empty(n, dtype=torch.bfloat16, device="cuda")
    for flags in (0, eq.AG_UNQUANTIZED, eq.RS_UNQUANTIZED, eq.SEMI_LOOP | eq.RING_ORDER):
        eq.equarx_reduce_variant_strided(dev, chunks, flags, out.fill_(5.0))
        assert (gpu.host_u16(out) == _oracle_variant_strided(oracle, x, chunks, flags)).all(), flags


@pytest.mark.parametrize("chunks,minishards,P", ((32, 127, 2), (32, 128, 2), (32, 160, 2), (32, 161, 2), (32, 192, 3), (32, 193, 3),
                                                 (32, 193, 4), (32, 200, 1), (32, 256, 2), (32, 257, 2), (64, 160, 2), (64, 161, 2), (64, 128, 4),
                                                 (64, 129, 4), (64, 136, 4), (64, 137, 4), (64, 192, 6), (64, 193, 6), (128, 48, 2),
                                                 (128, 49, 2), (128, 48, 9), (128, 49, 9), (128, 64, 3), (128, 65, 3), (128, 96, 4),
                                                 (128, 97, 3), (128, 128, 2), (128, 129, 2)))
def test_strided_sums_in_fp32(gpu, oracle, long_values, chunks, minishards, P):  # noqa: F811
    """Both sides of the lines of the reduce-scatter in fp32 that has a kernel of its own; a NaN, which fills its block, and an
    output that is one of the partials."""
    n = 1024 * chunks * minishards
    x = [np.resize(long_values[i % 3], n + i)[i:].copy() for i in range(P)]
    spoilt = np.zeros((minishards, 1, 1024), bool)
    for k, e in enumerate(np.random.default_rng(n + P).choice(n, 48, replace=False)):
        x[k % P][e] = (0x7FC0, 0xFFC0, 0x7F81)[k % 3]
        spoilt[e // (1024 * chunks), 0, e % 1024] = True
    spoilt = np.broadcast_to(spoilt, (minishards, chunks, 1024)).reshape(-1)
    for flags in (eq.RS_UNQUANTIZED, eq.RS_UNQUANTIZED | eq.RING_ORDER):
        dev = [gpu.dev_bf16(p) for p in x]
        eq.equarx_reduce_variant_strided(dev, chunks, flags, dev[P // 2])
        got = gpu.host_u16(dev[P // 2])
        assert (got[~spoilt] == _oracle_variant_strided(oracle, x, chunks, flags)[~spoilt]).all(), flags
        assert ((got[spoilt] & 0x7FFF) > 0x7F80).all(), flags


@pytest.mark.parametrize("chunks,minishards,P", ((32, 72, 4), (32, 73, 4), (32, 120, 4), (32, 129, 4), (32, 192, 5), (32, 193, 4), (32, 193, 5), (32, 288, 5), (32, 289, 5), (32, 400, 5), (32, 448, 4), (32, 448, 5),
                                                 (32, 511, 5), (32, 512, 5), (64, 129, 4), (64, 160, 4), (64, 161, 4), (64, 180, 4), (64, 181, 4), (64, 192, 4), (64, 193, 4),
                                                 (128, 95, 4), (128, 96, 5), (128, 97, 4),
                                                 (128, 111, 5), (128, 112, 4), (128, 112, 5), (128, 128, 5), (128, 129, 5),
                                                 (128, 8, 8), (128, 8, 9), (128, 9, 3), (128, 16, 2), (128, 17, 2), (128, 24, 2), (128, 25, 2), (128, 32, 2), (128, 33, 2)))
def test_strided_single_launch_rules(gpu, oracle, long_values, chunks, minishards, P):  # noqa: F811
    """Both sides of the lines that hang on rounds of workgroups and on partials: caps, layouts and runs of minishards."""
    n = 1024 * chunks * minishards
    x = [np.resize(long_values[i % 3], n + i)[i:].copy() for i in range(P)]
    dev = [gpu.dev_bf16(p) for p in x]
    out = torch.empty(n, dtype=torch.bfloat16, device="cuda")
    for flags in (0, eq.AG_UNQUANTIZED, eq.RS_UNQUANTIZED, eq.SEMI_LOOP, eq.SEMI_LOOP | eq.RING_ORDER | eq.AG_UNQUANTIZED):
        eq.equarx_reduce_variant_strided(dev, chunks, flags, out.fill_(5.0))
        assert (gpu.host_u16(out) == _oracle_variant_strided(oracle, x, chunks, flags)).all(), flags


@pytest.mark.parametrize("chunks,minishards,P", ((64, 159, 2), (64, 160, 2), (64, 203, 2), (64, 160, 3), (128, 79, 3), (128, 80, 4),
                                                 (128, 96, 3), (128, 96, 5), (128, 97, 2), (128, 101, 3), (128, 128, 5),
                                                 (128, 129, 3), (32, 223, 1), (32, 224, 1), (64, 95, 1), (64, 96, 1), (64, 129, 1),
                                                 (128, 79, 1), (128, 80, 1), (128, 128, 1), (128, 129, 1)))
def test_strided_hops_of_few_partials(gpu, oracle, long_values, chunks, minishards, P):  # noqa: F811
    """Around 10 Mi elements, from which few partials keep the parts of a minishard on all XCDs, and where the owner has lanes of
    its own."""
    n = 1024 * chunks * minishards
    x = [np.resize(long_values[i % 3], n + i)[i:].copy() for i in range(P)]
    for flags in (0, eq.RING_ORDER | eq.AG_UNQUANTIZED, eq.SEMI_LOOP, eq.SEMI_LOOP | eq.RING_ORDER):
        dev = [gpu.dev_bf16(p) for p in x]
        work = eq.alloc_variant_workspace(flags & ~eq.RING_ORDER, P, n, chunks)
        work = torch.empty(work.numel() + (5 << 16), dtype=torch.uint8, device="cuda")[5 << 16:]
        eq.equarx_reduce_variant_hops_strided(dev, chunks, flags, dev[0], work)
        assert (gpu.host_u16(dev[0]) == _oracle_variant_strided(oracle, x, chunks, flags)).all(), flags


@pytest.mark.parametrize("chunks,minishards", ((32, 191), (32, 192), (32, 193), (64, 97), (128, 48), (128, 49)))
def test_strided_dequantization_around_six_mi_elements(gpu, oracle, long_values, chunks, minishards):  # noqa: F811
    """Two tiles a lane and four, with a wire that begins between two runs."""
    n = 1024 * chunks * minishards
    codes, scales = oracle.quantize_bf16_strided(np.resize(long_values[0], n), chunks)
    c = torch.empty(n + (3 << 16), dtype=torch.int8, device="cuda")[3 << 16:]
    c.copy_(torch.from_numpy(codes))
    out = torch.full((n,), 5.0, dtype=torch.bfloat16, device="cuda")
    eq.equarx_dequantize_strided(c, torch.from_numpy(scales).cuda(), chunks, out)
    assert (gpu.host_u16(out) == oracle.dequantize_bf16_strided(codes, scales, chunks)).all()


@pytest.mark.parametrize("n,P", ((6_300_032, 3), (6_300_033, 7), (20 * 2 ** 20 + 64, 4), (20 * 2 ** 20 + 80, 4)))
def test_long_kept_wires(gpu, oracle, long_values, n, P):  # noqa: F811
    """Rows of the kept wire on 64-byte lines and off them, in both of the shapes that write them through the L2s."""
    x = [np.resize(long_values[i % 3], n + i)[i:].copy() for i in range(P)]
    want, wc, ws = oracle.reduce_chain(x, 64, keep_wire=True)
    got, c, s = gpu.gpu_chain_fused(x, 64)
    assert (got == want).all() and (c == wc).all() and (s.view(np.uint32) == ws.view(np.uint32)).all()


SMALL = 768 * 2048              # single-launch calls of few partials: up to here the batched kernel
ALL_SINGLE = SINGLE + (eq.SEMI_LOOP | eq.RING_ORDER, eq.AG_UNQUANTIZED | eq.RING_ORDER, eq.RS_UNQUANTIZED)


@pytest.mark.parametrize("flags", ALL_SINGLE)
@pytest.mark.parametrize("P", (3, 4, 5, 7, 8, 9, 15, 16, 17, 64))
def test_small_kernel_batches(gpu, oracle, P, flags):  # noqa: F811
    """Batches of 8 and 16 partials, one that loops, and what stays below or above them; odd and even lengths."""
    rng = np.random.default_rng(P + flags)
    for n, B in ((2048 * 33 + 9, 64), (2048 * 34, 512), (2048 * 40 + 6, 32), (5, 32)):
        x = [gpu.bf16_of(rng.standard_normal(n, dtype=np.float32)) for _ in range(P)]
        assert (gpu.gpu_variant(x, B, flags) == _oracle_variant(oracle, x, B, flags)).all(), (n, B)
        if flags == 0:
            want, wc, ws = oracle.reduce_chain(x, B, keep_wire=True)
            got, c, s = gpu.gpu_chain_fused(x, B)
            assert (got == want).all() and (c == wc).all() and (s.view(np.uint32) == ws.view(np.uint32)).all(), (n, B)


@pytest.mark.parametrize("n", (SMALL, SMALL + 1))
@pytest.mark.parametrize("flags", (0, eq.SEMI_LOOP | eq.RING_ORDER))
def test_single_launch_around_the_small_limit(gpu, oracle, values, n, flags):  # noqa: F811
    x = [values[i % 4][:n] for i in range(6)]
    assert (gpu.gpu_variant(x, 128, flags) == _oracle_variant(oracle, x, 128, flags)).all()


@pytest.mark.parametrize("tail", range(1, 17))
def test_ends_of_odd_length(gpu, oracle, tail):  # noqa: F811
    """Every remainder of the last words, at the end of a lane, a wave and a tile; nothing past the end is written."""
    rng = np.random.default_rng(tail)
    for n in (tail, 512 - 8 + tail, 2048 - 16 + tail, 2048 * 3 + tail):
        x = [gpu.bf16_of(rng.standard_normal(n, dtype=np.float32)) for _ in range(3)]
        dev = [gpu.dev_bf16(p) for p in x]
        room = n + 32
        nb = eq.num_blocks(n, 32)
        want, wc, ws = oracle.reduce_chain(x, 32, keep_wire=True)
        codes = torch.full((2, -(-room // 16) * 16), 77, dtype=torch.int8, device="cuda")
        scales = torch.full((2, -(-(nb + 8) // 4) * 4), -5.0, device="cuda")
        eq.equarx_quantize(dev[0], 32, codes[0], scales[0])
        eq.equarx_reduce_stage(codes[0], scales[0], dev[1], 32, codes[1], scales[1])
        eq.equarx_reduce_stage(codes[1], scales[1], dev[2], 32, codes[1], scales[1])        # in place
        assert (codes[0, :n].cpu().numpy() == wc[0]).all() and (codes[1, :n].cpu().numpy() == wc[2]).all(), n
        assert (_bits(scales[0, :nb]) == ws[0].view(np.uint32)).all() and (_bits(scales[1, :nb]) == ws[2].view(np.uint32)).all()
        assert (codes[:, n:] == 77).all() and (scales[:, nb:] == -5.0).all(), n
        twice = oracle.reduce_chain(x + x, 32)
        for expected, run in ((want, lambda o: eq.equarx_reduce_fused(dev, 32, o)),
                              (twice, lambda o: eq.equarx_reduce_fused(dev + dev, 32, o)),
                              (want, lambda o: eq.equarx_dequantize(codes[1, :n], scales[1, :nb], 32, o))):
            out = torch.full((room,), 3.0, dtype=torch.bfloat16, device="cuda")
            run(out)
            assert (gpu.host_u16(out[:n]) == expected).all() and (out[n:] == 3.0).all(), n
