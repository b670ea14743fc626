"""Performance cases: the calls a user of this library makes, over the range of message sizes they are made with.

A case names a call (or the calls one device makes per collective), the number of partial sums P, the tensor's
rows x hidden, the block size (or the chunks of the strided geometry), the flags and the distribution of the values.
`prepare` makes what the caller has in hand -- the partial sums, what arrived from other devices, the output buffers
and the workspace of that size -- and `run` makes the calls.  Shapes and distributions are those of
`paper_2506_17615_amd.workloads` and of the recorded size sweep; values are drawn on the GPU from the seed.

Every result is a single bit pattern (int8 codes, fp32 scales, and a bf16 output that follows from them by one
multiplication and one rounding), so the tolerance is exact.
"""
import torch

from paper_2506_17615_amd import binding as eq

SEMI, RS_OFF, AG_OFF, RING = eq.SEMI_LOOP, eq.RS_UNQUANTIZED, eq.AG_UNQUANTIZED, eq.RING_ORDER
CHUNK = 1024        # elements per chunk of the strided geometry
STRIDED = ("strided_fused", "strided_hops", "strided_variant", "strided_variant_hops")


def listed():
    return [
        # The smallest call in the tests and the benchmark: a 4096-element message, hop by hop.  Launches and host
        # time count, nothing else.
        dict(name="message_4k_hops", call="hops", P=4, rows=1, hidden=4096, block=256, flags=0, dist="normal"),
        # A decode step's AllReduce input (64 tokens x 5376) over 16 partials in the single launch a latency-bound
        # caller takes.
        dict(name="decode_fused", call="fused", P=16, rows=64, hidden=5376, block=128, flags=0, dist="normal"),
        # The same message hop by hop in a serving loop that holds no workspace of its own.
        dict(name="decode_static_hops", call="static", P=16, rows=64, hidden=5376, block=128, flags=0, dist="normal"),
        # One device's calls in a ring of 8 on the 27B-shaped prefill tensor (4096 x 5376): quantize, seven hops,
        # dequantize what the all-gather brought.
        dict(name="ring_device_27b", call="ring_device", P=8, rows=4096, hidden=5376, block=256, flags=0,
             dist="row_lognormal_outliers"),
        # One device's calls in the all-to-all form of the same reduction: batched quantize, flat reduce, dequantize.
        dict(name="alltoall_device_27b", call="alltoall_device", P=8, rows=4096, hidden=5376, block=256, flags=0,
             dist="row_lognormal_outliers"),
        # An odd-sized gradient-bucket-like message over an odd ring: semi-loop, per-shard ring order, small blocks.
        dict(name="ragged_semi_ring", call="variant", P=5, rows=1, hidden=1234567, block=64, flags=SEMI | RING,
             dist="normal"),
        # The 12B-shaped prefill activation (2048 tokens x 3840) in one launch.
        dict(name="prefill_12b_fused", call="fused", P=8, rows=2048, hidden=3840, block=256, flags=0,
             dist="row_lognormal"),
        # The paper's own setting (Sec. 4.1, Fig. 7): semi-loop, ring schedule, strided blocks of 64, (4096, 4096).
        dict(name="fig7_strided_semi_ring_hops", call="strided_variant_hops", P=8, rows=4096, hidden=4096, block=64,
             flags=SEMI | RING, dist="normal"),
        # The benchmark's headline: the 27B-shaped prefill activation, hop by hop.
        dict(name="prefill_27b_hops", call="hops", P=8, rows=4096, hidden=5376, block=256, flags=0,
             dist="row_lognormal_outliers"),
        # The same tensor in one launch in the paper's block geometry.
        dict(name="prefill_27b_strided_fused", call="strided_fused", P=8, rows=4096, hidden=5376, block=64, flags=0,
             dist="row_lognormal_outliers"),
        # The large-message end (64 MiB per partial, heavy tails) at the smallest block, ends fused.
        dict(name="large_b32_ends", call="ends", P=8, rows=1, hidden=33554432, block=32, flags=0, dist="student_t3"),
        # The longest prefill of the size sweep (16384 tokens x 5376) in one launch.
        dict(name="prefill_27b_16k_fused", call="fused", P=8, rows=16384, hidden=5376, block=256, flags=0,
             dist="row_lognormal_outliers"),
    ]


# What `draw` picks from: the call, how often, the flags it is used with, and the most (P + 1) * n elements of a case (a
# call that walks the wire through memory costs about twice a single launch of the same size).
_ONE_LAUNCH, _HOPS = 700_000_000, 270_000_000
_DRAWN = [
    ("fused", 3, [0], _ONE_LAUNCH),
    ("fused_kept_wire", 1, [0], _HOPS),
    ("hops", 3, [0], _HOPS),
    ("static", 1, [0], _HOPS),
    ("ends", 1, [0], _HOPS),
    ("variant", 2, [SEMI, SEMI | RING, RING, RS_OFF, AG_OFF, SEMI | AG_OFF, RING | AG_OFF], _ONE_LAUNCH),
    ("variant_hops", 1, [SEMI, SEMI | RING, RING, AG_OFF], _HOPS),
    ("ring_device", 2, [0], _ONE_LAUNCH),
    ("alltoall_device", 2, [0], _ONE_LAUNCH),
    ("strided_fused", 1, [0], _ONE_LAUNCH),
    ("strided_hops", 1, [0], _HOPS),
    ("strided_variant", 1, [SEMI, RING, AG_OFF, SEMI | RING], _ONE_LAUNCH),
    ("strided_variant_hops", 1, [SEMI, SEMI | RING, RING, AG_OFF], _HOPS),
]
_MOST_STATIC = 32 << 20     # elements the library's static wire buffers are promised to hold at block 32


def _log_uniform(rng, lo, hi):
    return int(lo * (hi / lo) ** rng.random())


def draw(rng):
    weights = [w for _, w, _, _ in _DRAWN]
    call, _, flags, most = rng.choices(_DRAWN, weights)[0]
    P = rng.randint(2, 16)
    most = most // (P + 1)
    if call == "static":
        most = min(most, _MOST_STATIC)
    if call in STRIDED:
        block = rng.choice([32, 64, 128])
        rows, hidden = _log_uniform(rng, 1, max(2, most // (CHUNK * block))), CHUNK * block
    else:
        block = rng.choice([32, 64, 128, 256, 512])
        n = _log_uniform(rng, 4096, most)
        if call in ("ring_device", "alltoall_device"):
            n = max(n, 2 * P * P * block)       # no device without a shard
        if rng.random() < 0.5:                  # an activation: whole rows
            hidden = rng.choice([2560, 3840, 4096, 5376, 8192])
            rows = max(1, n // hidden)
            if rows * hidden < n // 2 or call in ("ring_device", "alltoall_device"):
                rows += 1
        else:                                   # a flat message of any length
            rows, hidden = 1, n | rng.randint(0, 1)
    dist = rng.choice(["normal", "student_t3", "row_lognormal", "row_lognormal_outliers"]) if rows > 1 else \
        rng.choice(["normal", "student_t3"])
    return dict(call=call, P=P, rows=rows, hidden=hidden, block=block, flags=rng.choice(flags), dist=dist)


class _Values:
    """bf16 tensors of one distribution, drawn on the GPU in fp32 (the recipes of paper_2506_17615_amd.workloads)."""

    def __init__(self, case, seed):
        self.rows, self.hidden, self.dist = case["rows"], case["hidden"], case["dist"]
        self.gen = torch.Generator(device="cuda")
        self.gen.manual_seed(seed * 1_000_003 + 17)
        if self.dist.startswith("row_lognormal"):
            self.row = torch.exp(self._randn(self.rows, 1))     # per-token factor, shared by all partials
        if self.dist == "row_lognormal_outliers":
            k = max(1, round(0.001 * self.hidden))
            self.channels = torch.randperm(self.hidden, generator=self.gen, device="cuda")[:k]

    def _randn(self, *shape):
        return torch.randn(shape, generator=self.gen, device="cuda", dtype=torch.float32)

    def next(self, gain=1.0):
        v = self._randn(self.rows, self.hidden)
        if self.dist == "student_t3":
            chi2 = torch.zeros_like(v)
            for _ in range(3):
                chi2.addcmul_(*[self._randn(self.rows, self.hidden)] * 2)
            v /= torch.sqrt(chi2 / 3.0)
        elif self.dist != "normal":
            v *= self.row
            if self.dist == "row_lognormal_outliers":
                v[:, self.channels] *= 50.0
        return (v * gain).to(torch.bfloat16).reshape(-1)


def _empty(count, dtype):
    return torch.empty(count, dtype=dtype, device="cuda")


def _wire(n, block):
    return _empty(n, torch.int8), _empty(eq.num_blocks(n, block), torch.float32)


def _shards(n, P, block):
    """(first element, length) of each device's shard: ceil(nb / P) blocks, the last one shorter."""
    size = -(-eq.num_blocks(n, block) // P) * block
    return [(k * size, min(n, (k + 1) * size) - k * size) for k in range(P)]


def _received(x, block):
    """A wire as it arrives from another device: the quantized form of x."""
    codes, scales = _wire(x.numel(), block)
    eq.equarx_quantize(x, block, codes, scales)
    return codes, scales


def prepare(case, seed):
    call, P, block, flags = case["call"], case["P"], case["block"], case["flags"]
    n = case["rows"] * case["hidden"]
    values = _Values(case, seed)
    st = dict(call=call, block=block, flags=flags, out=_empty(n, torch.bfloat16))
    if call in ("ring_device", "alltoall_device"):
        local = values.next()                                   # this device's partial sum of the whole tensor
        shards = _shards(n, P, block)
        st["local"] = [local[lo:lo + size] for lo, size in shards]
        st["sends"] = [_wire(size, block) for _, size in shards]
        if call == "ring_device":                               # device 0: shards P-1, P-2, ..., 0 in turn
            st["received"] = []
            for i in range(1, P):                               # step i brings the running sum of i partials
                lo, size = shards[P - 1 - i]
                st["received"].append(_received(values.next(i ** 0.5)[lo:lo + size], block))
        else:                                                   # device 0 owns shard 0: one quantized shard per peer
            lo, size = shards[0]
            st["received"] = [_received(values.next()[lo:lo + size], block) for _ in range(1, P)]
        st["gathered"] = _received(values.next(P ** 0.5), block)        # what the all-gather brings
        return st
    st["partials"] = [values.next() for _ in range(P)]
    if call in ("hops", "ends", "strided_hops"):
        st["workspace"] = eq.alloc_workspace(P, n, block)
    elif call == "variant_hops":
        st["workspace"] = eq.alloc_variant_workspace(flags, P, n, block)
    elif call == "strided_variant_hops":
        st["workspace"] = eq.alloc_variant_workspace(flags & ~RING, P, n, block)
    elif call == "fused_kept_wire":                             # rows are padded: zeros there, written nowhere
        st["wire_codes"] = torch.zeros((P, eq.wire_row_codes(n)), dtype=torch.int8, device="cuda")
        st["wire_scales"] = torch.zeros((P, eq.wire_row_scales(n, block)), dtype=torch.float32, device="cuda")
    return st


def run(st):
    call, block, flags, out = st["call"], st["block"], st["flags"], st["out"]
    if call == "fused":
        eq.equarx_reduce_fused(st["partials"], block, out)
    elif call == "fused_kept_wire":
        eq.equarx_reduce_fused(st["partials"], block, out, st["wire_codes"], st["wire_scales"])
        return out, st["wire_codes"], st["wire_scales"]
    elif call == "hops":
        eq.equarx_reduce_quantized(st["partials"], block, out, st["workspace"])
    elif call == "static":
        eq.equarx_reduce_quantized_static(st["partials"], block, out)
    elif call == "ends":
        eq.equarx_reduce_quantized_fused_ends(st["partials"], block, out, st["workspace"])
    elif call == "variant":
        eq.equarx_reduce_variant(st["partials"], block, flags, out)
    elif call == "variant_hops":
        eq.equarx_reduce_variant_hops(st["partials"], block, flags, out, st["workspace"])
    elif call == "strided_fused":
        eq.equarx_reduce_fused_strided(st["partials"], block, out)
    elif call == "strided_hops":
        eq.equarx_reduce_quantized_strided(st["partials"], block, out, st["workspace"])
    elif call == "strided_variant":
        eq.equarx_reduce_variant_strided(st["partials"], block, flags, out)
    elif call == "strided_variant_hops":
        eq.equarx_reduce_variant_hops_strided(st["partials"], block, flags, out, st["workspace"])
    elif call == "ring_device":
        local, sends = st["local"], st["sends"]
        last = len(local) - 1
        eq.equarx_quantize(local[last], block, *sends[last])
        for i, (codes, scales) in enumerate(st["received"], 1):
            eq.equarx_reduce_stage(codes, scales, local[last - i], block, *sends[last - i])
        eq.equarx_dequantize(*st["gathered"], block, out)
        return out, sends
    elif call == "alltoall_device":
        local, sends, received = st["local"], st["sends"], st["received"]
        # the last shard may be shorter than the others and then goes out in a call of its own
        same = [k for k in range(1, len(local)) if local[k].numel() == local[0].numel()]
        eq.equarx_quantize_batch([local[k] for k in same], block, [sends[k][0] for k in same],
                                 [sends[k][1] for k in same])
        for k in range(1 + len(same), len(local)):
            eq.equarx_quantize(local[k], block, *sends[k])
        eq.equarx_reduce_flat(local[0], [c for c, _ in received], [s for _, s in received], block,
                              codes_out=sends[0][0], scales_out=sends[0][1])
        eq.equarx_dequantize(*st["gathered"], block, out)
        return out, sends
    return out


def work(case):
    """Inputs read once and outputs written once; a hop-by-hop call's wire buffers are neither and do not count.
    Operations per element and quantization: |.|, max, multiply, round, multiply-add (2)."""
    call, P, block = case["call"], case["P"], case["block"]
    n = case["rows"] * case["hidden"]
    wire = n * (1 + 4 / block)      # codes and scales of the whole tensor
    if call == "ring_device":       # in: the partial, P-1 received shards, the gathered wire; out: P sends, the result
        nbytes = 2 * n + wire * (P - 1) / P + wire + wire + 2 * n
        return {"bytes": nbytes, "flops": 6 * n}
    if call == "alltoall_device":   # the same with P-1 received copies of one shard
        nbytes = 2 * n + wire * (P - 1) / P + wire + wire + 2 * n
        return {"bytes": nbytes, "flops": 6 * n}
    nbytes = 2 * n * P + 2 * n + (P * wire if call == "fused_kept_wire" else 0)
    return {"bytes": nbytes, "flops": 6 * n * P}


def tolerance(case):
    return "exact"
