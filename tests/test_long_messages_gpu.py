"""Messages of more threads than a dimension of a grid holds (2^32): made in pieces, or refused; never cut short."""
import numpy as np
import pytest
import torch

from paper_2506_17615_amd import binding as eq
from test_parity_gpu import gpu  # noqa: F401  (the fixture that loads the library)

pytestmark = pytest.mark.gpu

W = 128 * 1024                  # a minishard of 128 chunks
LONG, LONGER = (1 << 35) + W, (1 << 36) + W      # beyond one piece; beyond what one launch of 512 threads x 2 tiles covers


class _Message:
    """x: zeros but for windows of random values at the start, on both sides of every piece's end and at the end."""

    def __init__(self, gpu, n):  # noqa: F811
        torch.cuda.empty_cache()
        if torch.cuda.mem_get_info()[0] < 3.2 * n:
            pytest.skip("not enough memory on this GPU")
        rng = np.random.default_rng(n % 1000)
        self.gpu, self.n = gpu, n
        self.at = sorted({0, n - W} | {e + d for e in range(1 << 35, n, 1 << 35) for d in (-W, 0)})
        self.host = {a: gpu.bf16_of(rng.standard_normal(W, dtype=np.float32)) for a in self.at}
        self.x = torch.zeros(n, dtype=torch.bfloat16, device="cuda")
        for a, v in self.host.items():
            self.x[a:a + W] = gpu.dev_bf16(v)
        self.codes = self.buffer(torch.int8)

    def buffer(self, dtype, count=None):
        return torch.empty(count or self.n, dtype=dtype, device="cuda")

    def holds(self, want, codes=None, scales=None, out=None, B=512):
        """want(window values) -> the oracle's (codes, scales) or bf16 bits."""
        for a, v in self.host.items():
            w = want(v)
            if out is not None:
                assert (self.gpu.host_u16(out[a:a + W]) == w).all(), a
            else:
                assert (codes[a:a + W].cpu().numpy() == w[0]).all(), a
                assert (scales[a // B:(a + W) // B].cpu().numpy().view(np.uint32) == w[1].view(np.uint32)).all(), a


@pytest.mark.parametrize("n", (LONG, LONGER))
def test_passes(gpu, oracle, n):  # noqa: F811
    m, B = _Message(gpu, n), 512
    x, c, s = m.x, m.codes, m.buffer(torch.float32, n // 512)
    eq.equarx_quantize_batch([x], B, [c], [s])
    m.holds(lambda v: oracle.quantize_bf16(v, B), c, s)
    c.zero_(), s.zero_()
    eq.equarx_reduce_flat(x, [], [], B, codes_out=c, scales_out=s)
    m.holds(lambda v: oracle.reduce_flat(v, [], [], B)[1:], c, s)
    c.zero_(), s.zero_()
    eq.equarx_quantize(x, B, c, s)
    m.holds(lambda v: oracle.quantize_bf16(v, B), c, s)
    eq.equarx_reduce_stage(c, s, x, B, c, s)                    # in place
    m.holds(lambda v: oracle.hop(*oracle.quantize_bf16(v, B), v, B), c, s)
    eq.equarx_dequantize(c, s, B, x)
    m.holds(lambda v: oracle.dequantize_bf16(*oracle.hop(*oracle.quantize_bf16(v, B), v, B), B), out=x)
    strided = torch.arange(1, 5, device="cuda", dtype=torch.float32).repeat(n // 128 // 4)
    eq.equarx_dequantize_strided(c, strided, 128, x)
    ones = strided[:W // 128].cpu().numpy()
    m.holds(lambda v: oracle.dequantize_bf16_strided(oracle.hop(*oracle.quantize_bf16(v, B), v, B)[0], ones, 128), out=x)


def test_received_wires_and_chains(gpu, oracle):  # noqa: F811
    m, B, n = _Message(gpu, LONG), 512, LONG
    c, s, c2, s2 = m.codes, m.buffer(torch.float32, n // B), m.buffer(torch.int8), m.buffer(torch.float32, n // B)
    eq.equarx_quantize(m.x, B, c, s)
    eq.equarx_reduce_flat(m.x, [c, c], [s, s], B, codes_out=c2, scales_out=s2)

    def flat(v):
        w, t = oracle.quantize_bf16(v, B)
        return oracle.reduce_flat(v, [w, w], [t, t], B)[1:]

    m.holds(flat, c2, s2)
    del c, s, c2, s2
    m.codes = None
    torch.cuda.empty_cache()
    work = torch.empty(eq.workspace_bytes(3, n, B), dtype=torch.uint8, device="cuda")
    out = m.buffer(torch.bfloat16)
    eq.equarx_reduce_quantized_fused_ends([m.x] * 3, B, out, work)
    m.holds(lambda v: oracle.reduce_chain([v] * 3, B), out=out)
    eq.equarx_reduce_variant_hops([m.x] * 2, B, eq.AG_UNQUANTIZED, out, work)
    m.holds(lambda v: oracle.reduce_stages([v] * 2, B, True, False), out=out)


@pytest.mark.parametrize("n", ((1 << 35) - 8192, (1 << 35) - 4096))
def test_around_the_last_length_of_1024_threads_by_one_tile(gpu, oracle, n):  # noqa: F811
    """The shape of few partials, of the semi-loop and of a long dequantization, as far as a grid holds its threads, and
    the first length beyond."""
    m, B = _Message(gpu, n), 512
    c, s, out = m.codes, m.buffer(torch.float32, n // B), m.buffer(torch.bfloat16).fill_(7.0)
    eq.equarx_quantize(m.x, B, c, s)
    eq.equarx_dequantize(c, s, B, out)
    m.holds(lambda v: oracle.dequantize_bf16(*oracle.quantize_bf16(v, B), B), out=out)
    eq.equarx_reduce_fused([m.x] * 2, B, out.fill_(7.0))
    m.holds(lambda v: oracle.reduce_chain([v] * 2, B), out=out)
    eq.equarx_reduce_variant([m.x] * 2, B, eq.SEMI_LOOP, out.fill_(7.0))
    m.holds(lambda v: oracle.reduce_semi_loop([v] * 2, B), out=out)


def test_semi_loop_in_one_launch(gpu, oracle):  # noqa: F811
    """In place, all partials one tensor: taken as far as one launch goes, and refused beyond."""
    m = _Message(gpu, LONG)
    eq.equarx_reduce_variant([m.x] * 2, 64, eq.SEMI_LOOP, m.x)
    m.holds(lambda v: oracle.reduce_semi_loop([v] * 2, 64), out=m.x)
    del m
    m = _Message(gpu, LONGER)
    with pytest.raises(eq.EquarxError) as e:
        eq.equarx_reduce_variant([m.x] * 2, 64, eq.SEMI_LOOP, m.x)
    assert e.value.status == eq.STATUS_DEVICE_ERROR
    m.holds(lambda v: v, out=m.x)
