"""The binding's native marshalling against the checks in Python: what one accepts and refuses the other does too."""
import os
import subprocess
import sys
import sysconfig

import pytest
import torch

from paper_2506_17615_amd import binding as eq


ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


class Subclass(torch.Tensor):
    pass


class _GeneralPath:
    """In place of the extension: hands every call back."""

    def __getattr__(self, name):
        return lambda *args: -1


def _calls(device):
    """name -> (call with every argument a plain tensor or number, its output tensors)."""
    n, B, P = 4096 + 40, 64, 3
    m = 1024 * 32 * 2
    gen = torch.Generator().manual_seed(5)

    def bf16(k):
        return torch.randn(k, generator=gen).to(torch.bfloat16).to(device)

    def wire(k, nb):
        return torch.randint(-127, 128, (k,), generator=gen).to(torch.int8).to(device), torch.rand(nb, generator=gen).to(device)

    nb = -(-n // B)
    x, xs = [bf16(n) for _ in range(P)], [bf16(m) for _ in range(P)]
    out, outs = bf16(n), bf16(m)
    (c0, s0), (c1, s1), (c2, s2) = wire(n, nb), wire(n, nb), wire(n, nb)
    (d0, t0), (d1, t1) = wire(m, m // 32), wire(m, m // 32)
    work = torch.zeros(1 << 20, dtype=torch.uint8, device=device)
    kept = (torch.zeros(P, -(-n // 16) * 16, dtype=torch.int8, device=device),
            torch.zeros(P, -(-nb // 4) * 4, dtype=torch.float32, device=device))
    return {
        "equarx_quantize": ((x[0], B, c0, s0), (c0, s0)),
        "equarx_quantize_batch": ((x[:2], B, [c0, c1], [s0, s1]), (c0, c1, s0, s1)),
        "equarx_dequantize": ((c0, s0, B, out), (out,)),
        "equarx_reduce_stage": ((c0, s0, x[0], B, c1, s1), (c1, s1)),
        "equarx_reduce_quantized": ((x, B, out, work, *kept), (out, *kept)),
        "equarx_reduce_quantized_static": ((tuple(x), B, out), (out,)),
        "equarx_reduce_quantized_fused_ends": ((x, B, out, work), (out,)),
        "equarx_reduce_fused": ((x, B, out, *kept), (out, *kept)),
        "equarx_reduce_variant": ((x, B, eq.SEMI_LOOP | eq.RING_ORDER, out), (out,)),
        "equarx_reduce_variant_hops": ((x, B, eq.SEMI_LOOP, out, work), (out,)),
        "equarx_reduce_flat": ((x[0], [c0, c1], [s0, s1], B, out, c2, s2), (out, c2, s2)),
        "equarx_quantize_strided": ((xs[0], 32, d0, t0), (d0, t0)),
        "equarx_dequantize_strided": ((d0, t0, 32, outs), (outs,)),
        "equarx_reduce_stage_strided": ((d0, t0, xs[0], 32, d1, t1), (d1, t1)),
        "equarx_reduce_quantized_strided": ((xs, 32, outs, work), (outs,)),
        "equarx_reduce_fused_strided": ((xs, 32, outs), (outs,)),
        "equarx_reduce_variant_strided": ((xs, 32, eq.AG_UNQUANTIZED, outs), (outs,)),
        "equarx_reduce_variant_hops_strided": ((xs, 32, eq.RING_ORDER, outs, work), (outs,)),
    }


NAMES = sorted(_calls("cpu"))


def _altered(args):
    """Argument lists a call has to refuse, or to take in another form than the plain one."""
    def swap(i, v):
        return args[:i] + (v,) + args[i + 1:]

    for i, a in enumerate(args):
        for j, t in enumerate([a] if torch.is_tensor(a) else a if isinstance(a, (list, tuple)) else []):
            for bad in (None, t.cpu(), t[:-8], t.view(-1).to(torch.float64), t.view(-1).repeat_interleave(2)[::2],
                        t.as_subclass(Subclass), torch.nn.Parameter(t, requires_grad=False)):
                yield swap(i, bad if torch.is_tensor(a) else list(a[:j]) + [bad] + list(a[j + 1:]))
        if isinstance(a, (list, tuple)):
            for bad in ([], list(a)[:1], list(a) * 33, iter(a)):
                yield swap(i, bad)
        if isinstance(a, int):
            for bad in (0, 1, 33, -1, 48, 512, 1024, 1 << 33, True, 64.0, "64"):
                yield swap(i, bad)


def test_every_entry_point_is_marshalled():
    assert set(NAMES) == {n for n in eq.SIGNATURES if n.startswith(("equarx_quantize", "equarx_dequantize", "equarx_reduce"))}


@pytest.mark.parametrize("name", NAMES)
def test_host_tensors_are_handed_back(name):
    eq.load()
    args, _ = _calls("cpu")[name]
    assert getattr(eq._native, name)(*args) == -1
    assert getattr(eq._native, name)(*args[:-1]) == -1
    with pytest.raises(ValueError):
        getattr(eq, name)(*args)


def _child(code):
    """Runs code in an interpreter of its own, on the CPU; what it printed."""
    env = dict(os.environ, PYTHONPATH=ROOT)
    run = subprocess.run([sys.executable, "-W", "always", "-c", code], env=env, capture_output=True, text=True, timeout=300, cwd=ROOT)
    assert run.returncode == 0, run.stdout + run.stderr
    return run.stdout


def test_an_unbound_extension_calls_nothing():
    assert _child("""
import torch
from paper_2506_17615_amd import _marshal
x = torch.zeros(64, dtype=torch.bfloat16)
try:
    print(_marshal.equarx_quantize(x, 32, x, x))
except RuntimeError as e:
    print(e)
""") == "not bound to a library\n"


def _load_child(setup):
    return _child(f"""
import warnings
import torch
from paper_2506_17615_amd import binding as eq, build
{setup}
with warnings.catch_warnings(record=True) as seen:
    warnings.simplefilter("always")
    eq.load()
    eq.load()
print([str(w.message).split(": ")[0] for w in seen], eq.num_blocks(1000, 32), eq._native.equarx_quantize(None, 32, None, None))
try:
    eq.equarx_quantize(torch.zeros(64, dtype=torch.bfloat16), 32, None, None)
except ValueError as e:
    print(str(e).split(":")[0])
""")


@pytest.mark.parametrize("setup", ("build.MARSHAL_PATH += '.gone'", "torch.__version__ = '1.0.0'",
                                   "build.MARSHAL_PATH = build.LIB_PATH"))
def test_without_its_extension_the_binding_marshals_in_python(setup):
    """None there, one for another torch, a file that is none: the library is all a call needs."""
    assert _load_child(setup) == "['calls are marshalled in Python, 5 to 11 us each'] 32 -1\nx_bf16\n"
    assert _load_child("") == "[] 32 -1\nx_bf16\n"


def test_an_extension_of_another_interpreter_or_compiler_abi_is_stale(monkeypatch):
    from paper_2506_17615_amd import build
    assert os.path.basename(build.MARSHAL_PATH) == "_marshal" + sysconfig.get_config_var("EXT_SUFFIX")
    now = build._marshal_digest()
    real = sysconfig.get_config_var
    with monkeypatch.context() as m:
        m.setattr(sysconfig, "get_config_var", lambda k: "cpython-399" if k == "SOABI" else real(k))
        assert build._marshal_digest() != now
    with monkeypatch.context() as m:
        m.setattr(torch._C, "_GLIBCXX_USE_CXX11_ABI", not torch._C._GLIBCXX_USE_CXX11_ABI)
        assert build._marshal_digest() != now
    assert build._marshal_digest() == now


def test_only_what_differs_is_built(monkeypatch):
    from paper_2506_17615_amd import build
    for library, extension in ((False, False), (True, False), (False, True)):
        made = []
        with monkeypatch.context() as m:
            m.setattr(build, "library_is_stale", lambda: library)
            m.setattr(build, "extension_is_stale", lambda: extension)
            m.setattr(build, "_build_library", lambda verbose: made.append("library"))
            m.setattr(build, "_build_marshal", lambda: made.append("extension"))
            build.build(force=False)
        assert made == ["library"] * library + ["extension"] * extension


def test_the_library_needs_no_torch_to_be_built():
    assert _child("""
import sys
sys.modules["torch"] = None
from paper_2506_17615_amd import build
build._build_library = lambda verbose: print("library")
print(build.extension_is_stale())
build.build()
""") == "False\nlibrary\ntorch is not installed: the library is built without the binding's extension\n"


@pytest.mark.gpu
@pytest.mark.parametrize("name", NAMES)
def test_plain_calls_are_taken_and_give_the_same(name):
    eq.load()
    args, outputs = _calls("cuda")[name]
    start = [o.clone() for o in outputs]
    results = []
    for _ in range(2):
        for o, s in zip(outputs, start):
            o.copy_(s)
        if not results:
            assert getattr(eq._native, name)(*args) == 0
        else:
            assert _general(name, args) is None
        results.append([o.clone().view(torch.uint8) for o in outputs])
    assert all(torch.equal(a, b) for a, b in zip(*results))


def _general(name, args):
    native, eq._native = eq._native, _GeneralPath()
    try:
        return getattr(eq, name)(*args)
    finally:
        eq._native = native


def _outcome(f):
    try:
        return f(), None
    except Exception as e:                                   # noqa: BLE001  (whatever it is, both must raise it)
        return None, (type(e), str(e))


@pytest.mark.gpu
@pytest.mark.parametrize("name", NAMES)
def test_altered_calls_end_the_same_way(name):
    """Wrong types, lengths, devices, layouts, numbers and containers: the same exception, or the same bits."""
    eq.load()
    args, outputs = _calls("cuda")[name]
    for bad in _altered(args):
        results = []
        for f in (lambda: getattr(eq, name)(*bad), lambda: _general(name, bad)):
            for o in outputs:
                o.zero_()
            results.append((_outcome(f), [o.clone().view(torch.uint8) for o in outputs]))
        (a, bits_a), (b, bits_b) = results
        assert a == b and all(torch.equal(p, q) for p, q in zip(bits_a, bits_b)), (name, a, b)
