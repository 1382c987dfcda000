"""CPU checks of the binding's extension: the plain calls it takes end as the ctypes calls do, and what it does not take is
handed back untouched and accepted or refused by ctypes as ever.  No call gets as far as a launch."""
import ctypes
import os

import numpy as np
import pytest
import torch

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
A = 0x1000                                       # an address nobody reads


@pytest.fixture(scope="module")
def nq():
    if not os.path.exists(os.path.join(ROOT, "paper_2506_17870_amd", "libnq.so")):
        from paper_2506_17870_amd import build
        build.build()
    import paper_2506_17870_amd as nq
    return nq


def weight(nq, n_bits=8, resident=1, N=32, K=64):
    big = 1 << 20
    return nq.nq_weight(nq.make_cfg(n_bits, 2), N, K, A, big, A, big, None, A, resident, 0, None, None, 0, 0, 0, 0)


def calls(nq, w, x, y, M=4, stream=0):
    """Every inference call that goes through the extension, and what the same arguments give through ctypes."""
    e, lib, by = nq.make_epilogue(0.5), nq.binding._lib, ctypes.byref
    sh, px, py = nq.nq_conv_shape(M, 1, 1, 64, 32, 1, 1, 1, 0), nq.binding._ptr(x), nq.binding._ptr(y)
    for kind in ("full", "part"):
        g, c, gc = (getattr(nq, f"nq_{n}_{kind}") for n in ("gemm", "conv", "gconv"))
        yield lambda g=g: g(x, M, w, e, y, stream), getattr(lib, f"nq_gemm_{kind}")(px, M, by(w), by(e), py, stream)
        yield lambda c=c: c(x, sh, w, e, y, stream), getattr(lib, f"nq_conv_{kind}")(px, by(sh), by(w), by(e), py, stream)
        yield lambda gc=gc: gc(x, sh, 1, w, e, y, stream), getattr(lib, f"nq_gconv_{kind}")(px, by(sh), 1, by(w), by(e), py, stream)
        full = kind == "full"
        args = (w, 0.5, None, None, 0.0, False, False, 1.0, y, stream)
        yield lambda full=full: nq.run_layer(full, x, M, *args), getattr(lib, f"nq_gemm_{kind}")(px, M, by(w), by(e), py, stream)
        yield (lambda full=full: nq.run_layer(full, x, (M, 1, 1, 64, 32, 1, 1, 0), *args),
               getattr(lib, f"nq_conv_{kind}")(px, by(sh), by(w), by(e), py, stream))


@pytest.mark.parametrize("case", ["bits", "paged out", "no input", "empty", "cpu tensors"])
def test_same_status_as_ctypes(nq, case):
    w = weight(nq, n_bits=7 if case == "bits" else 8, resident=0 if case == "paged out" else 1)
    x, y, M = A, A, 4
    if case == "paged out":
        w.N = 0                                   # part-bit: nothing to compute
    if case == "no input":
        x = None
    if case in ("empty", "cpu tensors"):
        M = 0
    if case == "cpu tensors":
        x, y = torch.zeros(4, 64, dtype=torch.int8), torch.zeros(4, 32)
    for call, status in calls(nq, w, x, y, M):
        if status == nq.NQ_OK:
            call()
        else:
            with pytest.raises(nq.NQError) as err:
                call()
            assert err.value.status == status


def test_what_is_not_plain(nq):
    w, e = weight(nq), nq.make_epilogue(0.5)
    fast = nq.binding._fast
    t = torch.zeros(8, 8)
    assert fast.gemm(1, t.t(), 0, w, e, A, 0) == -1               # not contiguous
    with pytest.raises(AssertionError):
        nq.nq_gemm_full(t.t(), 0, w, e, A, stream=0)
    assert fast.gemm(1, A, np.int64(0), w, e, A, 0) == -1         # ctypes takes it
    nq.nq_gemm_full(A, np.int64(0), w, e, A, stream=0)
    nq.nq_gemm_full(d_x=A, M=0, w=w, epi=e, d_y=A, stream=0)      # by name
    for bad in (dict(w=e), dict(epi=w), dict(M="4"), dict(M=1.5), dict(d_x="x")):
        args = dict(d_x=A, M=0, w=w, epi=e, d_y=A, stream=0)
        args.update(bad)
        assert fast.gemm(1, args["d_x"], args["M"], args["w"], args["epi"], A, 0) == -1
        with pytest.raises((ctypes.ArgumentError, TypeError, AttributeError)):
            nq.nq_gemm_full(**args)
    assert fast.gemm(1, A, 1 << 70, w, e, A, 0) == -1 and fast.gemm(1, A, 0, w, e, A) == -1
    assert fast.gconv(1, A, nq.nq_conv_shape(), 1 << 33, w, e, A, 0) == -1
    assert fast.layer(1, A, 0, (1, 1, 1, 64, 32, 1, 1), w, 0.5, None, None, 0.0, 0, 0, 1.0, A, 0) == -1   # seven sizes
    assert fast.layer(1, A, 0, None, w, "s", None, None, 0.0, 0, 0, 1.0, A, 0) == -1
    assert fast.quantize_pack(A, 0, 4, nq.make_cfg(), A, A, A, "s") == -1
    nq.nq_quantize_decompose_pack(A, 0, 4, nq.make_cfg(), A, A, A, stream=0)
    with pytest.raises(nq.NQError) as err:
        nq.nq_quantize_decompose_pack(A, 4, 4, nq.make_cfg(7, 2), A, A, A, stream=0)
    assert err.value.status == nq.NQ_ERR_UNSUPPORTED


def test_lists_of_weights(nq):
    ws = [weight(nq, N=n) for n in (1, 2, 3)]
    arr = nq.binding._wlist(ws)
    assert [arr[i].contents.N for i in range(3)] == [1, 2, 3] and len(nq.binding._wlist([])) == 0
    arr[1].contents.N = 7
    assert ws[1].N == 7


def test_replaced_functions_are_seen_through_the_package(nq, monkeypatch):
    own = nq.nq_gemm_full                         # looked up once: the package holds it
    with monkeypatch.context() as m:
        m.setattr(nq.binding, "nq_gemm_full", "mine")
        assert nq.nq_gemm_full == "mine"
        nq.nq_gemm_full = "here"                  # the package's own stays what its user made it
        m.setattr(nq.binding, "nq_gemm_full", "other")
        assert nq.nq_gemm_full == "here"
        del nq.nq_gemm_full
    assert nq.nq_gemm_full is own and nq.binding.nq_gemm_full is own
    nq.binding.extra = 1
    assert nq.extra == 1
    del nq.binding.extra
    with pytest.raises(AttributeError):
        nq.extra
    monkeypatch.setattr(nq.binding, "extra", None, raising=False)
    assert nq.extra is None
    monkeypatch.setattr(nq.binding, "extra", 2)
    assert nq.extra == 2


@pytest.mark.parametrize("full", [True, False])
@pytest.mark.parametrize("kind", ["conv", "gemm"])
def test_the_walkers_layers_reach_replaced_functions(nq, monkeypatch, kind, full):
    w, seen = weight(nq), []
    name = f"nq_{kind}_{'full' if full else 'part'}"
    monkeypatch.setattr(nq.binding, name, lambda *a: seen.append(a))
    for other in ("conv", "gemm"):
        sizes = 0 if other == "gemm" else (0, 4, 4, 64, 32, 1, 1, 0)
        nq.run_layer(full, A, sizes, w, 0.5, None, None, 0.0, True, True, 2.0, A, 0)      # empty: no launch
    assert len(seen) == 1
    x, what, wd, e, y, stream = seen[0]
    assert (what == 0 if kind == "gemm" else (what.H, what.Cout) == (4, 32)) and wd is w
    assert (x, y, stream, e.act_scale, e.relu, e.out_int8, e.inv_out_scale) == (A, A, 0, 0.5, 1, 1, 2.0)


def test_the_walkers_layers_reach_one_call_in_anothers_place(nq, monkeypatch):
    w = weight(nq, resident=False)
    args = (A, 1, w, 0.5, None, None, 0.0, True, True, 2.0, A, 0)
    with pytest.raises(nq.NQError) as err:
        nq.run_layer(True, *args)
    assert err.value.status == nq.NQ_ERR_NOT_RESIDENT
    seen = []
    monkeypatch.setattr(nq.binding, "run_layer_by_calls", lambda *a: seen.append(a))
    monkeypatch.setattr(nq.binding, "nq_gemm_full", nq.binding.nq_gemm_part)
    nq.run_layer(True, *args)
    assert len(seen) == 1


def test_an_extension_that_is_not_there_is_named(nq):
    import subprocess
    import sys
    code = ("import sys; sys.modules['paper_2506_17870_amd._nqcall'] = None\n"
            "import paper_2506_17870_amd as nq\n"
            "try: nq.nq_gemm_full\n"
            "except ImportError as e: sys.exit(0 if '-m paper_2506_17870_amd.build' in str(e) else 'no hint: %s' % e)\n"
            "sys.exit('it loads')")
    r = subprocess.run([sys.executable, "-c", code], cwd=ROOT, capture_output=True, text=True)
    assert r.returncode == 0, r.stderr


def test_the_extension_is_this_interpreters(nq):
    import sysconfig
    assert nq.binding._fast.__file__.endswith("_nqcall" + sysconfig.get_config_var("EXT_SUFFIX"))
