"""The extension module's marshalling against the Python one: the same results
for what both take (also on another stream, with fewer points, through views
and Parameters), and the same refusal for what the Python one refuses."""
import numpy as np
import pytest
import torch

from gpu_common import DTYPES, GAMMA, require_gpu, states
from paper_1809_09851_amd import fdbb as F

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    require_gpu()


def python_only(monkeypatch):
    for name in ("_run", "_char_apply", "_viscous_flux", "_empty_fields", "_empty_blocks"):
        monkeypatch.setattr(F, name, lambda *a: None)


def calls(dim, U, X, G, gT, dt):
    """(name, call(out...), shapes of the outputs) of every entry point."""
    K, n = dim + 2, U.shape[1]
    f = lambda k: F.empty_fields(k, n, dt).fill_(5.0)
    b = lambda: F.empty_blocks(dim, n, dt).fill_(5.0)
    flat = lambda: torch.full((n,), 5.0, dtype=dt, device="cuda")
    w = lambda k: torch.ones((k, n), dtype=dt, device="cuda")
    return {
        "cons2prim": (lambda V, **k: F.fdbb_cons2prim(dim, GAMMA, U, V, **k), lambda: [f(K)]),
        "prim2cons": (lambda V, **k: F.fdbb_prim2cons(dim, GAMMA, U, V, **k), lambda: [f(K)]),
        "eos": (lambda p, c, **k: F.fdbb_eos(dim, GAMMA, U, p, c, **k), lambda: [flat(), flat()]),
        "flux": (lambda o, **k: F.fdbb_flux(dim, GAMMA, U, o, **k), lambda: [f(K * dim)]),
        "flux_dir": (lambda o, **k: F.fdbb_flux_direction(dim, dim - 1, GAMMA, U, o, **k), lambda: [f(K)]),
        "flux_jacobian": (lambda A, **k: F.fdbb_flux_jacobian(dim, GAMMA, U, A, **k), lambda: [b()]),
        "riemann": (lambda R, **k: F.fdbb_riemann_invariants(dim, GAMMA, U, R, **k), lambda: [f(2 * dim + 1)]),
        "cons2char": (lambda W, **k: F.fdbb_cons2char(dim, 0, GAMMA, U, W, **k), lambda: [f(K)]),
        "fused": (lambda o, A, R, **k: F.fdbb_euler_fused(dim, GAMMA, U, o, A, R, **k),
                  lambda: [f(K * dim), b(), f(2 * dim + 1)]),
        "adjoint": (lambda o, **k: F.fdbb_flux_adjoint(dim, -1, GAMMA, U, w(K * dim), o, **k), lambda: [f(K)]),
        "adjoint_dir": (lambda o, **k: F.fdbb_flux_adjoint(dim, 0, GAMMA, U, X, o, **k), lambda: [f(K)]),
        "eigenvectors": (lambda L, R, **k: F.fdbb_eigenvectors(dim, GAMMA, U, L, R, **k), lambda: [b(), b()]),
        "char_apply": (lambda Y, **k: F.fdbb_char_apply(dim, 0, 1, GAMMA, U, X, Y, **k), lambda: [f(K)]),
        "roe": (lambda o, **k: F.fdbb_roe_average(dim, GAMMA, U, U, o, **k), lambda: [f(K)]),
        "viscous": (lambda o, **k: F.fdbb_viscous_flux(dim, 0.01, 0.02, U, G, gT, o, **k), lambda: [f(K * dim)]),
    }


@pytest.mark.parametrize("dt", ("f64", "f32"))
@pytest.mark.parametrize("dim", (1, 2, 3))
def test_same_results_both_ways(dim, dt, monkeypatch):
    n = 333
    _, U = states(dim, n + 2, 3, dt)
    U = torch.nn.Parameter(U.contiguous(), requires_grad=False)[:, 1:-1]
    X, G, gT = (torch.randn(k, n, device="cuda").to(DTYPES[dt]) for k in (dim + 2, dim * dim, dim))
    side = torch.cuda.Stream()
    table = calls(dim, U, X, G, gT, DTYPES[dt])
    native, python = {}, {}
    for into in (native, python):
        if into is python:
            python_only(monkeypatch)
        for name, (call, outs) in table.items():
            for label, kw in (("", {}), ("n", {"n": 200}), ("stream", {"stream": side}), ("handle", {"stream": side.cuda_stream})):
                o = outs()
                torch.cuda.synchronize()
                call(*o, **kw)
                torch.cuda.synchronize()
                into[name, label] = o
    for key, o in native.items():
        for x, y in zip(o, python[key]):
            assert torch.equal(x, y), key
            assert not bool((x == 5.0).all()), key
    for t, k in ((F.flux(U), dim * (dim + 2)), (F.cons2prim(U), dim + 2)):
        assert t.shape == (k, n) and t.stride() == (F.padded_ld(n), 1) and t.dtype == DTYPES[dt]
    monkeypatch.undo()
    for t, k in ((F.flux(U), dim * (dim + 2)), (F.cons2prim(U), dim + 2)):
        assert t.shape == (k, n) and t.stride() == (F.padded_ld(n), 1) and t.dtype == DTYPES[dt] and not t.requires_grad
    A = F.flux_jacobian(U)
    K = dim + 2
    assert A.shape == (dim, n, K, K) and A.stride(0) == F.padded_ld(n) * K * K


class Marked(torch.Tensor):
    pass


def test_same_refusals_both_ways(monkeypatch):
    _, U = states(3, 100, 3)
    V, P = F.empty_fields(5, 100), F.empty_fields(15, 100)
    A = F.empty_blocks(3, 100)
    bad = [
        lambda: F.fdbb_cons2prim(3, 1.4, U.cpu(), V),
        lambda: F.fdbb_cons2prim(3, 1.4, U, None),
        lambda: F.fdbb_cons2prim(3, 1.4, U, V[:4]),
        lambda: F.fdbb_cons2prim(3, 1.4, U.long(), V),
        lambda: F.fdbb_cons2prim(3, 1.4, U.t().contiguous().t(), V),
        lambda: F.fdbb_cons2prim(3, 0.9, U, V),
        lambda: F.fdbb_cons2prim(3, torch.tensor(1.4), U, V),
        lambda: F.fdbb_cons2prim(np.int64(3), 1.4, U, V),
        lambda: F.fdbb_cons2prim(3, "1.4", U, V),
        lambda: F.fdbb_cons2prim(3, 1.4, U, V, n=-1),
        lambda: F.fdbb_cons2prim(3, 1.4, U, V, n=101 * 64),
        lambda: F.fdbb_flux(3, 1.4, U, V),
        lambda: F.fdbb_flux(4, 1.4, U, P),
        lambda: F.fdbb_flux(3, 1.4, V, P[:, ::2]),
        lambda: F.fdbb_flux_direction(3, 3, 1.4, U, V),
        lambda: F.fdbb_flux_jacobian(3, 1.4, U, A.transpose(2, 3)),
        lambda: F.fdbb_euler_fused(3, 1.4, U),
        lambda: F.fdbb_flux_adjoint(3, -1, 1.4, U, V, V),
        lambda: F.fdbb_char_apply(3, 0, 2, 1.4, U, U, V),
        lambda: F.fdbb_viscous_flux(3, -1.0, 0.0, U, F.empty_fields(9, 100), F.empty_fields(3, 100), P),
        lambda: F.fdbb_roe_average(3, 1.4, U, U, U[:, 1:]),
    ]

    def refusals():
        got = []
        for call in bad:
            try:
                call()
                got.append("accepted")
            except Exception as e:
                got.append((type(e), str(e)))
        return got

    native = refusals()
    # ctypes converts a tensor to a double and a numpy integer to an int
    assert [k for k, got in enumerate(native) if got == "accepted"] == [6, 7]
    same = Marked(U.clone())
    F.fdbb_cons2prim(3, 1.4, same, V)  # a subclass takes the general path
    python_only(monkeypatch)
    assert refusals() == native
    W = F.empty_fields(5, 100)
    F.fdbb_cons2prim(3, 1.4, U, W)
    torch.cuda.synchronize()
    assert torch.equal(V, W)
