"""Batches whose (point, slot) workgroups hold more than the 2^32 threads of one grid dimension: they run as
several launches.  Every point is the same, so every row of a result has to equal that of a small batch."""
import numpy as np
import pytest
import torch

import synth

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def dev():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    return torch.device("cuda:0")


def _plan(B, max_ell, L, n_k, **kw):
    """One clustering tracer, n_chi = 256, one bias band; L of max_ell slots in use; B equal points."""
    from paper_2505_22718_amd.plan import Plan, device_inputs
    wl = synth.make_workload("cfg1")
    k = np.geomspace(wl["k"][0], wl["k"][-1], n_k)
    wl["pk"] = np.exp(np.interp(np.log(k), np.log(wl["k"]), np.log(wl["pk"][0])))[None]
    wl["k"], wl["n_chi"] = k, 256
    for n in ("kind", "nz", "bias"):
        wl[n] = np.ascontiguousarray(wl[n][:, :1])
    wl["n_tracers"], wl["n_ell"] = np.array([1], np.int32), np.array([L], np.int32)
    wl["ell_idx"] = np.resize(np.arange(0, 103, 7), max_ell).astype(np.int32)[None]
    wl["batch"] = 1
    t = {n: x.expand(B, *x.shape[1:]).contiguous() for n, x in device_inputs(wl, "cuda:0").items()}
    return Plan.for_workload(wl, max_batch=B, precision="fp32", band_ell_lo=(0.0,),
                             fftlog_b=((0.1,), (-1.5,), (-1.0,)), **kw), t


def test_projection(dev):
    """4200 points of 1024 multipole slots through k_windows_p: 4.3 million workgroups of 1024 threads."""
    p, t = _plan(4200, 1024, 1024, 64, rsd=True)
    C = p.cl(t)
    assert p.device_flags() == 0
    p1, t1 = _plan(3, 1024, 1024, 64, rsd=True)
    ref = p1.cl(t1)[:1]
    assert bool(ref.ne(0).all())
    assert bool((C == ref).all())


def test_fused_projection_and_windows(dev):
    """The same workgroups through k_windows_cl, for C_l and for the windows themselves."""
    p, t = _plan(4200, 1024, 1024, 64)
    p1, t1 = _plan(3, 1024, 1024, 64)
    ref = p1.cl(t1)[:1]
    assert bool(ref.ne(0).all())
    assert bool((p.cl(t) == ref).all())
    ref = p1.windows(t1)[:1]
    W = p.windows(t)
    assert p.device_flags() == 0
    for b in range(0, 4200, 600):
        assert bool((W[b:b + 600] == ref).all()), b


def test_rows_adjoint(dev):
    """16400 points of 256 multipole chunks through k_bwd_rows: 4.2 million workgroups of 1024 threads."""
    p, t = _plan(16400, 1024, 256, 256, rsd=True)
    g = p.backward(t, torch.ones((16400, 1024, 1), device=dev), want=("pk", "bias"))
    assert p.device_flags() == 0
    for name, x in g.items():
        assert bool(x[0].ne(0).any()), name
        assert bool((x == x[:1]).all()), name
    # C is linear in P: sum_k P_k dL/dP_k = L
    L = p.cl(t)[:, :256].double().sum((1, 2))
    assert float((((g["pk"] * t["pk"]).sum(1) - L) / L).abs().max()) < 1e-5


def test_limber(dev):
    """16400 points of 4096 slots (512 groups, 2 slots in use): 8.4 million workgroups of 512 threads."""
    p, t = _plan(16400, 4096, 2, 64)
    C = p.cl_limber(t)
    assert p.device_flags() == 0
    p1, t1 = _plan(3, 4096, 2, 64)
    ref = p1.cl_limber(t1)[:1]
    assert bool(ref[0, :2].ne(0).all()) and bool(ref[0, 2:].eq(0).all())
    assert bool((C == ref).all())
