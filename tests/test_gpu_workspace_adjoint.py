"""The adjoint through the workspace (k_bwd_wy, k_bwd_adj) at the edges of its shapes and across its point
chunks: every transform length, one and two tracers per wavefront, k grids that end inside a slab or a tile and
those that are no multiple of 4, RSD and magnification, more points than a chunk holds.  Identities of the
forward call: C is linear in P (sum_k P_k dL/dP_k = L) and quadratic in every bias (symmetric differences are
exact).  FP32 windows carry about 1e-6 of their row's scale, so L, a sum of n signed terms, is good to 1e-6 sum
|dC C|; a factor of 10 is left.  A point's sums do not depend on its chunk: equal bit for bit."""
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


@pytest.mark.parametrize("n_chi,n_k,T,used,L,B,rsd,mag,precision", [
    (256, 200, 32, 32, 20, 3, False, False, "fp32"),
    (256, 256, 17, 3, 5, 5, True, True, "fp32"),
    (512, 386, 17, 17, 40, 2, False, False, "split_bf16"),
    (512, 512, 31, 31, 103, 9, True, False, "fp32"),
    (1024, 1018, 31, 31, 30, 3, False, True, "fp32"),
    (1024, 1024, 32, 16, 7, 11, True, True, "split_bf16"),
    (2048, 1026, 16, 16, 12, 3, False, False, "fp32"),
    (2048, 2048, 15, 15, 12, 5, True, True, "fp32"),
    (2048, 1400, 1, 1, 3, 4, True, False, "fp32"),
    (2048, 1026, 32, 32, 12, 2, True, True, "fp32"),
])
def test_identities_and_point_chunks(dev, n_chi, n_k, T, used, L, B, rsd, mag, precision):
    from paper_2505_22718_amd.plan import Plan, device_inputs
    wl = synth.make_workload("cfg1")
    k = np.geomspace(wl["k"][0], wl["k"][-1], n_k)
    wl["pk"] = np.exp(np.interp(np.log(k), np.log(wl["k"]), np.log(wl["pk"][0])))[None]
    wl["k"], wl["n_chi"] = k, n_chi
    for n in ("kind", "nz", "bias"):
        wl[n] = wl[n][:, np.arange(T) % 15]
    wl["ell_idx"] = wl["ell_idx"][:, np.linspace(0, 102, L).round().astype(int)].astype(np.int32)
    wl["n_tracers"], wl["n_ell"] = np.array([used], np.int32), np.array([L], np.int32)
    if mag:
        wl["mag"] = np.where(wl["kind"] == 0, 0.3, 0.0)
    for n in ("n_tracers", "kind", "n_ell", "ell_idx", "chi_z", "D_z", "omega_m", "nz", "bias", "pk", "mag"):
        if n in wl:
            wl[n] = np.ascontiguousarray(np.repeat(wl[n], B, 0))
    wl["batch"] = B
    wl["bias"] = wl["bias"] * (1.0 + 0.1 * np.arange(B))[:, None]
    print(f"workspace adjoint n_chi={n_chi} n_k={n_k} T={used}/{T} L={L} B={B} rsd={rsd} mag={mag}", flush=True)
    p = Plan.for_workload(wl, precision=precision, rsd=rsd, magnification=mag)
    assert p.adjoint_mode == 2
    t = device_inputs(wl, dev)
    C = p.cl(t).double()
    dC = torch.randn(C.shape, generator=torch.Generator().manual_seed(5)).to(dev)
    assert p.workspace_points()["adjoint"] == B
    g = p.backward(t, dC, want=("pk", "bias"))
    for limit in (1, B - 1):
        assert p.workspace_points(limit)["adjoint"] == limit
        h = p.backward(t, dC, want=("pk", "bias"))
        for n in g:
            assert bool(torch.equal(g[n], h[n])), (n, limit)
    assert p.workspace_points(0)["adjoint"] == B
    assert p.device_flags() == 0
    # split plans project in bf16 hi + lo, the adjoint computes in FP32: their C is good to 1e-5 of its scale
    tol = 1e-5 if precision == "fp32" else 1e-4
    scale = (dC.double() * C).abs().sum((1, 2))
    e = ((g["pk"] * t["pk"]).sum(1) - (dC.double() * C).sum((1, 2))).abs() / scale
    print(f"  dP identity {e.max().item():.2e}", flush=True)
    assert e.max().item() < tol
    tr = min(4, used - 1)
    diff = []
    for f in (1.5, 0.5):
        b = t["bias"].clone()
        b[:, tr] *= f
        diff.append((dC.double() * p.cl(dict(t, bias=b)).double()).sum((1, 2)))
    e = (g["bias"][:, tr] * t["bias"][:, tr] - (diff[0] - diff[1])).abs() / scale
    print(f"  db of tracer {tr} {e.max().item():.2e}", flush=True)
    assert e.max().item() < tol


@pytest.mark.parametrize("n_chi,n_k,T,B,n_nodes,precision", [
    (256, 200, 15, 5, 20, "fp32"), (512, 512, 17, 3, 9, "split_bf16"), (1024, 1024, 32, 7, 40, "fp32"),
    (2048, 1400, 5, 2, 30, "fp32"), (2048, 2048, 18, 3, 12, "fp32")])
def test_growth_product_shapes_and_point_chunks(dev, n_chi, n_k, T, B, n_nodes, precision):
    """swiftcl_cl_kgrowth at every transform length and with more than 16 tracers, whole and in chunks of 1 and
    B - 1 points, against the node coefficients (1e-5 of sqrt(C^{ii} C^{jj}): two sums of about 1024 FP32
    roundings; split plans 2e-5 more, one bf16 hi + lo rounding of each operand per sum)."""
    from paper_2505_22718_amd.plan import Plan, device_inputs
    from tests.helpers import eps_metric, full_from_packed
    wl = synth.make_workload("cfg1")
    k = np.geomspace(wl["k"][0], wl["k"][-1], n_k)
    wl["pk"] = np.exp(np.interp(np.log(k), np.log(wl["k"]), np.log(wl["pk"][0])))[None]
    wl["k"], wl["n_chi"] = k, n_chi
    for n in ("kind", "nz", "bias"):
        wl[n] = wl[n][:, np.arange(T) % 15]
    wl["bias"] = wl["bias"] * (1.0 + 0.02 * np.arange(T))
    wl["ell_idx"] = np.ascontiguousarray(wl["ell_idx"][:, ::6])
    L = wl["ell_idx"].shape[1]
    wl["n_tracers"], wl["n_ell"] = np.array([T], np.int32), np.array([L], np.int32)
    synth.scale_dependent_growth(wl, n_nodes, f_nu=0.3)
    for n in ("n_tracers", "kind", "n_ell", "ell_idx", "chi_z", "D_z", "omega_m", "nz", "bias", "pk", "D_kz"):
        wl[n] = np.ascontiguousarray(np.repeat(wl[n], B, 0))
    wl["bias"] = wl["bias"] * (1.0 + 0.1 * np.arange(B))[:, None]
    wl["batch"] = B
    print(f"growth product n_chi={n_chi} n_k={n_k} T={T} B={B} nodes={n_nodes} {precision}", flush=True)
    p = Plan.for_workload(wl, precision=precision, n_interp=n_nodes)
    t = device_inputs(wl, dev)
    D = torch.as_tensor(wl["D_kz"], dtype=torch.float64, device=dev)
    ref = full_from_packed(p.cl_kgrowth_nodes(t, D).cpu().numpy().astype(np.float64), T)
    assert p.workspace_points()["growth"] == B
    for limit in (0, 1, B - 1):
        assert p.workspace_points(limit)["growth"] == (limit or B)
        C = full_from_packed(p.cl_kgrowth(t, D).cpu().numpy().astype(np.float64), T)
        e = max(eps_metric(C[b], ref[b]).max() for b in range(B))
        print(f"  chunks of {limit or B}: {e:.2e}", flush=True)
        assert e < (1e-5 if precision == "fp32" else 3e-5)
    assert p.device_flags() == 0
