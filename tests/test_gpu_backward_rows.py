"""The adjoint of RSD and magnification plans (k_bwd_rows) at the edges of its shapes: every transform length
it takes, k grids that end inside a 16-wide tile, 1, 15 and 16 tracers of more slots, fewer multipoles than
chunks, several points.  Identities of the forward call: C is linear in P (sum_k P_k dL/dP_k = L) and quadratic
in every bias (symmetric differences are exact).  FP32 windows carry about 1e-6 of their row's scale, so L, a
sum of n signed terms, is good to 1e-6 sum |dC C|; a factor of 10 is left."""
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


@pytest.mark.parametrize("n_chi,n_k,T,used,L,B", [(256, 256, 15, 15, 103, 3), (512, 386, 16, 16, 40, 2),
                                                  (1024, 1024, 16, 1, 2, 1), (1024, 1018, 15, 15, 103, 9)])
def test_rows_adjoint_identities(dev, n_chi, n_k, T, used, L, B):
    from paper_2505_22718_amd.plan import Plan, device_inputs
    wl = synth.make_workload("cfg1")
    k = np.geomspace(wl["k"][0], wl["k"][-1], n_k)
    wl["pk"] = np.exp(np.interp(np.log(k), np.log(wl["k"]), np.log(wl["pk"][0])))[None]
    wl["k"], wl["n_chi"] = k, n_chi
    for n in ("kind", "nz", "bias"):
        wl[n] = wl[n][:, np.arange(T) % 15]
    wl["ell_idx"] = wl["ell_idx"][:, np.linspace(0, 102, L).round().astype(int)].astype(np.int32)
    wl["n_tracers"], wl["n_ell"] = np.array([used], np.int32), np.array([L], np.int32)
    wl["mag"] = np.where(wl["kind"] == 0, 0.3, 0.0)
    for n in ("n_tracers", "kind", "n_ell", "ell_idx", "chi_z", "D_z", "omega_m", "nz", "bias", "pk", "mag"):
        wl[n] = np.ascontiguousarray(np.repeat(wl[n], B, 0))
    wl["batch"] = B
    wl["bias"] = wl["bias"] * (1.0 + 0.1 * np.arange(B))[:, None]
    print(f"rows adjoint n_chi={n_chi} n_k={n_k} T={used}/{T} L={L} B={B}", flush=True)
    p = Plan.for_workload(wl, precision="fp32", rsd=True, magnification=True)
    t = device_inputs(wl, dev)
    C = p.cl(t).double()
    dC = torch.randn(C.shape, generator=torch.Generator().manual_seed(5)).to(dev)
    g = p.backward(t, dC, want=("pk", "bias"))
    assert p.device_flags() == 0
    scale = (dC.double() * C).abs().sum((1, 2))
    e = ((g["pk"] * t["pk"]).sum(1) - (dC.double() * C).sum((1, 2))).abs() / scale
    print(f"  dP identity {e.max().item():.2e}", flush=True)
    assert e.max().item() < 1e-5
    tr = min(4, used - 1)
    diff = []
    for f in (1.5, 0.5):
        b = t["bias"].clone()
        b[:, tr] *= f
        diff.append((dC.double() * p.cl(dict(t, bias=b)).double()).sum((1, 2)))
    e = (g["bias"][:, tr] * t["bias"][:, tr] - (diff[0] - diff[1])).abs() / scale
    print(f"  db of tracer {tr} {e.max().item():.2e}", flush=True)
    assert e.max().item() < 1e-5
