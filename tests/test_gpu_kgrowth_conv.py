"""The product of swiftcl_cl_kgrowth at the edges of its tiles: 16 multipoles, 7 multipole tiles per
workgroup, 16 k nodes and one or two column tiles per wavefront, kinds with one tracer, points without a
kind, 2 nodes.  Against the FP64 oracle (1e-4, the FP32 target) and against the node-coefficient path
(swiftcl_cl_kgrowth_nodes): each window carries at most about sqrt(1024) FP32 roundings of its row's
scale, 2e-6, so two C_l differ by at most 1e-5 on the metric |dC^{ij}| / sqrt(C^{ii} C^{jj})."""
import sys

import numpy as np
import pytest
import torch

import synth
from oracle import fftlog, kgrowth
from tests.helpers import eps_metric, full_from_packed

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def dev():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    return torch.device("cuda:0")


def _workload(tracers, L, n_k, B, n_nodes):
    """cfg1 (10 clustering, 5 lensing tracers; 103 l) cut to `tracers`, L slots (repeated past 103) and n_k."""
    wl = synth.make_workload("cfg1")
    wl["k"], wl["pk"] = wl["k"][:n_k], wl["pk"][:, :n_k]
    slots = np.linspace(0, 102, L).round().astype(np.int32) if L <= 103 else np.arange(L, dtype=np.int32) % 103
    wl["ell_idx"] = wl["ell_idx"][:, slots]
    for n in ("kind", "nz", "bias"):
        wl[n] = wl[n][:, tracers]
    wl["n_tracers"], wl["n_ell"] = np.array([len(tracers)], np.int32), np.array([L], np.int32)
    synth.scale_dependent_growth(wl, n_nodes, f_nu=0.3)
    for n in ("n_tracers", "kind", "n_ell", "ell_idx", "chi_z", "D_z", "omega_m", "nz", "bias", "pk", "D_kz"):
        wl[n] = np.ascontiguousarray(np.repeat(wl[n], B, 0))
    wl["batch"] = B
    return wl


@pytest.mark.parametrize("tracers,L,n_k,B,n_nodes", [
    ([3], 1, 1024, 1, 2),                       # one tracer, one multipole
    ([10], 16, 1010, 1, 5),                     # one lensing tracer, a full row tile, a k tile of 2 nodes
    ([0, 12, 4], 17, 1022, 1, 17),              # kinds out of order, one row past a tile
    (list(range(7)), 103, 1024, 12, 40),        # two column tiles per wavefront, clustering only
    (list(range(15)), 113, 1024, 5, 64),        # two row groups
    (list(range(14, -1, -1)), 112, 1008, 1, 9), # seven full row tiles, lensing first
])
def test_kgrowth_product_tile_edges(dev, tracers, L, n_k, B, n_nodes):
    from paper_2505_22718_amd.plan import Plan, device_inputs
    wl = _workload(tracers, L, n_k, B, n_nodes)
    T = len(tracers)
    print(f"kgrowth product T={T} L={L} n_k={n_k} B={B} nodes={n_nodes}", flush=True)
    p = Plan.for_workload(wl, precision="fp32", n_interp=n_nodes)
    t = device_inputs(wl, dev)
    D = torch.as_tensor(wl["D_kz"], dtype=torch.float64, device=dev)
    C = p.cl_kgrowth(t, D).cpu().numpy().astype(np.float64)
    Cn = p.cl_kgrowth_nodes(t, D).cpu().numpy().astype(np.float64)
    assert p.device_flags() == 0
    for b in {0, B - 1}:
        e = eps_metric(full_from_packed(C[b], T), full_from_packed(Cn[b], T))
        print(f"  point {b}: against the node coefficients {e.max():.2e}", flush=True)
        assert e.max() < 1e-5
    slots = np.unique([0, L // 2, L - 1])
    m = fftlog.method_for(wl)
    W = kgrowth.windows_point(kgrowth.node_geometries(wl, 0), fftlog.point_ells(wl, 0)[slots], m)
    e = eps_metric(full_from_packed(C[0][slots], T), full_from_packed(fftlog.cl_from_windows(W, wl["pk"][0], m), T))
    print(f"  against the oracle {e.max():.2e}", flush=True)
    sys.stdout.flush()
    assert e.max() < 1e-4
