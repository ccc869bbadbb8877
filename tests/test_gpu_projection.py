"""The projection of plans beyond the fused kernel (k_windows_p: rows in registers, slabs of k through LDS)
at the edges of its shapes: every transform length, one and two tracers per wavefront (16, 17, 31 and 32
slots, fewer in use), k grids that end inside a slab, a padded multipole slot; FP32 and BF16 hi+lo against
the FP64 oracle (1e-4 and 1e-3 on |dC^{ij}| / sqrt(C^{ii} C^{jj}), the targets of the two precisions)."""
import numpy as np
import pytest
import torch

import synth
from oracle import fftlog
from tests.helpers import eps_metric, full_from_packed

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def dev():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    return torch.device("cuda:0")


def _workload(n_chi, n_k, T, used):
    """`used` of T tracer slots from the 15 tracers of cfg1 (cyclically, biases made distinct), 3 l of 4 slots."""
    wl = synth.make_workload("cfg1")
    k = np.geomspace(wl["k"][0], wl["k"][-1], n_k)
    wl["pk"] = np.exp(np.interp(np.log(k), np.log(wl["k"]), np.log(wl["pk"][0])))[None]
    wl["k"], wl["n_chi"] = k, n_chi
    sel = np.arange(T) % 15
    for n in ("kind", "nz", "bias"):
        wl[n] = np.ascontiguousarray(wl[n][:, sel])
    wl["bias"] = wl["bias"] * (1.0 + 0.01 * np.arange(T))
    wl["n_tracers"], wl["n_ell"] = np.array([used], np.int32), np.array([3], np.int32)
    wl["ell_idx"] = wl["ell_idx"][:, [0, 40, 102, 7]].copy()
    return wl


@pytest.mark.parametrize("n_chi,n_k,T,used,precision", [
    (256, 256, 17, 17, "fp32"), (256, 200, 32, 32, "split_bf16"),
    (512, 512, 31, 16, "split_bf16"), (512, 386, 32, 31, "fp32"),
    (1024, 1022, 17, 2, "fp32"), (1024, 1024, 32, 32, "split_bf16"),
    (2048, 2048, 16, 16, "fp32"), (2048, 1400, 16, 15, "split_bf16"), (2048, 1026, 32, 30, "fp32"),
])
def test_projection_edges(dev, n_chi, n_k, T, used, precision):
    from paper_2505_22718_amd.plan import Plan, device_inputs
    wl = _workload(n_chi, n_k, T, used)
    print(f"projection n_chi={n_chi} n_k={n_k} T={used}/{T} {precision}", flush=True)
    p = Plan.for_workload(wl, precision=precision)
    C = p.cl(device_inputs(wl, dev)).cpu().numpy().astype(np.float64)[0]
    assert p.device_flags() == 0
    assert np.all(C[3] == 0)
    full = full_from_packed(C[:3], T)
    assert np.all(full[:, used:, :] == 0)
    sub = dict(wl, **{n: np.ascontiguousarray(wl[n][:, :used]) for n in ("kind", "nz", "bias")},
               ell_idx=wl["ell_idx"][:, :3].copy())
    Cref = fftlog.cl(sub, 0)
    e = eps_metric(full[:, :used, :used], full_from_packed(Cref, used))
    print(f"  max eps {e.max():.3e}", flush=True)
    assert e.max() < (1e-4 if precision == "fp32" else 1e-3)
