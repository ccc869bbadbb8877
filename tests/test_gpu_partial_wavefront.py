"""The assembly's node loop where the support ends one node into a wavefront (64 q + 1 nodes): the last lane
works alone and takes every tracer's kind and bias.  All tracers of one and of two tracer groups against the
FP64 oracle (1e-4 on |dC^{ij}| / sqrt(C^{ii} C^{jj}), the FP32 target)."""
import numpy as np
import pytest
import torch

import synth
from oracle import fftlog
from tests.helpers import eps_metric, full_from_packed

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("T,q,n_chi", [(15, 1, 256), (15, 3, 512), (31, 5, 1024)])
def test_support_of_one_node_past_a_wavefront(T, q, n_chi):
    from paper_2505_22718_amd.plan import Plan, device_inputs
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    wl = synth.make_workload("cfg1")
    sel = np.arange(T) % 15
    for n in ("kind", "nz", "bias"):
        wl[n] = np.ascontiguousarray(wl[n][:, sel])
    wl["bias"] = wl["bias"] * (1.0 + 0.02 * np.arange(T))
    wl["n_tracers"] = np.array([T], np.int32)
    wl["ell_idx"] = np.ascontiguousarray(wl["ell_idx"][:, [0, 50, 102]])
    wl["n_ell"] = np.array([3], np.int32)
    # the step of ln k (and ln chi) that puts 64 q + 0.5 steps between the edges of the support
    chi = wl["chi_z"][0]
    delta = np.log(chi[-1] / chi[0]) / (64 * q + 0.5)
    n_k = min(n_chi, 2 * int(np.log(1e5) / delta / 2))
    k = 1e-4 * np.exp(delta * np.arange(n_k))
    wl["pk"] = np.exp(np.interp(np.log(k), np.log(wl["k"]), np.log(wl["pk"][0])))[None]
    wl["k"], wl["n_chi"] = k, n_chi
    m = fftlog.method_for(wl)
    from oracle.geometry import point_geometry
    assert len(fftlog.edge_weights(point_geometry(wl, 0), m)[0]) == 64 * q + 1
    print(f"partial wavefront T={T} nodes={64 * q + 1} n_k={n_k}", flush=True)
    p = Plan.for_workload(wl, precision="fp32")
    C = p.cl(device_inputs(wl, "cuda:0")).cpu().numpy().astype(np.float64)[0]
    assert p.device_flags() == 0
    e = eps_metric(full_from_packed(C, T), full_from_packed(fftlog.cl(wl, 0), T))
    print(f"  max eps {e.max():.2e}", flush=True)
    assert e.max() < 1e-4
