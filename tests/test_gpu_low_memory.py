"""Plans on a device with little free memory: the chunked workspace takes what is left after everything that the
plan cannot do without, and the results are those of the full workspace.  (The memory is held by tensors; every
kernel has run once before, so that the runtime's own allocations are made.)"""
import numpy as np
import pytest
import torch

import synth
from tests.helpers import eps_metric, full_from_packed

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def dev():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    return torch.device("cuda:0")


def _free():
    torch.cuda.synchronize()
    torch.cuda.empty_cache()
    return torch.cuda.mem_get_info()[0]


def _hold_all_but(target):
    held = []
    while _free() > target + (4 << 20):
        held.append(torch.empty(min(_free() - target, 32 << 30), dtype=torch.uint8, device="cuda:0"))
    return held


def _workload(T, B):
    """cfg1 with T tracers (cyclically) and B equal points."""
    wl = synth.make_workload("cfg1")
    for n in ("kind", "nz", "bias"):
        wl[n] = wl[n][:, np.arange(T) % 15]
    wl["bias"] = wl["bias"] * (1.0 + 0.01 * np.arange(T))
    wl["n_tracers"] = np.array([T], np.int32)
    for n in ("n_tracers", "kind", "n_ell", "ell_idx", "chi_z", "D_z", "omega_m", "nz", "bias", "pk"):
        wl[n] = np.ascontiguousarray(np.repeat(wl[n], B, 0))
    wl["bias"] *= (1.0 + 0.1 * np.arange(B) / B)[:, None]
    wl["batch"] = B
    return wl


def _roomy_and_tight(make, run, short):
    """run(plan) with all memory free, and on a plan built with `short` bytes less than that one took."""
    before = _free()
    p = make()
    size = before - _free()
    ref = run(p)
    p.close()
    print(f"  the full plan takes {size / 2**20:.0f} MiB; now {(size - short) / 2**20:.0f} MiB are free", flush=True)
    held = _hold_all_but(size - short)
    try:
        p = make()
    finally:
        del held
    got = run(p)
    assert p.device_flags() == 0
    return ref, got


def test_workspace_adjoint(dev):
    """30 tracers, 256 points at most: V rows of 256 points would take 3.5 GB of 4.9; 45 points of gradients."""
    from paper_2505_22718_amd.plan import Plan, device_inputs
    wl = _workload(30, 45)
    t = device_inputs(wl, dev)
    G = torch.randn((45, 103, 465), generator=torch.Generator().manual_seed(3)).to(dev)
    ref, got = _roomy_and_tight(lambda: Plan.for_workload(wl, precision="fp32", max_batch=256),
                                lambda p: p.backward(t, G, want=("pk", "bias")), 512 << 20)
    for n in ref:
        assert bool(torch.equal(ref[n], got[n])), n


def test_growth(dev):
    """Growth at 40 nodes, 48 points at most: the operands of the product shrink first."""
    from paper_2505_22718_amd.plan import Plan, device_inputs
    wl = _workload(15, 1)
    synth.scale_dependent_growth(wl, 40, f_nu=0.3)
    D = torch.as_tensor(wl["D_kz"], dtype=torch.float64, device=dev).expand(48, -1, -1).contiguous()
    wl = _workload(15, 48)
    t = device_inputs(wl, dev)
    ref, got = _roomy_and_tight(lambda: Plan.for_workload(wl, precision="fp32", n_interp=40),
                                lambda p: p.cl_kgrowth(t, D).cpu().numpy().astype(np.float64), 256 << 20)
    for b in (0, 20, 47):  # two sums of at most about 1024 FP32 roundings per window
        e = eps_metric(full_from_packed(got[b], 15), full_from_packed(ref[b], 15)).max()
        print(f"  point {b}: {e:.2e}", flush=True)
        assert e < 1e-5


def test_rows_adjoint_takes_no_workspace(dev):
    """RSD at 15 tracers and n_chi = 1024 keeps its rows in LDS: no V rows (0.5 GB) in memory."""
    from paper_2505_22718_amd.plan import Plan
    wl = _workload(15, 40)
    before = _free()
    p = Plan.for_workload(wl, precision="fp32", rsd=True)
    size = before - _free()
    print(f"  {size / 2**20:.0f} MiB", flush=True)
    p.close()
    assert size < 40 * 103 * 32 * 1024 * 4


def test_a_refused_plan_leaves_no_error_behind(dev):
    """A plan that no device holds (3 million points) is refused with E_NOMEM, its memory is given back, and the
    program's next GPU calls do not meet the failed allocation."""
    from paper_2505_22718_amd import binding as bd
    from paper_2505_22718_amd.plan import Plan
    wl = _workload(15, 1)
    before = _free()
    with pytest.raises(bd.SwiftclError) as err:
        Plan.for_workload(wl, precision="fp32", max_batch=3000000)
    assert err.value.status == bd.SWIFTCL_E_NOMEM
    assert float(torch.ones(8, device=dev).expand(4, 8).contiguous().sum()) == 32.0
    assert _free() >= before - (64 << 20)
