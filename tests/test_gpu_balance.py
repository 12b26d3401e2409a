"""Launches that share their templates out anew (plans with the default templates per block, more
workgroups than the device holds at once): the same bits as with blocks the caller fixed."""

import numpy as np
import pytest

import paper_1911_01353_amd as J

from gpu_helpers import build_bank, device, gpu_plane

pytestmark = pytest.mark.gpu


def _spec(n, seed):
    rng = np.random.default_rng(seed)
    x = ((rng.standard_normal(n) + 1j * rng.standard_normal(n)) / np.sqrt(2)).astype(np.complex64)
    x[n // 3] += 12.0
    return x


def _candidates(plan, bank, spec, k):
    import torch
    T = plan.info()["n_templates"]
    out = torch.zeros((1 << 20, 4), dtype=torch.int32, device="cuda")
    count = torch.zeros(1, dtype=torch.int64, device="cuda")
    stats = torch.zeros((T, 2), dtype=torch.float64, device="cuda")
    plan.search_candidates(bank, spec, k, None, out, count, stats=stats)
    torch.cuda.synchronize()
    assert int(count.item()) <= out.shape[0]
    return np.sort(J.candidates_numpy(out, count), order=["t", "p"]), stats.cpu().numpy()


@pytest.mark.parametrize("n,zmax,wmax", [((1 << 19) + 77, 200.0, 0.0), (1 << 18, 50.0, 150.0), (300001, 60.0, 60.0)])
def test_same_bits_as_fixed_blocks(n, zmax, wmax):
    import torch
    dev = device()
    spec_np = _spec(n, int(zmax))
    spec = torch.from_numpy(spec_np).to(dev)
    ref = None
    for tpb in (16, 0, 64):
        plan = J.Plan(n, zmax, wmax, path="fft", templates_per_block=tpb)
        bank = build_bank(plan)
        T = plan.info()["n_templates"]
        t0, t1 = T // 2 - 40, T // 2 + 41
        peaks = J.peaks_numpy(plan.search_peaks(bank, spec), T)
        found, stats = _candidates(plan, bank, spec, 9.0)
        planes = [torch.full((t1 - t0, 2 * m), float("nan"), dtype=torch.float32, device=dev) for m in (n, n // 2 + 1)]
        ws = torch.empty(plan.batch_workspace_bytes(2), dtype=torch.uint8, device=dev)
        plan.batch_search(bank, [(spec, planes[0], None), (spec[:n // 2 + 1], planes[1], None)], ws, t0, t1)
        torch.cuda.synchronize()
        slab = gpu_plane(plan, bank, spec_np, t0, t1)
        got = (peaks, found, stats, slab, planes[0].cpu().numpy(), planes[1].cpu().numpy())
        assert np.array_equal(got[3], got[4])
        assert len(found) > 0
        if ref is None:
            ref = got
        else:
            for a, b in zip(got, ref):
                assert a.tobytes() == b.tobytes(), tpb
        plan.close()
