"""GPU tests of the MFMA path across the width groups whose plane launches use the four-wave
kernel (48, 64 and 80 taps) and their neighbours (32 and 96 taps, one-wave kernels): whole
planes against the FP64 oracle, and the one-wave peak-key kernel against the planes."""

import numpy as np
import pytest

import paper_1911_01353_amd as J
from oracle import Grid, error_summary, oracle_plane, peak_index

from gpu_helpers import build_bank, device, gpu_plane

pytestmark = pytest.mark.gpu

ZMAX, WMAX = 40.0, 120.0  # 41 x 13 = 533 templates, groups of 32 ... 96 taps


def _spec(n, seed):
    rng = np.random.default_rng(seed)
    x = ((rng.standard_normal(n) + 1j * rng.standard_normal(n)) / np.sqrt(2)).astype(np.complex64)
    x[n // 3] += 8.0
    return x


@pytest.fixture(scope="module")
def ragged_case():
    n = 9001
    spec = _spec(n, 61)
    return spec, oracle_plane(spec, Grid(ZMAX, WMAX, 2.0, 20.0))


@pytest.mark.parametrize("path,tol", [("split_bf16", 1e-4), ("fp16", 1e-2)])
def test_all_groups_against_oracle(ragged_case, path, tol):
    """Every row of a 533-template plane over a ragged 9001-bin spectrum (several windows per
    workgroup, a partial last window, member ranges not filling the last block of 8)."""
    device()
    spec, ora = ragged_case
    n = spec.shape[0]
    plan = J.Plan(n, ZMAX, WMAX, 2.0, 20.0, path=path)
    taps = sorted({g["taps"] for g in plan.groups()})
    assert {48, 64, 80}.issubset(taps) and max(taps) >= 96
    got = gpu_plane(plan, build_bank(plan), spec)
    assert not np.isnan(got).any()
    s = error_summary(got, ora)
    print(f"[mfma groups] {path}: max {s['max']:.2e}, rms {s['rms']:.2e}", flush=True)
    assert s["max"] <= tol
    assert peak_index(got) == peak_index(ora)
    plan.close()


def test_peak_keys_equal_plane_row_maxima():
    """search_peaks (one-wave kernels with peak keys) equals the row argmax of the plane written
    by the four-wave kernels, bit for bit, on the 48-96-tap groups of a 2^18-bin spectrum."""
    import torch
    dev = device()
    n = 1 << 18
    spec_np = _spec(n, 62)
    plan = J.Plan(n, ZMAX, WMAX, 2.0, 20.0, path="split_bf16")
    bank = build_bank(plan)
    plane = gpu_plane(plan, bank, spec_np)
    spec = torch.from_numpy(spec_np).to(dev)
    pk = J.peaks_numpy(plan.search_peaks(bank, spec))
    idx = np.argmax(plane, axis=1)
    assert np.array_equal(pk["power"].view(np.uint32), plane[np.arange(plane.shape[0]), idx].view(np.uint32))
    assert np.array_equal(pk["p"].astype(np.int64), idx)
    plan.close()


@pytest.mark.parametrize("path,tol", [("fp16", 1e-2), ("split_bf16", 1e-4)])
@pytest.mark.parametrize("taps", list(range(16, 273, 16)))
def test_every_tap_count(taps, path, tol):
    """One kernel per tap count (the first tap count above them included): plane rows against the FP64
    correlation with the bank's taps, over several windows and a ragged end; row peaks against the
    plane's."""
    import torch
    from gpu_helpers import bank_taps
    dev = device()
    n = 701
    plan = J.Plan(n, 15.0, 0.0, 2.0, 20.0, path=path, margin=taps // 2 - 8, tap_quantum=taps)
    assert [g["taps"] for g in plan.groups()] == [taps]
    bank = build_bank(plan)
    rng = np.random.default_rng(taps)
    spec = ((rng.standard_normal(n) + 1j * rng.standard_normal(n)) / np.sqrt(2)).astype(np.complex64)
    plane = gpu_plane(plan, bank, spec)
    x = np.concatenate([np.zeros(taps // 2 - 1), spec.astype(np.complex128), np.zeros(taps // 2)])
    coef = bank_taps(plan, bank, 0)
    for k, t in enumerate(plan.members()):
        want = np.empty(2 * n)
        for phase in (0, 1):
            want[phase::2] = np.abs(np.correlate(x, np.conj(coef[k, phase]))) ** 2
        err = np.abs(plane[t] - want) / np.maximum(want, want.mean())
        assert err.max() <= tol, (t, err.max())
    got = J.peaks_numpy(plan.search_peaks(bank, torch.from_numpy(spec).to(dev)), plane.shape[0])
    torch.cuda.synchronize()
    assert np.array_equal(got["p"].astype(np.int64), plane.argmax(axis=1))
    assert np.array_equal(got["power"], plane.max(axis=1))
    plan.close()


@pytest.mark.parametrize("n", [701, 5000])
def test_wide_fp16_groups_share_launches(n):
    """FP16 groups of 32 to 240 taps (one launch of eight groups, one of six): the kernels a search
    queues, its plane against each group's own kernel (the same bits) and the FP64 correlation with
    the bank's taps, its row peaks against the plane's."""
    import torch
    from gpu_helpers import bank_taps, captured_kernels
    dev = device()
    plan = J.Plan(n, 200.0, 0.0, 2.0, 20.0, path="fp16")
    assert [g["taps"] for g in plan.groups()] == list(range(32, 241, 16))
    T = plan.info()["n_templates"]
    bank = build_bank(plan)
    spec_np = _spec(n, 63)
    spec = torch.from_numpy(spec_np).to(dev)
    plane = gpu_plane(plan, bank, spec_np)
    out = torch.full((T, 2 * n), float("nan"), dtype=torch.float32, device=dev)
    assert captured_kernels(lambda: plan.search(bank, spec, out)) == 2
    for gi in range(len(plan.groups())):
        plan.search_group(bank, spec, out, gi)
    torch.cuda.synchronize()
    assert np.array_equal(out.cpu().numpy().view(np.uint32), plane.view(np.uint32))
    members = plan.members()
    for gi, g in enumerate(plan.groups()):
        coef = bank_taps(plan, bank, gi)
        x = np.concatenate([np.zeros(g["taps"] // 2 - 1), spec_np.astype(np.complex128), np.zeros(g["taps"] // 2)])
        for k in range(g["n_members"]):
            t = members[g["first_member"] + k]
            want = np.empty(2 * n)
            for phase in (0, 1):
                want[phase::2] = np.abs(np.correlate(x, np.conj(coef[k, phase]))) ** 2
            err = np.abs(plane[t] - want) / np.maximum(want, want.mean())
            assert err.max() <= 1e-2, (t, err.max())
    got = J.peaks_numpy(plan.search_peaks(bank, spec), T)
    torch.cuda.synchronize()
    assert np.array_equal(got["p"].astype(np.int64), plane.argmax(axis=1))
    assert np.array_equal(got["power"], plane.max(axis=1))
    plan.close()


@pytest.fixture(scope="module")
def long_spectrum():
    return _spec((1 << 21) + 77, 64)


@pytest.mark.parametrize("taps", list(range(16, 257, 16)))
def test_fp16_several_windows_per_wave(long_spectrum, taps):
    """Every FP16 tap count on a spectrum long enough that a wave takes several windows (16 templates,
    at least 4 windows each): points at the ends of windows, at both ends of the spectrum and at random
    against the FP64 correlation with the bank's taps, row peaks against the plane's."""
    import torch
    from gpu_helpers import bank_taps
    dev = device()
    n = long_spectrum.shape[0]
    plan = J.Plan(n, 15.0, 0.0, 2.0, 20.0, path="fp16", margin=taps // 2 - 8, tap_quantum=taps)
    assert [(g["taps"], g["n_members"]) for g in plan.groups()] == [(taps, 16)]
    bank = build_bank(plan)
    spec = torch.from_numpy(long_spectrum).to(dev)
    plane = torch.full((16, 2 * n), float("nan"), dtype=torch.float32, device=dev)
    plan.search(bank, spec, plane)
    torch.cuda.synchronize()
    assert not torch.isnan(plane).any()
    rng = np.random.default_rng(taps)
    edges = np.concatenate([[w * 64 - 1, w * 64] for w in (*range(1, 40), *rng.integers(40, n // 64, 60))])
    at = np.unique(np.concatenate([[0, 1, n - 2, n - 1], edges, rng.integers(0, n, 100)]))
    hg = taps // 2
    x = np.concatenate([np.zeros(hg - 1), long_spectrum.astype(np.complex128), np.zeros(hg)])
    window = x[at[:, None] + np.arange(taps)[None, :]]  # (points, taps): tap j takes bin k0 - hg + 1 + j
    coef = bank_taps(plan, bank, 0)
    got = plane.cpu().numpy()
    for k, t in enumerate(plan.members()):
        for phase in (0, 1):
            want = np.abs(window @ coef[k, phase]) ** 2
            err = np.abs(got[t, 2 * at + phase] - want) / np.maximum(want, got[t].mean(dtype=np.float64))
            assert err.max() <= 1e-2, (t, phase, err.max())
    peaks = J.peaks_numpy(plan.search_peaks(bank, spec), 16)
    torch.cuda.synchronize()
    assert np.array_equal(peaks["p"].astype(np.int64), got.argmax(axis=1))
    assert np.array_equal(peaks["power"], got.max(axis=1))
    plan.close()
