"""Template bank at the edges of its generation: few and many width groups, group widths far above
the templates', windows without margin, ragged member counts, every segment length.

Taps are compared with the oracle's quadrature (both FP64, 1e-12 absolute; a sample of each
template's window), the spectra derived from them through a small plane, which must be the FP64
correlation with the bank's own taps (FP32 path: 1e-4 of the power or of its row's mean).
"""

import numpy as np
import pytest

import paper_1911_01353_amd as J
from oracle import Grid
from oracle.response import template_response

from gpu_helpers import bank_taps, build_bank, device, gpu_plane

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("zmax,wmax,dz,dw,margin,quantum,seg", [
    (1600.0, 0.0, 200.0, 20.0, 16, 0, 4096),  # wide templates, one or two to a group
    (700.0, 0.0, 20.0, 20.0, 16, 0, 2048),    # 36 width groups: more than one launch holds
    (7.0, 45.0, 2.0, 15.0, 0, 0, 512),        # no margin: windows of 2 to 16 taps
    (4.0, 0.0, 2.0, 20.0, 16, 512, 1024),     # groups of 512 taps around 36-tap windows
    (16.0, 0.0, 2.0, 20.0, 3, 0, 1024),       # 17 templates
])
def test_taps_and_spectra(zmax, wmax, dz, dw, margin, quantum, seg):
    device()
    n = 300
    plan = J.Plan(n, zmax, wmax, dz, dw, path="fft", margin=margin, seg_len=seg, tap_quantum=quantum)
    grid = Grid(zmax, wmax, dz, dw, margin)
    bank = build_bank(plan)
    members = plan.members()
    rng = np.random.default_rng(int(zmax))
    spec = ((rng.standard_normal(n) + 1j * rng.standard_normal(n)) / np.sqrt(2)).astype(np.complex64)
    plane = gpu_plane(plan, bank, spec)
    groups = plan.groups()
    for gi, g in enumerate(groups):
        taps = bank_taps(plan, bank, gi)
        hg = g["taps"] // 2
        x = np.concatenate([np.zeros(hg - 1), spec.astype(np.complex128), np.zeros(hg)])
        for k in range(g["n_members"]):
            t = int(members[g["first_member"] + k])
            zb, w, h = grid.params(t)
            inside = np.arange(hg - h, hg + h)
            outside = np.delete(np.arange(g["taps"]), inside)
            assert not taps[k][:, outside].any()
            if k in (0, g["n_members"] - 1) and gi in (0, 1, len(groups) // 2, len(groups) - 1):
                j = inside[np.unique(np.linspace(0, 2 * h - 1, 9).astype(int))]
                for phase in (0, 1):
                    want = np.conj(template_response(hg - 1 - j + phase / 2.0, zb, w))
                    assert np.max(np.abs(taps[k, phase, j] - want)) < 1e-12, (t, phase)
            want = np.empty(2 * n)
            for phase in (0, 1):
                want[phase::2] = np.abs(np.correlate(x, np.conj(taps[k, phase]))) ** 2
            err = np.abs(plane[t] - want) / np.maximum(want, want.mean())
            assert err.max() <= 1e-4, (t, err.max())
    plan.close()
