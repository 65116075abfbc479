"""Bin sums of the likelihood where the layout of lanes changes, against the FP64 oracle: the
cloudy/clear mixing with the sums in a kernel of their own (from 4096 wavenumbers on), and
narrow lane groups (8, 16 and 32 lanes a bin) within the sample's workgroup, with bin counts
that leave some of a wave's groups without a bin.

FP64 tolerances: lnL 1e-10 (rounding of 1e-16 times 1e3 for residuals at the noise level, and
room), gradients 1e-8 per component of at least 1e-3 of the largest (a further 1e2 for the
cancellation in r - b of the chord and 1e3 for the smaller components).
"""
import numpy as np
import pytest

import oracle
from parity_util import reduced

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


def _model(wl, batch):
    from paper_2602_19687_amd import ForwardModel
    return ForwardModel(wl, precision="fp64", batch_max=batch)


@pytest.mark.parametrize("n_nu,n_bins", [(4099, 41), (4200, 500)])
def test_partly_cloudy_with_split_sums(n_nu, n_bins):
    wl = reduced(6, n_nu=n_nu, n_bins=n_bins, batch=3, n_layers=6)
    print(f"[gpu] partly cloudy n_nu={n_nu} bins={n_bins}", flush=True)
    fm = _model(wl, 3)
    th = torch.tensor(wl["params"], dtype=torch.float64, device="cuda")
    lnl, g, st, spec = fm.grad(th, want_spectra=True)
    lnl, g, spec = lnl.cpu().numpy(), g.cpu().numpy(), spec.cpu().numpy()
    fm.close()
    assert torch.all(st == 0)
    for b in range(3):
        ref = oracle.forward(wl, wl["params"][b])
        assert np.max(np.abs(spec[b] / ref["spectrum"] - 1.0)) < 1e-10
        assert abs(lnl[b] - ref["lnL"]) <= 1e-10 * abs(ref["lnL"])
        gref = oracle.grad_complex_step(wl, wl["params"][b])
        assert np.max(np.abs(g[b] - gref) / np.maximum(np.abs(gref), 1e-3 * np.max(np.abs(gref)))) < 1e-8


# mean bin width: 8 to 15 wavenumbers 8 lanes, 16 to 31 16 lanes, 32 to 63 32 lanes; 64 / lanes
# groups a wave, 512 / lanes a workgroup, four bins of each in flight
@pytest.mark.parametrize("fcld", [False, True], ids=["plain", "partly-cloudy"])
@pytest.mark.parametrize("n_nu,n_bins", [(9, 1), (2330, 259), (700, 33), (3600, 131), (1400, 35)])
def test_narrow_lane_groups(n_nu, n_bins, fcld):
    wl = reduced(6 if fcld else 3, n_nu=n_nu, n_bins=n_bins, batch=2, n_layers=6)
    print(f"[gpu] lane groups n_nu={n_nu} bins={n_bins} fcld={fcld}", flush=True)
    fm = _model(wl, 2)
    _, lnl, st = fm.forward(torch.tensor(wl["params"], dtype=torch.float64, device="cuda"), want_spectra=False)
    lnl = lnl.cpu().numpy()
    fm.close()
    assert torch.all(st == 0)
    for b in range(2):
        ref = oracle.forward(wl, wl["params"][b])["lnL"]
        assert abs(lnl[b] - ref) <= 1e-10 * abs(ref)
