"""FP64 path at the ends of its range, against the FP64 oracle.

Tolerances: spectra and lnL 1e-10, gradients 1e-8 per component (of at least 1e-3 of the
largest): rounding of 1e-16 times about 1e2 for the cancellation in r - b of the chord,
1e3 for residuals at the noise level and 1e3 for the smaller components.
"""
import numpy as np
import pytest

import oracle
import oracle.model
from parity_util import reduced, rel_err

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


def _grad_err(g, ref):
    return np.max(np.abs(g - ref) / np.maximum(np.abs(ref), 1e-3 * np.max(np.abs(ref))))


def _model(wl, batch):
    from paper_2602_19687_amd import ForwardModel
    return ForwardModel(wl, precision="fp64", batch_max=batch)


@pytest.mark.parametrize("what", ["mixing-ratio", "table-floor"])
@pytest.mark.parametrize("cid,n_tp", [(3, 3), (2, 5)], ids=["trans", "emis"])
def test_absorber_without_absorption(cid, n_tp, what):
    """An absorber whose exponent is -inf adds nothing: a mixing ratio that underflows to
    zero (log10 X = -400), or cross sections at the lowest double."""
    wl = reduced(cid, n_nu=130, n_bins=7, batch=2, n_layers=40, step=97)
    if what == "mixing-ratio":
        wl["params"][0, n_tp + 1] = -400.0
    else:
        wl["log10_xsec"][1, ..., ::2] = np.finfo(np.float64).min
    print(f"[gpu] FP64 absorber without absorption cid={cid} {what}", flush=True)
    fm = _model(wl, 2)
    th = torch.tensor(wl["params"], dtype=torch.float64, device="cuda")
    spec, lnl, st = (x.cpu().numpy() for x in fm.forward(th))
    _, g, gst, _ = fm.grad(th)
    g, gst = g.cpu().numpy(), gst.cpu().numpy()
    fm.close()
    assert np.all(st == 0) and np.all(gst == 0)
    for b in range(2):
        with np.errstate(over="ignore", invalid="ignore"):
            ref = oracle.forward(wl, wl["params"][b])
            gref = oracle.grad_complex_step(wl, wl["params"][b])
        assert rel_err(spec[b], ref["spectrum"]) < 1e-10
        assert abs(lnl[b] - ref["lnL"]) <= 1e-10 * abs(ref["lnL"])
        # (the derivative by an underflowed X itself is 0 / 0)
        keep = wl["params"][b] > -400.0
        assert _grad_err(g[b][keep], gref[keep]) < 1e-8


@pytest.mark.parametrize("cid,n_tp", [(3, 3), (2, 5)], ids=["trans", "emis"])
def test_mixing_ratio_that_underflows_in_reduced_precision(cid, n_tp):
    """The reduced-precision record of a zero prefactor (a logarithm of -inf) adds nothing
    either: spectra to the 1e-3 of that path."""
    from paper_2602_19687_amd import ForwardModel
    wl = reduced(cid, n_nu=130, n_bins=7, batch=1, n_layers=40, step=97)
    wl["params"][0, n_tp + 1] = -400.0
    print(f"[gpu] reduced precision, underflowing mixing ratio cid={cid}", flush=True)
    fm = ForwardModel(wl, precision="mixed", batch_max=1)
    spec, lnl, st = fm.forward(torch.tensor(wl["params"], dtype=torch.float64, device="cuda"))
    spec = spec.double().cpu().numpy()
    fm.close()
    ref = oracle.forward(wl, wl["params"][0])
    assert int(st[0]) == 0 and rel_err(spec[0], ref["spectrum"]) < 1e-3
    assert abs(float(lnl[0]) - ref["lnL"]) <= 1e-3 * abs(ref["lnL"])


def test_gradient_of_a_thin_atmosphere(monkeypatch):
    """Slant optical depths near 1e-18, where 1 - e^-tau formed by subtraction is zero: the
    temperature moves such a spectrum through the annulus areas and the optical depths in
    equal parts.  p_ref is the bottom pressure, so the opaque core does not move."""
    def transit_depth(pm, dtau, r_lev, r_s):
        return (r_lev[0] ** 2 - (r_lev[1:] ** 2 - r_lev[:-1] ** 2) @ np.expm1(-(pm @ dtau))) / r_s ** 2

    monkeypatch.setattr(oracle.model, "transit_depth", transit_depth)
    wl = reduced(0, n_nu=200, n_bins=10, batch=1, n_layers=40, step=9)
    wl.update(p_ref_bar=wl["p_bot"], rayleigh=False, ray_h2=0.0, ray_he=0.0)
    wl["params"][0] = [1200.0, -27.0]
    print("[gpu] FP64 gradient of a thin atmosphere", flush=True)
    fm = _model(wl, 1)
    _, g, st, _ = fm.grad(torch.tensor(wl["params"], dtype=torch.float64, device="cuda"))
    g = g.cpu().numpy()[0]
    fm.close()
    assert int(st[0]) == 0
    # both components to the same relative accuracy, whatever their sizes
    assert rel_err(g, oracle.grad_complex_step(wl, wl["params"][0])) < 1e-8


def test_planck_intensity_of_a_cold_object():
    """An isothermal object's spectrum is B(T) / B(T_*).  With T and the wavenumbers powers of
    two, h c nu / k T is one rounded constant times a power of two, for the oracle too, so the
    intensities agree to their own roundings up to e^-368: 4e-15, some twenty roundings of
    1.1e-16 on either side.  An exponent rounded once more on the way is off by 2e-14."""
    wl = reduced(2, n_nu=4, n_bins=1, batch=1, n_layers=40)
    wl["nu"] = np.array([1024.0, 2048.0, 4096.0, 8192.0])
    wl.update(tp=0, n_knots=0, t_star=4096.0, params=np.concatenate([[[32.0]], wl["params"][:, 5:]], axis=1))
    print("[gpu] FP64 Planck intensity of a cold object", flush=True)
    fm = _model(wl, 1)
    spec, _, st = fm.forward(torch.tensor(wl["params"], dtype=torch.float64, device="cuda"))
    spec = spec.cpu().numpy()[0]
    fm.close()
    assert int(st[0]) == 0
    assert rel_err(spec, oracle.forward(wl, wl["params"][0])["spectrum"]) < 4e-15


def test_gradient_without_rayleigh():
    """Rayleigh scattering switched off with its coefficients left set: no term of it reaches
    the gradient through the H2 and He mixing ratios."""
    wl = reduced(0, n_nu=200, n_bins=10, batch=1, n_layers=40, step=9)
    wl["rayleigh"] = False
    wl["params"][0] = [1200.0, -8.0]
    print("[gpu] FP64 gradient without Rayleigh", flush=True)
    fm = _model(wl, 1)
    _, g, st, _ = fm.grad(torch.tensor(wl["params"], dtype=torch.float64, device="cuda"))
    g = g.cpu().numpy()[0]
    fm.close()
    assert int(st[0]) == 0
    assert rel_err(g, oracle.grad_complex_step(wl, wl["params"][0])) < 1e-8
