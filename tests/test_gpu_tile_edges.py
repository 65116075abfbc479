"""Sizes at which the tiled kernels change shape, against the FP64 oracle: 16-row blocks
and 32-layer chunks of the FP64 kernels, the quads and waves of the k-distribution
mixing, the likelihood's bin-sum paths and lane groups, and more samples than one pass
of the layer-count classes holds.

FP64 tolerance 1e-8 (per component as in the gradient tests): rounding of 1e-16, times
about 1e2 for the cancellation in r - b of the chord, 1e3 for residuals at the noise
level and 1e3 for components down to 1e-3 of the largest.  lnL in FP64 1e-10 (one
residual factor).  Correlated-k spectra 2e-5: FP32 mixing whose sort keys drop six bits
(4e-6 per merge at worst) and the bf16 hi/lo chord.  Reduced precision 1e-3 against FP64.
"""
import numpy as np
import pytest

import oracle
from parity_util import reduced, reduced_ck, rel_err

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


def _model(wl, precision, batch):
    from paper_2602_19687_amd import ForwardModel
    return ForwardModel(wl, precision=precision, batch_max=batch)


def _grad_err(g, ref):
    return np.max(np.abs(g - ref) / np.maximum(np.abs(ref), 1e-3 * np.max(np.abs(ref))))


@pytest.mark.parametrize("cid,lmax,layers", [
    (3, 128, [2, 15, 16, 17, 48, 112, 113, 128]),
    (3, 160, [3, 127, 129, 144, 145, 160]),
    (2, 160, [2, 31, 32, 33, 64, 65, 128, 160]),
], ids=["trans-128", "trans-160", "emis-160"])
def test_fp64_gradient_at_layer_edges(cid, lmax, layers):
    wl = reduced(cid, n_nu=130, n_bins=7, batch=len(layers), n_layers=lmax, step=97)
    print(f"[gpu] FP64 gradient cid={cid} layers={layers}", flush=True)
    fm = _model(wl, "fp64", len(layers))
    th = torch.tensor(wl["params"], dtype=torch.float64, device="cuda")
    lnl, g, st, _ = fm.grad(th, n_layers=np.array(layers, np.int32))
    lnl, g, st = lnl.cpu().numpy(), g.cpu().numpy(), st.cpu().numpy()
    fm.close()
    assert np.all(st == 0)
    for b, n in enumerate(layers):
        ref = oracle.forward(wl, wl["params"][b], n_layers=n)
        assert abs(lnl[b] - ref["lnL"]) <= 1e-10 * abs(ref["lnL"]), n
        err = _grad_err(g[b], oracle.grad_complex_step(wl, wl["params"][b], n_layers=n))
        print(f"layers {n}: lnL {lnl[b]:.6e} gradient err {err:.2e}")
        assert err < 1e-8, n


@pytest.mark.parametrize("cid,mix", [(8, 0), (7, 0), (7, 1)], ids=["emis-rorr", "trans-rorr", "trans-product"])
@pytest.mark.parametrize("n_ck,species", [(1, 6), (15, 1), (16, 2), (17, 6), (63, 3), (65, 6)])
def test_ck_at_bin_edges(cid, mix, n_ck, species):
    wl = reduced_ck(cid, n_ck=n_ck, n_bins=1, batch=3, step=29)
    n_tp = 3 if cid == 7 else 5
    drop = range(n_tp + species, n_tp + wl["n_species"])
    wl["params"] = np.delete(wl["params"], drop, axis=1)
    wl.update(ck_mix=mix, n_species=species, log10_xsec=np.ascontiguousarray(wl["log10_xsec"][:species]),
              species_mass=wl["species_mass"][:species])
    print(f"[gpu] ck cid={cid} mix={mix} bins={n_ck} species={species}", flush=True)
    fm = _model(wl, "mixed", 3)
    spec, _, st = fm.forward(torch.tensor(wl["params"], device="cuda"))
    spec = spec.double().cpu().numpy()
    fm.close()
    assert torch.all(st == 0)
    for b in range(3):
        ref = oracle.forward(wl, wl["params"][b])
        assert rel_err(spec[b], ref["spectrum"]) < 2e-5


@pytest.mark.parametrize("n_nu,n_bins", [(4095, 30), (4096, 500), (4097, 200), (4100, 100), (4223, 33), (300, 1)])
def test_likelihood_sums(n_nu, n_bins):
    """Both bin-sum paths (one kernel below 4096 wavenumbers) and every lane-group width."""
    wl = reduced(3, n_nu=n_nu, n_bins=n_bins, batch=2, n_layers=20)
    print(f"[gpu] likelihood n_nu={n_nu} bins={n_bins}", flush=True)
    fm = _model(wl, "fp64", 2)
    _, lnl, _ = fm.forward(torch.tensor(wl["params"], dtype=torch.float64, device="cuda"), want_spectra=False)
    lnl = lnl.cpu().numpy()
    fm.close()
    for b in range(2):
        ref = oracle.forward(wl, wl["params"][b])["lnL"]
        assert abs(lnl[b] - ref) <= 1e-10 * abs(ref)


def test_layer_classes_of_many_samples():
    """More samples than the class kernel ranks in one pass (256), with equal counts among them."""
    batch = 300
    wl = reduced(3, n_nu=200, n_bins=10, batch=batch, n_layers=150)
    layers = np.random.default_rng(5).integers(100, 151, batch).astype(np.int32)
    th = torch.tensor(wl["params"], dtype=torch.float64, device="cuda")
    print(f"[gpu] layer classes B={batch}", flush=True)
    spec = {}
    for precision in ("mixed", "fp64"):
        fm = _model(wl, precision, batch)
        s, _, st = fm.forward(th, n_layers=layers)
        assert torch.all(st == 0)
        spec[precision] = s.double().cpu().numpy()
        fm.close()
    assert rel_err(spec["mixed"], spec["fp64"]) < 1e-3
