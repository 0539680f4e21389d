"""Function-approximation weights of columns whose spectra lie far above the
common shift E0, against the oracle's eigenvector form: system spins that keep
their z-components (every column stays in its own sector), and quadratures of
single product columns at low temperature."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")
rdm = pytest.importorskip("paper_2204_08147_amd")

from oracle import lanczos as olz, product  # noqa: E402
from workloads import long_range_xx_zz, random_dense_terms  # noqa: E402

pytestmark = pytest.mark.gpu


def conserved(n_s, n_b, seed, beta, gap):
    """System spins coupled by J^z only, in z-fields: rho* is diagonal, its
    extreme eigenvalues about exp(-gap) apart."""
    inst = random_dense_terms(n_s, n_b, seed, k=30, betas=(beta,), n_v=3)
    inst.couplings = [(i, j, 0.0, 0.0, 0.1 * jz) if i < n_s else (i, j, jx, jy, jz)
                      for i, j, jx, jy, jz in inst.couplings]
    inst.hx[:n_s] = 0.0
    inst.hz[:n_s] = gap / (2.0 * n_s * beta) * (1.0 + 0.1 * np.arange(n_s))
    return inst


@pytest.mark.parametrize("n_s,n_b", [(1, 8), (2, 11)])
@pytest.mark.parametrize("gap", [10.0, 25.0, 30.0])
@pytest.mark.parametrize("mode", ["stored", "two_pass"])
def test_columns_of_a_high_sector(n_s, n_b, gap, mode):
    inst = conserved(n_s, n_b, 700 + n_b, 4.0, gap)
    want = olz.solve(inst)["results"][0]
    h_want = np.diag(want["h_star"])
    spread = inst.betas[0] * (h_want.max() - h_want.min())
    assert gap - 5.0 < spread < 36.0          # above the eigenvalues' floor of 2^-52
    got = rdm.solve(rdm.Hamiltonian.from_instance(inst), inst.betas, inst.n_v, inst.k, inst.seed, precision="fp64",
                    mode=mode)
    # the FP64 bar, held by every eigenvalue of rho* relative to itself
    # (beta dH* = d ln mu)
    assert np.abs(np.diag(got["h_star"][0]) - h_want).max() * inst.betas[0] < 1e-10
    assert np.abs(np.diag(got["rho"][0]) / np.diag(want["rho"]) - 1.0).max() < 1e-10


@pytest.mark.parametrize("n_s,n_b", [(1, 8), (2, 12)])
def test_product_samples_at_low_temperature(n_s, n_b):
    # few steps leave the columns' lowest Ritz values apart: at beta = 500 by
    # hundreds in the exponent
    inst = long_range_xx_zz(n_s, n_b, 0.5, 711, k=20, n_v=8)
    betas = [50.0, 100.0, 200.0, 500.0]
    want = product.lanczos_estimate(inst, betas, 8, 20, inst.seed)
    want["samples"] = want["log_z_t_samples"]
    got = rdm.product_trace(rdm.Hamiltonian.from_instance(inst), betas, 8, 20, inst.seed, precision="fp64")
    # beta times a Ritz value's rounding: 500 x 20 x 1e-14 absolute, 1e-10
    # relative to the logarithms of 1e3..1e4
    for key in ("samples", "log_z", "log_z_t", "log_z_b"):
        assert np.allclose(got[key], want[key], rtol=1e-10, atol=1e-10), key
