"""GPU solves at the edges of the device's function-approximation weights
(one, two and four rows of T per lane, and the host routine beyond; exponents
from nearly zero to large) against the oracle's eigenvector form."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")
rdm = pytest.importorskip("paper_2204_08147_amd")

from oracle import lanczos as olz  # noqa: E402
from workloads import random_dense_terms  # noqa: E402

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("k", [1, 2, 63, 64, 65, 128, 129, 256, 257])
def test_weights_match_oracle(k):
    inst = random_dense_terms(1, 8, 900 + k, k=k, betas=(1e-9, 1e-3, 0.7, 30.0), n_v=2)
    got = rdm.solve(rdm.Hamiltonian.from_instance(inst), inst.betas, inst.n_v, inst.k, inst.seed, precision="fp64")
    want = olz.solve(inst)["results"]
    for b, w in enumerate(want):
        # the FP64 parity bar; H* = -ln(..)/beta + .. loses 1 / beta of it
        assert np.linalg.norm(got["rho"][b] - w["rho"]) < 1e-10 * np.linalg.norm(w["rho"])
        tol = 1e-10 * max(1.0, 1e-5 / inst.betas[b])
        assert np.linalg.norm(got["h_star"][b] - w["h_star"]) < 10 * tol * max(1.0, np.linalg.norm(w["h_star"]))
        assert abs(got["log_z"][b] - w["log_z"]) < 1e-10 * max(1.0, abs(w["log_z"]))
        assert abs(got["entropy"][b] - w["entropy"]) < 1e-10


def test_many_temperatures_in_one_solve():
    # more than one launch's worth of temperatures, each as if solved alone
    inst = random_dense_terms(2, 7, 950, k=30, betas=tuple(0.05 * (b + 1) for b in range(37)), n_v=3)
    h = rdm.Hamiltonian.from_instance(inst)
    got = rdm.solve(h, inst.betas, inst.n_v, inst.k, inst.seed, precision="mixed")
    for b in (0, 15, 16, 31, 32, 36):
        one = rdm.solve(h, inst.betas[b:b + 1], inst.n_v, inst.k, inst.seed, precision="mixed")
        assert np.linalg.norm(got["rho"][b] - one["rho"][0]) < 1e-5 * np.linalg.norm(one["rho"][0])
        assert abs(got["log_z"][b] - one["log_z"][0]) < 1e-5


@pytest.mark.parametrize("k,n_beta", [(1, 4), (64, 4), (65, 4), (128, 18), (256, 4), (257, 4)])
def test_product_quadratures_match_oracle(k, n_beta):
    # both Hamiltonians' quadratures on the device (one, two and four rows per
    # lane, two launches' temperatures; the host beyond), temperatures from 0
    from oracle import product
    inst = random_dense_terms(2, 6, 960 + k)
    betas = [0.0, 1e-30, 1e-9] + [0.4 * (i + 1) for i in range(n_beta - 3)]
    want = product.lanczos_estimate(inst, betas, 3, k, 17)
    got = rdm.product_trace(rdm.Hamiltonian.from_instance(inst), betas, 3, k, 17, precision="fp64")
    want["samples"] = want["log_z_t_samples"]
    for key in ("samples", "log_z", "log_z_t", "log_z_b"):
        assert np.allclose(got[key], want[key], rtol=1e-10, atol=1e-10), key


@pytest.mark.parametrize("n_b,apply", [(7, "hops"), (12, "hops"), (15, "transform")])
@pytest.mark.parametrize("mode", ["stored", "two_pass"])
def test_no_result_depends_on_the_workspace_content(n_b, apply, mode):
    # a workspace of NaNs (all bits set) against one of zeros
    inst = random_dense_terms(1, n_b, 970 + n_b, k=24, betas=(0.5, 2.0), n_v=3)
    h = rdm.Hamiltonian.from_instance(inst, apply=apply)
    for precision in ("mixed", "fp64"):
        opts = dict(precision=precision, mode=mode)
        ws = torch.empty(rdm.workspace_size(h, len(inst.betas), inst.n_v, inst.k, **opts), dtype=torch.uint8,
                         device="cuda")
        got = []
        for fill in (0, 255):
            ws.fill_(fill)
            torch.cuda.synchronize()
            got.append(rdm.solve(h, inst.betas, inst.n_v, inst.k, inst.seed, workspace=ws, **opts))
        for key in ("rho", "h_star", "log_z", "entropy"):
            assert np.array_equal(got[0][key], got[1][key]), (precision, key)
