"""The coefficient histories hold k alphas and k - 1 betas per column: results
of solves whose weights the host forms (more than 256 steps) do not depend on
what the workspace held before, and the beta that no step computes is zero."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")
rdm = pytest.importorskip("paper_2204_08147_amd")

from workloads import random_dense_terms  # noqa: E402

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n_b", [9, 12])
@pytest.mark.parametrize("mode", ["stored", "two_pass"])
@pytest.mark.parametrize("precision", ["mixed", "fp64"])
def test_host_weights_ignore_the_workspace_content(n_b, mode, precision):
    # a workspace of NaNs (all bits set) against one of zeros
    inst = random_dense_terms(1, n_b, 720 + n_b, k=257, betas=(0.5, 2.0), n_v=2)
    h = rdm.Hamiltonian.from_instance(inst)
    opts = dict(precision=precision, mode=mode)
    ws = torch.empty(rdm.workspace_size(h, len(inst.betas), inst.n_v, inst.k, **opts), dtype=torch.uint8,
                     device="cuda")
    got = []
    for fill in (0, 255):
        ws.fill_(fill)
        torch.cuda.synchronize()
        got.append(rdm.solve(h, inst.betas, inst.n_v, inst.k, inst.seed, workspace=ws, **opts))
    for key in ("rho", "h_star", "log_z", "entropy"):
        assert np.array_equal(got[0][key], got[1][key]), key


@pytest.mark.parametrize("n_b,k", [(2, 1), (2, 12), (7, 9), (12, 9)])
@pytest.mark.parametrize("which", [0, 1])
def test_last_beta_of_a_recurrence_is_zero(n_b, k, which):
    # (2, 12): more steps than the space has dimensions
    inst = random_dense_terms(1, n_b, 730 + n_b, n_v=3)
    h = rdm.Hamiltonian.from_instance(inst)
    dirty = torch.full((1 << 24,), 255, dtype=torch.uint8, device="cuda")
    torch.cuda.synchronize()
    del dirty
    torch.cuda.empty_cache()
    alpha, beta, kc = rdm.lanczos(h, which=which, n_v=3, k=k, seed=5, precision="fp64")
    steps = min(k, 1 << (n_b + 1 - which))
    assert alpha.shape == beta.shape == (k, 6 if which == 0 else 3)
    assert np.isfinite(alpha).all() and np.all(beta[steps - 1:] == 0.0)
    for c in range(beta.shape[1]):
        assert np.all(beta[:kc[c] - 1, c] > 0.0)
