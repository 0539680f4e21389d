"""GPU block Lanczos at the edges of its update launches (rows per lane, one
column group or two per panel, a ragged last panel) against the oracle."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")
rdm = pytest.importorskip("paper_2204_08147_amd")

from oracle import block as oblk  # noqa: E402
from workloads import long_range_xx_zz, random_dense_terms  # noqa: E402

pytestmark = pytest.mark.gpu

CASES = [
    lambda: random_dense_terms(1, 6, 971, k=8, betas=(0.5, 2.0), n_v=1),   # half a tile of rows
    lambda: random_dense_terms(1, 8, 972, k=8, betas=(0.5, 2.0), n_v=3),   # two groups a panel, one ragged
    lambda: random_dense_terms(2, 8, 973, k=8, betas=(0.5, 2.0), n_v=3),
    lambda: random_dense_terms(3, 8, 974, k=6, betas=(0.5, 2.0), n_v=2),
]


@pytest.mark.parametrize("case", range(len(CASES)))
@pytest.mark.parametrize("prec,tol", [("fp64", 1e-10), ("mixed", 1e-5)])
def test_block_solve_matches_oracle(case, prec, tol):
    inst = CASES[case]()
    got = rdm.solve(rdm.Hamiltonian.from_instance(inst), inst.betas, inst.n_v, inst.k, inst.seed, precision=prec,
                    method="block")
    for b, w in enumerate(oblk.solve(inst)["results"]):
        assert np.linalg.norm(got["rho"][b] - w["rho"]) < tol * np.linalg.norm(w["rho"])
        assert abs(got["log_z"][b] - w["log_z"]) < tol * max(1.0, abs(w["log_z"]))


@pytest.mark.parametrize("n_s,n_v", [(1, 9), (2, 16), (3, 5)])
def test_several_rows_per_lane_agree_with_the_per_column_path(n_s, n_v):
    # 2^19 rows: up to 16 rows per lane; the two estimators agree at
    # convergence (28 steps at beta = 0.2)
    inst = long_range_xx_zz(n_s, 19 - n_s, 0.5, 975, betas=(0.2,), n_v=n_v, k=28)
    h = rdm.Hamiltonian.from_instance(inst)
    a = rdm.solve(h, inst.betas, n_v, inst.k, inst.seed, precision="fp64")
    b = rdm.solve(h, inst.betas, n_v, inst.k, inst.seed, precision="fp64", method="block")
    assert np.linalg.norm(a["rho"] - b["rho"]) < 1e-9 * np.linalg.norm(a["rho"])
    assert abs(a["log_z"][0] - b["log_z"][0]) < 1e-9 * abs(a["log_z"][0])
