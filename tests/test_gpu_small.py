"""GPU parity of the single-launch Lanczos run of small instances (1 to 11
sites: one to eight rows per lane) with the oracle, and with the kernel-per-phase
steps that timed and larger solves take."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")
rdm = pytest.importorskip("paper_2204_08147_amd")

from oracle import lanczos as olz  # noqa: E402
from workloads import nn_xxz_chain, random_dense_terms, random_sparse_xxz  # noqa: E402

pytestmark = pytest.mark.gpu

CASES = [
    lambda: random_dense_terms(1, 1, 981, k=4, n_v=1),
    lambda: random_dense_terms(2, 5, 982, k=20, betas=(0.5, 3.0), n_v=3),
    lambda: random_dense_terms(1, 7, 983, k=20, betas=(0.5, 3.0), n_v=5),    # 256 rows
    lambda: random_dense_terms(3, 6, 984, k=20, betas=(0.5, 3.0), n_v=2),    # 512
    lambda: nn_xxz_chain(1, 9, 985, n_v=3),                                  # 1024
    lambda: random_dense_terms(2, 9, 986, k=20, betas=(0.5, 3.0), n_v=3),    # 2048, every pair
]


def same(a, b):
    return all(np.array_equal(a[k], b[k]) for k in ("rho", "h_star", "log_z", "entropy"))


@pytest.mark.parametrize("case", range(len(CASES)))
@pytest.mark.parametrize("prec,tol", [("fp64", 1e-10), ("mixed", 1e-5)])
def test_small_solve_matches_oracle(case, prec, tol):
    inst = CASES[case]()
    h = rdm.Hamiltonian.from_instance(inst)
    args = (inst.betas, inst.n_v, inst.k, inst.seed)
    got = rdm.solve(h, *args, precision=prec)
    for b, w in enumerate(olz.solve(inst)["results"]):
        assert np.linalg.norm(got["rho"][b] - w["rho"]) < tol * np.linalg.norm(w["rho"])
        assert np.linalg.norm(got["h_star"][b] - w["h_star"]) < 10 * tol * np.linalg.norm(w["h_star"])
        assert abs(got["log_z"][b] - w["log_z"]) < tol * max(1.0, abs(w["log_z"]))
    # the regeneration pass and the launches without a graph repeat it exactly
    assert same(got, rdm.solve(h, *args, precision=prec, mode="two_pass"))
    assert same(got, rdm.solve(h, *args, precision=prec, eager=True))
    # timed steps are launched kernel by kernel
    assert same(got, rdm.solve(h, *args, precision=prec, profile=True))


@pytest.mark.parametrize("prec", ["fp64", "mixed"])
def test_small_instances_in_a_batch_equal_solo(prec):
    insts = [CASES[1](), random_sparse_xxz(3021, n_range=(13, 13), n_v=2, k=20), CASES[4](), CASES[5]()]
    hs = [rdm.Hamiltonian.from_instance(i) for i in insts]
    both = rdm.solve_batch([dict(h=h, betas=i.betas, n_v=i.n_v, k=i.k, seed=i.seed) for h, i in zip(hs, insts)],
                           precision=prec)
    for h, i, got in zip(hs, insts, both):
        assert same(got, rdm.solve(h, i.betas, i.n_v, i.k, i.seed, precision=prec))
