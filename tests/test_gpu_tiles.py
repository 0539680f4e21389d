"""GPU parity of the hop-table product on bit-set tiles at the edges of its
launch rules: segments with fewer tiles than CUs share a tile between several
workgroups when launched alone, and the workgroups' order over the XCDs has
whole runs and a remainder."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")
rdm = pytest.importorskip("paper_2204_08147_amd")

from oracle import spin  # noqa: E402
from workloads import long_range_xxz, random_dense_terms, random_sparse_xxz  # noqa: E402

pytestmark = pytest.mark.gpu

# (instance, columns): 1 tile; 16 tiles a panel, below / at / above 256 tiles
# in either panel width (4 FP32, 2 FP64 columns); 32 tiles a panel, above 512
# with and without a remainder
TILE_CASES = [
    (lambda: random_sparse_xxz(3007, n_range=(12, 12)), 1),
    (lambda: random_dense_terms(2, 11, 91, density=0.5), 6),
    (lambda: random_sparse_xxz(3007, n_range=(16, 16)), 3),
    (lambda: random_sparse_xxz(3007, n_range=(16, 16)), 33),
    (lambda: random_sparse_xxz(3007, n_range=(16, 16)), 64),
    (lambda: long_range_xxz(1, 15, 92), 30),
    (lambda: random_sparse_xxz(3009, n_range=(17, 17)), 64),
    (lambda: random_sparse_xxz(3009, n_range=(17, 17)), 77),
]


@pytest.mark.parametrize("case", range(len(TILE_CASES)))
@pytest.mark.parametrize("prec", ["fp64", "mixed"])
def test_bitset_product_matches_oracle(case, prec):
    make, n_cols = TILE_CASES[case]
    inst = make()
    h = rdm.Hamiltonian.from_instance(inst, apply="hops")
    assert h.info()["bitset_tiles"] == 1
    op = spin.sparse_hamiltonian(inst.n, inst.couplings, inst.hx, inst.hz)
    dt = torch.float64 if prec == "fp64" else torch.float32
    x = np.random.default_rng(case).normal(size=(inst.dim, n_cols))
    xd = rdm.to_panels(torch.tensor(x, dtype=dt, device="cuda"), prec)
    yd = torch.full_like(xd, float("nan"))
    rdm.apply(h, xd, yd, precision=prec, n_cols=n_cols)
    got = rdm.from_panels(yd, inst.dim, n_cols, prec).double().cpu().numpy()
    want = op.apply(x if prec == "fp64" else x.astype(np.float32).astype(np.float64))
    # the parity bar of the products: rounding of a sum of len(terms) products
    tol = 1e-13 if prec == "fp64" else 3e-6
    assert np.abs(got - want).max() < tol * np.abs(want).max() * max(1, np.sqrt(len(op.terms)))


@pytest.mark.parametrize("prec", ["fp64", "mixed"])
def test_small_instance_alone_equals_in_a_batch_that_fills_the_chip(prec):
    # alone its tiles are shared between workgroups, beside the larger
    # instance they are not
    insts = [random_sparse_xxz(3011, n_range=(14, 14), n_v=2, k=20),
             random_sparse_xxz(3012, n_range=(18, 18), n_v=8, k=20)]
    hs = [rdm.Hamiltonian.from_instance(i, apply="hops") for i in insts]
    items = [dict(h=h, betas=i.betas, n_v=i.n_v, k=i.k, seed=i.seed) for h, i in zip(hs, insts)]
    both = rdm.solve_batch(items, precision=prec)
    alone = rdm.solve(hs[0], insts[0].betas, insts[0].n_v, insts[0].k, insts[0].seed, precision=prec)
    for key in ("rho", "h_star", "log_z", "entropy"):
        assert np.array_equal(both[0][key], alone[key]), key
