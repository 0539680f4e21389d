"""The two launch forms of the product on bit-set tiles (a workgroup per tile,
and four of them in launches of fewer than 128 tiles) give the same result on
either side of the line: finite values bit for bit, and infinite entries of the
vector spread to the same rows."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")
rdm = pytest.importorskip("paper_2204_08147_amd")

from oracle import spin  # noqa: E402
from workloads import long_range_xxz, random_sparse_xxz  # noqa: E402

pytestmark = pytest.mark.gpu

SAME = ("rho", "h_star", "log_z", "entropy")


def product(h, x, prec):
    xd = rdm.to_panels(x, prec)
    yd = torch.full_like(xd, float("nan"))
    rdm.apply(h, xd, yd, precision=prec, n_cols=x.shape[1])
    return rdm.from_panels(yd, x.shape[0], x.shape[1], prec)


# 16 sites, 16 tiles a panel: 7 and 8 panels are 112 and 128 tiles
@pytest.mark.parametrize("family", ["dense", "sparse"])
@pytest.mark.parametrize("prec,width", [("mixed", 4), ("fp64", 2)])
def test_products_on_both_sides_of_the_line(family, prec, width):
    inst = long_range_xxz(2, 14, 741) if family == "dense" else random_sparse_xxz(3007, n_range=(16, 16))
    h = rdm.Hamiltonian.from_instance(inst, apply="hops")
    assert h.info()["bitset_tiles"] == 1
    dt = torch.float64 if prec == "fp64" else torch.float32
    x = torch.randn((inst.dim, 8 * width), generator=torch.Generator().manual_seed(3), dtype=dt).cuda()
    whole = product(h, x, prec)
    split = product(h, x[:, :7 * width].contiguous(), prec)
    assert torch.equal(split, whole[:, :7 * width])
    op = spin.sparse_hamiltonian(inst.n, inst.couplings, inst.hx, inst.hz)
    want = op.apply(x.double().cpu().numpy())
    # rounding of a sum of len(terms) products
    tol = 1e-13 if prec == "fp64" else 3e-6
    err = np.abs(whole.double().cpu().numpy() - want).max()
    assert err < tol * np.abs(want).max() * max(1, np.sqrt(len(op.terms)))


@pytest.mark.parametrize("prec,width", [("mixed", 4), ("fp64", 2)])
def test_infinite_entries_reach_the_same_rows(prec, width):
    # XX + YY couplings only: rows with equal spins on a pair have no matrix element
    inst = long_range_xxz(2, 14, 742)
    inst.hx[:] = 0.0
    h = rdm.Hamiltonian.from_instance(inst, apply="hops")
    assert h.info()["bitset_tiles"] == 1
    dt = torch.float64 if prec == "fp64" else torch.float32
    x = torch.randn((inst.dim, 8 * width), generator=torch.Generator().manual_seed(4), dtype=dt).cuda()
    for c, row in enumerate((0, inst.dim - 1, 0x5A5A, 0x0FF0)):
        x[row, c % width] = float("inf")
    whole = product(h, x, prec)[:, :width]
    split = product(h, x[:, :width].contiguous(), prec)
    assert torch.equal(torch.isfinite(split), torch.isfinite(whole))
    assert torch.equal(torch.nan_to_num(split), torch.nan_to_num(whole))


# four columns a vector: one FP32 panel, two FP64 panels, 16 tiles each; the
# bath's 14 bits add 4 tiles a panel (104 / 120 and 136 tiles alone)
@pytest.mark.parametrize("prec,n_v", [("mixed", 7), ("mixed", 8), ("fp64", 3), ("fp64", 4)])
def test_solves_on_both_sides_of_the_line(prec, n_v):
    inst = random_sparse_xxz(3013, n_range=(16, 16), n_s_choices=(2,), n_v=n_v, k=12)
    big = random_sparse_xxz(3012, n_range=(17, 17), n_v=8, k=12)
    hs = [rdm.Hamiltonian.from_instance(i, apply="hops") for i in (inst, big)]
    alone = rdm.solve(hs[0], inst.betas, inst.n_v, inst.k, inst.seed, precision=prec)
    both = rdm.solve_batch([dict(h=h, betas=i.betas, n_v=i.n_v, k=i.k, seed=i.seed) for h, i in zip(hs, (inst, big))],
                           precision=prec)
    for key in SAME:
        assert np.array_equal(both[0][key], alone[key]), key
