"""Plain products from several threads and streams at once on one Hamiltonian:
one call uses the descriptor kept with the operator's tables, the others their
own; results equal those of single calls bit for bit."""
import threading

import pytest

torch = pytest.importorskip("torch")
rdm = pytest.importorskip("paper_2204_08147_amd")

from workloads import random_dense_terms  # noqa: E402

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n_b,apply", [(6, "hops"), (13, "hops"), (16, "transform")])
@pytest.mark.parametrize("precision", ["mixed", "fp64"])
def test_concurrent_products_equal_single_ones(n_b, apply, precision):
    inst = random_dense_terms(1, n_b, 40 + n_b)
    h = rdm.Hamiltonian.from_instance(inst, apply=apply)
    gen = torch.Generator(device="cuda").manual_seed(n_b)
    w, dtype = (2, torch.float64) if precision == "fp64" else (4, torch.float32)
    cols = (1, 3, 8, 13)
    xs = [torch.randn((1 << (n_b + 1)) * (-(-c // w) * w), generator=gen, device="cuda", dtype=dtype) for c in cols]

    def product(i):
        y = torch.empty_like(xs[i])
        rdm.apply(h, xs[i], y, precision=precision, n_cols=cols[i])
        return y

    want = [product(i) for i in range(len(xs))]
    torch.cuda.synchronize()
    got = [[] for _ in xs]

    def calls(i):
        with torch.cuda.stream(torch.cuda.Stream()):
            for _ in range(5):
                got[i].append(product(i))

    threads = [threading.Thread(target=calls, args=(i,)) for i in range(len(xs))]
    for t in threads:
        t.start()
    for t in threads:
        t.join()
    torch.cuda.synchronize()
    for i, w in enumerate(want):
        assert len(got[i]) == 5
        for y in got[i]:
            assert torch.equal(y, w)
