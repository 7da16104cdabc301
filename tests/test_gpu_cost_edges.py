"""Cost diagonals at the edges of the cost kernel's waves and clause lists,
against the oracle, every entry: sizes around one wave's states (2^11, and
2^13 from 2^25 states on), clause counts around a list chunk (192) and a multiple of
four or sixteen patterns, and clause sets that sit wholly in one list."""
import numpy as np
import pytest

import oracle
from workloads import instances as inst

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def q():
    import torch
    assert torch.cuda.is_available(), "GPU tests need a ROCm device"
    import paper_2401_02852_amd as q
    q.load_library()
    return q


def check(q, cl, n, pred="nae"):
    print(f"\n[cost] n={n} m={cl.shape[0]} k={cl.shape[1]} {pred}", flush=True)
    ref = oracle.cost(cl, n, pred)
    c, sols = q.build_cost_diagonal(cl, n, predicate=pred, count_solutions=True)
    assert np.array_equal(c.cpu().numpy().astype(np.int64), ref)
    assert sols == int((ref == 0).sum())
    (cb,) = q.build_cost_diagonals([cl], [n], predicate=pred)
    assert np.array_equal(cb.cpu().numpy().astype(np.int64), ref)


@pytest.mark.parametrize("n,m", [(3, 5), (4, 16), (5, 17), (10, 3), (11, 191), (11, 192), (12, 193), (13, 255), (13, 256),
                                 (14, 385), (17, 60), (23, 40), (24, 33), (24, 260), (25, 9), (25, 260)])
@pytest.mark.parametrize("pred", ["nae", "sat"])
def test_waves_and_chunks(q, n, m, pred):
    check(q, inst.instance(n, 3, m, 1000 * n + m), n, pred)


# variables of every clause drawn from one range: the pattern list, the list
# of clauses constant over a run, those constant over a wave, and high bits only
@pytest.mark.parametrize("lo,hi", [(0, 5), (5, 11), (11, 13), (13, 24), (0, 24)])
@pytest.mark.parametrize("n,m", [(24, 200), (24, 1), (25, 200)])
def test_clauses_of_one_list(q, lo, hi, n, m):
    rng = np.random.default_rng(lo * 100 + hi + m)
    k = min(3, hi - lo)
    v = np.stack([rng.choice(np.arange(lo, hi), k, replace=False) for _ in range(m)])
    cl = np.where(rng.integers(0, 2, (m, k)) == 1, -(v + 1), v + 1).astype(np.int32)
    check(q, cl, n)


# one clause repeated: the largest counts an 8-bit and a 16-bit diagonal hold in a test's time
@pytest.mark.parametrize("m", [255, 256, 4095, 4096, 65535])
def test_repeated_clause(q, m):
    for lits in ([1, -2, 3], [9, 10, -11], [12, 13, 14], [2, 8, -14]):
        check(q, np.tile(np.array(lits, dtype=np.int32), (m, 1)), 14)
