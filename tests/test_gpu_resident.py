"""One-workgroup circuits on both sides of every size that has a kernel of its
own (n = 9 .. 14), against the FP64 oracle with whole final states, and the same
instances in one batch, whose workgroups hold more waves than most of them use:
8- and 16-bit costs, both directions of the relabelling, tables in the kernel
arguments, in LDS and too long for it."""
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


def setup(n, m, p, pred, u16, cots, seed):
    import torch
    cost = oracle.cost(inst.instance(n, min(n, 3), min(m, 250), seed), n, pred)
    rng = np.random.default_rng(seed)
    b = rng.uniform(-0.7, 0.7, p)
    b[:cots] = 1.2
    dev = torch.from_numpy(cost.astype(np.uint16 if u16 else np.uint8)).cuda()
    return cost, dev, rng.uniform(-1, 1, p), b


def check(got, psi, cost, n, g, b):
    ref, ref_psi = oracle.qaoa(cost, n, g, b), oracle.state(cost, n, g, b)
    assert abs(got[0] - ref[0]) <= 1e-5
    assert abs(got[1] - ref[1]) <= 1e-5 * ref[1] + 1e-9
    assert abs(got[2] - 1.0) <= 1e-5
    # FP32: a few rounding errors of 6e-8 per layer and qubit on the amplitude scale
    assert np.max(np.abs(psi.cpu().numpy() - ref_psi)) <= 6e-8 * 4 * n * max(len(g), 1) * np.max(np.abs(ref_psi))


# (m, p): tables in the kernel arguments; in LDS; longer than that
SHAPES = [(40, 3), (40, 0), (100, 8), (250, 12)]


@pytest.mark.parametrize("n", [1, 6, 9, 10, 11, 12, 13, 14])
@pytest.mark.parametrize("m,p", SHAPES)
@pytest.mark.parametrize("u16", [False, True])
def test_single_and_batched(q, n, m, p, u16):
    import torch
    jobs = []
    for i, pred in enumerate(("nae", "sat", "sat")):
        cost, dev, g, b = setup(n, m, p, pred, u16, min(i, p), 100 * n + i)
        psi = torch.full((1 << n,), 7.0, dtype=torch.complex64, device="cuda")
        r = q.qaoa_run(dev, n, m, g, b, state=psi)
        check((r.p_success, r.expected_cost, r.norm), psi, cost, n, g, b)
        jobs.append((dev, g, b, r, psi))
    states = [torch.full((1 << n,), 7.0, dtype=torch.complex64, device="cuda") for _ in jobs]
    got = q.qaoa_run_batched([j[0] for j in jobs], [n] * 3, [m] * 3, [j[1] for j in jobs], [j[2] for j in jobs],
                             states=states)
    for (dev, g, b, r, psi), st, x in zip(jobs, states, got):
        assert torch.equal(st, psi)
        assert abs(x.p_success - r.p_success) <= 1e-12 and abs(x.expected_cost - r.expected_cost) <= 1e-12 * (1 + m)


# (m, p, checkpoint_every): short and long phase tables, with and without checkpoints
@pytest.mark.parametrize("n", [9, 10, 11, 12, 13])
@pytest.mark.parametrize("m,p,every", [(40, 0, 0), (40, 1, 0), (40, 7, 3), (250, 12, 0), (2600, 5, 2)])
@pytest.mark.parametrize("u16", [False, True])
def test_gradients(q, n, m, p, every, u16):
    if m > 255 and not u16:
        m = 255
    for i, pred in enumerate(("nae", "sat")):
        cost, dev, g, b = setup(n, m, p, pred, u16, min(i, p), 7 * n + i)
        dg, db, r = q.qaoa_grad(dev, n, m, g, b, w_psucc=1.0, w_energy=0.1, checkpoint_every=every)
        ref = oracle.qaoa(cost, n, g, b)
        assert abs(r.p_success - ref[0]) <= 1e-5
        assert abs(r.expected_cost - ref[1]) <= 1e-5 * ref[1] + 1e-9
        assert abs(r.norm - 1.0) <= 1e-5
        if p == 0:
            continue
        rg, rb, _ = oracle.qaoa_grad(cost, n, g, b, 1.0, 0.1)
        scale = max(np.max(np.abs(rg)), np.max(np.abs(rb)))
        # the two states carry a few rounding errors of 6e-8 per layer and qubit: below 6e-8 * 4 * 13 * 12 of the scale
        assert np.max(np.abs(dg - rg)) <= 1e-4 * scale + 1e-5
        assert np.max(np.abs(db - rb)) <= 1e-4 * scale + 1e-5


# Row lengths around what one thread fetches of the next phase row (256 threads at n = 12, 512
# at n = 13), the last that fits the LDS row and the first that does not; p rows
# that do not all fit, so rows come one at a time. Every entry of a row is read.
@pytest.mark.parametrize("n", [11, 12, 13])
@pytest.mark.parametrize("rows", [256, 257, 512, 513, 1025, 2304, 2305, 2559, 2560, 2561])
def test_gradients_with_long_phase_rows(q, n, rows):
    import torch
    m, p = rows - 1, 12
    rng = np.random.default_rng(rows + n)
    cost = rng.integers(0, rows, 1 << n)
    cost[rng.permutation(1 << n)[:rows]] = np.arange(rows)[: 1 << n]
    dev = torch.from_numpy(cost.astype(np.uint16)).cuda()
    g, b = rng.uniform(-1, 1, p), rng.uniform(-0.7, 0.7, p)
    b[p // 2] = 1.2
    # (the weights keep E[C], about m / 2, and p_succ of one scale)
    we = 1.0 / m
    dg, db, r = q.qaoa_grad(dev, n, m, g, b, w_psucc=1.0, w_energy=we, checkpoint_every=3)
    ref = oracle.qaoa(cost, n, g, b)
    assert abs(r.p_success - ref[0]) <= 1e-5
    assert abs(r.expected_cost - ref[1]) <= 1e-5 * ref[1]
    assert abs(r.norm - 1.0) <= 1e-5
    rg, rb, _ = oracle.qaoa_grad(cost, n, g, b, 1.0, we)
    scale = max(np.max(np.abs(rg)), np.max(np.abs(rb)))
    # as test_gradients: 6e-8 * 4 * 13 * 12 of the scale, with its room
    assert np.max(np.abs(dg - rg)) <= 1e-4 * scale + 1e-5
    assert np.max(np.abs(db - rb)) <= 1e-4 * scale + 1e-5
    # side by side with others: the same, bit for bit
    one = q.qaoa_grad_batched([dev] * 3, [n] * 3, [m] * 3, [g] * 3, [b] * 3, w_psucc=1.0, w_energy=we, checkpoint_every=3)
    for x, y in zip(one[0], one[1]):
        assert np.array_equal(x, dg) and np.array_equal(y, db)
