"""Runs and gradients of whole cost diagonals that turn out flip-symmetric use
half the state: against the FP64 oracle on both sides of every size limit of
that choice, and with one entry of a symmetric diagonal changed, where the
whole state has to be used."""
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


def angles(p, seed):
    """Both butterfly forms: |tan beta| <= 1 and > 1 (an odd number of them)."""
    rng = np.random.default_rng(seed)
    b = rng.uniform(-0.7, 0.7, p)
    b[p // 2] = 1.3
    return rng.uniform(-1, 1, p), b


def check_run(q, cost_np, n, m, p, u16, ctx):
    import torch
    g, b = angles(p, n)
    cost = torch.from_numpy(cost_np.astype(np.uint16 if u16 else np.uint8)).cuda()
    ref, ref_psi = oracle.qaoa(cost_np, n, g, b), oracle.state(cost_np, n, g, b)
    psi = torch.full((1 << n,), 7.0, dtype=torch.complex64, device="cuda")
    for state in (None, psi):
        got = q.qaoa_run(cost, n, m, g, b, state=state, ctx=ctx)
        assert abs(got.p_success - ref[0]) <= 1e-5
        assert abs(got.expected_cost - ref[1]) <= 1e-5 * ref[1] + 1e-9
        assert abs(got.norm - 1.0) <= 1e-5
    # FP32 butterflies: a few rounding errors of 6e-8 per layer and qubit on the amplitude scale
    assert np.max(np.abs(psi.cpu().numpy() - ref_psi)) <= 6e-8 * 4 * n * p * np.max(np.abs(ref_psi))
    dg, db, r = q.qaoa_grad(cost, n, m, g, b, w_psucc=1.0, w_energy=0.1, ctx=ctx)
    rg, rb, _ = oracle.qaoa_grad(cost_np, n, g, b, 1.0, 0.1)
    scale = max(np.max(np.abs(rg)), np.max(np.abs(rb)))
    assert np.max(np.abs(dg - rg)) <= 1e-4 * scale + 1e-5
    assert np.max(np.abs(db - rb)) <= 1e-4 * scale + 1e-5
    assert abs(r.norm - 1.0) <= 1e-5


# n = 20: the smallest checked size; up to 22 the first sweep is launched ahead of
# the check's answer, above after it; tile sizes with two and three groups
@pytest.mark.parametrize("n,u16,tb", [(19, False, 13), (20, False, 12), (20, True, 13), (21, False, 14), (22, True, 12),
                                      (24, False, 14), (25, False, 13)])
def test_symmetric_and_nearly_symmetric(q, n, u16, tb):
    m = 300 if u16 else 40
    p = 3
    base = oracle.cost(inst.instance(n, 3, m, n), n)
    ctx = q.Context()
    ctx.set_tune(n, {"tile_bits": tb, "low_run_bits": 4, "page_bit": 18, "split": 0}, "u16" if u16 else "u8")
    # symmetric; first, last, middle and one random entry different from its mirror
    rng = np.random.default_rng(n)
    spots = [None, 0, (1 << n) - 1, 1 << (n - 1), int(rng.integers(1 << n))]
    for at in spots if n < 24 else spots[:2]:
        print(f"\n[flip] n={n} u16={u16} tb={tb} at={at}", flush=True)
        cost = base.copy()
        if at is not None:
            cost[at] = (cost[at] + 1) % (m + 1)
        check_run(q, cost, n, m, p, u16, ctx)
    ctx.close()


# n = 22 and 23: the last size whose first sweep is launched ahead of the check's
# answer, and the first that waits for it
@pytest.mark.parametrize("n,u16,tb", [(22, False, 13), (23, False, 13), (23, True, 14), (23, False, 12)])
def test_both_sides_of_the_wait(q, n, u16, tb):
    m = 300 if u16 else 40
    base = oracle.cost(inst.instance(n, 3, m, n + tb), n)
    ctx = q.Context()
    ctx.set_tune(n, {"tile_bits": tb, "low_run_bits": 4, "page_bit": 18, "split": 0}, "u16" if u16 else "u8")
    for at in (None, (1 << (n - 1)) - 1):  # symmetric; the last pair in the middle differs
        print(f"\n[flip] n={n} u16={u16} tb={tb} at={at}", flush=True)
        cost = base.copy()
        if at is not None:
            cost[at] = (cost[at] + 1) % (m + 1)
        check_run(q, cost, n, m, 2, u16, ctx)
    ctx.close()
