"""Sweep kernels of every tile size against the FP64 oracle, whole final states
included: the smallest tiled states, both directions of the state's relabelling
(an odd and an even number of layers beyond |tan beta| = 1), 8- and 16-bit
costs, and both sides of the size (2^24 stored amplitudes) from which the middle
sweeps exchange through LDS in another way; then batches on both sides of the
size from which their diagonals are checked for flip symmetry."""
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


def device_cost(cost, u16):
    import torch
    return torch.from_numpy(cost.astype(np.uint16 if u16 else np.uint8)).cuda()


def angles(p, cots, seed):
    rng = np.random.default_rng(seed)
    b = rng.uniform(-0.7, 0.7, p)
    b[:cots] = 1.2
    return rng.uniform(-1, 1, p), b


def state_bound(n, p, ref):
    """FP32 butterflies: a few rounding errors of 6e-8 per layer and qubit on the amplitude scale."""
    return 6e-8 * 4 * n * p * np.max(np.abs(ref))


CASES = [(n, pred, tb, low, cots, u16)
         for tb, low in ((12, 4), (12, 6), (13, 4), (13, 5), (14, 4), (14, 6))
         for n, pred, cots, u16 in ((15, "sat", 1, False), (16, "nae", 2, True), (20, "sat", 1, True), (21, "nae", 1, False))]
CASES += [(24, "sat", 13, 4, 1, False), (25, "sat", 12, 4, 1, False), (25, "sat", 13, 4, 0, True),
          (25, "nae", 13, 4, 1, False), (26, "nae", 12, 4, 1, False), (26, "nae", 13, 5, 1, True)]


@pytest.mark.parametrize("n,pred,tb,low,cots,u16", CASES)
def test_states_of_every_tile(q, n, pred, tb, low, cots, u16):
    import torch
    m, p = 30, 3
    cost = oracle.cost(inst.instance(n, 3, m, n), n, pred)
    g, b = angles(p, cots, n)
    print(f"\n[tiles] n={n} {pred} tb={tb} low={low} u16={u16}", flush=True)
    ctx = q.Context()
    ctx.set_tune(n, {"tile_bits": tb, "low_run_bits": low, "page_bit": 18, "split": 0}, "u16" if u16 else "u8")
    psi = torch.full((1 << n,), 7.0, dtype=torch.complex64, device="cuda")
    got = q.qaoa_run(device_cost(cost, u16), n, m, g, b, state=psi, ctx=ctx)
    ref, ref_psi = oracle.qaoa(cost, n, g, b), oracle.state(cost, n, g, b)
    assert abs(got.p_success - ref[0]) <= 1e-5
    assert abs(got.expected_cost - ref[1]) <= 1e-5 * ref[1] + 1e-9
    assert abs(got.norm - 1.0) <= 1e-5
    assert np.max(np.abs(psi.cpu().numpy() - ref_psi)) <= state_bound(n, p, ref_psi)
    ctx.close()


@pytest.mark.parametrize("u16", [False, True])
@pytest.mark.parametrize("sizes", [[20, 19, 17, 20, 15, 16, 12, 3],            # below 2^23 amplitudes: not checked
                                   [20, 19, 17, 20, 15, 16, 12, 3, 22, 20, 20]])   # from there on: checked
def test_batches_of_symmetric_and_nearly_symmetric(q, sizes, u16):
    """Symmetric diagonals, diagonals with one entry changed and 3-SAT ones in one
    launch, states kept, run three times (the later ones replay a graph) with
    other angles and, for the last, another diagonal in the same buffer."""
    import torch
    m, p = 40, 3
    costs = [oracle.cost(inst.instance(n, 3, m, 7 * n + i), n, "sat" if i % 4 == 2 else "nae") for i, n in enumerate(sizes)]
    for i, n in enumerate(sizes):
        if i % 4 == 3:
            at = (1 << n) - 1 - i
            costs[i][at] = (costs[i][at] + 1) % (m + 1)
    dev = [device_cost(c, u16) for c in costs]
    states = [torch.empty(1 << n, dtype=torch.complex64, device="cuda") for n in sizes]
    run = q.PreparedBatch(dev, sizes, [m] * len(sizes), [p] * len(sizes), states=states)
    for turn in range(3):
        if turn == 2:  # a symmetric one loses its symmetry in place
            costs[0][5] = (costs[0][5] + 1) % (m + 1)
            dev[0].copy_(device_cost(costs[0], u16))
        a = [angles(p, (turn + i) % 3, 10 * turn + i) for i in range(len(sizes))]
        got = np.asarray(run.run([x[0] for x in a], [x[1] for x in a]))
        for i, n in enumerate(sizes):
            print(f"[batch] turn={turn} i={i} n={n}", flush=True)
            ref, ref_psi = oracle.qaoa(costs[i], n, *a[i]), oracle.state(costs[i], n, *a[i])
            assert abs(got[i][0] - ref[0]) <= 1e-5
            assert abs(got[i][1] - ref[1]) <= 1e-5 * ref[1] + 1e-9
            assert abs(got[i][2] - 1.0) <= 1e-5
            assert np.max(np.abs(states[i].cpu().numpy() - ref_psi)) <= state_bound(n, p, ref_psi)
