"""One workspace, several users: what a call leaves there must not be taken for what a plan keeps there."""
import numpy as np
import pytest

from workloads.bitstrings import random_bitstrings
from workloads.circuits import generate
from workloads.plans import region_plan, sweep_plan

pytestmark = pytest.mark.gpu


def _say(msg):
    print(msg, flush=True)


def _plan(ctx, kind, precision="fp32"):
    """A plan and its number of qubits: chains of small tensors (one workgroup each), of larger ones one at a
    time, or in launches of two."""
    from paper_1905_00444_amd import Circuit, Plan
    if kind == "small":
        c = generate(4, 4, 8, 0)
        return Plan(ctx, Circuit(ctx, c.to_text()), sweep_plan(c, open_qubits=[15, 14]), precision), 16
    c = generate(4, 5, 24, 2)
    qid = c.qubit_of()
    plan, _ = region_plan(c, 2, 2, [[qid[(1, 3)], qid[(2, 3)], 0, 2]], [(3, 4), (2, 4)])
    return Plan(ctx, Circuit(ctx, c.to_text()), plan, precision, batch=2 if kind == "batched" else 1), 20


@pytest.mark.parametrize("kind", ["small", "one chain", "batched"])
@pytest.mark.parametrize("M,N,K", [(64, 64, 4096), (100, 90, 5000)])
def test_split_products_between_a_plans_calls(kind, M, N, K):
    """A product that splits K puts its partial tiles where the plan's tables and world-lines were: the
    plan's next call gives the same bits as the one before."""
    import torch
    from paper_1905_00444_amd import Context, cgemm
    _say(f"split product between calls of a plan: {kind} {M}x{N}x{K}")
    ctx = Context(0)
    ctx.ensure_workspace(64 << 20)
    p, n = _plan(ctx, kind)
    bits = random_bitstrings(3, n, 1)
    want = p.amplitudes(bits)
    rng = np.random.default_rng(K)
    a, b = (torch.from_numpy((rng.standard_normal((r, K)) + 1j * rng.standard_normal((r, K))).astype(np.complex64)).cuda()
            for r in (M, N))
    cgemm(ctx, a, b)
    got = p.amplitudes(bits)
    torch.cuda.synchronize()
    assert np.array_equal(got.cpu().numpy(), want.cpu().numpy())
