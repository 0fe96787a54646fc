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


@pytest.mark.parametrize("kind", ["small", "one chain"])
@pytest.mark.parametrize("roomy", [True, False])
def test_captured_call_survives_calls_of_other_sizes(kind, roomy):
    """A caller's own graph of a one-chain call, with calls of one and of several chains and a change of the
    gates between its replays: every replay gives what an eager call gives.  roomy: the workspace holds
    the largest of these calls from the start; else they get a buffer of their own."""
    import torch
    from paper_1905_00444_amd import Context
    _say(f"captured call among others: {kind}, roomy {roomy}")
    ctx = Context(0, stream=torch.cuda.Stream())
    if roomy:
        ctx.ensure_workspace(128 << 20)
    p, n = _plan(ctx, kind)
    bits = torch.from_numpy(random_bitstrings(40, n, 1)).cuda()
    torch.cuda.synchronize()
    one = bits[:1]

    def eager(b):
        got = p.amplitudes(b)
        ctx.synchronize()
        return got.cpu().numpy()

    want = eager(one)
    out = torch.zeros((1, 4), dtype=torch.complex128, device="cuda")
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph, stream=ctx.stream):
        out.zero_()
        p.amplitudes(one, out=out)

    def replay():
        torch.cuda.synchronize()
        graph.replay()
        torch.cuda.synchronize()
        return out.cpu().numpy()

    assert np.array_equal(replay(), want)
    many = eager(bits)
    assert np.array_equal(many[:1], want)
    litter = [torch.full((1 << 20,), 255, dtype=torch.uint8, device="cuda") for _ in range(32)]  # what was given back
    assert np.array_equal(replay(), want)
    values = p.circuit.values
    p.circuit.set_values(values * np.complex64(0.5))
    half = eager(one)
    assert not np.array_equal(half, want)
    assert np.array_equal(replay(), half)
    p.circuit.set_values(values)
    assert np.array_equal(eager(bits), many)
    assert np.array_equal(replay(), want)
    assert litter[0][0] == 255


def test_captured_call_of_several_chains():
    """Captured after an eager call of one chain only: the workspace does not move under the capture."""
    import torch
    from paper_1905_00444_amd import Context
    _say("captured call of several chains")
    for kind in ("small", "one chain"):
        ctx = Context(0, stream=torch.cuda.Stream())
        p, n = _plan(ctx, kind)
        bits = torch.from_numpy(random_bitstrings(3, n, 1)).cuda()
        torch.cuda.synchronize()
        want = [p.amplitudes(bits[i:i + 1]) for i in range(3)]
        ctx.synchronize()
        want = torch.cat(want)
        out = torch.zeros((3, 4), dtype=torch.complex128, device="cuda")
        torch.cuda.synchronize()
        graph = torch.cuda.CUDAGraph()
        with torch.cuda.graph(graph, stream=ctx.stream):
            p.amplitudes(bits, out=out)
        for _ in range(2):
            with torch.cuda.stream(ctx.stream):
                out.zero_()
            torch.cuda.synchronize()
            graph.replay()
            torch.cuda.synchronize()
            assert np.array_equal(out.cpu().numpy(), want.cpu().numpy())
            p.amplitudes(bits)
            ctx.synchronize()
