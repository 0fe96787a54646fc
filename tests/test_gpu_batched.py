"""Batched chains (G bitstring x slice pairs per launch) and their hipGraph replay: identical
to the one-chain-at-a-time path, and correct against the oracle and closed forms, including
the 70-qubit (8x9 minus two corners, 1+24+1) workload's shapes."""
import numpy as np
import pytest

from oracle import sv
from oracle.metrics import rel_err
from workloads.bitstrings import random_bitstrings
from workloads.circuits import generate, identity_cz
from workloads.plans import region_plan, sweep_plan, plan_8x9, C5_REMOVED

pytestmark = pytest.mark.gpu


def _say(msg):
    print(msg, flush=True)


@pytest.fixture(scope="module")
def ctx():
    import torch
    from paper_1905_00444_amd import Context
    assert torch.cuda.is_available()
    return Context(0)


@pytest.fixture(scope="module")
def gctx():
    """A context on a non-default stream (graph capture needs one)."""
    import torch
    from paper_1905_00444_amd import Context
    return Context(0, stream=torch.cuda.Stream())


def _setup_4x5():
    c = generate(4, 5, 32, 2)
    qid = c.qubit_of()
    cuts = [[qid[(1, 3)], qid[(2, 3)], 0, 2], [qid[(3, 1)], qid[(3, 2)], 1, 2]]
    plan, _ = region_plan(c, 2, 2, cuts, [(3, 4), (2, 4)])
    return c, plan


@pytest.mark.parametrize("precision", ["fp32", "bf16x3"])
@pytest.mark.parametrize("G", [2, 8])
def test_batched_equals_sequential_bitwise(ctx, precision, G):
    """With group hoisting off, the batched path runs every step of every chain with the same
    kernels and shapes as the one-chain path: bitwise equal."""
    import torch
    from paper_1905_00444_amd import Circuit, Plan
    _say(f"batched G={G} {precision}")
    c, plan = _setup_4x5()
    bits = random_bitstrings(3, 20, 5)  # 3 x 16 = 48 chains: 48 / 8 leaves no tail, 48 / 32 would
    circ = Circuit(ctx, c.to_text())
    seq = Plan(ctx, circ, plan, precision, hoist=False).amplitudes(bits)
    bat = Plan(ctx, circ, plan, precision, batch=G, hoist=False).amplitudes(bits)
    torch.cuda.synchronize()
    assert np.array_equal(seq.cpu().numpy(), bat.cpu().numpy())


@pytest.mark.parametrize("precision", ["fp32", "bf16x3"])
@pytest.mark.parametrize("G", [2, 8, 32])
def test_group_hoisting_matches_sequential_and_state_vector(ctx, precision, G):
    """Batched plans with cuts (default): the steps that depend on no cut run once per launch
    group, a shared operand is taken as B and the group's chains stack along M.  Different GEMM
    shapes and operand roles accumulate in another order and split their operands in other
    kernels, so the comparison with the one-chain path is within rounding: FP32 2e-6 norm-wise,
    split-BF16 2e-5 (each operand is represented to about 2^-17 relative, and the two paths
    round their splits independently); both meet the state-vector bounds."""
    import torch
    from paper_1905_00444_amd import Circuit, Plan
    _say(f"group hoisting G={G} {precision}")
    c, plan = _setup_4x5()
    bits = random_bitstrings(3, 20, 5)
    circ = Circuit(ctx, c.to_text())
    seq = Plan(ctx, circ, plan, precision).amplitudes(bits)
    bp = Plan(ctx, circ, plan, precision, batch=G)
    bat = bp.amplitudes(bits)
    torch.cuda.synchronize()
    seq, bat = seq.cpu().numpy(), bat.cpu().numpy()
    assert rel_err(bat, seq) <= {"fp32": 2e-6, "bf16x3": 2e-5}[precision]
    ref = sv.open_amplitudes(c.to_text(), bits, plan["open"])
    bound = 1e-5 if precision == "fp32" else 1e-4
    assert rel_err(seq, ref) <= bound and rel_err(bat, ref) <= bound
    # the executed flops count each group's cut-independent steps once
    S = bp.info()["n_slices"]
    assert bp.flops(0, S) < S * bp.info()["flops_per_slice"]


@pytest.mark.parametrize("precision", ["fp32", "bf16x3"])
@pytest.mark.parametrize("cuts,hoist,n,rng", [(True, True, 3, (0, 16)), (True, True, 1, (3, 10)), (True, False, 5, (2, 5)),
                                              (False, True, 7, (0, 1)), (False, True, 70, (0, 1))])
def test_call_of_several_chains_equals_single_chains_bitwise(precision, cuts, hoist, n, rng):
    """A one-chain plan runs a call of several chains with several per launch: the same bits as one call
    per bitstring and slice."""
    import torch
    from paper_1905_00444_amd import Context, Circuit, Plan
    _say(f"several chains per call {precision} cuts {cuts} hoist {hoist} n {n} slices {rng}")
    c, plan = _setup_4x5()
    if not cuts:
        c = generate(4, 5, 16, 2)
        plan, _ = region_plan(c, 2, 2, [], [(3, 4), (2, 4)])
    bits = random_bitstrings(n, 20, 8)
    one = Context(0)
    seq = Plan(one, Circuit(one, c.to_text()), plan, precision, hoist=hoist)
    want = torch.zeros((n, 4), dtype=torch.complex128, device="cuda")
    for b in range(n):
        for s in range(*rng):
            seq.amplitudes(bits[b:b + 1], s, s + 1, out=want[b:b + 1])
    many = Context(0)
    p = Plan(many, Circuit(many, c.to_text()), plan, precision, hoist=hoist)
    got = p.amplitudes(bits, *rng)
    again = p.amplitudes(bits[:1], *rng)  # fewer chains on the same layout
    torch.cuda.synchronize()
    assert many.ws.numel() > one.ws.numel()
    assert np.array_equal(got.cpu().numpy(), want.cpu().numpy())
    assert np.array_equal(again.cpu().numpy(), want[:1].cpu().numpy())


@pytest.mark.parametrize("rows,cols,depth,n_open,n,precision", [
    (2, 1, 8, 0, 1, "fp32"), (1, 5, 23, 1, 3, "bf16x3"), (3, 3, 16, 2, 65, "fp16"), (3, 4, 20, 3, 7, "fp32"),
    (4, 4, 8, 3, 600, "fp32"), (3, 1, 43, 0, 2, "bf16x3")])
def test_plans_of_small_tensors_vs_state_vector(ctx, rows, cols, depth, n_open, n, precision):
    """Plans whose chains run whole in a workgroup: FP32 products of at most 2^11 terms in at most 15 steps,
    norm-wise 15 x 8 x 2^-24 = 7.2e-6; and one chain at a time (a workspace of one chain) the same bits as
    all at once.  600 chains are more than a launch takes; tensors from 2 elements to 2^11."""
    import torch
    from paper_1905_00444_amd import Circuit, Plan
    _say(f"small {rows}x{cols} d{depth} open {n_open} n {n} {precision}")
    c = generate(rows, cols, depth, 5)
    plan = sweep_plan(c, range(rows * cols - n_open, rows * cols), by="row" if cols <= rows else "col")
    bits = random_bitstrings(n, rows * cols, 3)
    p = Plan(ctx, Circuit(ctx, c.to_text()), plan, precision)
    shapes = [(s["m_bits"], s["n_bits"], s["k_bits"]) for s in p.steps()]
    assert max(max(M + K, N + K, M + N) for M, N, K in shapes) <= 11
    got = p.amplitudes(bits)
    one = torch.cat([p.amplitudes(bits[i:i + 1]) for i in range(min(n, 5))])
    torch.cuda.synchronize()
    assert rel_err(got.cpu().numpy(), sv.open_amplitudes(c.to_text(), bits, plan["open"])) <= 7.2e-6
    assert np.array_equal(got[:5].cpu().numpy(), one.cpu().numpy())


@pytest.mark.parametrize("precision", ["fp32", "bf16x3"])
@pytest.mark.parametrize("depth,cut_bits,n,batch", [(16, 0, 1, 1), (20, 1, 3, 1), (24, 0, 40, 64), (27, 2, 2, 4), (32, 0, 2, 1),
                                                    (32, 2, 5, 16)])
def test_products_that_read_reordered_operands_in_place(ctx, precision, depth, cut_bits, n, batch):
    """Regions whose joins read one or both results in another order than they lie in, through every tile that
    depths 16 to 32 give (bonds of 2 to 4 bits), single chains and groups.  15 steps, the plan tests' bounds."""
    import torch
    from paper_1905_00444_amd import Circuit, Plan
    _say(f"reordered operands d{depth} cut {cut_bits} n {n} batch {batch} {precision}")
    c = generate(4, 4, depth, 6)
    qid = c.qubit_of()
    plan, _ = region_plan(c, 2, 2, [[qid[(1, 3)], qid[(2, 3)], 0, cut_bits]] if cut_bits else [], [(3, 3)])
    bits = random_bitstrings(n, 16, 5)
    p = Plan(ctx, Circuit(ctx, c.to_text()), plan, precision, batch=batch)
    nodes = [(s["a_node"], s["a_reordered"]) for s in p.steps()] + [(s["b_node"], s["b_reordered"]) for s in p.steps()]
    assert any(node >= 16 and reordered for node, reordered in nodes)
    got = p.amplitudes(bits)
    torch.cuda.synchronize()
    assert rel_err(got.cpu().numpy(), sv.open_amplitudes(c.to_text(), bits, plan["open"])) <= {"fp32": 1e-5, "bf16x3": 1e-4}[precision]


def test_batched_tail_and_slice_subrange(ctx):
    """Chains that do not fill the last group are masked; slice sub-ranges compose.  Group
    hoisting puts each bitstring's slices in groups of their own (7 slices of 3 bitstrings in
    groups of 8: one partly idle group per bitstring)."""
    import torch
    from paper_1905_00444_amd import Circuit, Plan
    _say("batched tail")
    c, plan = _setup_4x5()
    bits = random_bitstrings(3, 20, 6)
    circ = Circuit(ctx, c.to_text())
    seq = Plan(ctx, circ, plan, "fp32", hoist=False).amplitudes(bits, 3, 10)  # 21 chains
    bat = Plan(ctx, circ, plan, "fp32", batch=8, hoist=False).amplitudes(bits, 3, 10)
    hst = Plan(ctx, circ, plan, "fp32", batch=8).amplitudes(bits, 3, 10)
    torch.cuda.synchronize()
    assert np.array_equal(seq.cpu().numpy(), bat.cpu().numpy())
    assert rel_err(hst.cpu().numpy(), seq.cpu().numpy()) <= 2e-6
    ref = sv.open_amplitudes(c.to_text(), bits, plan["open"])
    full = Plan(ctx, circ, plan, "fp32", batch=8)
    parts = full.amplitudes(bits, 0, 5)
    full.amplitudes(bits, 5, 16, out=parts)
    whole = full.amplitudes(bits)
    torch.cuda.synchronize()
    assert rel_err(whole.cpu().numpy(), ref) <= 1e-5
    assert rel_err(parts.cpu().numpy(), whole.cpu().numpy()) <= 2e-6


def test_graph_replays_match_eager(gctx):
    import torch
    from paper_1905_00444_amd import Circuit, Plan
    _say("graph replay")
    c, plan = _setup_4x5()
    bits = random_bitstrings(4, 20, 7)
    circ = Circuit(gctx, c.to_text())
    eager = Plan(gctx, circ, plan, "bf16x3", batch=4)
    graph = Plan(gctx, circ, plan, "bf16x3", batch=4, graph=True)
    ref = eager.amplitudes(bits)
    gctx.synchronize()
    ref = ref.cpu().numpy()
    bits_t = torch.from_numpy(bits).to(gctx.device)
    with torch.cuda.stream(gctx.stream):
        out = torch.zeros((4, 4), dtype=torch.complex128, device=gctx.device)
    n_chains = 4 * graph.info()["n_slices"]
    assert n_chains // 4 >= 8  # several groups of 4 chains per call
    for rep in range(4):
        with torch.cuda.stream(gctx.stream):
            out.zero_()
        graph.amplitudes(bits_t, out=out)  # same pointers every time: the captured graph is replayed
        gctx.synchronize()
        assert np.array_equal(out.cpu().numpy(), ref), rep
        # the whole call, every group of 4 chains, is one graph launch
        launches, nodes = graph.graph_info()
        assert launches == rep + 1
        assert nodes > n_chains // 4
        # eager work between replays
        eager.amplitudes(bits)
        gctx.synchronize()


def _product_slice(circ, plan, bits_row, s):
    from oracle import gates
    total = sum(x[3] for x in plan["cuts"])
    fixed = {}
    off = total
    for q0, q1, lo, nb in plan["cuts"]:
        off -= nb
        v = (s >> off) & ((1 << nb) - 1)
        for i in range(nb):
            fixed[(q0, q1, lo + i)] = (v >> (nb - 1 - i)) & 1
    vecs = [np.array([1, 0], dtype=np.complex128) for _ in range(circ.n_qubits)]
    seen = {}
    for op in circ.ops:
        if len(op.qubits) == 1:
            vecs[op.qubits[0]] = gates.one_qubit(op.name) @ vecs[op.qubits[0]]
        else:
            j = seen.get(op.qubits, 0)
            seen[op.qubits] = j + 1
            if op.qubits + (j,) in fixed:
                q0 = op.qubits[0]
                vecs[q0] = vecs[q0] * (np.arange(2) == fixed[op.qubits + (j,)])
    return np.prod([vecs[q][bits_row[q]] for q in range(circ.n_qubits)])


def _clifford_batch(base, plan, n, seed):
    """Clifford product circuit (CZ -> identity, T -> S) and n bitstrings with nonzero slice-0
    amplitudes: the larger component of every qubit, then random flips of the qubits whose two
    components are equal in magnitude (see the 7x7 product test for why split-BF16 needs it)."""
    from test_gpu_amplitudes import _product_vectors
    from workloads.circuits import clifford_substitute
    c = clifford_substitute(identity_cz(base))
    vecs = _product_vectors(c, plan, 0)
    first = np.array([int(np.argmax(np.abs(v))) for v in vecs], dtype=np.uint8)
    cut_q = {q for cut in plan["cuts"] for q in cut[:2]}
    free = [q for q, v in enumerate(vecs) if q not in cut_q and abs(abs(v[0]) - abs(v[1])) < 1e-12]
    rng = np.random.default_rng(seed)
    bits = np.tile(first, (n, 1))
    for b in range(1, n):
        bits[b, free] ^= rng.integers(0, 2, len(free)).astype(np.uint8)
    return c, bits


@pytest.mark.parametrize("precision", ["fp32", "bf16x3"])
def test_70_qubit_product_circuit_batched_graph(gctx, precision):
    """8x9 minus two corners, (1+24+1), every CZ -> identity: each chain has a closed form.
    16 bitstrings x slices 0..7 run as 128 chains, 32 per launch, through the captured graph.
    Split-BF16 runs the Clifford variant."""
    import torch
    from paper_1905_00444_amd import Circuit, Plan
    _say(f"70 qubits product circuit {precision}")
    base = generate(8, 9, 24, 0, C5_REMOVED)
    plan, _ = plan_8x9(base)
    if precision == "bf16x3":
        c, bits = _clifford_batch(base, plan, 16, 1)
    else:
        c = identity_cz(base)
        bits = random_bitstrings(16, 70, 1)
    p = Plan(gctx, Circuit(gctx, c.to_text()), plan, precision, batch=32, graph=True)
    got = p.amplitudes(bits, 0, 8)
    gctx.synchronize()
    ref = np.array([sum(_product_slice(c, plan, bits[b], s) for s in range(8)) for b in range(16)])
    assert np.count_nonzero(ref) >= 8
    assert rel_err(got.cpu().numpy()[:, 0], ref) <= (1e-5 if precision == "fp32" else 1e-4)


def test_70_qubit_random_circuit_batched_vs_oracle_one_chain(gctx):
    """One chain (bitstring 0, slice 5) of the random 70-qubit circuit against the FP64
    tensor-network oracle, through the batched graph path."""
    import torch
    from oracle import tn
    from paper_1905_00444_amd import Circuit, Plan
    _say("70 qubits random, one chain vs oracle")
    c = generate(8, 9, 24, 0, C5_REMOVED)
    plan, _ = plan_8x9(c)
    bits = random_bitstrings(1, 70, 1)
    p = Plan(gctx, Circuit(gctx, c.to_text()), plan, "fp32", batch=2, graph=True)
    got = p.amplitudes(bits, 5, 6)
    gctx.synchronize()
    ref = tn.amplitudes(c.to_text(), bits, plan, slices=[5])
    assert rel_err(got.cpu().numpy(), ref) <= 1e-5


@pytest.mark.parametrize("precision", ["fp32", "bf16x3"])
@pytest.mark.parametrize("cuts", [False, True])
def test_chains_of_one_call_keep_scales_of_their_own(precision, cuts):
    """Four qubits whose bit 1 is weighed by 1e-12: bitstrings with these bits set have amplitudes below FP32's range
    beside those without, in the same call.  The same bits as one call per bitstring, and weighed by
    1e-48 against the plain circuit (20 qubits, the plan tests' bounds)."""
    import torch
    from paper_1905_00444_amd import Context, Circuit, Plan
    _say(f"scales of chains {precision} cuts {cuts}")
    c, plan = _setup_4x5()
    if not cuts:
        c = generate(4, 5, 24, 2)
        plan, _ = region_plan(c, 2, 2, [], [(3, 4), (2, 4)])
    heavy = [q for q in (0, 6, 11, 17) if q not in plan["open"]]
    assert len(heavy) == 4
    bits = random_bitstrings(6, 20, 8)
    bits[:3, heavy] = 0
    bits[3:, heavy] = 1
    ctx = Context(0)
    circ = Circuit(ctx, c.to_text())
    p = Plan(ctx, circ, plan, precision)
    plain = p.amplitudes(bits)
    values = circ.values.copy()
    for q in heavy:
        last = max(i for i, op in enumerate(circ.ops) if op[2] == (q,))
        values[last, 2:] *= np.complex64(1e-12)
    circ.set_values(values)
    one = [p.amplitudes(bits[i:i + 1]) for i in range(6)]
    all_ = p.amplitudes(bits)
    torch.cuda.synchronize()
    plain, one, all_ = plain.cpu().numpy(), torch.cat(one).cpu().numpy(), all_.cpu().numpy()
    bound = 1e-5 if precision == "fp32" else 1e-4
    assert rel_err(one[:3], plain[:3]) <= bound
    assert rel_err(one[3:] * 1e48, plain[3:]) <= bound
    assert np.array_equal(all_, one)


@pytest.mark.parametrize("n,rng", [(3, (0, 1)), (67, (0, 1)), (2, (0, 11)), (1, (2, 7))])
def test_calls_run_the_chains_they_have(n, rng):
    """The flops of the largest products that a call of several chains launches: those of its chains, as one at a
    time (three chains, or 67 in launches of 64, ran as four and as 128)."""
    import torch
    from paper_1905_00444_amd import Context, Circuit, Plan, profile_enable, profile_read
    _say(f"chains run by a call n {n} slices {rng}")
    c, plan = _setup_4x5()
    if rng[1] - rng[0] == 1:
        c = generate(4, 5, 24, 2)
        plan, _ = region_plan(c, 2, 2, [], [(3, 4), (2, 4)])
    bits = random_bitstrings(n, 20, 8)
    ctx = Context(0)
    p = Plan(ctx, Circuit(ctx, c.to_text()), plan, "fp32")
    largest = [s for s in p.steps() if s["flops"] == max(x["flops"] for x in p.steps())]
    profile_enable(ctx)
    p.amplitudes(bits, *rng)
    torch.cuda.synchronize()
    _, _, flops = profile_read(ctx)
    profile_enable(ctx, False)
    chains = n * (rng[1] - rng[0])
    assert flops <= chains * sum(s["flops"] for s in largest)
    assert flops >= sum(s["flops"] for s in largest)
