"""The split kernels (small vectors and plans: the members of a unit divided
over the waves of a workgroup) against the oracle, at the edges of their slabs
of 256 elements, of their size rule and of their batches; and the kernels with
one lane tile per workgroup at the small sizes that the split kernels serve by
default (two passes per workgroup select them)."""
import contextlib

import numpy as np
import pytest
import torch

import oracle
import test_lars_gpu as lars
import test_parity_gpu as parity
import workloads

pytestmark = pytest.mark.gpu

if torch.cuda.device_count() > 0:
    import paper_1906_05936_amd as lsgd
else:
    lsgd = None

LIMIT = 1 << 18   # flat steps up to here take the split kernels whatever the grouping


@contextlib.contextmanager
def passes_per_workgroup(k):
    c, b, u = lsgd.get_launch_shape()
    lsgd.set_launch_shape(c, b, k)
    try:
        yield
    finally:
        lsgd.set_launch_shape(c, b, u)


def step_against_oracle(sizes, gdt, n, R, rdt, literal=False, bcast=False, seed=0):
    rng = np.random.default_rng([seed, n, len(sizes), R])
    gow = [j for j, c in enumerate(sizes) for _ in range(c)]
    rng.shuffle(gow)
    gh = [parity.rand_host(rng, n, 1e-2, gdt) for _ in gow]
    p_ref = (rng.standard_normal(n) * 0.05).astype(np.float32)
    m_ref = (rng.standard_normal(n) * 0.01).astype(np.float32)
    p, m, grads = parity.to_dev(p_ref), parity.to_dev(m_ref), [parity.to_dev(g) for g in gh]
    rtd = torch.bfloat16 if rdt == "bf16" else torch.float32
    reps = [torch.full((n,), float("nan"), device=parity.DEV, dtype=rtd) for _ in range(R)]
    lsgd.step(p, m, grads, gow, len(sizes), 0.1, 0.9, 1e-4, reps,
              reduction="literal" if literal else "mean_of_means", broadcast_grad=bcast)
    rr = [np.zeros(n, np.uint16 if rdt == "bf16" else np.float32) for _ in range(R)]
    ort = oracle.BF16 if rdt == "bf16" else oracle.F32
    gbar = None
    if literal:
        oracle.lsgd_step_literal(p_ref, m_ref, gh, gow, len(sizes), 0.1, 0.9, 1e-4, rr, ort, broadcast_grad=bcast)
    else:
        if bcast:
            gbar = oracle.global_mean(oracle.group_means(gh, gow, len(sizes)))
        oracle.lsgd_step(p_ref, m_ref, gh, gow, len(sizes), 0.1, 0.9, 1e-4, rr, ort)
    torch.cuda.synchronize()
    parity.assert_close(parity.to_host(p), p_ref, "params")
    parity.assert_close(parity.to_host(m), m_ref, "momentum")
    for r in range(R):
        assert np.array_equal(parity.to_host(reps[r]), rr[r]), r
    if bcast:
        for w in range(len(gow)):
            assert np.array_equal(parity.to_host(grads[w]), gh[w] if literal else gbar), w


# every batch form: whole groups of 1 to 4 packed with remainders, single
# batches of 5 to 8, groups of several batches with every remainder, one group
# of one member, unequal groups (and more batches than the LDS holds)
LAYOUTS = [([1] * 7, True), ([1] * 13, False), ([2] * 5, False), ([3] * 5, False), ([4] * 3, True), ([5] * 3, False),
           ([6] * 2, True), ([7], False), ([8] * 9, False), ([9] * 3, False), ([20] * 3, False), ([43] * 2, True),
           ([1], False), ([2, 3, 5, 6], True), ([17, 1, 8, 30], True), ([1] * 99 + [2], True)]


@pytest.mark.parametrize("sizes,literal", LAYOUTS)
@pytest.mark.parametrize("gdt", ["f32", "bf16"])
def test_batch_forms(sizes, literal, gdt):
    for n, R in ((1, 1), (259, 3), (1027, 0)):
        step_against_oracle(sizes, gdt, n, R, "bf16" if n == 259 else "f32", literal)


@pytest.mark.parametrize("n", [2, 3, 4, 5, 255, 256, 257, 260, 511, 4 * 256 + 3, 8 * 512 * 256 + 1])
def test_slab_edges(n):
    step_against_oracle([4] * 4, "f32", n if n < 1 << 20 else LIMIT - 1, 5, "f32")
    step_against_oracle([8] * 5, "f32", n, 2, "bf16")      # 2^20 + 1: beyond the rule for many workers
    step_against_oracle([4] * 2, "bf16", min(n, LIMIT), 9, "bf16")


@pytest.mark.parametrize("n,R", [(1003, 4), (LIMIT, 16), (LIMIT + 1, 1), (LIMIT - 1, 70)])
def test_broadcast_and_copies(n, R):
    """The broadcast and the copies in the kernel, and (70 replicas of 1 MB) in
    passes of their own."""
    step_against_oracle([4] * 4, "f32", n, R, "f32", literal=True, bcast=True)
    step_against_oracle([3] * 3, "f32", n, R, "f32", bcast=True)


def test_replayed_graph_of_split_steps_matches_eager():
    """A captured split step and LARS step, replayed with other work between,
    give the eager results each time."""
    gen = torch.Generator(device=parity.DEV)
    gen.manual_seed(3)
    sizes = [1000, 3, 257, 4096]
    new = lambda s, k: torch.randn(s, device=parity.DEV, generator=gen) * k
    p, m = [new(s, 0.05) for s in sizes], [new(s, 0.01) for s in sizes]
    g = [[new(s, 0.01) for s in sizes] for _ in range(10)]
    r = [[torch.zeros(s, device=parity.DEV) for s in sizes] for _ in range(3)]
    plan = lsgd.Plan(p, m, g, [w // 2 for w in range(10)], 5, r)
    fp, fm, fg = new(5003, 0.05), new(5003, 0.01), [new(5003, 0.01) for _ in range(10)]

    def work():
        plan.step(0.1, 0.9, 1e-4)
        plan.lars_step_noalloc(0.1, 0.9, 1e-4, 1e-3)
        lsgd.step(fp, fm, fg, [w // 2 for w in range(10)], 5, 0.1, 0.9, 1e-4)

    state = p + m + [fp, fm] + [x for row in r for x in row]
    start = [x.clone() for x in state]
    want = []
    for _ in range(4):
        work()
        torch.cuda.synchronize()
        want.append([x.clone() for x in state])
    for x, y in zip(state, start):
        x.copy_(y)
    side = torch.cuda.Stream()
    side.wait_stream(torch.cuda.current_stream())
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph, stream=side):
        work()
    for k in range(4):
        graph.replay()
        torch.cuda.synchronize()
        assert all(torch.equal(x, y) for x, y in zip(state, want[k])), k
        (fp * 2).sum().item()
    plan.close()


@pytest.mark.parametrize("case", [c for c in parity.STEP_CASES if c[3] < 1 << 20], ids=lambda c: "%dx%d-%s-%d" % c[:4])
def test_other_kernels_at_small_sizes(case):
    with passes_per_workgroup(2):
        parity.test_fused_step_matches_oracle(*case)


@pytest.mark.parametrize("G,W,gdt,R,rdt", [(4, 4, "f32", 16, "f32"), (8, 8, "bf16", 3, "bf16"), (3, 5, "f32", 1, "bf16"),
                                           (16, 8, "f32", 2, "f32"), (20, 3, "bf16", 0, "f32"), (32, 4, "f32", 2, "f32")])
def test_other_plan_kernels_at_small_sizes(G, W, gdt, R, rdt):
    with passes_per_workgroup(2):
        parity.test_plan_matches_oracle(G, W, gdt, R, rdt)
        lars.test_lars_plan_matches_oracle(G, W, gdt, R, rdt)
