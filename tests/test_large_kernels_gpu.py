"""The kernels that serve large vectors and plans by default (compile-time and
stream kernels, LARS norms and update over a plan's pieces) at the sizes, options
and values of the other tests, which the split kernels serve by default: two
passes per workgroup select them. And what only larger sizes reach: four-unit
stream tiles (a round of them more than half full, 129 to 256 tiles), the forms
of the means, and plans of many small tensors."""
import numpy as np
import pytest
import torch

import oracle
import test_lars_gpu as lars
import test_parity_gpu as parity
import test_randomized_gpu as randomized
import test_split_gpu as split
import workloads

pytestmark = pytest.mark.gpu

if torch.cuda.device_count() > 0:
    import paper_1906_05936_amd as lsgd
else:
    lsgd = None

TILE = 4096


@pytest.fixture
def two_passes():
    with split.passes_per_workgroup(2):
        yield


@pytest.mark.parametrize("k", range(96))
def test_random_case(two_passes, k):
    randomized.test_random_case_matches_oracle(k)


@pytest.mark.parametrize("case", [c for c in parity.LITERAL_CASES if c[3] < 1 << 19], ids=lambda c: "%s-%s-%d-%s" % (c[1], c[2], c[3], c[5]))
def test_literal_reduction(two_passes, case):
    parity.test_literal_reduction_matches_oracle(*case)


@pytest.mark.parametrize("gdt", ["f32", "bf16"])
def test_range_extremes(two_passes, gdt):
    """The compile-time kernels, flat and plan."""
    parity.test_literal_power_of_two_groups_at_range_extremes(gdt)


@pytest.mark.parametrize("sizes,literal", [([9], False), ([3] * 20, True), ([2, 3, 5, 6], True)])
@pytest.mark.parametrize("gdt", ["f32", "bf16"])
def test_range_extremes_stream(two_passes, sizes, literal, gdt):
    """Subnormal, near-overflow and non-finite sums in the stream kernels."""
    n, G = 9_003, len(sizes)
    rng = np.random.default_rng(G)
    gow = [j for j, c in enumerate(sizes) for _ in range(c)]
    gh = parity.extreme_grads(rng, n, len(gow), gdt)
    ph = (rng.standard_normal(n) * 0.05).astype(np.float32)
    mh = np.zeros(n, np.float32)
    p, m = parity.to_dev(ph), torch.zeros(n, device=parity.DEV)
    lsgd.step(p, m, [parity.to_dev(x) for x in gh], gow, G, 0.5, 0.0, 0.0, reduction="literal" if literal else "mean_of_means")
    if literal:
        oracle.lsgd_step_literal(ph, mh, [x.copy() for x in gh], gow, G, 0.5, 0.0, 0.0, [])
    else:
        oracle.lsgd_step(ph, mh, gh, gow, G, 0.5, 0.0, 0.0)
    parity.assert_close(parity.to_host(p), ph, "params")
    parity.assert_close(parity.to_host(m), mh, "momentum")


@pytest.mark.parametrize("G,W", [(4, 4), (3, 5), (2, 16), (10, 4), (1, 9)])
def test_broadcast_with_mean_of_means(two_passes, G, W):
    parity.test_gradient_broadcast_with_mean_of_means(G, W)


@pytest.mark.parametrize("case", [(4, 4, "f32", 33, "f32", 100_003), (2, 2, "bf16", 9, "bf16", 77_777), (8, 8, "f32", 3, "f32", 65_539),
                                  (3, 5, "f32", 20, "bf16", 4_099), (10, 4, "f32", 7, "f32", 30_001), (1, 11, "bf16", 5, "f32", 30_001)])
def test_copy_out_modes(two_passes, case):
    parity.test_copy_out_pass_matches_oracle_in_every_mode(*case)


PLAN_LITERAL = [([0, 0, 1, 1, 1, 2, 2, 2, 2, 2, 3, 3, 3, 3, 3, 3], 4, "f32", 3, False), ([2, 0, 1, 1, 0, 2, 1], 3, "bf16", 2, False),
                ([0, 0, 1, 1, 1, 2, 2, 2, 2, 2, 3, 3, 3, 3, 3, 3], 4, "f32", 1, True), ([0, 1] * 8, 2, "f32", 16, True),
                (list(range(5)), 5, "bf16", 1, False), (list(range(9)), 9, "f32", 2, True)]


@pytest.mark.parametrize("case", PLAN_LITERAL, ids=lambda c: "%dx-%s-%s" % (c[1], c[2], c[4]))
def test_plan_literal_and_broadcast(two_passes, case):
    parity.test_plan_literal_reduction_and_broadcast_match_oracle(*case)


@pytest.mark.parametrize("gdt,G,W,R,rdt", [("f32", 2, 2, 1, "f32"), ("bf16", 4, 4, 2, "bf16"), ("f32", 3, 5, 1, "f32"), ("f32", 8, 4, 2, "f32"),
                                           ("bf16", 10, 4, 1, "f32"), ("f32", 1, 9, 1, "bf16")])
def test_every_tail_size_flat(two_passes, gdt, G, W, R, rdt):
    parity.test_every_tail_size_flat(gdt, G, W, R, rdt)


@pytest.mark.parametrize("gdt,G,W", [("f32", 2, 4), ("bf16", 2, 4), ("f32", 8, 4), ("bf16", 10, 4), ("f32", 9, 1)])
def test_every_tail_size_as_plan_tensors(two_passes, gdt, G, W):
    parity.test_every_tail_size_as_plan_tensors(gdt, G, W)


@pytest.mark.parametrize("G,W,gdt,R,rdt", [(10, 4, "f32", 2, "f32"), (9, 3, "f32", 1, "bf16"), (1, 11, "f32", 0, "f32"), (9, 1, "f32", 1, "f32"),
                                           (10, 4, "bf16", 2, "bf16"), (8, 8, "f32", 1, "f32")])
def test_lars_plan(two_passes, G, W, gdt, R, rdt):
    """The LARS norms stream kernel for both types, and the compile-time one in
    four-unit tiles."""
    lars.test_lars_plan_matches_oracle(G, W, gdt, R, rdt)


@pytest.mark.parametrize("mode", [0, 1])
@pytest.mark.parametrize("sizes", [[4] * 10, [2, 3, 5, 6], [9]])
def test_stream_broadcast_tile_edges(two_passes, sizes, mode):
    """The gradient broadcast in the stream kernels: lanes past the end read
    units that other lanes overwrite, and store nothing."""
    lsgd.set_copy_out_mode(mode)
    try:
        for n in (1, 3, 7, 8, 2047, 2048, 2049, 4096 + 5, 3 * 2048 - 4):
            split.step_against_oracle(sizes, "f32", n, 2, "f32", literal=True, bcast=True)
        parity.test_plan_literal_reduction_and_broadcast_match_oracle([j for j, c in enumerate(sizes) for _ in range(c)], len(sizes), "f32", 1, True)
    finally:
        lsgd.set_copy_out_mode(lsgd.COPY_OUT_AUTO)


# 131 tiles of 4096 elements: more than half of a round, so four units per lane
@pytest.mark.parametrize("extra", [1, 4, TILE - 4, TILE - 1])
@pytest.mark.parametrize("sizes,literal,bcast", [([4] * 5, False, False), ([3] * 6, True, True), ([2, 3, 5, 9], True, False)])
def test_four_unit_tiles(sizes, literal, bcast, extra):
    split.step_against_oracle(sizes, "f32", 131 * TILE + extra, 2, "f32", literal, bcast)


def test_four_unit_plan_pieces_match_flat():
    """Plan pieces of 4096 elements, their copies over 2048: the flat step's bits."""
    sizes = [TILE * 140 + 4, 20_000, 36, TILE * 2]
    gow, G, R = [w // 4 for w in range(20)], 5, 3
    gen = torch.Generator(device=parity.DEV)
    gen.manual_seed(5)
    new = lambda s, k: torch.randn(s, device=parity.DEV, generator=gen) * k
    p, m = [new(s, 0.05) for s in sizes], [new(s, 0.01) for s in sizes]
    g = [[new(s, 0.01) for s in sizes] for _ in gow]
    want = []
    for t, s in enumerate(sizes):
        a, b, r = p[t].clone(), m[t].clone(), torch.zeros(s, device=parity.DEV)
        lsgd.step(a, b, [row[t] for row in g], gow, G, 0.1, 0.9, 1e-4, [r])
        want.append((a, b, r))
    for mode in (lsgd.COPY_OUT_FUSED, lsgd.COPY_OUT_SEPARATE):
        pp, mm = [x.clone() for x in p], [x.clone() for x in m]
        reps = [[torch.zeros(s, device=parity.DEV) for s in sizes] for _ in range(R)]
        lsgd.set_copy_out_mode(mode)
        try:
            plan = lsgd.Plan(pp, mm, g, gow, G, reps)
            plan.step(0.1, 0.9, 1e-4)
            torch.cuda.synchronize()
        finally:
            lsgd.set_copy_out_mode(lsgd.COPY_OUT_AUTO)
        for t in range(len(sizes)):
            assert torch.equal(pp[t], want[t][0]) and torch.equal(mm[t], want[t][1]), (mode, t)
            assert all(torch.equal(row[t], want[t][2]) for row in reps), (mode, t)
        plan.close()


def test_deepest_stack():
    """The layout with the most partial sums waiting in LDS (9 levels, 144 KB):
    63 single workers, then a group of 65."""
    sizes = [1] * 63 + [65]
    split.step_against_oracle(sizes, "f32", 130 * TILE, 1, "f32", literal=True)
    with split.passes_per_workgroup(2):
        split.step_against_oracle(sizes, "bf16", TILE + 3, 1, "bf16", literal=True)


@pytest.mark.parametrize("W,n", [(9, (1 << 19) + 5), (40, (1 << 19) + 5), (40, (1 << 22) + 1)])
@pytest.mark.parametrize("gdt", ["f32", "bf16"])
def test_mean_forms(W, n, gdt):
    rng = np.random.default_rng(W)
    base = parity.rand_host(rng, n, 1e-2, gdt)
    gh = [np.roll(base, 977 * w) for w in range(W)]
    out = [torch.full((n,), float("nan"), device=parity.DEV)]
    lsgd.group_mean([parity.to_dev(g) for g in gh], [0] * W, 1, out)
    torch.cuda.synchronize()
    assert np.array_equal(parity.to_host(out[0]), oracle.group_means(gh, [0] * W, 1)[0])


@pytest.mark.parametrize("G,W,gdt,R,rdt,each,T", [(10, 4, "f32", 3, "f32", 203, 5_400), (2, 2, "f32", 5, "f32", 601, 1_900),
                                                  (2, 2, "bf16", 5, "bf16", 602, 1_900), (3, 3, "bf16", 0, "f32", 5, 220_000),
                                                  (10, 4, "f32", 2, "bf16", 1_501, 800)])
def test_plan_of_small_tensors(G, W, gdt, R, rdt, each, T):
    """Plans beyond the split kernels' sizes whose tensors leave most of a piece
    empty (split kernels, a copy pass of several replicas per workgroup) or end
    ragged (two-unit stream tiles): step and LARS against the oracle's step over
    all tensors as one vector, and per tensor."""
    rng = np.random.default_rng(T)
    n, N = each * T, G * W
    gow = workloads.shuffled_groups(G, W, 3)
    base = parity.rand_host(rng, n, 1e-2, gdt)
    gh = [np.roll(base, 1_009 * w) for w in range(N)]
    ph = (rng.standard_normal(n) * 0.05).astype(np.float32)
    mh = np.zeros(n, np.float32)
    step = -(-each // 8) * 8          # every tensor on a 16-byte boundary

    def padded(x):
        t = parity.to_dev(x).view(T, each)
        out = torch.zeros((T, step), device=parity.DEV, dtype=t.dtype)
        out[:, :each] = t
        return out

    rows = lambda x: [x[t, :each] for t in range(T)]
    p, m, g = padded(ph), padded(mh), [padded(x) for x in gh]
    rtd = torch.bfloat16 if rdt == "bf16" else torch.float32
    reps = [torch.zeros((T, step), device=parity.DEV, dtype=rtd) for _ in range(R)]
    plan = lsgd.Plan(rows(p), rows(m), [rows(x) for x in g], gow, G, [rows(x) for x in reps])
    plan.step(0.1, 0.9, 1e-4)
    torch.cuda.synchronize()
    rr = [np.zeros(n, np.uint16 if rdt == "bf16" else np.float32) for _ in range(R)]
    oracle.lsgd_step(ph, mh, gh, gow, G, 0.1, 0.9, 1e-4, rr, oracle.BF16 if rdt == "bf16" else oracle.F32)
    flat = lambda x: parity.to_host(x[:, :each].reshape(-1))
    assert np.array_equal(flat(p), ph) and np.array_equal(flat(m), mh)
    for r in range(R):
        assert np.array_equal(flat(reps[r]), rr[r]), r
    assert all(not x[:, each:].any() for x in [p, m] + reps)
    trust = torch.zeros(T, device=parity.DEV)
    plan.lars_step(0.1, 0.9, 1e-4, 1e-3, trust_out=trust)
    torch.cuda.synchronize()
    tg, pg = parity.to_host(trust), flat(p)
    for t in list(range(0, T, max(1, T // 40))) + [T - 1]:
        sl = slice(t * each, (t + 1) * each)
        p1, m1 = ph[sl].copy(), mh[sl].copy()
        tr = oracle.lars_step(p1, m1, [x[sl] for x in gh], gow, G, 0.1, 0.9, 1e-4, 1e-3)
        assert lars.ulps(tg[t], tr) <= 1, (t, tg[t], tr)
        if np.float32(tg[t]) == np.float32(tr):
            assert np.array_equal(pg[sl], p1), t
            for r in range(R):
                want = oracle.f32_to_bf16(p1) if rdt == "bf16" else p1
                assert np.array_equal(parity.to_host(reps[r][t, :each]), want), (t, r)
    plan.close()
