"""The stream kernels (group layouts and input counts without a compile-time
kernel) against the oracle, bit for bit, at the edges of their tiles of 4096
elements: one element, less than a unit, a ragged end alone and after a whole
tile, the last unit repeated by the lanes past the end. Group and global means
also at the counts on both sides of the compile-time ones."""
import numpy as np
import pytest
import torch

import oracle
import test_parity_gpu as parity
import test_split_gpu as split

pytestmark = pytest.mark.gpu

if torch.cuda.device_count() > 0:
    import paper_1906_05936_amd as lsgd
else:
    lsgd = None

TILE = 4096
EDGES = [1, 3, 7, 8, TILE - 1, TILE, TILE + 1, 2 * TILE + 8, 3 * TILE - 4]


@pytest.mark.parametrize("n", EDGES)
@pytest.mark.parametrize("sizes,gdt,literal", [([4] * 10, "f32", False), ([4] * 10, "bf16", True), ([2, 3, 5, 6], "bf16", True),
                                               ([17], "f32", False), ([3] * 20, "bf16", False)])
def test_step_tile_edges(n, sizes, gdt, literal):
    with split.passes_per_workgroup(2):   # past the split kernels, which serve small sizes by default
        split.step_against_oracle(sizes, gdt, n, 3, "f32", literal)
        split.step_against_oracle(sizes, gdt, n, 1, "bf16", literal)


@pytest.mark.parametrize("G,W", [(1, 1), (1, 3), (3, 8), (2, 9), (9, 1), (12, 5), (10, 12), (2, 16), (7, 17), (128, 1), (1, 128)])
@pytest.mark.parametrize("gdt", ["f32", "bf16"])
def test_means(G, W, gdt):
    for n in (1, 7, TILE - 1, TILE + 1, 2 * TILE):
        rng = np.random.default_rng([G, W, n])
        gow = [j for j in range(G) for _ in range(W)]
        rng.shuffle(gow)
        gh = [parity.rand_host(rng, n, 1e-2, gdt) for _ in gow]
        means = [torch.full((n,), float("nan"), device=parity.DEV) for _ in range(G)]
        mean = torch.full((n,), float("nan"), device=parity.DEV)
        lsgd.group_mean([parity.to_dev(g) for g in gh], gow, G, means)
        lsgd.global_mean(means, mean)
        torch.cuda.synchronize()
        want = oracle.group_means(gh, gow, G)
        for j in range(G):
            assert np.array_equal(parity.to_host(means[j]), want[j]), (n, j)
        assert np.array_equal(parity.to_host(mean), oracle.global_mean(want)), n
