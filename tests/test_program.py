"""The reduction programs of lsgd_program.hpp (host C++, no GPU): both forms of
a program, the additions by tree level and the stack of partial sums, are
evaluated symbolically and must be the two-level pairwise mean, addition for
addition and division for division, for every equal grouping of up to 128
workers in both reductions and for random partitions. Additions of one level
touch no common slot (the kernel runs them without a barrier between)."""
import os
import random
import subprocess

import pytest

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_1906_05936_amd", "csrc")

MAX_STACK = 9   # kMaxStack: a lane's partial sums in LDS, 16 KB a level

DUMP = r"""
#include <cstdio>
#include <vector>
#include "lsgd_program.hpp"
int main() {
    int literal, G;
    while (std::scanf("%d %d", &literal, &G) == 2) {
        std::vector<int32_t> start(G + 1, 0);
        for (int j = 0; j < G; ++j) { int s; if (std::scanf("%d", &s) != 1) return 1; start[j + 1] = start[j] + s; }
        static lsgd::Program p;
        lsgd::build_program(G, start.data(), literal != 0, p);
        std::printf("%d %d %d %g %g %g", p.n_batches, p.n_levels, p.stack_depth, p.group_div, p.group_scale, p.total_div);
        for (int i = 0; i < p.n_batches; ++i) {
            const lsgd::Batch& b = p.batch[i];
            std::printf(" %d %d %d %d %d %d", b.first, b.count, b.sub, b.pre, b.post, b.div);
        }
        int at = 0;
        for (int l = 0; l < p.n_levels; ++l) {
            std::printf(" %d", p.level_end[l] - at);
            for (; at < p.level_end[l]; ++at) std::printf(" %d %d %d", p.op[at].dst, p.op[at].src, p.op[at].div);
        }
        std::printf("\n");
    }
    return 0;
}
"""


def pw(x):
    if len(x) == 1:
        return x[0]
    h = 1
    while 2 * h < len(x):
        h *= 2
    return (pw(x[:h]), pw(x[h:]))


def over(x, d):
    return x if d == 1 else (x, "/", int(d))   # x / 1 is x


def reference(sizes, literal):
    n, at, means = sum(sizes), 0, []
    for s in sizes:
        means.append(over(pw(list(range(at, at + s))), n if literal else s))
        at += s
    return pw(means) if literal else over(pw(means), len(sizes))


def check(sizes, literal, line):
    f = line.split()
    nb, levels, depth = (int(x) for x in f[:3])
    div, scale, total = (float(x) for x in f[3:6])
    assert scale in (0.0, 1.0 / div) and (scale != 0.0) == (int(div) & (int(div) - 1) == 0)
    f = [int(x) for x in f[6:]]
    batches = [f[6 * i:6 * i + 6] for i in range(nb)]
    f = f[6 * nb:]

    def batch_sum(first, count, sub):
        m = list(range(first, first + count))
        if sub == 0:
            return pw(m)
        assert count % sub == 0
        return pw([over(pw(m[k:k + sub]), div) for k in range(0, count, sub)])

    assert [m for b in batches for m in range(b[0], b[0] + b[1])] == list(range(sum(sizes)))
    # the tree form
    slots = []
    for first, count, sub, pre, post, d in batches:
        x = batch_sum(first, count, sub)
        slots.append(over(x, div) if d and pre == 0 else x)
    for _ in range(levels):
        k, f = f[0], f[1:]
        used = []
        for _ in range(k):
            dst, src, d = f[:3]
            f = f[3:]
            used += [dst, src]
            slots[dst] = (slots[dst], slots[src])
            if d:
                slots[dst] = over(slots[dst], div)
        assert len(used) == len(set(used))
    assert f == []
    want = reference(sizes, literal)
    assert over(slots[0], total) == want
    # the stack form
    stack, most = [], 0
    for first, count, sub, pre, post, d in batches:
        x = batch_sum(first, count, sub)
        for _ in range(pre):
            x = (stack.pop(), x)
        if d:
            x = over(x, div)
        for _ in range(post):
            x = (stack.pop(), x)
        stack.append(x)
        most = max(most, len(stack))
    assert len(stack) == 1 and most == depth <= MAX_STACK
    assert over(stack[0], total) == want


@pytest.fixture(scope="module")
def dump(tmp_path_factory):
    d = tmp_path_factory.mktemp("program")
    (d / "dump.cpp").write_text(DUMP)
    exe = str(d / "dump")
    subprocess.run(["g++", "-std=c++17", "-O1", "-Wall", "-Werror", "-I" + CSRC, str(d / "dump.cpp"), "-o", exe], check=True)

    def run(layouts):
        text = "\n".join("%d %d %s" % (lit, len(s), " ".join(map(str, s))) for s, lit in layouts)
        r = subprocess.run([exe], input=text, capture_output=True, text=True, check=True)
        return r.stdout.splitlines()

    return run


def test_every_equal_grouping(dump):
    layouts = [([w] * g, lit) for g in range(1, 129) for w in range(1, 128 // g + 1) for lit in (False, True)]
    lines = dump(layouts)
    assert len(lines) == len(layouts)
    for (sizes, lit), line in zip(layouts, lines):
        check(sizes, lit, line)


def test_random_partitions(dump):
    rng = random.Random(1906)
    layouts = []
    for _ in range(3000):
        sizes = [1] * rng.randint(1, 128)
        for _ in range(rng.randint(0, 128 - len(sizes))):
            sizes[rng.randrange(len(sizes))] += 1
        layouts.append((sizes, True))
    for (sizes, lit), line in zip(layouts, dump(layouts)):
        check(sizes, lit, line)


def test_deepest_stacks(dump):
    """A group of every size after every count of single workers that fits (the
    partial sums of the groups before wait while a group's own pile up)."""
    layouts = [([1] * k + [s], True) for k in range(1, 128) for s in range(1, 129 - k)]
    depths = [int(line.split()[2]) for line in dump(layouts)]
    assert max(depths) == MAX_STACK
    for (sizes, lit), d, line in zip(layouts, depths, dump(layouts)):
        if d == MAX_STACK:
            check(sizes, lit, line)
