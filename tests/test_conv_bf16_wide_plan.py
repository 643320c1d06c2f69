"""How layers share a launch of wide tiles (csrc/conv_bf16_wide_plan.h), compiled for the host: where there is a plan, every layer and the pooling step have
workgroups and all of them together fit the compute units; where these do not suffice for a workgroup per filter block, there is none."""
import os
import random
import subprocess

import pytest

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_1708_04728_amd", "csrc")

PROGRAM = r"""
#include <cstdio>
#include "conv_bf16_wide_plan.h"
int main()
{
    int cus, pool, n;
    while (scanf("%d %d %d", &cus, &pool, &n) == 3) {
        dr::WideLayer l[dr::WIDE_LAYERS];
        for (int i = 0; i < n; ++i)
            if (scanf("%d %d %d", &l[i].K, &l[i].Ng, &l[i].slices) != 3) return 1;
        dr::WidePlan p{};
        const bool found = dr::wide_plan(l, n, pool, cus, &p);
        printf("%d %d", found, p.pool_share);
        for (int i = 0; i < n; ++i) printf(" %d %d %d", dr::WIDE_TILES[p.tile[i]][0], dr::WIDE_TILES[p.tile[i]][1], p.gn[i]);
        printf("\n");
    }
}
"""


@pytest.fixture(scope="module")
def plans(tmp_path_factory):
    d = tmp_path_factory.mktemp("wide_plan")
    (d / "plan.cpp").write_text(PROGRAM)
    subprocess.check_call(["g++", "-std=c++17", "-O1", "-fsanitize=undefined", "-fno-sanitize-recover=undefined", "-I", CSRC, str(d / "plan.cpp"), "-o", str(d / "plan")])

    def ask(cases):
        """cases: (compute units, groups of pooling items, layers (K, Ng, slices))"""
        text = "\n".join("%d %d %d " % (cus, pool, len(ls)) + " ".join("%d %d %d" % v for v in ls) for cus, pool, ls in cases)
        out = subprocess.run([str(d / "plan")], input=text, capture_output=True, text=True, check=True, timeout=60).stdout.splitlines()
        assert len(out) == len(cases)
        return [[int(v) for v in line.split()] for line in out]
    return ask


def eights(v):
    return -(-v // 8) * 8


def fewest(pool, layers):
    """Workgroups that the layers take at least: one per block of 224 filters, in whole eights."""
    return (8 if pool else 0) + sum(eights(-(-K // 224)) for K, _, _ in layers)


def check(case, plan):
    cus, pool, layers = case
    found, share, *per = plan
    assert bool(found) == (fewest(pool, layers) <= cus), case
    if not found:
        return
    total = share
    assert share % 8 == 0 and (0 < share <= eights(pool) if pool else share == 0), case
    for i, (K, Ng, _) in enumerate(layers):
        tm, tn, gn = per[3 * i:3 * i + 3]
        assert 1 <= gn <= -(-Ng // (32 * tn)), (case, plan)
        total += eights(gn * -(-K // (32 * tm)))
    assert total <= cus, (case, plan)


@pytest.mark.parametrize("cus,pool,layers", [
    (256, 0, [(28600, 196, 1)] * 2),
    (256, 0, [(28700, 196, 1)] * 2),              # 129 blocks, 136 workgroups, each
    (256, 0, [(28700, 49, 1)] * 2),               # ... on one pixel tile
    (256, 0, [(30000, 196, 1)] * 2),
    (256, 0, [(20000, 3000, 4)] * 3),
    (256, 0, [(14400, 3000, 4)] * 4),
    (256, 0, [(14336, 3000, 4)] * 4),             # 64 blocks each: all of the compute units
    (256, 5, [(57400, 49, 1)]),                   # a single one beside a pooling step
    (256, 5, [(55552, 49, 1)]),                   # 248 blocks and a workgroup for each of the five groups
    (256, 0, [(1 << 20, 49, 1)]),
    (32, 7, [(64, 784, 8)] * 4),                  # four layers and a pooling step on few compute units
    (32, 0, [(64, 784, 8)] * 4),
    (8, 0, [(64, 784, 8)]),
])
def test_at_the_line(plans, cus, pool, layers):
    check((cus, pool, layers), plans([(cus, pool, layers)])[0])


def test_drawn_layers(plans):
    rng, cases = random.Random(8), []
    log = lambda lo, hi: int(lo * (hi / lo) ** rng.random())
    for _ in range(2000):
        layers = [(8 * log(1, 6000), log(1, 1 << 23), log(1, 128)) for _ in range(rng.randint(1, 4))]
        cases.append((rng.choice((256, 256, 256, 304, 64, 32)), rng.choice((0, 0, 1, log(2, 448))), layers))
    got = plans(cases)
    for case, plan in zip(cases, got):
        check(case, plan)
    assert 200 < sum(not p[0] for p in got) < 1000
