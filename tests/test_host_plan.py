"""Launch plans of the passes (host code without a GPU)."""
import os
import random
import subprocess

import pytest

from conftest import ROOT

SRC = r"""
#include <cstdio>
#include <vector>
#include "pass_plan.h"
int main()
{
    // per line: count rows_per_block rp per_cu, then across, along and room for splits per tensor
    unsigned count, rpb, rp, per_cu;
    while (std::scanf("%u %u %u %u", &count, &rpb, &rp, &per_cu) == 4) {
        std::vector<uint32_t> across(count), along(count);
        std::vector<uint64_t> most(count);
        double d_bytes = 0.0;
        for (unsigned i = 0; i < count; ++i) {
            if (std::scanf("%u %u %lu", &across[i], &along[i], &most[i]) != 3) return 1;
            d_bytes += 4.0 * across[i] * rpb * along[i] * 64.0;
        }
        std::printf("%u\n", edgc::pass_p_step(count, across.data(), along.data(), most.data(), rpb, rp, d_bytes, 256, per_cu));
    }
}
"""


DECOMPRESS = r"""
#include <cstdio>
#include "pass_plan.h"
int main()
{
    for (unsigned stages = 1; stages <= 300; ++stages)
        for (unsigned splits = 1; splits <= stages; ++splits)
            std::printf("%u %u %u %u\n", stages, splits, edgc::decompress_step(stages, splits, false),
                        edgc::decompress_step(stages, splits, true));
}
"""


@pytest.fixture(scope="module")
def plan(tmp_path_factory):
    d = tmp_path_factory.mktemp("plan")
    (d / "plan.cpp").write_text(SRC)
    subprocess.run(["g++", "-std=c++17", "-Wall", "-Werror", "-I" + os.path.join(ROOT, "paper_2511_10333_amd", "csrc"),
                    str(d / "plan.cpp"), "-o", str(d / "plan")], check=True)

    def run(groups):
        text = "\n".join(" ".join(map(str, [len(t), rpb, rp, per_cu, *[v for s in t for v in s]])) for t, rpb, rp, per_cu in groups)
        out = subprocess.run([str(d / "plan")], input=text, check=True, capture_output=True, text=True).stdout
        return [int(x) for x in out.split()]
    return run


def _cdiv(a, b):
    return -(-a // b)


def _group(shapes, rpb, rp, per_cu=0, most=1 << 40):
    return [(_cdiv(m, rpb), _cdiv(n, 64), most) for m, n in shapes], rpb, rp, per_cu


def _blocks(group, step):
    return sum(a * _cdiv(k, step) for a, k, _ in group[0])


def test_p_pass_plan_bounds(plan):
    rng = random.Random(3)
    groups = []
    for _ in range(3000):
        shapes = [(int(2 ** rng.uniform(4, 17)), int(2 ** rng.uniform(4, 16))) for _ in range(rng.randint(1, 16))]
        groups.append(_group(shapes, rng.choice([128, 128, 256]), rng.choice([32, 64, 128]), rng.choice([0, 0, 0, 1, 3])))
    for g, step in zip(groups, plan(groups)):
        tensors, rpb, rp, per_cu = g
        assert 1 <= step <= max(k for _, k, _ in tensors)
        single = sum(a for a, _, _ in tensors)              # every tensor in one split
        most = per_cu or (2 if rpb == 256 else 8)
        assert _blocks(g, step) <= max(256 * most, single), g
        if not per_cu and 8 * step < rp:
            # blocks so short that their partials weigh: at most four per CU
            assert _blocks(g, step) <= max(256 * 4, single), g


@pytest.mark.parametrize("m,n,most", [(662, 13048, 612), (1381, 9200, 792), (5003, 777, 520), (1024, 50257, 1024)])
def test_p_pass_plan_does_not_trade_partials_for_the_last_places(plan, m, n, most):
    """Shapes at which no count of blocks fills the CUs evenly: not more splits than blocks in proportion (four per CU)."""
    for rp in (32, 64, 128):
        g = _group([(m, n)], 128, rp)
        assert _blocks(g, plan([g])[0]) <= most


def test_p_pass_plan_fits_the_scratch_it_was_given(plan):
    """The partials of a context made for exactly the shape and rank hold about four blocks of 128 rows per CU: a plan with
    more splits than that would be cut back to another one than was chosen."""
    rng = random.Random(4)
    groups = []
    for _ in range(2000):
        m, n, rp = int(2 ** rng.uniform(5, 17)), int(2 ** rng.uniform(5, 17)), rng.choice([32, 64, 128])
        room = (max(m, 128 * 1024) + m) * rp // (m * rp) if rng.random() < 0.7 else rng.randint(1, 8)
        groups.append(_group([(m, n)], rng.choice([128, 256]), rp, most=room))
    for g, step in zip(groups, plan(groups)):
        (_, k, room), = g[0]
        assert _cdiv(k, step) <= room, g


def test_decompress_plan_is_the_one_asked_for(tmp_path):
    """Blocks of at most eight stages by the rule; with a count of blocks per CU asked for, its splits and no more."""
    (tmp_path / "d.cpp").write_text(DECOMPRESS)
    subprocess.run(["g++", "-std=c++17", "-Wall", "-Werror", "-I" + os.path.join(ROOT, "paper_2511_10333_amd", "csrc"),
                    str(tmp_path / "d.cpp"), "-o", str(tmp_path / "d")], check=True)
    for line in subprocess.run([str(tmp_path / "d")], check=True, capture_output=True, text=True).stdout.splitlines():
        stages, splits, rule, asked = map(int, line.split())
        assert asked == _cdiv(stages, splits) and rule == min(asked, 8)


CACHING = r"""
#include <cstdio>
#include "pass_plan.h"
int main()
{
    using edgc::Caching;
    const auto at = [](uint64_t a) { return reinterpret_cast<const void*>(a); };
    // k_pass_p by the size of its group; the kernels of the deferred form where D is to stay cached and cannot beside G
    const auto past = [](double mb, uint32_t esz, bool pairs, bool defer) { return edgc::gradient_past(mb * 1048576.0, esz, pairs, defer); };
    for (double mb : {0.001, 16.0, 40.0, 41.0, 53.0, 54.0, 63.9, 64.1, 127.9, 128.1, 170.0, 171.0, 256.0, 257.0, 4000.0}) {
        const bool want[] = {mb > 40.0, mb > 80.0 / 1.5, mb > 64.0 && mb <= 256.0, mb > 48.0 && mb <= 128.0, mb > 64.0 && mb <= 170.5};
        const bool got[] = {past(mb, 4, false, false), past(mb, 2, false, false), past(mb, 2, true, false), past(mb, 4, true, true),
                            past(mb, 2, true, true)};
        for (int i = 0; i < 5; ++i)
            if (want[i] != got[i]) return 2;
    }
    std::printf("%d %d %d %d %d\n", edgc::whole_lines(at(4096), 256), edgc::whole_lines(at(4096), 8224), edgc::whole_lines(at(4100), 256),
                edgc::whole_lines(at(4096 + 64), 128), edgc::whole_lines(at(128), 1u << 30));
    for (uint32_t count = 1; count <= 16; ++count)
        for (uint32_t past = 0; past <= count; ++past)
            for (double mb : {1.0, 40.0, 40.1})
                if (edgc::group_caching(past, count, mb * 1048576.0) !=
                    (past == count ? Caching::past : past ? Caching::by_tensor : mb <= 40.0 ? Caching::small : Caching::through))
                    return 1;
}
"""


def test_a_tensor_of_ragged_rows_does_not_decide_for_its_group(tmp_path):
    """Each tensor's rows are looked at by themselves, and only groups of one kind get one form for all."""
    (tmp_path / "c.cpp").write_text(CACHING)
    subprocess.run(["g++", "-std=c++17", "-Wall", "-Werror", "-I" + os.path.join(ROOT, "paper_2511_10333_amd", "csrc"),
                    str(tmp_path / "c.cpp"), "-o", str(tmp_path / "c")], check=True)
    out = subprocess.run([str(tmp_path / "c")], check=True, capture_output=True, text=True).stdout
    assert out.split() == ["1", "0", "0", "0", "1"]
