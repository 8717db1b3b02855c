"""The plan that cuts an attention launch over its keys (csrc/attention_plan.h), built for the CPU: the parts never take
more than the memory they are given, every part is long enough for its first key to be visible to its whole query tile,
and the launches that the GPU tests of the cut form use are in fact cut."""
import os
import resource
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
PART_BUDGET = 256 << 20


@pytest.fixture(scope="module")
def plan(tmp_path_factory):
    cxx = shutil.which("g++") or shutil.which("c++")
    if cxx is None:
        pytest.skip("no host C++ compiler")
    exe = str(tmp_path_factory.mktemp("plan") / "dump")
    subprocess.run([cxx, "-std=c++17", "-O2", os.path.join(ROOT, "tests", "host", "attention_plan_dump.cpp"), "-o", exe], check=True)

    def run(launches):
        """launches: (heads, max_parts, [(new, cached), ...]) -> [(part size, parts, smallest part)]"""
        text = "\n".join(" ".join(map(str, [h, mx, len(seqs), *(v for s in seqs for v in s)])) for h, mx, seqs in launches)
        out = subprocess.run([exe], input=text + "\n", stdout=subprocess.PIPE, text=True, check=True, timeout=300).stdout
        return [tuple(map(int, line.split())) for line in out.splitlines()]
    return run


def _max_parts(heads, head_dim):
    return PART_BUDGET // (heads * 256 * (head_dim + 2) * 4)


def test_parts_stay_within_their_memory_and_are_never_too_short(plan):
    """Chunks and prompts of up to 12000 tokens behind up to 130000, alone and in pairs: the uncapped plan asked for up to
    0.75 GB here."""
    lengths, cached = [1, 37, 128, 300, 700, 1100, 2048, 3300, 4600, 6369, 7187, 9000, 12000], [0, 256, 1100, 3000, 8000, 24576, 50000, 100000, 130000]
    launches = [(h, _max_parts(h, d), seqs) for h in (2, 5, 8, 14, 32, 40, 64, 128) for d in (64, 128)
                for n in lengths for c in cached for seqs in ([(n, c)], [(n, c), (300, 20000)])]
    results = plan(launches)
    assert any(parts for _, parts, _ in results)
    for (heads, max_parts, seqs), (limit, parts, least) in zip(launches, results):
        assert parts <= max_parts, (heads, seqs, parts, max_parts)
        assert (limit == 0) == (parts == 0), (heads, seqs)
        assert parts == 0 or least >= 5, (heads, seqs, least)   # 5 tiles of 64 keys: 256 queries and one key before them


def test_a_tight_budget_leaves_the_tiles_whole(plan):
    free, none, few = plan([(32, 1 << 30, [(512, 15872)]), (32, 0, [(512, 15872)]), (32, 3, [(512, 15872)])])
    assert free[1] > 0 and none == (0, 0, 0) and few == (0, 0, 0)


def test_launches_of_the_gpu_tests_are_cut_or_whole_as_meant(plan):
    cut = [[(1, 1023)], [(257, 1008), (40, 3000)], [(700, 2400)], [(2100, 0)], [(32, 1328)]]
    whole = [[(1, 0)], [(1, 64)], [(65, 0)], [(129, 50)], [(300, 7), (40, 100)], [(640, 63)]]
    results = plan([(4, _max_parts(4, d), seqs) for d in (64, 128) for seqs in cut + whole])
    for i, (limit, parts, _) in enumerate(results):
        assert (parts > 1) == (i % len(cut + whole) < len(cut)), (i, limit, parts)


def _plain_plan(tiles, heads, max_parts):
    """The plan as its comment states it, gone through place by place."""
    places = min(64, max(1, 256 // heads))
    if not tiles or len(tiles) > 4 * places or tiles[0] < 16:
        return 0

    def end_of(limit):
        at, stored = [0] * places, 0
        for n in tiles:
            parts = -(-n // limit) if limit else 1
            stored += parts if parts > 1 else 0
            for _ in range(parts):
                at[at.index(min(at))] += -(-n // parts) + (5 if parts > 1 else 3)
        return max(at) + (4 + stored * heads // 50 if stored else 0), stored

    end = end_of(0)[0]
    best, best_end, last = 0, end - end // 16, 0
    for parts in range(2, 17):
        limit = max(15, -(-tiles[0] // parts))
        if limit != last and limit < tiles[0]:
            end, stored = end_of(limit)
            if stored <= max_parts and end < best_end:
                best, best_end = limit, end
            last = limit
    return best


def test_the_plan_is_the_one_its_comment_states(plan):
    launches = [(h, mx, [(n, c)]) for h in (1, 4, 7, 32, 64, 200) for mx in (20, 1 << 30)
                for n, c in ((1, 1023), (300, 2048), (512, 15872), (1500, 0), (2100, 0), (2048, 24576), (5000, 30000), (9000, 7000))]
    for (heads, max_parts, [(n, c)]), (limit, _, _) in zip(launches, plan(launches)):
        tiles = sorted(((c + min(n, q + 256) + 63) // 64 for q in range(0, n, 256)), reverse=True)
        assert limit == _plain_plan(tiles, heads, max_parts), (heads, max_parts, n, c)


def test_planning_a_long_prompt_takes_microseconds(plan):
    """begin() plans before its first launch: 100 plans of 254 query tiles take 3 ms; going through every candidate place by
    place they took 180."""
    def cpu():
        usage = resource.getrusage(resource.RUSAGE_CHILDREN)
        return usage.ru_utime
    plan([(2, 1 << 30, [(1, 0)])])
    start = cpu()
    plan([(2, 1 << 30, [(65000, 30000)])] * 100)
    assert cpu() - start < 0.1
