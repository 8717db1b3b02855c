"""The rules that choose a GEMM's tile (csrc/gemm_plan.h), built for the CPU."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


@pytest.fixture(scope="module")
def rules(tmp_path_factory):
    cxx = shutil.which("g++") or shutil.which("c++")
    if cxx is None:
        pytest.skip("no host C++ compiler")
    exe = str(tmp_path_factory.mktemp("plan") / "dump")
    subprocess.run([cxx, "-std=c++17", "-O2", os.path.join(ROOT, "tests", "host", "gemm_plan_dump.cpp"), "-o", exe], check=True)

    def run(lines):
        out = subprocess.run([exe], input="\n".join(lines) + "\n", stdout=subprocess.PIPE, text=True, check=True, timeout=60).stdout
        return out.split()
    return run


def test_expert_matrices_beyond_32_bit_offsets_stay_on_the_large_tile(rules):
    """The small tiles reach an expert's up rows through byte offsets of up to (ffn + 64) x hidden x 2, where 2^31 means
    "outside": from there on only the 256-row tile, with a base for gate and one for up, may be chosen."""
    sizes = [(768, 2048), (14336, 4096), (16384, 32768), (32512, 32768), (32576, 32768), (65536, 16384), (1 << 18, 8192)]
    asked = [(rows, f, d) for f, d in sizes for rows in (1, 18, 40, 90, 500)]
    for (rows, f, d), tile in zip(asked, rules([f"moe {r} {f} {d}" for r, f, d in asked])):
        fits = (f + 64) * d * 2 < 1 << 31
        assert int(tile) in (32, 64, 128, 256) and (fits or int(tile) == 256), (rows, f, d, tile)
    assert rules(["moe 18 768 2048", "moe 40 14336 4096", "moe 500 768 2048"]) == ["32", "64", "256"]


def test_the_gpu_tests_reach_every_tile(rules):
    """Which tile the problems of tests/test_gpu_ops.py and tests/test_gpu_prefill.py run on."""
    odd_k = [(3329, 3080, 8), (3329, 3080, 72), (3329, 3080, 136), (3329, 3080, 200), (3329, 3080, 632), (4100, 2568, 1016), (8200, 1288, 2040)]
    assert set(rules([f"tile {m} {n} {k} {r}" for m, n, k in odd_k for r in (0, 1)])) == {"large"}
    about_100 = [(2560, 2560, 8), (2305, 2568, 72), (2304, 2816, 136), (2305, 2568, 200), (2049, 3080, 632), (4100, 1544, 1016), (8200, 520, 2040)]
    assert set(rules([f"tile {m} {n} {k} 0" for m, n, k in about_100])) == {"any128"}
    assert set(rules([f"tile {m} {n} {k} 1" for m, n, k in about_100])) == {"large", "ring128"}
    small = [(1, 8, 8), (37, 520, 264), (300, 1408, 256), (256, 256, 704), (1000, 256, 704), (513, 776, 1000)]
    assert rules([f"tile {m} {n} {k} 0" for m, n, k in small]) == ["any128", "ring32", "ring32", "ring32", "ring32", "ring32"]
    assert rules([f"swiglu {m} {f} {k}" for m, f, k in [(200, 704, 256), (1, 704, 256), (97, 200, 264), (700, 1032, 320)]]) == ["32", "32", "32", "64"]


def test_wide_problems_of_short_k_do_not_run_on_the_smallest_tiles(rules):
    """A round of small tiles costs more than its share of the outputs: many rounds of them lose to one or two rounds of
    128x128 (measured, us, 32x64 tiles against the choice: 31.6/11.1, 38/21, 20.9/14, 28.6/13.4)."""
    problems = [(725, 7104, 256), (1168, 2648, 1312), (1330, 1848, 704), (953, 3728, 576)]
    assert set(rules([f"tile {m} {n} {k} 0" for m, n, k in problems])) <= {"ring128", "any128"}
    # Up to two rounds of 128x128 tiles for odd K: two of their workgroups share a CU, the large tile leaves half the CUs idle.
    assert set(rules([f"tile {m} {n} {k} 0" for m, n, k in [(2012, 2840, 2552), (3779, 1648, 784), (1596, 4520, 856)]])) == {"any128"}
    assert rules(["tile 4072 2472 3736 0", "tile 8192 8192 2056 0"]) == ["large", "large"]


@pytest.mark.parametrize("k", [8, 64, 1000, 1 << 21, (1 << 21) + 8, 1 << 24])
def test_sizes_beyond_32_bit_offsets_run_on_the_kernel_without_them(rules, k):
    tiles = set(rules([f"tile {m} {n} {k} {r}" for m, n in ((8, 8), (4096, 4096), (70000, 70000)) for r in (0, 1)]))
    assert tiles == {"any128"} if k > 1 << 21 else tiles <= {"ring32", "ring64", "ring128", "any128", "large"}
    assert "large" not in rules([f"tile 4096 {(1 << 21) + 8} {k} 0"])


def test_expert_tiles_leave_room_for_uneven_counts(rules):
    """Counts spread by about the root of their mean: a tile is chosen only where two such deviations still fit it, since an
    expert with a second tile reads its weights twice (130 rows on 128-row tiles, 8 experts of 14336 x 4096: 1020 us, 738 on
    256-row ones; 52 rows on 64-row tiles, 64 experts of 1408 x 2048: 234 us, 223 on 128-row ones)."""
    means = list(range(1, 400))
    for mean, tile in zip(means, map(int, rules([f"moe {m} 14336 4096" for m in means]))):
        assert tile == 256 or mean + 2 * mean ** 0.5 <= tile, (mean, tile)


def test_the_gpu_tests_reach_every_height_of_the_large_tile(rules):
    from tests.test_gpu_ops import LARGE_TILE_SIZES
    got = rules([f"rows {m} {n} {k} {epilogue}" for _, epilogue, m, n, k in LARGE_TILE_SIZES])
    assert [int(r) for r in got] == [rows for rows, *_ in LARGE_TILE_SIZES]
    for _, epilogue, m, n, _ in LARGE_TILE_SIZES:             # none of them is cut over K or left to the small tiles
        assert (m + 255) // 256 * ((n + (127 if epilogue == "swiglu" else 255)) // (128 if epilogue == "swiglu" else 256)) >= 160


def test_the_gpu_tests_reach_every_fp32_tile(rules):
    from tests.test_gpu_ops import F32_TILE_SIZES
    got = rules([f"f32 {m} {n} {k} {residual}" for _, m, n, k, residual in F32_TILE_SIZES])
    assert [int(r) for r in got] == [rows for rows, *_ in F32_TILE_SIZES]
    assert {int(r) for r in got} == {16, 32, 48, 64, 80, 128}


def test_the_l2_warm_up_asks_for_shared_lines_only(rules):
    """Every line of a W panel is asked for by one of the row tiles that share it, and by nobody where one row tile is alone."""
    shares = [int(n) for n in rules([f"warm {n}" for n in range(1, 9)])]
    assert shares[0] == 0 and all(n / 2 < s <= n for n, s in enumerate(shares[1:], 2)), shares


def test_three_stages_ask_for_the_warm_up_where_it_was_measured_to_gain(rules):
    """Time with over time without it, measured means: 0.92 to 0.98 for 3 and 5 times 512 to 4096 (SwiGLU 0.95 to 1.02), 0.98 to
    1.06 for factors of 9 and more, where 5120 columns of 27648 gain 2 % (SwiGLU 1.02 to 1.08); 1.01 to 1.08 for powers of two,
    0.97 to 1.04 for smaller powers.  The GPU tests run both sides of the rule."""
    small, larger = (1536, 2560, 3072, 3584, 5120, 6144, 10240, 14336), (4608, 5632, 6656, 7680, 9216, 11264, 13824, 18944, 27648)
    never = (64, 832, 896, 1024, 4096, 8192, 16384, 1280, 2304, 3328, 4160, 4480)
    assert rules([f"warm3 {k} 0" for k in small + larger + never]) == ["1"] * 17 + ["0"] * len(never)
    assert rules([f"warm3 {k} 1" for k in small + larger + never]) == ["1"] * 8 + ["0"] * (9 + len(never))
    from tests.test_gpu_ops import LARGE_TILE_SIZES
    three = {(rows, epilogue, k) for rows, epilogue, _, _, k in LARGE_TILE_SIZES if rows <= 160}
    for rows in (128, 160):
        for epilogue in ("bf16", "residual", "swiglu"):
            # k-tiles behind the last whole turn of six: one and two (832, 896), none and a half with the warm-up (1536, 2560)
            assert {(rows, epilogue, k) for k in (64, 576, 832, 896, 1536, 2560)} <= three


def test_wide_projections_of_65_to_128_rows_stay_on_the_few_rows_kernel(rules):
    """Measured, us, few-rows kernel / large kernel: 110 / 137, 244 / 288, 107 / 131, 124 / 130, 128 / 135 -- and, a short K
    in one round of large tiles, the other way round."""
    wide = [(65, 49152, 5120), (65, 128256, 5120), (65, 41000, 5120), (65, 65536, 4096), (65, 128256, 2048)]
    assert rules([f"few {m} {n} {k}" for m, n, k in wide]) == ["1"] * 5
    assert rules(["few 128 41000 512", "few 128 65536 1024", "few 65 40704 5120", "few 129 49152 5120", "few 64 8 8"]) == ["0", "0", "0", "0", "1"]


def test_columns_start_elsewhere_only_where_either_form_does(rules):
    """A projection fused with SiLU*up and the plain one of the same matrix take the same starts, whichever tile they run on: none
    for problems that could be on a tile without them (the 256-column one, 65 to 128 rows of a long K on the few-rows one)."""
    asked = [(m, n, k) for m in (1, 64, 65, 128, 129, 256, 257, 512, 513) for n in (12544, 14336, 28672, 40704, 40960, 57344) for k in (1024, 2048, 4096, 16384, 16512)]
    for (m, n, k), groups, few in zip(asked, rules([f"starts {m} {n} {k}" for m, n, k in asked]), rules([f"few {m} {n} {k}" for m, n, k in asked])):
        narrow = m <= 512 and (m + 255) // 256 * (n // 256) < 160
        assert int(groups) == (n // 256 if narrow and 2048 <= k <= 16384 else 0), (m, n, k, groups)
        assert int(groups) == 0 or m <= 64 or few == "0", (m, n, k)
    assert rules(["starts 50 28680 4096", "starts 50 28672 4160", "starts 50 128 4096"]) == ["0", "0", "0"]


@pytest.mark.parametrize("aligned", [1, 0])
def test_the_fused_and_the_plain_form_start_alike_on_the_tiles_they_take(rules, aligned):
    """The dispatch itself, operands on the 16-byte grid or off it (then nothing runs on the few-rows kernel): wherever the fused
    projection exists and the plain one is not cut, every output's gate, up and fused column start at one k."""
    outputs = [128 * g + 8 * d for g in (15, 47, 48, 49, 50, 56, 63, 64, 79, 80, 81, 95, 96, 110, 111, 112, 127, 128, 159, 160, 161, 319, 320) for d in (0, 1, 8)]
    # Workspace: none, and enough to cut whatever the rules cut (three and four row tiles may come out uncut of that).
    asked = [(m, f, k, ws, aligned) for m in (1, 32, 33, 64, 65, 96, 128, 129, 256, 257, 384, 512, 513, 768, 1024) for f in outputs
             for k in (64, 1024, 1920, 2048, 2112, 3072, 4096, 6144, 16384, 16512, 17408) for ws in (0, 1 << 40)]
    answers = rules([f"forms {m} {f} {k} {ws} {a}" for m, f, k, ws, a in asked])
    answers = [tuple(map(int, answers[i:i + 4])) for i in range(0, len(answers), 4)]
    compared = 0
    for case, (plain, fused, alike, form) in zip(asked, answers):
        if form == 0:
            assert plain == fused and alike, (case, plain, fused)
            compared += fused > 0
    assert compared > 500
