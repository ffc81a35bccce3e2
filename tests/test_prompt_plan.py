"""How long prompt passes and the training step's contractions are cut into workgroups (csrc/prompt_plan.h), on the CPU: the header is host
arithmetic, compiled here with g++ and asked for every projection of a range of widths and pass lengths."""
import os
import shutil
import subprocess

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)
PART_ROWS, SLICES, CUS_PER_XCD = 4096, 8, 32


@pytest.fixture(scope="module")
def plan(tmp_path_factory):
    """What the plan picks for a list of (weight tiles, k-steps, rows, may be cut): those, then tiles, pairs and slices."""
    if shutil.which("g++") is None:
        pytest.skip("g++ not available")
    exe = str(tmp_path_factory.mktemp("plan") / "plan")
    res = subprocess.run(["g++", "-O2", "-std=c++17", "-I", os.path.join(ROOT, "paper_2404_18911_amd", "csrc"),
                          os.path.join(HERE, "native", "prompt_plan_driver.cpp"), "-o", exe], capture_output=True, text=True)
    assert res.returncode == 0, res.stderr[-2000:]

    def ask(asked, *mode):
        out = subprocess.run([exe, *mode], input="\n".join(" ".join(map(str, a)) for a in asked), capture_output=True, text=True, timeout=120).stdout
        rows = [tuple(map(int, l.split())) for l in out.splitlines()]
        assert [r[:len(a)] for r, a in zip(rows, asked)] == asked and len(rows) == len(asked)
        return rows
    return ask


def _projections(d, f, T):
    return [(3 * d // 16, d // 32, T, 0), (2 * f // 16, d // 32, T, 0), (d // 16, d // 32, T, 1), (d // 16, (f + 31) // 32, T, 1)]


@pytest.fixture(scope="module")
def picks(plan):
    asked = []
    for d in list(range(512, 8193, 256)):
        f = d * 43 // 16 // 16 * 16
        for T in list(range(97, 1100, 13)) + [1200, 1465, 2001, 3000, 4096]:
            asked += _projections(d, f, T)
    return plan(asked)


def test_picked_slices_fit_the_buffers_and_the_projection(picks):
    for NT, KS, T, split, tiles, pairs, S in picks:
        assert tiles in (6, 8, 12, 16, 32) and 5 <= pairs <= 8 and (tiles > 6 or pairs == 8)
        assert 1 <= S <= (SLICES if split else 1)
        if S > 1:
            assert S * T <= PART_ROWS and KS >= 8 * S and tiles < 32


def test_no_slicing_leaves_an_xcd_with_a_few_workgroups_more_than_whole_rounds(picks):
    """A slice's workgroups are dealt out to the 8 XCDs in equal shares (the larger share decides), so S slices put S * ceil(w / 8)
    workgroups on one XCD.  A plan that counts compute units of the whole device instead took such launches for one round."""
    cut = 0
    for NT, KS, T, split, tiles, pairs, S in picks:
        if S == 1:
            continue
        cut += 1
        w = -(-((T + 15) // 16) // pairs) * -(-NT // tiles)
        on_one = S * -(-w // 8)
        rest = on_one % CUS_PER_XCD
        assert on_one < CUS_PER_XCD or rest == 0 or rest >= CUS_PER_XCD // 4, (NT, KS, T, tiles, pairs, S, on_one)
    assert cut > 1000


def test_the_gpu_prompt_tests_reach_every_variant_and_number_of_slices(plan):
    """The passes of tests/test_gpu_prompt_kernels.py run every tile size with every number of pairs, and every number of slices."""
    from tests.test_gpu_prompt_kernels import LENGTHS, SHAPES
    asked = []
    for s in SHAPES.values():
        for T in LENGTHS:
            if T > (192 if s.d_model <= 2048 else 96):          # shorter ones are weight streams
                asked += _projections(s.d_model, s.d_ffn, T)
    rows = plan(asked)
    assert {r[4:6] for r in rows} == {(6, 8)} | {(t, p) for t in (8, 12, 16, 32) for p in (5, 6, 7, 8)}
    assert {r[6] for r in rows} == set(range(1, SLICES + 1))


def test_slices_of_a_training_contraction_hold_every_k_once(plan):
    """None empty, none beyond the partial sums' buffer, each a whole number of steps but the last, and no launch cut that fills its rounds."""
    asked = []
    for d in (64, 384, 640, 1024, 4096, 5120, 6656):
        f, V = d * 43 // 16 // 16 * 16, 32000
        for T in (1, 33, 129, 256, 300, 777, 1000, 1400, 2048):
            part = SLICES * min(T, 256) * 3 * d
            asked += [(T, n, k, t16, part) for t16 in (0, 1) for n, k in ((3 * d, d), (d, 3 * d), (d, d), (f, d), (d, f), (V, d), (d, V))]
            asked += [(n, k, T, 0, part) for n, k in ((3 * d, d), (d, d), (f, d), (d, f), (V, d))]
    seen = set()
    for M, N, K, t16, part, S, chunk in plan(asked, "train"):
        seen.add(S)
        assert 1 <= S <= SLICES and chunk % 32 == 0 and (S - 1) * chunk < K <= S * chunk
        assert S == 1 or (S * M * N <= part and K // S >= 128)
        assert S == 1 or (-(-M // 128) * -(-N // 256)) % 256 != 0
    assert seen == set(range(1, SLICES + 1))


def test_slices_of_a_training_contraction_are_counted_on_the_busiest_xcd(plan):
    """The tiles of column c of C go to XCD c % 8 (with 16 columns or more, or a multiple of 8): of 20 columns some XCDs have three, and 36 tiles are two rounds
    on the 32 compute units of one where 240 would be one on the device.  The steps of the chosen number of slices against those of the best one:
    at most a third more, which the partial sums may be worth."""
    asked = [(T, d, k, t16, SLICES * min(T, 256) * 3 * d) for d in (2048, 4096, 5120, 6656, 8192) for T in (100, 150, 256, 333, 450, 500, 700, 1000, 1400)
             for k, t16 in ((d, 0), (3 * d, 0), (d * 43 // 16, 0), (32000, 1))]
    for M, N, K, t16, part, S, chunk in plan(asked, "train"):
        gm, gn = -(-M // 128), -(-N // 256)
        assert gn % 8 == 0 or gn >= 16

        def steps(n):
            return -(-gm * -(-gn // 8) * n // 32) * -(-(-(-K // n)) // 32)
        best = min(steps(n) for n in range(1, SLICES + 1) if n == 1 or (K // n >= 128 and n * M * N <= part))
        assert steps(S) <= 4 / 3 * best, (M, N, K, S, steps(S), best)
