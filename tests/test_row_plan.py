"""Which kernel a call of the automatic choice runs on: the rules of flashd_plan.h, compiled for the host,
and the shapes of the GPU tests that mean to reach a certain kernel."""
import os
import shutil
import subprocess

import pytest

from paper_2505_14201_amd import flashd

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(os.path.dirname(HERE), "paper_2505_14201_amd", "csrc")

PROGRAM = r"""
#include <cstdio>
#include "flashd_plan.h"
using namespace flashd;
int main() {
    Shape s;
    int causal, shift, splits, states, fp8;
    while (std::scanf("%d %d %d %d %d %d %d %d %d %d %d %d", &s.B, &s.Hq, &s.Hkv, &s.Lq, &s.Lk, &s.d, &s.dtype,
                      &causal, &shift, &splits, &states, &fp8) == 12) {
        if (s.dtype == 0) {
            std::printf("f32 %d\n", f32_runs_whole(s, causal != 0, shift, states != 0, splits) ? 1 : splits);
        } else if ((long)(s.Hq / s.Hkv) * s.Lq <= 32) {
            std::printf("decode %d\n", states == 0 && decode_on_eight(s, fp8 != 0, splits) ? 8 : 4);
        } else {
            const RowPlan p = row_plan(s, causal != 0, shift, splits, states, fp8 != 0);
            std::printf("%s %d\n", p.kernel == RowKernel::Short ? "32" : p.kernel == RowKernel::Tile64 ? "64" : "128",
                        p.splits);
        }
    }
}
"""


@pytest.fixture(scope="module")
def plan(tmp_path_factory):
    """plan(calls, dtype) -> [(kernel, splits or wavefronts)]; a call is (B, Hq, Hkv, Lq, Lk, d, causal) and
    optionally shift, states (how many states are read and written) and fp8."""
    if shutil.which("g++") is None:
        pytest.skip("needs g++ to compile the header")
    tmp = tmp_path_factory.mktemp("plan")
    src, exe = tmp / "plan.cpp", tmp / "plan"
    src.write_text(PROGRAM)
    subprocess.run(["g++", "-O1", "-std=c++17", "-Wall", "-I", CSRC, "-o", str(exe), str(src)], check=True)

    def ask(calls, dtype=flashd.BF16):
        lines, wide = [], []
        for B, Hq, Hkv, Lq, Lk, d, causal, *more in calls:
            shift, states, fp8 = (more + [None, 0, 0][len(more):])
            shift = Lk - Lq if shift is None else max(min(shift, Lk), -Lq - 1)
            sp = flashd.auto_splits(B, Hq, Hkv, Lq, Lk, d, dtype)
            lines.append(f"{B} {Hq} {Hkv} {Lq} {Lk} {d} {dtype} {int(causal)} {shift} {sp} {states} {int(fp8)}")
            wide.append(not states and not fp8 and flashd.auto_variant(B, Hq, Hkv, Lq, Lk, d, dtype, causal)
                        == flashd.VARIANT_TILE_256)
        out = subprocess.run([str(exe)], input="\n".join(lines), capture_output=True, text=True, check=True).stdout
        got = [(k, int(n)) for k, n in (l.split() for l in out.splitlines())]
        assert len(got) == len(calls)
        return [("256", 1) if w else g for w, g in zip(wide, got)]
    return ask


BOTH, MASKS = (64, 128), (False, True)


def test_shapes_for_32_rows_per_workgroup(plan):
    from tests.test_gpu_row_kernels import SHORT
    calls = [(*s, d, c) for s in SHORT for d in BOTH for c in MASKS]
    calls += [(*s, d, True, None, 0, 1) for s in SHORT for d in BOTH]                       # fp8
    calls += [(*s[:4], s[4] // 2 + 1, d, True, s[4] - s[3], 1) for s in SHORT for d in BOTH]     # a first chunk
    for call, (kernel, splits) in zip(calls, plan(calls)):
        assert kernel == "32", call
        assert (splits > 1) == (call[4] > 1000), call


def test_shapes_for_64_rows_per_workgroup(plan):
    from tests.test_gpu_row_kernels import FEW_KEYS, TILE64_ALL, TILE64_STATES
    calls = [(*s, d, c) for d in TILE64_ALL for s in TILE64_ALL[d] for c in MASKS]
    for d in TILE64_STATES:
        for B, Hq, Hkv, Lq, Lk in TILE64_STATES[d]:
            cut = Lk // 2 + 1
            calls += [(B, Hq, Hkv, Lq, cut, d, True, Lk - Lq, 1), (B, Hq, Hkv, Lq, Lk - cut, d, True, Lk - Lq - cut, 2)]
    calls += [(*FEW_KEYS[-1], d, c) for d in BOTH for c in MASKS] + [(*FEW_KEYS[-1], 128, True, None, 0, 1)]
    for call, got in zip(calls, plan(calls)):
        assert got == ("64", 1), call


def test_shapes_of_at_most_two_key_tiles(plan):
    from tests.test_gpu_row_kernels import FEW_KEYS
    for s, d128 in zip(FEW_KEYS, ("128", "128", "32", "32", "64")):
        d64 = "64" if d128 == "64" else "32"
        assert [k for k, _ in plan([(*s, d, c) for d in BOTH for c in MASKS])] == [d64, d64, d128, d128], s
        assert [k for k, _ in plan([(*s, d, True, None, 0, 1) for d in BOTH])] == [d64, d64], s        # fp8


def test_shapes_for_the_128_row_kernel(plan):
    from tests import test_gpu_tile_state as t
    calls = [(2, 16, 16, 2200, 320, d, True, -n, 2) for d in BOTH for n in (2200, 1900)]    # test_gpu_state_rows.py
    for B, Hq, Hkv, Lq, Lk, cuts, shift in t.CHUNKS:
        k0 = 0
        for k1 in (*cuts, Lk):
            calls += [(B, Hq, Hkv, Lq, k1 - k0, d, c, shift - k0, 2 if k0 else 1) for d in BOTH for c in MASKS]
            k0 = k1
        calls += [(B, Hq, Hkv, Lq, Lk - cuts[-1], d, c, shift - cuts[-1], 1) for d in BOTH for c in MASKS]
    calls += [(*s, d, c, None, 0, 1) for s in t.FP8 for d in BOTH for c in MASKS]
    for call, got in zip(calls, plan(calls)):
        assert got == ("128", 1), call


def test_shapes_of_the_precision_tests(plan):
    from tests import test_gpu_row_precision as t
    calls = [(B, H, H, Lq, b - a, d, False, None, 2 if a else 1) for B, H, Lq, Lk in t.SHAPES for d in BOTH
             for chunks in (1, 2) for a, b in t.cuts(Lk, chunks)]
    calls += [(B, H, H, Lq, Lk, d, c, None, 1) for B, H, Lq, Lk in t.MASKED for d in BOTH for c in MASKS]
    assert not [c for c, (k, _) in zip(calls, plan(calls)) if k == "128"]


def test_shapes_that_carry_states(plan):
    from tests.test_gpu_state_rows import EMPTY
    calls = [(B, H, H, Lq, Lk, d, True, -(Lq - Lq // 3), 2) for B, H, Lq, Lk, d, _ in EMPTY[:4]]
    assert [k for k, _ in plan(calls)] == ["128", "128", "64", "32"]


def test_shapes_for_decode_on_eight_wavefronts(plan):
    from tests.test_gpu_decode_eight import ON_FP8, SHAPES
    calls = [(*s, True) for s in SHAPES] + [(*s, True, None, 0, 1) for s in ON_FP8]
    assert plan(calls) == [("decode", 8)] * len(calls)
    # many units over long ranges have HBM as their bound
    calls = [(13, 64, 16, 1, 65536, 64, False), (19, 44, 11, 1, 8192, 64, False), (19, 44, 11, 1, 8193, 64, False)]
    assert plan(calls) == [("decode", n) for n in (8, 8, 4)]


def test_large_keys_and_values_stay_on_the_128_row_kernel(plan):
    """More than 100 MB of K and V, which every round of workgroups reads again; the next ones are on either side of
    a line (bytes, workgroups) of the rule."""
    calls = [(13, 24, 8, 46, 5093, 128, True), (25, 96, 8, 11, 9065, 64, True), (16, 5, 5, 155, 5306, 128, True),
             (4, 64, 64, 152, 1223, 128, True), (34, 12, 12, 147, 2012, 128, True)]
    assert [k for k, _ in plan(calls)] == ["128"] * 5
    assert plan([(13, 24, 8, 46, 1800, 128, True), (13, 24, 8, 42, 2500, 128, True)]) == [("32", 1), ("32", 1)]
    assert [k for k, _ in plan([(B, 12, 12, 145, 1779, 128, True) for B in (14, 15)])] == ["64", "128"]
    # fp8: half the bytes, and the 128-row kernel would need them widened
    assert plan([(13, 24, 8, 46, 5093, 128, True, None, 0, 1)])[0][0] == "32"


@pytest.mark.parametrize("H,Lq,Lk,d,causal,whole,with_state", [
    # as many rounds of row tiles in splits: whole, a single one up to 2000 keys
    (256, 1, 1999, 64, 0, 1, 1), (256, 1, 2000, 64, 0, 0, 0), (64, 63, 13491, 64, 0, 0, 0),
    (8, 1000, 8192, 64, 0, 1, 1), (8, 1000, 8192, 64, 1, 1, 1), (700, 1, 2000, 128, 0, 1, 1),
    # nearly as many: by splits, keys and d
    (400, 1, 2000, 64, 0, 1, 0), (400, 1, 2000, 128, 0, 0, 0), (400, 1, 1300, 128, 0, 1, 0),
    (637, 1, 999, 64, 0, 1, 0), (637, 1, 1000, 64, 0, 0, 0), (637, 1, 999, 128, 0, 0, 0),
    # fewer: split, but under a mask that rows see unequally of, and up to 600 keys
    (8, 545, 1306, 64, 0, 0, 0), (8, 545, 8192, 64, 1, 0, 0), (8, 545, 1000, 64, 1, 1, 0), (8, 545, 1306, 64, 1, 1, 0),
    (8, 545, 1364, 64, 1, 0, 0), (32, 130, 601, 64, 0, 0, 0), (32, 130, 600, 64, 0, 1, 0),
    # rows that see no key
    (7, 1094, 542, 64, 1, 1, 1), (2, 2073, 1176, 64, 1, 0, 0),
])
def test_fp32_calls_that_run_whole(plan, H, Lq, Lk, d, causal, whole, with_state):
    call = (1, H, H, Lq, Lk, d, causal)
    assert flashd.auto_splits(*call[:6], flashd.F32) > 1
    assert (plan([call], flashd.F32)[0][1] == 1) == bool(whole)
    assert (plan([(*call, None, 2)], flashd.F32)[0][1] == 1) == bool(with_state)


HAND_OUT_PROGRAM = r"""
#include <cstdio>
#include "flashd_plan.h"
int main() {
    long m_tiles, units, slots;
    int Lk, d;
    double mb;
    while (std::scanf("%ld %ld %ld %d %d %lf", &m_tiles, &units, &slots, &Lk, &d, &mb) == 6)
        std::printf("%d\n", flashd::rows_in_pairs(m_tiles, units, slots, Lk, d, mb) ? 1 : 0);
}
"""


def test_shapes_in_pairs_and_one_by_one(tmp_path):
    """The shapes of test_gpu_wide.HAND_OUT reach the hand-out that they are meant for."""
    from tests.test_gpu_wide import HAND_OUT, WIDE
    if shutil.which("g++") is None:
        pytest.skip("needs g++ to compile the header")
    src, exe = tmp_path / "pairs.cpp", tmp_path / "pairs"
    src.write_text(HAND_OUT_PROGRAM)
    subprocess.run(["g++", "-O1", "-std=c++17", "-Wall", "-I", CSRC, "-o", str(exe), str(src)], check=True)
    lines = []
    for variant, B, Hq, Hkv, Lq, Lk, d, _ in HAND_OUT:
        rows, slots = (256, 256) if variant == WIDE else (128, 512 if d == 128 else 768)
        g = 1 if variant == WIDE else Hq // Hkv       # the 128-row kernel runs these heads of a group as one
        lines.append(f"{(g * Lq + rows - 1) // rows} {B * Hq // g} {slots} {Lk} {d} {B * Hkv * Lk * d * 4e-6}")
    out = subprocess.run([str(exe)], input="\n".join(lines), capture_output=True, text=True, check=True).stdout
    assert [bool(int(x)) for x in out.split()] == [h[-1] for h in HAND_OUT]
    pairs = [h for h in HAND_OUT if h[-1]]
    odd = [h for h in pairs if (h[2] // h[3] * h[4] + 127) // 128 % 2 and h[0] != WIDE]
    assert {h[6] for h in odd} == {64, 128} and any(h[2] != h[3] for h in odd)
