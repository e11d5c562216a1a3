"""How many workgroups of the causal attention share a CU (csrc/zo_attn_items.h), compiled for the host: whatever is chosen, every
query tile of every (sequence, head) pair is worked exactly once, and the choice is about the faster one of those measured."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

# for each line "seq heads sequences CUs d_head": workgroups a CU, slots and fill of the plan, whether each item comes once
PROGRAM = r"""
#include "zo_attn_items.h"
#include <cstdio>
#include <vector>
int main()
{
    int seq, heads, n_seq, cus, d_head;
    while (scanf("%d %d %d %d %d", &seq, &heads, &n_seq, &cus, &d_head) == 5) {
        const int n_qt = (seq + zo::kAttnRows - 1) / zo::kAttnRows;
        const zo::AttnPlan plan = zo::attention_plan_on((long long)heads * n_seq, n_qt, cus, d_head);
        const zo::AttnItems list(seq, heads, n_seq, plan.fill);
        std::vector<int> seen((size_t)heads * n_seq * n_qt, 0);
        bool good = true;
        for (int xcd = 0; xcd < 8; ++xcd)
            for (int slot = 0; slot < plan.slots; ++slot)
                for (int round = 0; round * plan.slots < list.n_lin; ++round) {
                    int qt = -1;
                    const int pair = list.pair_at(round * plan.slots + (round & 1 ? plan.slots - 1 - slot : slot), xcd, qt);
                    if (pair < 0) continue;
                    good = good && pair < heads * n_seq && pair % 8 == xcd && qt >= 0 && qt < n_qt;
                    if (good) ++seen[(size_t)pair * n_qt + qt];
                }
        for (int s : seen) good = good && s == 1;
        printf("%d %d %d %d\n", plan.per_cu, plan.slots, plan.fill, (int)good);
    }
    return 0;
}
"""


@pytest.fixture(scope="module")
def plans(tmp_path_factory):
    cxx = shutil.which("g++") or shutil.which("c++")
    rocm = next((p for p in (os.environ.get("ROCM_PATH"), "/opt/rocm") if p and os.path.exists(os.path.join(p, "include", "hip"))), None)
    if not cxx or not rocm:
        pytest.skip("no host compiler or no HIP headers")
    folder = tmp_path_factory.mktemp("residency")
    src, exe = folder / "residency.cpp", folder / "residency"
    src.write_text(PROGRAM)
    subprocess.run([cxx, "-O1", "-std=c++17", "-D__HIP_PLATFORM_AMD__", "-I", os.path.join(ROOT, "paper_2507_03211_amd", "csrc"),
                    "-I", os.path.join(rocm, "include"), str(src), "-o", str(exe)], check=True, timeout=120)

    def ask(rows):
        run = subprocess.run([str(exe)], input="\n".join(" ".join(map(str, r)) for r in rows), capture_output=True, text=True, timeout=120, check=True)
        return [tuple(map(int, line.split())) for line in run.stdout.splitlines()]

    return ask


def test_every_item_comes_once(plans):
    rows = [(seq, heads, n_seq, cus, dh) for dh in (64, 80, 96, 128) for cus in (1, 5, 32) for seq in (1, 129, 300, 512, 600, 768, 1023, 1500, 2048, 4200, 8320)
            for heads, n_seq in ((1, 1), (3, 3), (5, 8), (17, 2), (12, 24), (40, 8), (32, 32)) if heads * n_seq * seq <= 1200000]
    room = {64: 4, 80: 3}
    for row, (per_cu, slots, fill, good) in zip(rows, plans(rows)):
        assert good and slots >= 1 and fill >= 1, row
        assert per_cu in (room.get(row[4], 2), max(2, room.get(row[4], 2) - 1)), row


# d_head, tokens, pairs, us with one workgroup a CU less than there is room for, with all of them (bf16, 256 CUs)
MEASURED = [
    (64, 331, 1024, 50.1, 51.1), (64, 512, 976, 77.5, 80.9), (64, 379, 2048, 105.2, 110.7), (64, 512, 272, 26.5, 29.4), (64, 256, 1760, 59.0, 61.3), (64, 238, 444, 18.2, 15.6),
    (64, 277, 288, 17.9, 14.8), (64, 768, 144, 29.9, 23.3), (64, 221, 512, 18.5, 16.7), (64, 2048, 256, 188.0, 173.5), (64, 1987, 168, 122.1, 114.0), (64, 1024, 512, 114.0, 106.9),
    (64, 909, 2048, 368.6, 349.0), (64, 766, 512, 68.4, 68.5), (80, 2048, 128, 158.4, 150.5), (80, 847, 124, 40.8, 35.3), (80, 1071, 156, 65.4, 61.7), (80, 331, 512, 40.7, 39.0),
    (80, 512, 448, 56.2, 52.3), (80, 199, 312, 18.3, 15.2), (80, 384, 512, 45.6, 42.8), (80, 768, 400, 88.2, 92.3), (80, 128, 832, 22.5, 23.5), (80, 388, 248, 26.1, 27.6), (80, 1280, 64, 36.5, 37.9),
    (80, 128, 1024, 23.7, 24.7), (80, 1280, 736, 386.7, 358.4), (80, 608, 816, 126.6, 126.0),
]


def test_the_choice_is_about_the_faster_one(plans):
    got = plans([(seq, 1, pairs, 32, dh) for dh, seq, pairs, *_ in MEASURED])
    for (dh, seq, pairs, fewer, full), (per_cu, *_) in zip(MEASURED, got):
        # 2 % and more is what repeated measurements of one size differ by
        assert (full if per_cu == (4 if dh == 64 else 3) else fewer) <= 1.025 * min(fewer, full), (dh, seq, pairs)


# d_head, tokens, pairs, us with one workgroup a CU less than there is room for: persistent, a workgroup per item in groups of pairs, the same
# in one group; the three with all of them (bf16, 256 CUs)
PLANS = [
    (64, 1024, 104, (31.6, 32.7, 24.6, 25.1, 25.1, 25.1)),
    (64, 1024, 128, (32.8, 34.7, 30.1, 27.5, 27.6, 27.6)),
    (64, 1024, 136, (34.2, 36.9, 31.7, 39.6, 39.6, 30.2)),
    (64, 1024, 176, (39.9, 42.1, 37.5, 42.5, 44.4, 37.0)),
    (64, 1024, 256, (51.7, 58.5, 55.1, 53.7, 56.8, 54.2)),
    (64, 1024, 288, (59.8, 61.6, 62.1, 58.8, 63.3, 61.6)),
    (64, 1024, 344, (73.5, 73.7, 74.9, 68.6, 73.5, 74.4)),
    (64, 1024, 464, (94.2, 94.2, 105.2, 96.9, 92.5, 105.6)),
    (64, 768, 192, (31.4, 32.3, 28.7, 41.3, 34.4, 30.1)),
    (64, 768, 320, (43.3, 47.7, 45.2, 52.0, 47.5, 44.9)),
    (64, 768, 464, (63.5, 62.9, 66.9, 64.6, 62.7, 67.0)),
    (64, 896, 288, (53.2, 52.5, 50.8, 58.4, 53.7, 50.1)),
    (64, 896, 392, (80.5, 66.2, 70.7, 69.7, 68.1, 70.0)),
    (64, 1152, 88, (29.7, 29.7, 25.6, 26.0, 26.0, 25.9)),
    (64, 1152, 320, (98.6, 79.8, 84.9, 86.0, 81.9, 84.3)),
    (64, 1152, 368, (100.7, 93.5, 98.9, 114.5, 91.4, 98.5)),
    (64, 1280, 128, (53.9, 45.0, 39.0, 53.4, 49.9, 38.8)),
    (64, 1408, 264, (118.3, 99.3, 100.5, 100.0, 96.2, 97.5)),
    (64, 1536, 160, (67.8, 75.3, 65.2, 81.9, 73.0, 63.1)),
    (64, 1536, 256, (104.7, 103.4, 108.4, 112.6, 108.3, 108.4)),
    (64, 2048, 200, (141.7, 144.4, 132.3, 147.0, 144.2, 129.0)),
    (64, 2048, 240, (169.1, 167.0, 167.2, 166.4, 158.5, 167.4)),
    (64, 2560, 176, (201.6, 183.3, 173.1, 210.6, 175.6, 168.6)),
    (64, 4096, 112, (280.6, 291.7, 263.9, 280.2, 280.0, 257.8)),
    (64, 8192, 120, (1173.7, 1145.2, 1143.0, 1140.0, 1119.5, 1105.4)),
    (64, 8192, 152, (1486.1, 1439.2, 1488.2, 1450.7, 1405.5, 1449.2)),
    (80, 640, 160, (39.3, 32.7, 31.1, 42.4, 32.4, 27.9)),
    (80, 640, 232, (44.8, 44.0, 46.3, 47.2, 48.5, 42.1)),
    (80, 640, 288, (51.8, 48.1, 55.0, 55.3, 51.1, 49.5)),
    (80, 640, 304, (52.0, 54.5, 57.4, 56.0, 52.8, 54.3)),
    (80, 640, 416, (75.2, 70.4, 77.3, 72.4, 68.2, 73.0)),
]


def test_the_plan_over_few_rounds_is_about_the_fastest(plans):
    got = plans([(seq, 1, pairs, 32, dh) for dh, seq, pairs, _ in PLANS])
    for (dh, seq, pairs, us), (per_cu, slots, fill, _) in zip(PLANS, got):
        items, full = pairs // 8 * -(-seq // 128), {64: 4, 80: 3}[dh]
        shape = 2 if fill == items else 0 if slots == 32 * per_cu else 1
        # repeated measurements differ by 2 %; lines that hold for every number of tiles cost up to 5 % at some
        assert us[3 * (per_cu == full) + shape] <= 1.055 * min(us), (dh, seq, pairs)


def test_the_gpu_tests_cases_take_the_plans_they_are_there_for(plans):
    import test_gpu_attention_items as items
    import test_gpu_attention_residency as residency
    cases = items.CASES + residency.CASES
    for case, (per_cu, slots, fill, _) in zip(cases, plans([(seq, heads, n_seq, 32, dh) for n_seq, seq, heads, dh, *_ in cases])):
        n_seq, seq, heads, dh, want_cu, want = case
        count = -(-n_seq * heads // 8) * -(-seq // 128)
        kind = "all" if count <= 32 * per_cu else "one" if fill == count else "persistent" if slots == 32 * per_cu else "groups"
        assert (per_cu, kind) == (want_cu, want), case
