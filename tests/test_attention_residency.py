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
