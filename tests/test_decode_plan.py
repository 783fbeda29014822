"""The split plan of a decode call (csrc/planner.cpp), compiled for the host and run on shapes at its edges."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2606_13097_amd", "csrc")
MAX_SEQS = 64   # sequences of a launch
CUS = 256

MAIN = r"""
#include <cstdio>
#include "planner.hpp"
int main() {  // hq hkv d n len...  ->  split_keys max_slots ring
  int hq, hkv, d, n;
  while (std::scanf("%d %d %d %d", &hq, &hkv, &d, &n) == 4) {
    std::vector<int32_t> pos(n);
    for (int32_t& p : pos) if (std::scanf("%d", &p) != 1) return 1;
    const fcg_model_desc desc{1, hq, hkv, d, 1e6, FCG_BF16, 0};
    const fcg::DecodePlan p = fcg::plan_decode(desc, pos, @MAX@);
    std::printf("%lld %d %d\n", (long long)p.split_keys, p.max_slots, p.ring);
  }
}
"""


@pytest.fixture(scope="module")
def plan(tmp_path_factory):
    gxx = shutil.which("g++")
    if not gxx:
        pytest.skip("no host compiler")
    tmp = tmp_path_factory.mktemp("plan")
    src, exe = tmp / "main.cpp", tmp / "plan"
    src.write_text(MAIN.replace("@MAX@", str(MAX_SEQS)))
    subprocess.run([gxx, "-std=c++17", "-O1", "-I", CSRC, "-I", os.path.join(ROOT, "include"), str(src),
                    os.path.join(CSRC, "planner.cpp"), "-o", str(exe)], check=True)

    def run(hq, hkv, d, lens):
        line = " ".join(map(str, [hq, hkv, d, len(lens), *lens]))
        out = subprocess.run([str(exe)], input=line, capture_output=True, text=True, check=True).stdout
        return [int(x) for x in out.split()]
    return run


def _grids(hkv, lens, sk):
    """Blocks of each launch, the empty ones of shorter sequences included."""
    for i in range(0, len(lens), MAX_SEQS):
        part = lens[i:i + MAX_SEQS]
        yield len(part) * max(p // sk + 1 for p in part) * hkv


@pytest.mark.parametrize("hq,hkv,d", [(32, 8, 128), (64, 8, 128), (8, 8, 64), (16, 1, 64)])
@pytest.mark.parametrize("lens", [[1], [4100], [2000], [8190], [30] * 32, [30] * 33, [100] * 64, [50] * 128, [250] * 32,
                                  [300, 3000], [6000] + [90] * 20, [16000], [63, 64, 127, 128], [1000] * 65, [7] * 64])
def test_ring_and_splits(plan, hq, hkv, d, lens):
    """The four-tile ring (128 KB of LDS at D 128, one block per compute unit) only where there are at
    most 256 keys for each unit and the whole launch, empty blocks included, fits one block per compute unit; splits are whole 64-key chunks, at
    most 256 per sequence, and the partial slots cover every launch."""
    sk, slots, ring = plan(hq, hkv, d, lens)
    assert sk >= 64 and sk % 64 == 0
    assert max(p // sk + 1 for p in lens) <= 256
    assert slots == max(sum(p // sk + 1 for p in lens[i:i + MAX_SEQS]) for i in range(0, len(lens), MAX_SEQS))
    few_keys = sum(p + 1 for p in lens) * hkv <= 256 * CUS
    assert ring == (4 if few_keys and max(_grids(hkv, lens, sk)) <= CUS else 2)
