"""The launch plan's arithmetic (csrc/nmc_internal.h), compiled for the host: a
queue grab takes at most 1/64 of a work-group's even share among the
work-groups that the launch has, chunk otherwise; every unit is covered; the
autotuner's candidates are different launches."""
import os
import subprocess

import pytest

from paper_2601_00976_amd import autotune as AT

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

SRC = """
#include <cstdio>
#include "nmc_internal.h"
int main() {
  long long units, rounds;
  int per_cu, cu, bpc, chunk, persistent;
  while (scanf("%lld %d %d %d %d %d %lld", &units, &per_cu, &cu, &bpc, &chunk, &persistent, &rounds) == 7) {
    const nmc_launch L = {bpc, chunk, persistent, 0};
    const nmc::LaunchPlan p = nmc::plan_launch(L, units, per_cu, cu, rounds);
    printf("%lld %d %d\\n", (long long)p.grid, p.chunk, (int)p.queue);
  }
}
"""


@pytest.fixture(scope="module")
def plan(tmp_path_factory):
    d = tmp_path_factory.mktemp("plan")
    (d / "plan.cpp").write_text(SRC)
    inc = [os.path.join(ROOT, "include"), os.path.join(ROOT, "paper_2601_00976_amd", "csrc"), "/opt/rocm/include"]
    subprocess.run(["g++", "-std=c++17", "-D__HIP_PLATFORM_AMD__", *[f"-I{i}" for i in inc], str(d / "plan.cpp"), "-o",
                    str(d / "plan")], check=True, capture_output=True)

    def run(rows):
        text = "\n".join(" ".join(str(int(x)) for x in r) for r in rows)
        out = subprocess.run([str(d / "plan")], input=text, check=True, capture_output=True, text=True).stdout
        return [tuple(int(x) for x in line.split()) for line in out.splitlines()]
    return run


def test_plan(plan):
    rows = [(units, per_cu, cu, bpc, chunk, persistent, rounds)
            for units in (1, 3, 2047, 16384, 32768, 32769, 65536, 262144, 1 << 22) for per_cu in (4, 8) for cu in (1, 256)
            for bpc in (0, 1, 2, 8, 64) for chunk in (1, 3, 4, 4096) for persistent in (0, 1) for rounds in (4, 16)]
    for r, (grid, c, queue) in zip(rows, plan(rows)):
        units, per_cu, cu, bpc, chunk, persistent, rounds = r
        assert 1 <= c <= chunk and grid >= 1, r
        if not persistent:
            assert not queue and c == chunk and (grid - 1) * c < units <= grid * c, r
        elif queue:
            groups = (bpc or per_cu) * cu
            assert c == max(1, min(chunk, units // (64 * groups))), (r, c)
            assert grid <= (bpc or 2 * per_cu) * cu and (grid - 1) * c < units, r
        else:
            assert bpc == 0 and c == 1 and grid == units <= rounds * per_cu * cu, r


@pytest.mark.parametrize("P", [1 << 16, 1 << 22])
def test_candidates_are_different_launches(plan, P):
    cands = [c for c in AT.candidates(P=P) if c.kernel_store == 0]
    plans = plan([((P + 1) // 2, 8, 256, c.blocks_per_cu, c.chunk, c.persistent, 16) for c in cands])
    assert all(q for _, _, q in plans)
    assert len({(c.blocks_per_cu, chunk) for c, (_, chunk, _) in zip(cands, plans)}) == len(cands)
