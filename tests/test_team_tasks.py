"""The order in which the kernel that does the teams' work again hands out its tasks (csrc/team_tasks.h), replayed on the host: every part of
every problem once in each phase, and nothing that a task waits for behind it, or the kernel would wait for ever."""
import os
import subprocess

import pytest

from paper_2604_10235_amd import build

# Arguments: problems, places for their sums, most parts, whole, workgroups.  Prints the number of tasks; what is wrong, and exits with 1.
REPLAY = r"""
#include <cstdio>
#include <cstdlib>
#include <map>
#include <set>
#include <vector>
#include "team_tasks.h"
using namespace codecomp;
int wrong(const char* what, int phase, int at) { std::printf("%s: phase %d of %d\n", what, phase, at); return 1; }
int main(int, char** argv) {
  const int problems = std::atoi(argv[1]), slots = std::atoi(argv[2]), most = std::atoi(argv[3]), workgroups = std::atoi(argv[5]);
  const bool whole = std::atoi(argv[4]) != 0;
  const TeamTasks t = TeamTasks::make(problems, slots, most, whole, workgroups);
  const int first = whole ? kTeamSums : kTeamLargest;
  std::map<int, std::vector<int>> numbers[4];
  std::map<int, std::set<int>> parts[4];
  int n = 0;
  for (;; ++n) {
    const TeamTaskAt x = t.at(n);
    if (x.at < 0) break;
    if (n > 20000000 || x.phase < first || x.phase > kTeamMasses || x.at >= problems || x.first >= x.last || x.last > most) return wrong("out of bounds", x.phase, x.at);
    numbers[x.phase][x.at].push_back(n);
    for (int p = x.first; p < x.last; ++p) if (!parts[x.phase][x.at].insert(p).second) return wrong("twice", x.phase, x.at);
  }
  for (int more = 0; more < 4 * workgroups; ++more) if (t.at(n + more).at >= 0) return wrong("after the end", 0, n + more);
  for (int at = 0; at < problems; ++at)
    for (int phase = first; phase <= kTeamMasses; ++phase) {
      if ((int)parts[phase][at].size() != most) return wrong("parts left out", phase, at);
      if ((int)numbers[phase][at].size() != t.tasks_of(most, phase)) return wrong("tasks that are counted", phase, at);
      if (phase > first && numbers[phase][at].front() < numbers[phase - 1][at].back()) return wrong("before the phase it waits for", phase, at);
      if (phase == first && at >= slots && numbers[phase][at].front() < numbers[kTeamMasses][at - slots].back()) return wrong("before its place is free", phase, at);
    }
  std::printf("%d\n", n);
}
"""


@pytest.fixture(scope="module")
def replay(tmp_path_factory):
    d = tmp_path_factory.mktemp("tasks")
    src, exe = d / "replay.cpp", d / "replay"
    src.write_text(REPLAY)
    subprocess.run(["g++", "-std=c++17", "-O1", "-D__HIP_PLATFORM_AMD__", "-I", os.path.join(build.ROCM, "include"), "-I", build.CSRC,
                    str(src), "-o", str(exe)], check=True)

    def run(*args):
        r = subprocess.run([str(exe), *map(str, args)], capture_output=True, text=True)
        assert r.returncode == 0, (args, r.stdout)
        return int(r.stdout)
    return run


# One problem; as many places as problems, one less, two and three times fewer, the fewest that the plan leaves; groups that come out even or
# do not; one part and the most (256 half members).
@pytest.mark.parametrize("whole", [0, 1])
@pytest.mark.parametrize("problems,slots", [(1, 1), (2, 2), (3, 3), (7, 7), (8, 7), (112, 38), (112, 37), (113, 36), (256, 16), (300, 8), (100, 3), (1040, 1040), (1040, 1029)])
@pytest.mark.parametrize("most", [2, 6, 128, 256])
def test_tasks(replay, problems, slots, most, whole):
    replay(problems, slots, most, whole, 512)


def test_large_tasks_where_groups_allow_them(replay):
    assert replay(1040, 1029, 6, 1, 512) < 4 * 1040 * 6 and replay(112, 38, 128, 1, 512) == 112 * (64 + 16 + 16 + 64)
    assert replay(16, 16, 80, 0, 512) == 16 * 80 * 3
