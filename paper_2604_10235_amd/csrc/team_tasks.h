// Tasks of the kernel that does the teams' work again (score_team_again_kernel): a counter hands out numbers, and this says what each
// stands for.  Integers only, so that the same function runs on the host.
#pragma once
#include <hip/hip_runtime.h>

namespace codecomp {

// What is done for a problem, in this order.  A task waits only for tasks of smaller numbers.
enum {
  kTeamSums = 0,       // row sums over a part's keys, to memory; who finishes the last of a problem adds them up: weights of the rows, to memory
  kTeamLargest = 1,    // where a row of the problem is out of range: its largest logits become the references
  kTeamSumsAgain = 2,  // ... and the sums are formed again
  kTeamMasses = 3,     // masses of a part's keys
};

struct TeamTaskAt {
  int phase, at;       // at: position of the problem among those that are done (-1: no task is left)
  int first, last;     // parts [first, last) of the problem
};

// The sums of `slots` problems have a place at a time (problem `at` that of problem at - slots, when that has its masses), each with up
// to `most` parts.  whole: all problems from the start; else only those with rows out of range, without their first phase.
struct TeamTasks {
  int problems, slots, most;
  bool whole;
  int group;           // problems whose tasks of a phase come together
  int common, rare;    // parts that one task takes: of the phases that every problem needs, and of the two that few need
  int tasks_common, tasks_rare, groups, full;      // tasks of a problem in such a phase; groups; tasks of a step in which all stages have a whole group

  // The phases of a group come in stages, each beside the next stage of the groups before, so that nobody waits for a group's last sums
  // while there is other work: whole: sums of group k, then what is left of group k - 1; else largest logits of group k, sums of k - 1, masses of k - 2.
  __host__ __device__ int stages() const { return whole ? 2 : 3; }
  __host__ __device__ static TeamTasks make(int problems, int slots, int most, bool whole, int workgroups) {
    TeamTasks t = {problems, slots, most, whole, 1, 1, 1, 0, 0, 0, 0};
    if (slots >= t.stages()) t.group = slots / t.stages();             // (fewer slots: as many as problems, none waits for its place)
    // More parts to a task where a group still has two tasks for every workgroup: numbers and counters take a few us of a task.
    const int fill = t.group * most / (2 * workgroups);
    t.common = fill < 1 ? 1 : fill < 8 ? fill : 8;
    t.rare = whole ? 8 : t.common;
    t.tasks_common = t.tasks_of(most, kTeamMasses);
    t.tasks_rare = t.tasks_of(most, kTeamLargest);
    t.groups = (problems + t.group - 1) / t.group;
    t.full = t.group * ((whole ? 2 : 1) * t.tasks_common + 2 * t.tasks_rare);
    return t;
  }
  __host__ __device__ static bool is_rare(int phase) { return phase == kTeamLargest || phase == kTeamSumsAgain; }
  __host__ __device__ int tasks_of(int parts, int phase) const {
    const int size = is_rare(phase) ? rare : common;
    return (parts + size - 1) / size;
  }
  __host__ __device__ int group_size(int g) const {
    const int left = problems - g * group;
    return g < 0 || left <= 0 ? 0 : left < group ? left : group;
  }
  // first and last phase of a stage
  __host__ __device__ int phase0(int stage) const { return whole ? stage : stage + 1; }
  __host__ __device__ int phase1(int stage) const { return whole && stage == 1 ? kTeamMasses : phase0(stage); }
  __host__ __device__ TeamTaskAt at(int number) const {
    int x = number;
    for (int step = 0; step < groups + stages() - 1; ++step) {
      if (step == stages() - 1 && groups > stages()) {                 // steps up to the one before the last group's are alike
        const int alike = groups - stages(), skip = x / full < alike ? x / full : alike;
        x -= skip * full;
        step += skip;
      }
      for (int s = 0; s < stages(); ++s) {
        const int g = step - s, here = group_size(g);
        for (int phase = phase0(s); phase <= phase1(s); ++phase) {
          const int tasks = is_rare(phase) ? tasks_rare : tasks_common;
          if (x < here * tasks) {
            const int size = is_rare(phase) ? rare : common, i = x / tasks, first = (x - i * tasks) * size;
            return {phase, g * group + i, first, first + size < most ? first + size : most};
          }
          x -= here * tasks;
        }
      }
    }
    return {0, -1, 0, 0};
  }
};

}  // namespace codecomp
