// The task queue of k_topk_general: which tasks a draw stands for, when a task may begin and for how long it waits.  Plain
// functions of numbers, so that the queue can be gone through on the host as well.
#pragma once

#include <stdint.h>

namespace compams {

// The part of the general route that a problem is at: the parts before it are done.
enum : uint32_t { kPhaseLevel0 = 0, kPhaseLevel1 = 1, kPhaseLevel2 = 2, kPhaseCount = 3, kGeneralParts = 4 };

struct GeneralTasks {
  uint32_t groups[kGeneralParts];  // (a selection per row) workgroups per row, for each part
  uint32_t total[kGeneralParts];   // tasks of each part
};

// Tasks first, first + stride, ... below total of a part.
struct TaskShare {
  uint32_t part, first, stride, total;
};

// What draw number `drawn` stands for: every part is cut into as many shares as there are workgroups (or tasks, if they are fewer),
// all of one part's before the next one's.  False: nothing is left.  total: tasks of the parts.
__host__ __device__ inline bool share_of(uint32_t drawn, uint32_t workgroups, uint32_t total0, uint32_t total1, uint32_t total2,
                                         uint32_t total3, TaskShare& s) {
  s.part = kPhaseLevel0;
  s.first = drawn;
  s.total = total0;
  s.stride = total0 < workgroups ? total0 : workgroups;
  auto next_part = [&](uint32_t total) {
    if (s.first < s.stride) return;
    s.first -= s.stride;
    ++s.part;
    s.total = total;
    s.stride = total < workgroups ? total : workgroups;
  };
  next_part(total1);
  if (s.part == kPhaseLevel1) next_part(total2);
  if (s.part == kPhaseLevel2) next_part(total3);
  return s.first < s.stride;
}

// The phase in which level 0 leaves a problem.  resolved: it has done level 1's work as well.
__host__ __device__ inline uint32_t phase_after_level0(bool resolved) { return resolved ? kPhaseLevel2 : kPhaseLevel1; }

// A task of a part looks at its problem's phase until the part before is done, but no more than kMostLooks times.  A part takes
// milliseconds at most and a look half a microsecond at least, so the limit, of seconds, is met only if the control blocks are written by
// somebody else meanwhile (calls of compams_step_static that overlap in time): the kernel then ends with wrong results, where without
// a limit it would hold the GPU for good.  Returns the phase that was seen last.
constexpr uint32_t kMostLooks = 1u << 22;
template <typename Look>
__host__ __device__ inline uint32_t wait_for_part(uint32_t part, uint32_t most_looks, Look&& look) {
  uint32_t at = look();
  for (uint32_t looks = 1; at < part && looks < most_looks; ++looks) at = look();
  return at;
}

// What a task of a part does at that phase.
enum TaskTurn { kTurnRun, kTurnSkip, kTurnStop };
__host__ __device__ inline TaskTurn turn_of(uint32_t part, uint32_t at) {
  if (at < part) return kTurnStop;                           // it has given up waiting
  return part == kPhaseLevel1 && at > part ? kTurnSkip : kTurnRun;  // level 0 has done it
}

}  // namespace compams
