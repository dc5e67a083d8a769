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

// Tasks first .. end - 1 of a part.
struct TaskRange {
  uint32_t first, end;
};

// Every part is cut into as many shares as there are workgroups.  Consecutive tasks: a share is then much the same
// problem in every part.  (A part has 4096 tasks at most.)
__host__ __device__ inline TaskRange tasks_of(uint32_t share, uint32_t shares, uint32_t total) {
  return TaskRange{share * total / shares, (share + 1) * total / shares};
}

// Shares are drawn from kQueues counters, as many shares from each as there are workgroups that begin with it: draws from
// one counter follow one another 13 ns apart.  (512 of them: the last workgroup began 8 us after the launch.)
constexpr uint32_t kQueues = 16;
__host__ __device__ inline uint32_t queue_shares(uint32_t queue, uint32_t shares) {
  return (shares + kQueues - 1 - queue) / kQueues;
}

// The next share for a workgroup: its first one from its own queue; further ones, after level 0's tasks of that, only if
// there are queues with some left, so that all shares belong to workgroups that are running before anybody waits.
// left(): the queues with some left, a bit each; draw(q): how many were drawn from q before.  Returns `shares` if there
// is none.
template <typename Left, typename Draw>
__host__ __device__ inline uint32_t next_share(uint32_t workgroup, bool first, uint32_t shares, Left&& left, Draw&& draw) {
  uint32_t q = workgroup % kQueues;
  for (;;) {
    if (!first) {
      const uint32_t some = left();
      if (!some) return shares;
      q = static_cast<uint32_t>(__builtin_ctz(some));
    }
    first = false;
    const uint32_t drawn = draw(q);
    if (drawn < queue_shares(q, shares)) return drawn * kQueues + q;
  }
}

// The phase in which level 0 leaves a problem.  resolved: it has done level 1's work as well.
__host__ __device__ inline uint32_t phase_after_level0(bool resolved) { return resolved ? kPhaseLevel2 : kPhaseLevel1; }

// A task of a part looks at its problem's phase until the part before is done, but no more than kMostLooks times.  A part
// takes milliseconds at most and a look half a microsecond at least, so the limit, of seconds, is met only if the control
// blocks are written by somebody else meanwhile (calls of compams_step_static that overlap in time): the kernel then ends
// with wrong results, where without a limit it would hold the GPU for good.  Returns the phase that was seen last.
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
