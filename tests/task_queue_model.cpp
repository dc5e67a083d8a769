// Goes through the task queue of the one-launch selection on the host: a thread stands for a workgroup.  Arguments: seed, workgroups,
// problems, disturb (0 or 1).  Undisturbed, every task runs once, after its problem's part before, and level 1's only where level 0 has
// left it; disturbed, the phases and the queue are set back meanwhile, and every workgroup has to end all the same.
#define __host__
#define __device__
#include "compams_tasks.h"

#include <atomic>
#include <cstdio>
#include <cstdlib>
#include <random>
#include <thread>
#include <vector>

using namespace compams;

struct Problem {
  bool fast, resolved;  // found by the band kernel; level 0 does level 1's work
  std::atomic<uint32_t> phase{kPhaseLevel0}, begun[kGeneralParts]{}, done[kGeneralParts]{};
};

int main(int, char** argv) {
  const uint32_t seed = std::atoi(argv[1]), workgroups = std::atoi(argv[2]), n = std::atoi(argv[3]);
  const bool disturb = std::atoi(argv[4]) != 0;
  std::mt19937 rng(seed);
  std::vector<Problem> problems(n);
  for (Problem& p : problems) { p.fast = rng() % 3 == 0; p.resolved = rng() % 2 == 0; }
  GeneralTasks tasks;
  for (uint32_t part = 0; part < kGeneralParts; ++part) {
    tasks.groups[part] = 1 + rng() % 9;
    tasks.total[part] = tasks.groups[part] * n;
  }
  std::atomic<uint32_t> queue{0}, wrong{0}, gave_up{0}, ended{0};
  auto workgroup = [&] {
    for (;;) {
      TaskShare s;
      if (!share_of(queue.fetch_add(1), workgroups, tasks.total[0], tasks.total[1], tasks.total[2], tasks.total[3], s)) return;
      for (uint32_t q = s.first; q < s.total; q += s.stride) {
        Problem& p = problems[q / tasks.groups[s.part]];
        if (p.fast) continue;
        if (s.part) {
          const uint32_t at = wait_for_part(s.part, disturb ? 2000u : kMostLooks, [&] {
            std::this_thread::yield();
            return p.phase.load();
          });
          const TaskTurn turn = turn_of(s.part, at);
          if (turn == kTurnStop) { ++gave_up; return; }
          if (turn == kTurnSkip) {
            if (!p.resolved) ++wrong;
            continue;
          }
          const uint32_t before = s.part - 1 - (s.part == kPhaseLevel2 && p.resolved ? 1u : 0u);
          if (p.done[before] < tasks.groups[before]) ++wrong;
        }
        ++p.begun[s.part];
        if (q % 5 == seed % 5) std::this_thread::yield();
        if (++p.done[s.part] == tasks.groups[s.part] && s.part < kPhaseCount)
          p.phase = s.part == kPhaseLevel0 ? phase_after_level0(p.resolved) : s.part + 1;
      }
    }
  };
  std::vector<std::thread> threads;
  for (uint32_t w = 0; w < workgroups; ++w) threads.emplace_back([&] { workgroup(); ++ended; });
  for (int i = 0; disturb && i < 50 && ended < workgroups; ++i) {
    for (Problem& p : problems) p.phase = kPhaseLevel0;
    queue = 0;
    std::this_thread::yield();
  }
  for (std::thread& t : threads) t.join();
  if (!disturb)
    for (Problem& p : problems)
      for (uint32_t part = 0; part < kGeneralParts; ++part)
        if (p.begun[part] != (p.fast || (part == kPhaseLevel1 && p.resolved) ? 0u : tasks.groups[part])) ++wrong;
  std::printf("wrong %u gave_up %u\n", wrong.load(), gave_up.load());
  return !disturb && (wrong || gave_up) ? 1 : 0;
}
