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
  const bool disturb = std::atoi(argv[4]) != 0, late = seed % 2;
  std::mt19937 rng(seed);
  std::vector<Problem> problems(n);
  for (Problem& p : problems) { p.fast = rng() % 3 == 0; p.resolved = rng() % 2 == 0; }
  GeneralTasks tasks;
  for (uint32_t part = 0; part < kGeneralParts; ++part) {
    tasks.groups[part] = 1 + rng() % 9;
    tasks.total[part] = tasks.groups[part] * n;
  }
  std::atomic<uint32_t> queues[kQueues]{}, wrong{0}, gave_up{0}, ended{0};
  auto workgroup = [&](uint32_t w) {
    std::vector<uint32_t> held;
    for (uint32_t part = 0; part < kGeneralParts; ++part) {
      for (uint32_t i = 0; part == 0 || i < held.size(); ++i) {
        if (part == 0) {
          if (held.size() == workgroups) break;
          auto left = [&] {
            uint32_t some = 0;
            for (uint32_t queue = 0; queue < kQueues; ++queue) some |= (queues[queue] < queue_shares(queue, workgroups) ? 1u : 0u) << queue;
            return some;
          };
          const uint32_t share = next_share(w, i == 0, workgroups, left, [&](uint32_t queue) { return queues[queue].fetch_add(1); });
          if (share >= workgroups) break;
          held.push_back(share);
        }
        const TaskRange range = tasks_of(held[i], workgroups, tasks.total[part]);
        for (uint32_t q = range.first; q < range.end; ++q) {
          Problem& p = problems[q / tasks.groups[part]];
          if (p.fast) continue;
          uint32_t at = 0;
          if (part)
            at = wait_for_part(part, disturb ? 2000u : kMostLooks, [&] {
              std::this_thread::yield();
              return p.phase.load();
            });
          const TaskTurn turn = turn_of(part, at);
          if (turn == kTurnStop) { ++gave_up; return; }
          if (turn == kTurnSkip) {
            if (!p.resolved && !disturb) ++wrong;
            continue;
          }
          if (part && !disturb) {
            const uint32_t before = part - 1 - (part == kPhaseLevel2 && p.resolved ? 1u : 0u);
            if (p.done[before] < tasks.groups[before]) ++wrong;
          }
          ++p.begun[part];
          if (q % 5 == seed % 5) std::this_thread::yield();
          if (++p.done[part] == tasks.groups[part] && part < kPhaseCount)
            p.phase = part == kPhaseLevel0 ? phase_after_level0(p.resolved) : part + 1;
        }
      }
    }
  };
  std::vector<std::thread> threads;
  // (late: every second workgroup finds no place to run until another one has ended)
  for (uint32_t w = 0; w < workgroups; ++w)
    threads.emplace_back([&, w] {
      while (late && w % 2 && !ended) std::this_thread::yield();
      workgroup(w);
      ++ended;
    });
  for (int i = 0; disturb && i < 50 && ended < workgroups; ++i) {
    for (Problem& p : problems) p.phase = kPhaseLevel0;
    for (auto& queue : queues) queue = 0;
    std::this_thread::yield();
  }
  for (std::thread& t : threads) t.join();
  if (!disturb)
    for (Problem& p : problems)
      for (uint32_t part = 0; part < kGeneralParts; ++part)
        if (p.begun[part] != (p.fast || (part == kPhaseLevel1 && p.resolved) ? 0u : tasks.groups[part])) ++wrong;
  std::printf("wrong %u gave_up %u\n", wrong.load(), gave_up.load());
  return wrong || (!disturb && gave_up) ? 1 : 0;
}
