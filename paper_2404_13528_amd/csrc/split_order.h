// Order of the tasks of the chained split Linears (k_split.hip), apart from the kernel so that the host can run it too: an
// XCD's workgroups take numbers from a counter, every run of group_tasks numbers belongs to a group of rows that the workgroup
// with the run's first number claims, and a task waits until the tasks before it have arrived.
//
// The counters lie in the caller's workspace and are cleared in front of every launch.  Two calls that overlap on one
// workspace (which the interface forbids) overwrite each other's, so nothing read from them is trusted: whatever they hold,
// a group and a task are in range, and every wait ends after `spins` looks (about a second; a task takes microseconds, and a
// wait covers a few of them).  A workgroup whose wait ended that way takes no further task: values are wrong then, as with any
// overlap, but the launch ends.
#pragma once

#if defined(__HIPCC__)
#define SPLIT_HD __host__ __device__ __forceinline__
#else
#define SPLIT_HD inline
#endif

namespace sm {

constexpr int SPLIT_LINE = 32;                    // words of a cache line
constexpr unsigned SPLIT_SPINS = 1u << 21;

struct TaskOrder {
  int* claimed;                                   // groups claimed so far, on all XCDs
  int* mine;                                      // this XCD's line: numbers handed out, then 1 + the group of every run of numbers
  unsigned group_tasks; int n_groups;
  unsigned spins;
  unsigned run_known; int group_known;            // of this workgroup's last number
  bool lost;                                      // a wait was given up
};

// Mem: take(p, v) adds at the XCD's own L2 and look(p) reads there, take_device(p, v) adds for all XCDs; pause()
template <typename Mem> SPLIT_HD int wait_nonzero(TaskOrder& o, int* p) {
  for (unsigned i = 0; i < o.spins; ++i) {
    const int v = Mem::look(p);
    if (v) return v;
    Mem::pause();
  }
  o.lost = true;
  return 0;
}
template <typename Mem> SPLIT_HD void wait_arrivals(TaskOrder& o, int* arrived, int want) {
  for (unsigned i = 0; i < o.spins; ++i) {
    if (Mem::look(arrived) >= want) return;
    Mem::pause();
  }
  o.lost = true;
}
// number n -> task to[0] (-1: no more) of group to[1]
template <typename Mem> SPLIT_HD void task_of(TaskOrder& o, unsigned n, int* to) {
  const unsigned run = n / o.group_tasks, k = n - run * o.group_tasks;
  if (run != o.run_known) {
    int* claim = o.mine + 1 + (run < SPLIT_LINE - 2 ? run : SPLIT_LINE - 2);
    if (k == 0) {
      o.group_known = Mem::take_device(o.claimed, 1);
      Mem::take(claim, (int)((unsigned)o.group_known + 1u));
    } else {
      o.group_known = (int)((unsigned)wait_nonzero<Mem>(o, claim) - 1u);      // the run's first number is with a running workgroup
    }
    o.run_known = run;
  }
  to[0] = !o.lost && (unsigned)o.group_known < (unsigned)o.n_groups ? (int)k : -1;
  to[1] = o.group_known;
}

}  // namespace sm
