// Threads of GPU workgroups as fibers of one CPU thread, for tests of code in
// which many threads take part: a fiber runs until it gives way (at a barrier,
// or wherever its environment calls give_way), and a scheduler picks the next.
//
//  ROUND_ROBIN  one after another
//  PRIORITY     the runnable fiber of the highest priority; priorities are
//               random, change at random (one in 64 steps) and fall to the
//               bottom when a fiber naps in a wait, so that a thread can be as
//               late, at any one point, as it can be on a GPU
#pragma once
#include <setjmp.h>
#include <stdint.h>
#include <sys/mman.h>
#include <ucontext.h>

#include <vector>

namespace fibers {

enum { ROUND_ROBIN = 0, PRIORITY = 1 };
enum { OK = 0, MISMATCH = -100, HANG = -101 };

struct Barrier {
  uint32_t size = 0, in = 0;
  uint64_t passed = 0;
  int line = 0;  // where the threads now waiting called it
};

class Pool {
 public:
  Pool(int policy, uint64_t seed, uint64_t max_steps)
      : policy_(policy), rng_(seed * 2654435761u + 88172645463325252ull), max_steps_(max_steps) {}
  ~Pool() {
    for (Fiber& f : f_) munmap(f.stack, STACK);
  }

  // body(i) for every i < n, each on a fiber; OK, MISMATCH (threads of one
  // barrier at different calls of it) or HANG (max_steps passed).
  template <class F>
  int run(uint32_t n, F& body) {
    call_ = [](void* b, uint32_t i) { (*static_cast<F*>(b))(i); };
    body_ = &body;
    f_.resize(n);
    for (Fiber& f : f_) {
      f.stack = mmap(nullptr, STACK, PROT_READ | PROT_WRITE, MAP_PRIVATE | MAP_ANONYMOUS, -1, 0);
      f.prio = (int64_t)(random() >> 2);
    }
    uint32_t left = n;
    current = 0;
    self() = this;
    while (left && !failed_) {
      if (++steps > max_steps_) return HANG;
      const int i = pick();
      if (i < 0) return HANG;  // every one waits at a barrier
      current = (uint32_t)i;
      resume(f_[current]);
      if (f_[current].done) --left;
    }
    return failed_;
  }

  void give_way() { leave(f_[current]); }
  // A step of a wait: the others first.
  void nap() {
    f_[current].prio = --lowest_;
    give_way();
  }
  // The barrier `b`, called at `line`.
  void wait(Barrier& b, int line) {
    if (b.in && b.line != line) fail(MISMATCH);
    b.line = line;
    if (++b.in == b.size) {
      b.in = 0;
      ++b.passed;
      give_way();
    } else {
      f_[current].at = &b;
      f_[current].seen = b.passed;
      give_way();
    }
  }
  void fail(int code) {
    if (!failed_) failed_ = code;
    give_way();
  }
  uint64_t random() {
    rng_ ^= rng_ << 13;
    rng_ ^= rng_ >> 7;
    return rng_ ^= rng_ << 17;
  }

  uint32_t current = 0;
  uint64_t steps = 0;

 private:
  static constexpr size_t STACK = 256 << 10;
  struct Fiber {
    ucontext_t uc;
    jmp_buf jb;
    void* stack = nullptr;
    bool started = false, done = false;
    const Barrier* at = nullptr;
    uint64_t seen = 0;
    int64_t prio = 0;
  };
  static Pool*& self() {
    static thread_local Pool* p;
    return p;
  }
  static void start() {
    Pool* p = self();
    p->call_(p->body_, p->current);
    p->f_[p->current].done = true;
    p->leave(p->f_[p->current]);
  }
  bool runnable(Fiber& f) {
    if (f.at && f.at->passed != f.seen) f.at = nullptr;
    return !f.done && !f.at;
  }
  int pick() {
    const uint32_t n = (uint32_t)f_.size();
    if (policy_ == ROUND_ROBIN) {
      for (uint32_t k = 1; k <= n; ++k)
        if (runnable(f_[(current + k) % n])) return (int)((current + k) % n);
      return -1;
    }
    if (random() % 64 == 0) f_[random() % n].prio = (int64_t)(random() >> 2);
    int best = -1;
    for (uint32_t i = 0; i < n; ++i)
      if (runnable(f_[i]) && (best < 0 || f_[i].prio > f_[best].prio)) best = (int)i;
    return best;
  }
  // (a context is made once; switches are setjmp's, without system calls)
  __attribute__((noinline)) void resume(Fiber& f) {
    if (_setjmp(back_)) return;
    if (f.started) _longjmp(f.jb, 1);
    f.started = true;
    getcontext(&f.uc);
    f.uc.uc_stack.ss_sp = f.stack;
    f.uc.uc_stack.ss_size = STACK;
    f.uc.uc_link = nullptr;
    makecontext(&f.uc, start, 0);
    setcontext(&f.uc);
  }
  __attribute__((noinline)) void leave(Fiber& f) {
    if (!_setjmp(f.jb)) _longjmp(back_, 1);
  }

  int policy_;
  uint64_t rng_, max_steps_;
  int failed_ = 0;
  int64_t lowest_ = 0;
  std::vector<Fiber> f_;
  jmp_buf back_;
  void (*call_)(void*, uint32_t) = nullptr;
  void* body_ = nullptr;
};

}  // namespace fibers
