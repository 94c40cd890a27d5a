// The bound of a mailbox wait (plain C++, no device code, so it can be
// checked on its own).
//
// A round of a wait is a gather past the caches, whose time depends on the
// graph and on how many wavefronts wait with it (1 us to some 20 us), so the
// bound is a time: about a second of the device's constant-rate clock, looked
// at every kWaitCheck rounds together with the launch's failure flag.  The
// clock starts at the first look, so a wait of fewer rounds never reads it.
#pragma once

#ifdef __HIPCC__
#define FM_HOST_DEVICE __host__ __device__
#else
#define FM_HOST_DEVICE
#endif

constexpr unsigned kWaitCheck = 256;                     // rounds between two looks
constexpr unsigned long long kWaitTicks = 100000000ull;  // one second of the 100 MHz clock

struct WaitBound {
  unsigned rounds = 0;
  bool timed = false;
  unsigned long long start = 0;

  // After a round that did not find what it waits for: whether to go on.
  // `now` reads the clock, `failed` whether some wavefront of the launch has
  // given up (true ends the wait too).
  template <typename Now, typename Failed>
  FM_HOST_DEVICE bool go_on(Now now, Failed failed) {
    if (++rounds % kWaitCheck != 0) return true;
    const unsigned long long t = now();
    if (!timed) {
      timed = true;
      start = t;
    }
    return t - start < kWaitTicks && !failed();
  }
};
