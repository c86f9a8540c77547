// Host side of the mailboxes that solver kernels post to (Mail, vecops.hpp).
#pragma once

#include <hip/hip_runtime.h>

#include <cstring>
#include <thread>

#include "vecops.hpp"

namespace vd {

// Whether mailbox m holds the whole of post number seq.  The words arrive in any
// order; one that is still the last post's does not fit the check.  A post orders
// nothing but its own words: whatever else a kernel stores to pinned memory is
// read after the stream has been waited for.
inline bool mail_here(const Mail* m, unsigned long long seq) {
  if (__atomic_load_n(&m->seq, __ATOMIC_ACQUIRE) != seq) return false;
  unsigned long long w[2];
  for (int i = 0; i < 2; ++i) w[i] = __atomic_load_n((const unsigned long long*)&m->v[i], __ATOMIC_ACQUIRE);
  const unsigned long long flags = __atomic_load_n(&m->flags, __ATOMIC_ACQUIRE);
  return __atomic_load_n(&m->check, __ATOMIC_ACQUIRE) == mail_check(w[0], w[1], flags, seq);
}

// Waits until mailbox m holds post number seq, which work already on stream st
// will post.  Polls the pinned memory; every few ten microseconds it also asks
// the stream, so that a device error, or a stream that has ended without
// posting, ends the wait (false).
inline bool wait_mail(const Mail* m, unsigned long long seq, hipStream_t st) {
  for (unsigned spin = 1;; ++spin) {
    if (mail_here(m, seq)) return true;
#if defined(__x86_64__)
    __builtin_ia32_pause();
#endif
    if (spin % 1024) continue;
    const hipError_t before = hipPeekAtLastError();
    const hipError_t q = hipStreamQuery(st);
    if (q == hipErrorNotReady) {
      if (before == hipSuccess) (void)hipGetLastError();  // "not ready" is no error of the library's work
      std::this_thread::yield();
      continue;
    }
    return q == hipSuccess && mail_here(m, seq);
  }
}

// The state that a Krylov step posted.
struct StepState {
  double resid = 0, nrm2 = 0;
  bool bad = false, halt = false;
  int nreorth = 0;
};
inline bool wait_step(const Mail* mail, int j, unsigned long long run, hipStream_t st, StepState* t) {
  const Mail& m = mail[MAIL_STEP + (j & 1)];
  if (!wait_mail(&m, run + j + 1, st)) return false;
  t->resid = m.v[0];
  t->nrm2 = m.v[1];
  t->bad = m.flags & 1;
  t->halt = (m.flags >> 1) & 1;
  t->nreorth = (int)(m.flags >> 2);
  return true;
}

// The pinned mailboxes of a new solver state, announced to it on stream st (the
// state's memory must be cleared on that stream before).
inline hipError_t make_mail(Mail** mail, DevState* dst, hipStream_t st) {
  void* dev = nullptr;
  hipError_t e = hipHostMalloc(mail, kMails * sizeof(Mail));
  if (e != hipSuccess) return e;
  std::memset((void*)*mail, 0, kMails * sizeof(Mail));
  e = hipHostGetDevicePointer(&dev, *mail, 0);
  if (e != hipSuccess) return e;
  set_mail(dst, (Mail*)dev, st);
  return hipSuccess;
}

}  // namespace vd
