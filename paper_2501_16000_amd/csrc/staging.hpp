// staging.hpp -- copies from the device to a caller's pageable array, and the
// check of the fields that come in.
//
// A pageable hipMemcpyAsync brings 18.9 MB (the populations of 512^2) back in 1050
// us; the link takes 340 us.  Larger copies therefore go through a few pinned
// pieces, so that the link fills one while the host empties another: populations
// of 512^2 1210 -> 760 us, of 2000^2 27.2 -> 22.0 ms (most of it the caller's new
// pages), moments of 2000^2 5.4 -> 3.8 ms.  To the device the runtime's own path
// is as fast as these pieces (520 us).
//
// Small results (sums, profiles, moments of the smallest lattices) go through one
// pinned block: one wait for the stream, then a copy by the host.  lb_diagnostics of
// 32^2, us alone / behind 10 / 50 steps: a pageable copy 32 / 41 / 88, one after a wait
// for the stream 43 / 51 / 88, pinned 25 / 33 / 69; moments of 16^2 (6 KB) 30 / 35 / 49,
// 39 / 45 / 59 and 20 / 27 / 42; of 32^2 (24 KB) 28 / 36 / 92, 28 / 37 / 68 and 28 / 35 /
// 78, so larger results wait first.  The block costs 25 us when it is allocated: a
// lattice that is read once has its pageable copy.
#pragma once

#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>
#include <cstdint>
#include <cstring>
#include <limits>

namespace oreg {

// The pinned memory of one lattice: a block for small results, from the second one
// on, and pieces for larger ones, each allocated by the first copy that takes it and
// freed with the lattice.  If they cannot be had, copies stay pageable.
struct PinnedPieces {
  static constexpr int kPieces = 4;
  static constexpr size_t kBytes = 1 << 20, kSmall = 16 << 10;
  char* base = nullptr;
  hipEvent_t done[kPieces] = {};
  bool refused = false;
  char* small = nullptr;
  bool small_refused = false, small_read = false;

  bool small_ready() {
    if (small || small_refused) return small != nullptr;
    if (!small_read) {  // the first one
      small_read = true;
      return false;
    }
    if (hipHostMalloc((void**)&small, kSmall, hipHostMallocDefault) == hipSuccess) return true;
    (void)hipGetLastError();  // not an error of the caller's
    small = nullptr;
    small_refused = true;
    return false;
  }

  bool ready() {
    if (base || refused) return base != nullptr;
    int made = 0;
    if (hipHostMalloc((void**)&base, kPieces * kBytes, hipHostMallocDefault) == hipSuccess) {
      while (made < kPieces &&
             hipEventCreateWithFlags(&done[made], hipEventDisableTiming) == hipSuccess)
        ++made;
      if (made == kPieces) return true;
    } else {
      base = nullptr;
    }
    (void)hipGetLastError();  // not an error of the caller's
    while (made > 0) (void)hipEventDestroy(done[--made]);
    if (base) (void)hipHostFree(base);
    base = nullptr;
    refused = true;
    return false;
  }
  void release() {
    if (small) (void)hipHostFree(small);
    small = nullptr;
    if (!base) return;
    for (int i = 0; i < kPieces; ++i) (void)hipEventDestroy(done[i]);
    (void)hipHostFree(base);
    base = nullptr;
  }
};

// The copies of one call on one stream, to consecutive places.  to_host may return
// before the data is in dst: finish() completes it.  A call that fails in between leaves nothing in
// flight behind.
class HostTransfer {
 public:
  // bytes: what the call moves in all.  Between the small block and 1.5 MB the
  // runtime's own path is faster (moments of 200^2, 0.96 MB: 65 against 72 us; of
  // 256^2: 105 against 101), and no memory is pinned for it.
  HostTransfer(PinnedPieces& p, hipStream_t s, size_t bytes)
      : p_(p),
        s_(s),
        few_(bytes <= PinnedPieces::kSmall),
        small_(few_ && p.small_ready()),
        pinned_(bytes >= 1500000 && p.ready()) {}
  ~HostTransfer() {
    if (busy_) (void)hipStreamSynchronize(s_);
  }
  HostTransfer(const HostTransfer&) = delete;
  HostTransfer& operator=(const HostTransfer&) = delete;

  hipError_t to_host(void* dst, const void* src, size_t bytes) {
    if (small_) {
      if (used_ + bytes > PinnedPieces::kSmall) return hipErrorInvalidValue;
      busy_ = true;
      if (used_ == 0) first_ = static_cast<char*>(dst);
      const hipError_t e = hipMemcpyAsync(p_.small + used_, src, bytes, hipMemcpyDeviceToHost, s_);
      used_ += bytes;
      return e;
    }
    if (!pinned_) {
      // The runtime waits for the stream by itself, but 25 us longer from seven
      // queued launches on (32^2, 50 steps and moments: 89 us, 66 with the wait
      // here), unless there is little to copy.
      const hipError_t e = few_ ? hipSuccess : hipStreamSynchronize(s_);
      return e != hipSuccess ? e : hipMemcpyAsync(dst, src, bytes, hipMemcpyDeviceToHost, s_);
    }
    busy_ = true;
    for (size_t at = 0; at < bytes; at += PinnedPieces::kBytes) {
      const size_t n = std::min(PinnedPieces::kBytes, bytes - at);
      const int i = next_;
      next_ = (next_ + 1) % PinnedPieces::kPieces;
      hipError_t e = empty(i);
      if (e != hipSuccess) return e;
      e = hipMemcpyAsync(p_.base + i * PinnedPieces::kBytes, static_cast<const char*>(src) + at, n,
                         hipMemcpyDeviceToHost, s_);
      if (e == hipSuccess) e = hipEventRecord(p_.done[i], s_);
      if (e != hipSuccess) return e;
      to_[i] = static_cast<char*>(dst) + at;
      count_[i] = n;
    }
    return hipSuccess;
  }
  hipError_t finish() {
    for (int i = 0; i < PinnedPieces::kPieces; ++i) {
      const hipError_t e = empty(next_);
      if (e != hipSuccess) return e;
      next_ = (next_ + 1) % PinnedPieces::kPieces;
    }
    const hipError_t e = hipStreamSynchronize(s_);
    if (e == hipSuccess) busy_ = false;
    if (e == hipSuccess && used_ > 0) std::memcpy(first_, p_.small, used_);
    return e;
  }

 private:
  // Waits for piece i and moves what it brought to its place.
  hipError_t empty(int i) {
    if (!to_[i]) return hipSuccess;
    const hipError_t e = hipEventSynchronize(p_.done[i]);
    if (e == hipSuccess) std::memcpy(to_[i], p_.base + i * PinnedPieces::kBytes, count_[i]);
    to_[i] = nullptr;
    return e;
  }

  PinnedPieces& p_;
  hipStream_t s_;
  bool few_, small_, pinned_, busy_ = false;
  size_t used_ = 0;        // bytes of the small block
  char* first_ = nullptr;  // where they go
  int next_ = 0;
  char* to_[PinnedPieces::kPieces] = {};
  size_t count_[PinnedPieces::kPieces] = {};
};

// First node from which fields have to be looked at one by one (one with a value
// that is not finite or rho <= 0 is among the next kCheck nodes), or n.  Without
// an early exit per node the check runs on vectors.  All arrays in one loop: one
// after the other in blocks of kCheck, the check waited for memory (12.0 ms for
// 2048^2 nodes, 8.7 with an exit per node, 6.4 like this).
constexpr int64_t kCheck = 1024;
template <int D>
inline int64_t first_suspect_fields(const double* rho, const double* const (&u)[D], int64_t n) {
  constexpr double most = std::numeric_limits<double>::max();
  for (int64_t c0 = 0; c0 < n; c0 += kCheck) {
    const int64_t end = std::min(c0 + kCheck, n);
    int bad = 0;
    for (int64_t c = c0; c < end; ++c) {
      int b = (int)!(rho[c] > 0.0) | (int)!(rho[c] <= most);
#pragma unroll
      for (int a = 0; a < D; ++a) b |= (int)!(std::fabs(u[a][c]) <= most);
      bad |= b;
    }
    if (bad) return c0;
  }
  return n;
}

}  // namespace oreg
