// What a context remembers of its recent eager calls to choose the launches of
// the next: plain host code over words that the device stores into host-mapped
// memory, read back without waiting.
#pragma once

#include <stdint.h>

namespace fgbd {

// What predicts the sweeps that a call needs: the entry point, the clouds in
// the call and the magnitude (power of two) of its size.  Calls of one kind follow each
// other's counts only: with one record for the whole context, a 1M-point frame
// of 4 sweeps after a batch that needed 31 was given 32 launches for its next
// eight calls.
enum CallEntry { kCallDenoise = 0, kCallBatched, kCallFilter };
struct CallKind {
  int32_t entry, clouds, magnitude;
  bool operator==(const CallKind &o) const {
    return entry == o.entry && clouds == o.clouds && magnitude == o.magnitude;
  }
};
inline CallKind call_kind(int entry, int clouds, int64_t n) {
  int32_t m = 0;
  for (; n > 1; n >>= 1) ++m;
  return {entry, clouds, m};
}

// Sweep counts of recent calls.  The last finalising launch of a call that
// asked for it stores each cloud's count and the call's tag in one word; a
// later call reads them once every cloud's word carries the tag.  (No events:
// each one recorded left the GPU idle for about 6 us.)
class SweepCounts {
 public:
  static constexpr int kKinds = 8;   // records kept, the least recently used goes
  static constexpr int kRecent = 8;  // counts per record

  bool pending() const { return pending_; }

  // Takes the outstanding counts into their record once they are all there.
  void poll(const int32_t *words) {
    if (!pending_) return;
    int32_t most = 0;
    for (int i = 0; i < clouds_; ++i) {
      const int32_t v = __atomic_load_n(&words[i], __ATOMIC_ACQUIRE);
      if (tag_of(v) != tag_) return;
      most = (v & 0xffff) > most ? v & 0xffff : most;
    }
    Record &r = record(asked_);
    r.recent[r.at] = most;
    r.at = (r.at + 1) % kRecent;
    r.count += r.count < kRecent ? 1 : 0;
    pending_ = false;
  }

  // A call of this kind asks for its counts (none may be outstanding).
  // Returns the tag for its words, which are cleared: tags come round again,
  // and a word that a larger batch left long ago must not pass for a new one.
  int32_t ask(const CallKind &kind, int clouds, int32_t *words) {
    tag_ = tag_ == 0x7fff0000u ? 0x10000u : tag_ + 0x10000u;
    for (int i = 0; i < clouds; ++i) __atomic_store_n(&words[i], 0, __ATOMIC_RELEASE);
    pending_ = true;
    asked_ = kind;
    clouds_ = clouds;
    return (int32_t)tag_;
  }

  // The call that asked failed: its launches may or may not have been
  // enqueued, so later calls ask anew, and the words are in use until the
  // device has been waited for.
  void cancel() {
    pending_ = false;
    unsure_ = true;
  }

  // Whether a wait for the device has to come before the words are freed
  // whatever they hold, and whether launches may still store counts.
  bool unsure() const { return unsure_; }
  bool outstanding(const int32_t *words) const {
    for (int i = 0; pending_ && i < clouds_; ++i)
      if (tag_of(__atomic_load_n(&words[i], __ATOMIC_ACQUIRE)) != tag_) return true;
    return false;
  }

  // Separate sweep launches for a call of this kind: the most that its recent
  // calls needed where those agree, one more where they do not, within
  // 1..limit; `unknown` before any count was read.
  int launches(const CallKind &kind, int unknown, int limit) {
    const Record &r = record(kind);
    if (r.count == 0) return unknown;
    int32_t most = 0, least = INT32_MAX;
    for (int i = 0; i < r.count; ++i) {
      most = r.recent[i] > most ? r.recent[i] : most;
      least = r.recent[i] < least ? r.recent[i] : least;
    }
    const int want = (r.count >= 2 && least == most) ? most : most + 1;  // steady counts: no spare launch
    return want < 1 ? 1 : (want < limit ? want : limit);
  }

 private:
  static uint32_t tag_of(int32_t word) { return (uint32_t)word & ~0xffffu; }
  struct Record {
    CallKind kind = {-1, 0, 0};
    int32_t recent[kRecent] = {0};
    int32_t count = 0, at = 0;
    uint64_t used = 0;
  };
  Record &record(const CallKind &kind) {
    Record *old = &records_[0];
    for (Record &r : records_) {
      if (r.kind == kind) {
        r.used = ++clock_;
        return r;
      }
      if (r.used < old->used) old = &r;
    }
    *old = Record();
    old->kind = kind;
    old->used = ++clock_;
    return *old;
  }
  Record records_[kKinds];
  uint64_t clock_ = 0;
  bool pending_ = false, unsure_ = false;
  uint32_t tag_ = 0;  // of the outstanding counts: 15 bits above the count's 16
  CallKind asked_ = {-1, 0, 0};
  int clouds_ = 0;
};

// The mark that a context's schedule was chosen, over trials of candidates: set
// while they run (they bound the trial calls' sweep launches), and after them
// only if a schedule was kept; a tuning that fails leaves the mark as it was.
class ScheduleTrial {
 public:
  explicit ScheduleTrial(bool &chosen) : chosen_(chosen), before_(chosen) {}
  ~ScheduleTrial() { chosen_ = kept_ || before_; }
  ScheduleTrial(const ScheduleTrial &) = delete;
  ScheduleTrial &operator=(const ScheduleTrial &) = delete;
  void start() { chosen_ = true; }
  void keep() { kept_ = true; }

 private:
  bool &chosen_;
  const bool before_;
  bool kept_ = false;
};

// The radix sort's route.  words[0] is set by the local sort of a call that
// asked when it found a very large range (points crowded into few top code
// digits, such as a plane normal to a scan axis), words[1] by the launch after
// that sort, to the call's number.  Once a call was found crowded, the next
// ones sort by LSD passes, until one that asks again is not: every kCalls'th
// does, and those that are made before its answer is there keep to the passes
// (calls made ahead of the GPU, half of them, took the crowded route at first:
// 924 us a call for a million points in one plane on a 2^11 grid, 400 so).
class SortWatch {
 public:
  static constexpr int kCalls = 32;

  // Whether a call sorts by LSD passes.
  bool lsd(const int32_t *words) {
    const bool crowded = last_crowded(words);
    if (left_ == 0) return crowded && pending_;
    --left_;
    return true;
  }

  // Whether the last call that asked was crowded (a captured call goes by that).
  bool last_crowded(const int32_t *words) {
    if (pending_ && __atomic_load_n(&words[1], __ATOMIC_ACQUIRE) == seq_) {
      crowded_ = __atomic_load_n(&words[0], __ATOMIC_RELAXED) != 0;
      left_ = crowded_ ? kCalls : 0;
      pending_ = false;
    }
    return crowded_;
  }

  bool pending() const { return pending_; }

  // A call asks (none may be outstanding).  Returns its number.
  int32_t ask(int32_t *words) {
    __atomic_store_n(&words[0], 0, __ATOMIC_RELEASE);
    seq_ = seq_ == INT32_MAX ? 1 : seq_ + 1;
    pending_ = true;
    return seq_;
  }

  // As in SweepCounts.
  void cancel() {
    pending_ = false;
    unsure_ = true;
  }
  bool unsure() const { return unsure_; }
  bool outstanding(const int32_t *words) const {
    return pending_ && __atomic_load_n(&words[1], __ATOMIC_ACQUIRE) != seq_;
  }

 private:
  int32_t seq_ = 0, left_ = 0;
  bool pending_ = false, unsure_ = false, crowded_ = false;
};

}  // namespace fgbd
