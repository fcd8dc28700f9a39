// The host's upper bound on a table's live count (host arithmetic only).
//
// Every insert call gets a 16-bit tag; its last front-end kernel stores
// (tag << 48) | exact live count to pinned host memory, and `ids_at` remembers
// how many ids all calls up to that one brought.  A call inserts at most its
// ids, so "count published by call T + ids enqueued after T" bounds the live
// count once every enqueued call has run, whichever published count is read,
// however often it is read, and whatever the bound was before.
#pragma once

#include <stdint.h>

#include <algorithm>

namespace rs {

struct LiveBound {
  static constexpr int kTags = 64;
  int64_t bound = 0;
  int64_t tag = 0;   // the newest call's, 1 ... 65535 (0: nothing published)
  int64_t last = 0;  // the newest enqueued call's
  int64_t ids = 0;  // ids of all enqueued calls
  int64_t ids_at[kTags];

  LiveBound() { std::fill(ids_at, ids_at + kTags, int64_t(-1)); }

  // A new call's tag; no refresh from it before `enqueued`.
  int64_t next_tag() {
    tag = tag == 0xFFFF ? 1 : tag + 1;
    ids_at[tag % kTags] = -1;
    return tag;
  }

  // The newest tag's call, of n ids, has been enqueued: the bound is `after`.
  void enqueued(int64_t n, int64_t after) {
    ids += n;
    ids_at[tag % kTags] = ids;
    last = tag;
    bound = after;
  }

  // No enqueued call has yet to publish: the bound can fall no further.
  bool settled(int64_t word) const { return last == 0 || ((word >> 48) & 0xFFFF) == last; }

  // Lower the bound with a published word.
  void refresh(int64_t word) {
    const int64_t t = (word >> 48) & 0xFFFF;
    if (t == 0 || ((tag - t) & 0xFFFF) >= kTags) return;
    const int64_t at = ids_at[t % kTags];
    if (at < 0) return;
    bound = std::min(bound, (word & ((int64_t(1) << 48) - 1)) + (ids - at));
  }
};

}  // namespace rs
