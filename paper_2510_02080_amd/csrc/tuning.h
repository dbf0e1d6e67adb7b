// Launch shapes of the point passes, and the shapes that autotuning has kept: host
// code without HIP, so that the rule below can be checked without a GPU.
#pragma once

#include <stdint.h>

#include <algorithm>
#include <vector>

namespace s3a {

struct LaunchCfg {
  int wg = 256;
  int items = 4;
  int occupancy = 4;  // workgroups per CU (0: one per tile)
  int window = 0;     // pairs per window in the persistent launch (0: all)
};

inline int size_class(int64_t n_points) {
  int c = 0;
  while (n_points > 65536 && c < 12) {
    n_points >>= 2;
    ++c;
  }
  return c;
}

// 1, up to 4, 16, 64, ... pairs.
inline int pair_class(int64_t n_pairs) {
  int c = 0;
  for (; n_pairs > 1; n_pairs = (n_pairs + 3) / 4) ++c;
  return c;
}

// What autotuning found for the kinds of calls it was run on: a shape, or that the
// untuned call was fastest. A call takes what was found for its own kind (input type,
// points, pairs, persistent launch or not). One whose kind was not tuned takes the shape
// found last for its type and points, as before kinds were told apart by pairs, unless
// its passes can solve for themselves, which no shape's do: that is worth a seventh to a
// sixth of such a call (one pair of 3,072 points 99 us against 119, 20 of 200,000 260
// against 299), and a batch of another kind says nothing about it.
class TuneTable {
 public:
  void record(int dtype, int64_t n_points, int64_t n_pairs, bool persistent, const LaunchCfg* shape) {
    const Entry e{dtype, size_class(n_points), pair_class(n_pairs), persistent, shape != nullptr,
                  shape ? *shape : LaunchCfg{}};
    entries_.erase(std::remove_if(entries_.begin(), entries_.end(), [&](const Entry& o) { return o.same_kind(e); }),
                   entries_.end());
    entries_.push_back(e);
  }

  // The shape of a call, or null: untuned. solving: its passes could solve for themselves.
  const LaunchCfg* find(int dtype, int64_t n_points, int64_t n_pairs, bool persistent, bool solving) const {
    const Entry k{dtype, size_class(n_points), pair_class(n_pairs), persistent, false, LaunchCfg{}};
    for (const Entry& e : entries_)
      if (e.same_kind(k)) return e.shaped ? &e.cfg : nullptr;
    return solving ? nullptr : last(dtype, n_points);
  }

  // The shape found last for calls of this type and points, or null.
  const LaunchCfg* last(int dtype, int64_t n_points) const {
    for (auto e = entries_.rbegin(); e != entries_.rend(); ++e)
      if (e->dtype == dtype && e->size == size_class(n_points)) return e->shaped ? &e->cfg : nullptr;
    return nullptr;
  }

 private:
  struct Entry {
    int dtype, size, pairs;
    bool persistent, shaped;
    LaunchCfg cfg;
    bool same_kind(const Entry& o) const {
      return dtype == o.dtype && size == o.size && pairs == o.pairs && persistent == o.persistent;
    }
  };
  std::vector<Entry> entries_;
};

}  // namespace s3a
