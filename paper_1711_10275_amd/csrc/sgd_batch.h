// Which of a list of parameter tensors one launch of the update may take (host
// code without HIP, so that a test can run it on made-up addresses).
#pragma once

#include <algorithm>
#include <cstdint>

namespace sscn {

// Tensors of one launch: their table is 2.8 KB of the 4 KB that a kernel's
// arguments may have.
constexpr int kSgdTensors = 64;
// Elements of a tensor per workgroup.
constexpr int kSgdPer = 1024;
// Workgroups of one launch (1G elements; a grid may have 2^32 threads, 2^24
// workgroups).  A tensor of more goes alone.
constexpr int64_t kSgdGroups = 1 << 20;

inline int64_t sgd_groups(int64_t count) { return (count + kSgdPer - 1) / kSgdPer; }

// The number of leading tensors (n >= 1 of them, empty ones included) that one
// launch updates as if one after another: at most kSgdTensors of kSgdGroups
// workgroups in all, and none that shares memory with an earlier one, unless
// both only read there.
template <class Tensor>
int sgd_batch(const Tensor* t, int n) {
  struct Range {
    uintptr_t lo, hi;
    bool written;
    int tensor;
  };
  Range r[4 * kSgdTensors];
  int ranges = 0, taken = 0, k = 0;
  int64_t groups = 0;
  const auto add = [&](const void* p, int64_t bytes, bool written) {
    const uintptr_t lo = reinterpret_cast<uintptr_t>(p);
    r[ranges++] = Range{lo, lo + (uintptr_t)bytes, written, k};
  };
  for (; k < n && taken < kSgdTensors; ++k) {
    if (t[k].count == 0) continue;
    groups += sgd_groups(t[k].count);
    if (taken > 0 && groups > kSgdGroups) break;
    ++taken;
    add(t[k].params, 4 * t[k].count, true);
    add(t[k].grads, 4 * t[k].count, false);
    add(t[k].momentum_buf, 4 * t[k].count, true);
    if (t[k].params_bf16) add(t[k].params_bf16, 2 * t[k].count, true);
  }
  // As a rule nothing meets: one pass over the ranges by their starts shows it.
  Range s[4 * kSgdTensors];
  std::copy(r, r + ranges, s);
  std::sort(s, s + ranges, [](const Range& a, const Range& b) { return a.lo < b.lo; });
  uintptr_t written_to = 0, read_to = 0;
  bool meets = false;
  for (int i = 0; i < ranges && !meets; ++i) {
    meets = s[i].lo < written_to || (s[i].written && s[i].lo < read_to);
    uintptr_t& to = s[i].written ? written_to : read_to;
    to = std::max(to, s[i].hi);
  }
  if (!meets) return k;
  for (int i = 1; i < ranges; ++i)  // by tensors: the first that meets an earlier one
    for (int j = 0; j < i; ++j)
      if (r[j].tensor != r[i].tensor && (r[i].written || r[j].written) && r[i].lo < r[j].hi && r[j].lo < r[i].hi)
        return r[i].tensor;
  return k;
}

}  // namespace sscn
