// Which of several mappings of one matrix sprnn_create keeps: no device code and no HIP, so that every course it can take is
// followed on the CPU with made-up times (tests/mapping_contest.cpp).
#ifndef SPRNN_CONTEST_H
#define SPRNN_CONTEST_H

#include <algorithm>

namespace sprnn {

// The calls that a handle offers and that its mapping decides (forward passes it always offers).
struct Abilities {
  bool backward = false;          // sprnn_backward
  bool backward_weights = false;  // sprnn_*_backward*_with_weights
  bool weights = false;           // sprnn_weight_gradient
  bool noalloc = false;           // sprnn_forward_noalloc

  // Everything that `other` can do.
  bool cover(const Abilities& other) const {
    return (backward || !other.backward) && (backward_weights || !other.backward_weights) && (weights || !other.weights) && (noalloc || !other.noalloc);
  }
};

// A second mapping worth measuring against the library's own choice (0 = none): fewer, larger workgroups that fit one
// XCD, or more wavefronts per workgroup so that the copy of h issues fewer surplus loads.
struct Alternative {
  int grid = 0;
  int fill_waves = 0;
  bool any() const { return grid != 0 || fill_waves != 0; }
};

struct Request {   // what is asked of a contending mapping (0: the packer's choice)
  int parts = 1, lanes = 0;
  Alternative alternative;
};

struct Facts {     // what is known of a mapping that was built and measured
  int parts = 1, lanes = 1;
  bool compact = false;
  float us = 0.0f, with_weights_us = 0.0f;   // per step (0: not measured)
  Abilities can;
};

// Shorter by enough to count.  Like with like: by the plain pass alone unless both were measured with the weight gradient as well.
inline bool is_faster(const Facts& a, const Facts& b) {
  const bool both = a.with_weights_us > 0.0f && b.with_weights_us > 0.0f;
  return a.us > 0.0f && a.us + (both ? a.with_weights_us : 0.0f) < 0.98f * (b.us + (both ? b.with_weights_us : 0.0f));
}

template <class Handle>
struct Winner {
  Handle* kept = nullptr;
  Handle* whole = nullptr;   // `kept` has several parts: the handle of the same lanes with all samples in one
};

// `Builder`: Handle* build(const Request&, const Handle* incumbent, Alternative*) (null: that mapping cannot be had),
// Facts facts(const Handle*), void release(Handle*).  `first` is the packer's own mapping, `alternative` what it proposed beside it.
// Whatever fails, `first` or something faster is kept; nothing that `first` can do is lost by another one's being faster, so which
// calls a handle offers does not depend on times; and a mapping of several parts is kept only when the handle behind it is there.
template <class Handle, class Builder>
Winner<Handle> contest(Builder& builder, Handle* first, const Alternative& alternative, int batch, int most_lanes) {
  const Abilities needed = builder.facts(first).can;
  // the fastest handle of each number of lanes (2^i) with all samples in one part, and the fastest of these
  Handle* whole[8] = {};
  auto slot = [&](int lanes) -> Handle*& {
    int i = 0;
    while (i < 7 && (1 << i) < lanes) ++i;
    return whole[i];
  };
  slot(builder.facts(first).lanes) = first;
  Handle* best = first;
  auto contend_whole = [&](const Request& request) {
    Handle* const other = builder.build(request, best, nullptr);
    if (!other) return;
    const Facts f = builder.facts(other);
    Handle*& same_lanes = slot(f.lanes);
    if (!f.can.cover(needed) || (same_lanes && !is_faster(f, builder.facts(same_lanes)))) { builder.release(other); return; }
    if (is_faster(f, builder.facts(best))) best = other;
    if (same_lanes) builder.release(same_lanes);   // (if that was the best, `other` is faster than it)
    same_lanes = other;
  };
  // (1) fewer, larger workgroups on one XCD, or a wavefront count that copies h with fewer loads
  if (alternative.any()) contend_whole({1, 0, alternative});
  // (2) The lanes a row is spread over: the packer's rule of thumb (at least eight nonzeros per lane) is not the best
  // for every shape; twice and half as many lanes are measured too, each with the mapping the packer picks for it.
  auto other_lanes = [&](int lanes, auto&& contend) {
    for (const int l : {lanes * 2, lanes / 2})
      if (l >= batch && l >= 1 && l <= most_lanes) contend(l);
  };
  other_lanes(builder.facts(best).lanes, [&](int l) { contend_whole({1, l, Alternative()}); });
  // (3) The samples shared out to several groups of workgroups (see persistent_kernel): every number that the batch can be
  // divided into, each with the packer's mapping and its alternative; then the lanes of the best.  All the handle's calls add a
  // row's products in one order, which is that of all samples in one part with these lanes: only lanes of which there is
  // such a handle come into question, and not where it copies only the columns that its rows read (the order then follows
  // their places).
  Handle* split = nullptr;
  auto contend_split = [&](const Request& request, Alternative* proposed) {
    Handle* const other = builder.build(request, split ? split : best, proposed);
    if (!other) return;
    const Facts f = builder.facts(other);
    const Handle* const behind = slot(f.lanes);
    Abilities can = f.can;   // (the weight gradients are the other handle's)
    if (behind) { can.weights = builder.facts(behind).can.weights; can.backward_weights = builder.facts(behind).can.backward_weights; }
    if (!behind || builder.facts(behind).compact || !can.cover(needed) || !is_faster(f, builder.facts(split ? split : best))) {
      builder.release(other);
      return;
    }
    if (split) builder.release(split);
    split = other;
  };
  for (int parts = 2; parts <= batch; parts *= 2) {
    Alternative proposed;
    contend_split({parts, 0, Alternative()}, &proposed);
    if (proposed.any()) contend_split({parts, 0, proposed}, nullptr);
  }
  if (split) {
    const Facts f = builder.facts(split);
    other_lanes(f.lanes, [&](int l) { contend_split({f.parts, l, Alternative()}, nullptr); });
  }
  Winner<Handle> w;
  w.kept = split ? split : best;
  w.whole = split ? slot(builder.facts(split).lanes) : nullptr;
  for (Handle*& h : whole)
    if (h && h != w.kept && h != w.whole) builder.release(h);
  return w;
}

}  // namespace sprnn
#endif
