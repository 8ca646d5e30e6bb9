// Follows csrc/sprnn_contest.h with made-up mappings.  Standard input: batch, most lanes, then one mapping a line,
//   parts lanes grid  compact us  backward backward_weights weights noalloc  proposed_grid
// (lanes 0 and grid 0 of a request stand for the first line that fits; the first line of all is the packer's own mapping).  A
// request that no line answers cannot be had.  Prints what is kept, what is behind it, every request, and handles not released.
#include <cstdio>
#include <vector>

#include "sprnn_contest.h"

struct Made { sprnn::Facts facts; int grid = 0, proposed = 0; };
struct Handle { const Made* made; };

struct Builder {
  const std::vector<Made>& made;
  int alive = 0, live_at_most = 0;
  Handle* take(const Made& m) { alive += 1; if (alive > live_at_most) live_at_most = alive; return new Handle{&m}; }
  Handle* build(const sprnn::Request& r, const Handle* incumbent, sprnn::Alternative* proposed) {
    std::printf("asked parts %d lanes %d grid %d against %d/%d\n", r.parts, r.lanes, r.alternative.grid, incumbent->made->facts.parts, incumbent->made->facts.lanes);
    for (const Made& m : made)
      if (m.facts.parts == r.parts && (r.lanes == 0 || m.facts.lanes == r.lanes) && m.grid == r.alternative.grid) {
        if (proposed) proposed->grid = m.proposed;
        return take(m);
      }
    return nullptr;
  }
  sprnn::Facts facts(const Handle* h) const { return h->made->facts; }
  void release(Handle* h) { alive -= 1; delete h; }
};

int main() {
  int batch = 0, most = 0;
  if (std::scanf("%d %d", &batch, &most) != 2) return 1;
  std::vector<Made> made;
  int compact, b, bw, w, n;
  for (Made m; std::scanf("%d %d %d %d %f %d %d %d %d %d", &m.facts.parts, &m.facts.lanes, &m.grid, &compact, &m.facts.us, &b, &bw, &w, &n, &m.proposed) == 10;) {
    m.facts.compact = compact; m.facts.can.backward = b; m.facts.can.backward_weights = bw; m.facts.can.weights = w; m.facts.can.noalloc = n;
    made.push_back(m);
  }
  Builder builder{made};
  Handle* const first = builder.take(made.at(0));
  sprnn::Alternative alternative;
  alternative.grid = made[0].proposed;
  const sprnn::Winner<Handle> winner = sprnn::contest(builder, first, alternative, batch, most);
  const sprnn::Facts& k = winner.kept->made->facts;
  std::printf("kept parts %d lanes %d grid %d us %.2f\n", k.parts, k.lanes, winner.kept->made->grid, k.us);
  if (winner.whole) std::printf("behind parts %d lanes %d grid %d us %.2f\n", winner.whole->made->facts.parts, winner.whole->made->facts.lanes, winner.whole->made->grid, winner.whole->made->facts.us);
  std::printf("left %d\n", builder.alive - 1 - (winner.whole ? 1 : 0));
  delete winner.whole;
  delete winner.kept;
  return 0;
}
