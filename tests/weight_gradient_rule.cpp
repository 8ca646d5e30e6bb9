// Prints which way sprnn_weight_gradient takes for each call on standard input: rows cols cus batch steps, one a line.
#include <cstdio>

#include "sprnn_wgrad_rule.h"

int main() {
  sprnn::WGradCall c;
  long long steps = 0;
  while (std::scanf("%d %d %d %d %lld", &c.rows, &c.cols, &c.num_cus, &c.batch, &steps) == 5) {
    c.steps = steps;
    c.tile = sprnn::choose_weight_gradient_tile(c.rows, c.cols, c.num_cus);
    std::puts(sprnn::lane_sums_are_faster(c) ? "lanes" : "product");
  }
  return 0;
}
