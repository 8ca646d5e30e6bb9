// Prints which way sprnn_weight_gradient takes for each call on standard input: rows cols cus batch block steps, one a line.
#include <cstdio>

#include "sprnn_wgrad_rule.h"

int main() {
  sprnn::WGradCall c;
  long long steps = 0;
  while (std::scanf("%d %d %d %d %d %lld", &c.rows, &c.cols, &c.num_cus, &c.batch, &c.block, &steps) == 6) {
    c.steps = steps;
    c.h_bytes = ((long long)c.cols * c.batch * 4 + 15) / 16 * 16;
    c.tile = sprnn::choose_weight_gradient_tile(c.rows, c.cols, c.num_cus);
    std::puts(sprnn::lane_sums_are_faster(c) ? "lanes" : "product");
  }
  return 0;
}
