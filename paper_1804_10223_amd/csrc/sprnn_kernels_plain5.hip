// Device code of libsprnn: the persistent kernel without run-time options, for layers whose h takes
// more than four rounds of the copy: forward passes of the vanilla cells, also with binary16 activations, of the LSTM and the GRU,
// and the backward passes.
#include "sprnn_persistent.h"

namespace sprnn {

const void* persistent_plain5_kernel_for(int batch, int template_words, int cell, bool half) {
  return pick_plain<kFormLong>(batch, template_words, cell, half);
}

}  // namespace sprnn
