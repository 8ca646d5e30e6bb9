// Device code of libsprnn: the persistent kernel without run-time options for layers of a single workgroup (or one per part):
// forward passes of the vanilla cells, the LSTM and the GRU.
#include "sprnn_persistent.h"

namespace sprnn {

const void* persistent_solo_kernel_for(int batch, int template_words, int cell) { return pick_plain<kFormSolo>(batch, template_words, cell, false); }

}  // namespace sprnn
