// Instantiations of the decode kernel (decode_impl.h) for models whose keys and values
// of one sample and layer exceed 32-bit offsets.
#include "decode_impl.h"

namespace fvan {

FVAN_DECODE_WIDE_LIST(FVAN_DECODE_WIDE_INST)

}  // namespace fvan
