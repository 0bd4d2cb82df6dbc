// Encoder on 16-lane rows: Rslm4Lite, with a 2-bit RSLM second stage.
#include "encode_rows.h"

namespace rslm {

template void launch_encode_rows<4, true, true>(const EncodeArgs &, hipStream_t);

}  // namespace rslm
