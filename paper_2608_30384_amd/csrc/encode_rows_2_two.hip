// Encoder on 16-lane rows: 2-bit codec, with a 2-bit RSLM second stage.
#include "encode_rows.h"

namespace rslm {

template void launch_encode_rows<2, false, true>(const EncodeArgs &, hipStream_t);

}  // namespace rslm
