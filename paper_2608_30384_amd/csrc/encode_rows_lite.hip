// Encoder on 16-lane rows: Rslm4Lite, alone or with the second residual (floats, SQ8).
#include "encode_rows.h"

namespace rslm {

template void launch_encode_rows<4, true, false>(const EncodeArgs &, hipStream_t);

}  // namespace rslm
