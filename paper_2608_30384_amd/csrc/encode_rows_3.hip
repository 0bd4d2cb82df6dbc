// Encoder on 16-lane rows: 3-bit codec, alone or with the second residual (floats, SQ8).
#include "encode_rows.h"

namespace rslm {

template void launch_encode_rows<3, false, false>(const EncodeArgs &, hipStream_t);

}  // namespace rslm
