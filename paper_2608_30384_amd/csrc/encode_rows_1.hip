// Encoder on 16-lane rows: 1-bit codec, alone or with the second residual (floats, SQ8).
#include "encode_rows.h"

namespace rslm {

template void launch_encode_rows<1, false, false>(const EncodeArgs &, hipStream_t);

}  // namespace rslm
