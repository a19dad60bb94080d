// Instances of the encoder kernel (FP32 form, D = 128).
#include "encode_kernel.h"

namespace veckm {

template int launch_layout<4, 8>(const EncArgs&, const EncodeTables&, int, int, hipStream_t);

}  // namespace veckm
