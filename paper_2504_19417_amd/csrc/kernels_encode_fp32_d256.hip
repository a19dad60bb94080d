// Instances of the encoder kernel (FP32 form, D = 256).
#include "encode_kernel.h"

namespace veckm {

template int launch_layout<4, 16>(const EncArgs&, const EncodeTables&, int, int, hipStream_t);

}  // namespace veckm
