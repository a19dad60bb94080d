// Instances of the encoder kernel (FP32 form, D = 64).
#include "encode_kernel.h"

namespace veckm {

template int launch_layout<4, 4>(const EncArgs&, const EncodeTables&, int, int, hipStream_t);

}  // namespace veckm
