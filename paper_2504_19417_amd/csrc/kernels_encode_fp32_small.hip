// Instances of the encoder kernel (FP32 form, D = 16, 32 and 48).
#include "encode_kernel.h"

namespace veckm {

template int launch_layout<4, 1>(const EncArgs&, const EncodeTables&, int, int, hipStream_t);
template int launch_layout<4, 2>(const EncArgs&, const EncodeTables&, int, int, hipStream_t);
template int launch_layout<4, 3>(const EncArgs&, const EncodeTables&, int, int, hipStream_t);

}  // namespace veckm
