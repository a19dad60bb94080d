// Instances of the encoder kernel (FP16 form, D = 64).
#include "encode_kernel.h"

namespace veckm {

template int launch_layout<2, 4>(const EncArgs&, const EncodeTables&, int, int, hipStream_t);

}  // namespace veckm
