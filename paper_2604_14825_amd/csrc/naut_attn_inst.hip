// naut_attn_inst.hip -- the kernel instantiations of one (input type, output type) pair and some head widths.
//
// Compiled once per pair and widths with -DNAUT_INST_IN=<naut_dtype> -DNAUT_INST_OUT=<naut_dtype> (bf16/bf16,
// bf16/f32, f16/f16, f16/f32) -DNAUT_INST_W=64|96|128|256 (96: both 80 and 96; 256: both 192 and 256), so that they build in parallel; naut_attn.hip declares
// these launchers extern and holds none of the kernels.
#include "naut_attn_kernels.h"

#if !defined(NAUT_INST_IN) || !defined(NAUT_INST_OUT) || !defined(NAUT_INST_W)  // a bare compile of this file
#undef NAUT_INST_IN
#undef NAUT_INST_OUT
#undef NAUT_INST_W
#define NAUT_INST_IN NAUT_BF16
#define NAUT_INST_OUT NAUT_BF16
#define NAUT_INST_W 128
#endif

namespace naut_k {

#if NAUT_INST_W == 64
template int launch<64, NAUT_INST_IN, NAUT_INST_OUT>(Params, int, hipStream_t);
#elif NAUT_INST_W == 96
template int launch<80, NAUT_INST_IN, NAUT_INST_OUT>(Params, int, hipStream_t);
template int launch<96, NAUT_INST_IN, NAUT_INST_OUT>(Params, int, hipStream_t);
#elif NAUT_INST_W == 128
template int launch<128, NAUT_INST_IN, NAUT_INST_OUT>(Params, int, hipStream_t);
#else
template int launch<192, NAUT_INST_IN, NAUT_INST_OUT>(Params, int, hipStream_t);
template int launch<256, NAUT_INST_IN, NAUT_INST_OUT>(Params, int, hipStream_t);
#endif

}  // namespace naut_k
