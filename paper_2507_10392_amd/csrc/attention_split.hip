// The matrix-core attention kernels for 16-bit heads below 128, bf16: the same source with split probabilities and dS.
#define ZS_ATTN_SPLIT 1
#include "attention_mfma.hip"
