// The matrix-core attention kernels for 16-bit heads below 128, IEEE half.
#define ZS_ATTN_SPLIT 1
#define ZS_ATTN_F16 1
#include "attention_mfma.hip"
