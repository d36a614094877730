// The fused inner-grouped kernels for the contiguous store, groups of 64 (see attention_inner.hip).
#define INNERQ_PAGED_STORE 0
#define INNERQ_INNER_JOIN 0
#define INNERQ_INNER_LAUNCH launch_inner_g64
#define INNERQ_INNER_GROUP 64
#include "attention_inner.hip"
