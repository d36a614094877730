// The fused inner-grouped kernels that join their partials, for a paged store, groups of 64 (see attention_inner.hip).
#define INNERQ_PAGED_STORE 1
#define INNERQ_INNER_JOIN 1
#define INNERQ_INNER_LAUNCH launch_join_paged_g64
#define INNERQ_INNER_GROUP 64
#include "attention_inner.hip"
