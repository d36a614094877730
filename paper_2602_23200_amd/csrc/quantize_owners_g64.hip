// Ring owners for groups of 64 (see quantize_owners.hip; a translation unit of its own to compile in parallel).
#define INNERQ_OWNERS_GROUP 64
#include "quantize_owners.hip"
