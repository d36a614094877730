// The bulk quantiser for groups of 64 (see quantize_bulk.hip; a translation unit of its own to compile in parallel).
#define INNERQ_BULK_GROUP 64
#include "quantize_bulk.hip"
