// The grouped angle quantizer's attention with 4-bit values.
#define PQ_GROUPED_VB 4
#define PQ_GROUPED_LAUNCH launch_attention_grouped_v4
#include "pq_decode_grouped.hip"
