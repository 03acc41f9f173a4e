// The grouped angle quantizer's attention with 2-bit values.
#define PQ_GROUPED_VB 2
#define PQ_GROUPED_LAUNCH launch_attention_grouped_v2
#include "pq_decode_grouped.hip"
