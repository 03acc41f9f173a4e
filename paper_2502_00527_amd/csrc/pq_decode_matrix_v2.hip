// The attention kernels of pq_decode_matrix.hip for 2-bit quantized values.
#define PQ_MATRIX_VB 2
#define PQ_MATRIX_LAUNCH launch_attention_matrix_v2
#include "pq_decode_matrix.hip"
