// The attention kernels of pq_decode_matrix.hip for 4-bit quantized values.
#define PQ_MATRIX_VB 4
#define PQ_MATRIX_LAUNCH launch_attention_matrix_v4
#include "pq_decode_matrix.hip"
