// Interface of the long-prompt kernels (pv_kernels_prefill.hip).
#pragma once
#include "pv_internal.h"

#define PV_PRE_MIN 64           // up to this many rows the kernels of the running block are the better ones (they take no more)

struct pv_pre_out { const uint16_t *xop; const float *ssq; };   // LM-head operand and sums of squares of the kept rows

size_t pv_pre_bytes(const pv_model *m, int rows);         // buffers of passes of up to `rows` rows (a multiple of 64; 0: no long-prompt path)
int pv_pre_init(const pv_model *m);
// rows tokens through all layers; the first rows - keep are committed, the last `keep` (a multiple of 16 rows behind the
// start) are left as the cache's running block
int pv_pre_block(pv_cache *c, const int32_t *d_host_tokens, int rows, int keep, pv_pre_out *out, hipStream_t s);
