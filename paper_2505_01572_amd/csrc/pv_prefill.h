// Interface of the long-prompt kernels (pv_kernels_prefill.hip).
#pragma once
#include "pv_internal.h"

#define PV_PRE_MIN 64           // up to this many rows the kernels of the running block are the better ones (they take no more)

struct pv_pre_out { const uint16_t *xop; const float *ssq; };   // LM-head operand and sums of squares of the kept rows

int pv_pre_rows(const pv_model *m, int max_tokens);       // rows a cache's buffers are laid out for (0: no long-prompt path)
size_t pv_pre_bytes(const pv_model *m, int max_tokens);
int pv_pre_init(const pv_model *m);
// rows tokens through all layers; the first rows - keep are committed, the last `keep` (a multiple of 16 rows behind the
// start) are left as the cache's running block
int pv_pre_block(pv_cache *c, char *base, const int32_t *d_host_tokens, int rows, int keep, pv_pre_out *out, hipStream_t s);
