// Shared by the translation units of the products with a dense matrix.
#pragma once
#include "common.h"

namespace us {

// spmm_panels.hip: Y (+)= A X over entries grouped by row.  row: the row of every entry, or null with `rows` instead.  Rows with
// entries are stored (add: added to), the others left as they are.
void panel_spmm(Env &env, const us_formatted &A, const int32_t *row, const StoredRows *rows, const int32_t *col, const char *name,
                const float *X, int64_t N, int64_t ldx, float *Y, int64_t ldy, bool add);

// ELL: all rows are stored (add: added to)
void panel_ell_spmm(Env &env, const us_formatted &A, const float *X, int64_t N, int64_t ldx, float *Y, int64_t ldy, bool add);

}  // namespace us
