// The row kernels (row.hip) built a third time for short rows: 256 threads per row, rows of at most
// kRowShortMaxN ids in windows of at most kRowShortMaxL positions.  See the note at the head of row.hip.
#define SCD_ROW_SHORT 1
#include "row.hip"
