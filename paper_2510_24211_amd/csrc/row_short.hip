// The row kernels (row.hip) built a third time for short rows: 256 threads per row, rows of at most
// 2048 ids.  See the note at the head of row.hip.
#define SCD_ROW_SHORT 1
#include "row.hip"
