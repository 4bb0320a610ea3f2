// The row kernel on rows of any start and length (rowkl.hip, kRagged), as a
// translation unit of its own.
#define TURNKL_RAGGED_ROWS 1
#include "rowkl.hip"
