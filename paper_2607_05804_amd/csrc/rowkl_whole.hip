// The row kernel with one workgroup per row (rowkl.hip, kWhole), as a
// translation unit of its own.
#define TURNKL_WHOLE_ROWS 1
#include "rowkl.hip"
