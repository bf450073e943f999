// FP64 windowed-lane instances, r = 2, unit-stride rows.
#include "win.h"

namespace cb {

static const WinKernel kTable[] = {CB_WIN_X(2, 8),
                                   CB_WIN_X(2, 10),
                                   CB_WIN_X(2, 12),
                                   CB_WIN_X(2, 16),
                                   CB_WIN_X(2, 20),
                                   CB_WIN_X(2, 24)};

const WinKernel *win_table_r2_x(int *count) {
  *count = (int)(sizeof(kTable) / sizeof(kTable[0]));
  return kTable;
}

}  // namespace cb
