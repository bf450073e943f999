// FP64 windowed-lane instances, r = 1, unit-stride rows.
#include "win.h"

namespace cb {

static const WinKernel kTable[] = {CB_WIN_X(1, 8),
                                   CB_WIN_X(1, 10),
                                   CB_WIN_X(1, 12),
                                   CB_WIN_X(1, 16),
                                   CB_WIN_X(1, 20),
                                   CB_WIN_X(1, 24)};

const WinKernel *win_table_r1_x(int *count) {
  *count = (int)(sizeof(kTable) / sizeof(kTable[0]));
  return kTable;
}

}  // namespace cb
