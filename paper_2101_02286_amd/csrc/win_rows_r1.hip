// Windowed-lane instances with coefficients for each lane, r = 1.
#include "win.h"

namespace cb {

static const WinKernel kTable[] = {CB_WIN_ROWS(1, 8, MODE_X),
                                   CB_WIN_ROWS(1, 12, MODE_X),
                                   CB_WIN_ROWS(1, 16, MODE_X),
                                   CB_WIN_ROWS(1, 8, MODE_S),
                                   CB_WIN_ROWS(1, 12, MODE_S),
                                   CB_WIN_ROWS(1, 16, MODE_S)};

const WinKernel *win_table_rows_r1(int *count) {
  *count = (int)(sizeof(kTable) / sizeof(kTable[0]));
  return kTable;
}

}  // namespace cb
