// Windowed-lane instances with coefficients for each lane, r = 2.
#include "win.h"

namespace cb {

static const WinKernel kTable[] = {CB_WIN_ROWS(2, 8, MODE_X),
                                   CB_WIN_ROWS(2, 12, MODE_X),
                                   CB_WIN_ROWS(2, 16, MODE_X),
                                   CB_WIN_ROWS(2, 8, MODE_S),
                                   CB_WIN_ROWS(2, 12, MODE_S),
                                   CB_WIN_ROWS(2, 16, MODE_S)};

const WinKernel *win_table_rows_r2(int *count) {
  *count = (int)(sizeof(kTable) / sizeof(kTable[0]));
  return kTable;
}

}  // namespace cb
