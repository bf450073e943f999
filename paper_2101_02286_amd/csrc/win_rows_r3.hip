// Windowed-lane instances with coefficients for each lane, r = 3.
#include "win.h"

namespace cb {

static const WinKernel kTable[] = {CB_WIN_ROWS(3, 12, MODE_X),
                                   CB_WIN_ROWS(3, 16, MODE_X),
                                   CB_WIN_ROWS(3, 12, MODE_S),
                                   CB_WIN_ROWS(3, 16, MODE_S)};

const WinKernel *win_table_rows_r3(int *count) {
  *count = (int)(sizeof(kTable) / sizeof(kTable[0]));
  return kTable;
}

}  // namespace cb
