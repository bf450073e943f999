// FP64 windowed-lane instances, r = 2, strided rows.
#include "win.h"

namespace cb {

static const WinKernel kTable[] = {CB_WIN_S(2, 8),
                                   CB_WIN_S(2, 12),
                                   CB_WIN_S(2, 16)};

const WinKernel *win_table_r2_s(int *count) {
  *count = (int)(sizeof(kTable) / sizeof(kTable[0]));
  return kTable;
}

}  // namespace cb
