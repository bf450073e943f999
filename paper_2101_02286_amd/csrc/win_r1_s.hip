// FP64 windowed-lane instances, r = 1, strided rows.
#include "win.h"

namespace cb {

static const WinKernel kTable[] = {CB_WIN_S(1, 8),
                                   CB_WIN_S(1, 12),
                                   CB_WIN_S(1, 16)};

const WinKernel *win_table_r1_s(int *count) {
  *count = (int)(sizeof(kTable) / sizeof(kTable[0]));
  return kTable;
}

}  // namespace cb
