// FP64 windowed-lane instances, r = 3, unit-stride rows.
#include "win.h"

namespace cb {

static const WinKernel kTable[] = {CB_WIN_X(3, 16)};

const WinKernel *win_table_r3_x(int *count) {
  *count = (int)(sizeof(kTable) / sizeof(kTable[0]));
  return kTable;
}

}  // namespace cb
