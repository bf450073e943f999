// FP64 windowed-lane instances, r = 3, strided rows.
#include "win.h"

namespace cb {

static const WinKernel kTable[] = {CB_WIN_S(3, 16)};

const WinKernel *win_table_r3_s(int *count) {
  *count = (int)(sizeof(kTable) / sizeof(kTable[0]));
  return kTable;
}

}  // namespace cb
