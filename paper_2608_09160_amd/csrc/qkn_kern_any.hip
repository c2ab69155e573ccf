// libqkn: the register-resident kernels for rows of any width and alignment (the kernel templates are in qkn_kernels.h).

#include "qkn_kernels.h"

namespace qkn_dev {

#define QKN_ANY_ROW(F, M, A)                                                                     \
  {qkn_rows<F, A, 0, M, 0, true>, qkn_rows<F, A, 1, M, 0, true>, qkn_rows<F, A, 2, M, 0, true>, \
   qkn_rows<F, A, 4, M, 0, true>
#define QKN_ANY_ROW16(M, A) QKN_ANY_ROW(FmtBf16, M, A), qkn_rows<FmtBf16, A, 8, M, 0, true>}
#define QKN_ANY_ROW8(M, A) QKN_ANY_ROW(FmtFp8, M, A), nullptr}
#define QKN_ANY_ONE16(M)                                                              \
  {qkn_rows<FmtBf16, 1, 0, M, 0, true>, qkn_rows<FmtBf16, 2, 0, M, 0, true>,         \
   qkn_rows<FmtBf16, 4, 0, M, 0, true>, qkn_rows<FmtBf16, 8, 0, M, 0, true>}
#define QKN_ANY_ONE8(M)                                                           \
  {qkn_rows<FmtFp8, 1, 0, M, 0, true>, qkn_rows<FmtFp8, 2, 0, M, 0, true>,       \
   qkn_rows<FmtFp8, 4, 0, M, 0, true>, nullptr}

const RowsFn kAnyFusedTable[2][4][5] = {
    {QKN_ANY_ROW16(kFused, 1), QKN_ANY_ROW16(kFused, 2), QKN_ANY_ROW16(kFused, 4),
     QKN_ANY_ROW16(kFused, 8)},
    {QKN_ANY_ROW8(kFused, 1), QKN_ANY_ROW8(kFused, 2), QKN_ANY_ROW8(kFused, 4),
     {nullptr, nullptr, nullptr, nullptr, nullptr}}};
const RowsFn kAnyApplyTable[2][4] = {QKN_ANY_ONE16(kApply), QKN_ANY_ONE8(kApply)};
const RowsFn kAnyPartialTable[2][4] = {QKN_ANY_ONE16(kPartial), QKN_ANY_ONE8(kPartial)};

}  // namespace qkn_dev
