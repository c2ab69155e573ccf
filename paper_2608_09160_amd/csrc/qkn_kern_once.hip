// libqkn: the register-path kernels of one token per wavefront (the kernel templates are in qkn_kernels.h).

#include "qkn_kernels.h"

namespace qkn_dev {

#define QKN_ONCE_ROW(F, A)                                                                                      \
  {qkn_rows_once<F, A, 0, kFused>, qkn_rows_once<F, A, 1, kFused>, qkn_rows_once<F, A, 2, kFused>, \
   qkn_rows_once<F, A, 4, kFused>
#define QKN_ONCE_ROW16(A) QKN_ONCE_ROW(FmtBf16, A), qkn_rows_once<FmtBf16, A, 8, kFused>}
#define QKN_ONCE_ROW8(A) QKN_ONCE_ROW(FmtFp8, A), nullptr}
#define QKN_ONCE_SET16(M)                                                    \
  {qkn_rows_once<FmtBf16, 1, 0, M>, qkn_rows_once<FmtBf16, 2, 0, M>, \
   qkn_rows_once<FmtBf16, 4, 0, M>, qkn_rows_once<FmtBf16, 8, 0, M>}
#define QKN_ONCE_SET8(M) \
  {qkn_rows_once<FmtFp8, 1, 0, M>, qkn_rows_once<FmtFp8, 2, 0, M>, qkn_rows_once<FmtFp8, 4, 0, M>, nullptr}

const RowsFn kOnceFusedTable[2][4][5] = {
    {QKN_ONCE_ROW16(1), QKN_ONCE_ROW16(2), QKN_ONCE_ROW16(4), QKN_ONCE_ROW16(8)},
    {QKN_ONCE_ROW8(1), QKN_ONCE_ROW8(2), QKN_ONCE_ROW8(4), {nullptr, nullptr, nullptr, nullptr, nullptr}}};
const RowsFn kOnceApplyTable[2][4] = {QKN_ONCE_SET16(kApply), QKN_ONCE_SET8(kApply)};
const RowsFn kOncePartialTable[2][4] = {QKN_ONCE_SET16(kPartial), QKN_ONCE_SET8(kPartial)};

}  // namespace qkn_dev
