// The setup kernel for matrices of aligned runs of three columns (rows_b.hpp): its instances
// and their choice.
#include "rows_b.hpp"

namespace afsai {

template <int GS, int MMAX, int CAPT, int NB, int WPE>
static RowsKernel b_inst(int mm, int *gs, size_t *lds) {
    *gs = GS;
    *lds = (size_t)(64 / GS) * (size_t)bform::Layout<GS, MMAX, CAPT, NB>::bytes(mm);
    return bform::k_rows_b<GS, MMAX, CAPT, NB, WPE>;
}

RowsKernel rows_kernel_b(int mmax, int maxlen, int *gs_out, size_t *lds_out) {
    if (maxlen > 3 * bform::kRunRow || mmax > 64) return nullptr;
    if (mmax <= 24) return b_inst<32, 24, 128, 2, 3>(mmax, gs_out, lds_out);
    if (mmax <= 32) return b_inst<32, 32, 160, 4, 3>(mmax, gs_out, lds_out);
    if (mmax <= 48) return b_inst<64, 48, 176, 4, 3>(mmax, gs_out, lds_out);
    return b_inst<64, 64, 256, 4, 2>(mmax, gs_out, lds_out);
}

}  // namespace afsai
