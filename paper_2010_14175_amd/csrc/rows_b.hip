// The setup kernel for matrices of aligned runs of three columns (rows_b.hpp): its instances
// and their choice.
#include "rows_b.hpp"

namespace afsai {

template <int GS, int MMAX, int CAPT, int NB, int WPE>
static RowsKernel b_inst(int mm, int s, int *gs, size_t *lds) {
    *gs = GS;
    *lds = (size_t)(64 / GS) * (size_t)bform::Layout<GS, MMAX, CAPT, NB>::bytes(mm, s);
    return bform::k_rows_b<GS, MMAX, CAPT, NB, WPE>;
}

// nb: new rows per block of the general form for the same rows (rows_w_block)
RowsKernel rows_kernel_b(int n, int mmax, int s, int maxlen, int nb, int *gs_out, size_t *lds_out) {
    if (maxlen > 3 * bform::kRunRow || mmax > 64) return nullptr;
    // Table slots: what the patterns of the 27-point operators touch (99.9% of their rows: 56 runs
    // for 11 positions, 90 for 21, 148 for 46), no more: fewer slots are fewer bytes of LDS (64^3:
    // 12.3 ms with 128 slots, 10.4 ms with 92, 16 wavefronts per CU) and fewer to scan.  150^3: 618 ms
    // with 176 slots, 654 with 192 (10 wavefronts per CU), 625 with 160 (longer probes).  Rows that
    // touch more are redone (rows_kernel_b_large).  New rows per block: the general form's (1, 2, 4),
    // 3 instead of 4 for three or fewer rows a step (the same blocks).  48^3, whole setups, this and the general form: 49 positions 27.3,
    // 40.4 ms; 61 (s = 4, 5) 37.9, 69.1 and 49.4, 72.9; 64 54.3, 105.9.
    // Small systems take the next larger table: redoing even a few rows costs 0.15 ms (a launch and its
    // host round trip), more than 128 slots cost at 24,000 rows (21 positions: kernel 0.39 -> 0.46 ms,
    // setup 0.92 -> 0.84 ms) and less than they cost at 100,000.
    const bool roomy = n < 65536;
    if (nb == 1 && !roomy) return b_inst<32, 24, 64, 1, 4>(mmax, s, gs_out, lds_out);
    if (nb == 1) return b_inst<32, 24, 92, 1, 4>(mmax, s, gs_out, lds_out);
    if (mmax <= 12 && !roomy) return b_inst<32, 24, 64, 2, 4>(mmax, s, gs_out, lds_out);
    if (mmax <= 12) return b_inst<32, 24, 92, 2, 4>(mmax, s, gs_out, lds_out);
    if (mmax <= 24 && roomy) return b_inst<32, 24, 128, 2, 3>(mmax, s, gs_out, lds_out);
    if (mmax <= 24) return b_inst<32, 24, 92, 2, 4>(mmax, s, gs_out, lds_out);
    if (mmax <= 32)
        return s <= 3 ? b_inst<32, 32, 128, 3, 3>(mmax, s, gs_out, lds_out) : b_inst<32, 32, 128, 4, 3>(mmax, s, gs_out, lds_out);
    if (mmax <= 48)
        return s <= 3 ? b_inst<64, 48, 176, 3, 3>(mmax, s, gs_out, lds_out) : b_inst<64, 48, 176, 4, 3>(mmax, s, gs_out, lds_out);
    return s <= 3 ? b_inst<64, 64, 256, 3, 2>(mmax, s, gs_out, lds_out) : b_inst<64, 64, 256, 4, 2>(mmax, s, gs_out, lds_out);
}

// The instance for the rows that overflowed a table of fewer than 176 slots (nullptr: none).  176 runs hold whatever
// the general form's first table (512 entries) does; patterns on other node orders and on irregular meshes touch more
// runs than the first table was made for, and the general form's second table is sized for the worst case, one row to
// a wavefront.  64^3 randomly numbered, 21 positions, 12% of the rows redone: 21.2 -> 15.9 ms (the general form
// alone 26.1; with 256 slots 16.5); a graph of 13 runs a row, 31 positions, 91% of 120,000 rows redone: 18.8 -> 8.9 ms
// (14.8; with 176 slots 10.1).  Where most rows touch more than that too, the pass is lost (27 runs a row, 21 positions:
// 10.9 -> 13.1 ms, the general form alone 16.9).
RowsKernel rows_kernel_b_large(int mmax, int s, int nb, int *gs_out, size_t *lds_out) {
    if (nb == 1) return b_inst<32, 24, 176, 1, 2>(mmax, s, gs_out, lds_out);
    if (mmax <= 24) return b_inst<32, 24, 176, 2, 2>(mmax, s, gs_out, lds_out);
    if (mmax > 32) return nullptr;
    return s <= 3 ? b_inst<64, 48, 256, 3, 2>(mmax, s, gs_out, lds_out) : b_inst<64, 48, 256, 4, 2>(mmax, s, gs_out, lds_out);
}

}  // namespace afsai
