// Instantiates the EM kernels for D = 1 with float iterations.
#include "gm_compress_impl.h"

namespace gm {

int launch_compress_d1_float(int kmax_tpl, int per_thread, int mode, int waves, const CompressArgs& a, int grid,
                          hipStream_t st)
{
    return launch_bucket_dr<1, float>(kmax_tpl, per_thread, mode, waves, a, grid, st);
}

int grid_compress_d1_float(int kmax_tpl, int per_thread, int mode, int waves)
{
    return grid_dr<1, float>(kmax_tpl, per_thread, mode, waves);
}

int launch_compress_pre_d1(const CompressArgs& a, hipStream_t st) { return launch_pre_dr<1>(a, st); }

int launch_compress_requeue_d1(const CompressArgs& a, hipStream_t st) { return launch_requeue_dr<1>(a, st); }

int launch_compress_finish_d1(int kmax_tpl, const CompressArgs& a, hipStream_t st)
{
    return launch_finish_dr<1>(kmax_tpl, a, st);
}


int launch_compress_big_d1_float(int kmax_tpl, const CompressArgs& a, int grid, hipStream_t st)
{
    return launch_big_dr<1, float>(kmax_tpl, a, grid, st);
}

int launch_compress_span_d1_float(int kmax_tpl, const CompressArgs& a, int waves, int b_hi, int b_lo, int b_help,
                                int64_t n_cells, hipStream_t st)
{
    return launch_span_dr<1, float>(kmax_tpl, a, waves, b_hi, b_lo, b_help, n_cells, st);
}

}  // namespace gm
