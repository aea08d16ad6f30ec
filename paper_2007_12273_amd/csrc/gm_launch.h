// gm_launch.h -- internal launch interface between the C ABI layer and the
// kernel translation units of libgmcr.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include "../../include/gmcr.h"

namespace gm {

// ---- compress ------------------------------------------------------------
struct CompressArgs;

// Length buckets: cell n -> first bucket with n <= max_n.  In a plan that
// launches per bucket, each is run by one persistent launch of 64 * waves
// threads per workgroup, each thread holding `per_thread` particles (the
// built-in plan's launches walk several, em_default below).  `store_e` buckets
// keep every density term in registers, so the particles per thread depend
// on the number of component slots (KMAX): the register file holds
// (KMAX + D + 2) values per particle.
struct Bucket {
    int max_n;
    int per_thread;
    int waves;
    bool store_e;
};
constexpr int kNumBuckets = 12;
// KMAX = 8: 8 register-resident particles per thread up to 8 waves (4096
// particles), then the recompute mode.
constexpr Bucket kBuckets8[kNumBuckets] = {
    {64, 1, 1, true},    {128, 2, 1, true},   {256, 4, 1, true},    {512, 8, 1, true},
    {1024, 8, 2, true},  {1536, 8, 3, true},  {2048, 8, 4, true},   {2560, 8, 5, true},
    {3072, 8, 6, true},  {3584, 8, 7, true},  {4096, 8, 8, true},   {8192, 16, 8, false},
};
// KMAX = 16: 4 register-resident particles per thread, one bucket per wave
// count up to 8 waves (2048 particles), then the recompute mode; cells of
// 2049-4096 particles in two buckets (their FP32 launch plans keep 5 and 8
// particles per thread in registers).  Cells of up to 128 particles share
// one bucket (two particles per thread; such cells are rare in the
// workloads that use 16 slots).
constexpr Bucket kBuckets16[kNumBuckets] = {
    {128, 2, 1, true},   {256, 4, 1, true},   {512, 4, 2, true},    {768, 4, 3, true},
    {1024, 4, 4, true},  {1280, 4, 5, true},  {1536, 4, 6, true},   {1792, 4, 7, true},
    {2048, 4, 8, true},  {2560, 8, 5, false}, {4096, 8, 8, false},  {8192, 16, 8, false},
};
__host__ __device__ constexpr const Bucket& bucket_cfg(int kmax_tpl, int b)
{
    return kmax_tpl == 8 ? kBuckets8[b] : kBuckets16[b];
}
// largest cell of the register-resident launches; larger cells go to k_em_big
constexpr int kMaxCellParticles = 8192;

// Launch variants a bucket can run with (the autotuner picks among them):
// particles per thread, whether the density terms stay in registers, and
// the build: standard (workgroups of up to 512 threads, up to 256 VGPRs per
// lane, two waves per SIMD; three for FP32 with one register-resident
// particle per thread) or lean (up to 1024 threads, at most 128 VGPRs, four
// waves per SIMD: more cells in flight per CU, and 16-wave workgroups for
// the largest cells).  Lean builds exist for FP32 iterations
// only.  A variant fits a bucket when 64 * waves * per_thread >= max_n with
// waves = ceil(max_n / (64 * per_thread)) <= the build's waves.
// Register-resident densities with 8 particles per thread are built for
// kmax 8 only (16 slots x 8 particles do not fit the register file); with
// 5, 6 and 7 for FP32 iterations at kmax 16 only, so that the cells of
// 1025-1792 particles run as four waves, one per SIMD: with five to seven
// waves some SIMD carries two of the cell's waves and every component
// update waits for it.
// Launch mode bits: kModeStoreE (densities in registers), kModeLean.
constexpr int kModeStoreE = 1;
constexpr int kModeLean = 2;
struct EmVariant {
    int per_thread;
    bool store_e;
    bool lean;
};
constexpr int kNumVariants = 13;
constexpr EmVariant kVariants[kNumVariants] = {{1, true, false}, {2, true, false}, {4, true, false},
                                              {8, true, false}, {8, false, false}, {16, false, false},
                                              {1, true, true},  {2, true, true},  {4, false, true},
                                              {8, false, true}, {5, true, false}, {6, true, false},
                                              {7, true, false}};
// the 5-, 6- and 7-particle register-resident builds exist for FP32 at
// kmax 16 only; the 8-particle one for kmax 8, and for FP32 at kmax 16
__host__ __device__ constexpr bool em_variant_built(int D, int kt, bool fp64, int per_thread, bool store_e)
{
    return (void)D, !store_e || (per_thread >= 5 && per_thread <= 7 ? (kt == 16 && !fp64)
                                 : per_thread == 8              ? (kt == 8 || !fp64)
                                                                : true);
}
constexpr int kEmMaxThreads = 512;
constexpr int kEmLeanThreads = 1024;
__host__ __device__ constexpr int em_max_waves(bool lean) { return (lean ? kEmLeanThreads : kEmMaxThreads) / 64; }
constexpr int kEmMaxWaves = kEmLeanThreads / 64;
// The built-in plan's variant of bucket b, as the plan reports it
// (em_reported) and as its launches run it (em_default).
struct EmDefault {
    int per_thread;  // most particles per thread any cell of the bucket needs
    int waves;
    int mode;
    bool span;       // in the launches that walk several buckets (k_em_span)
};

// Buckets of cells above 2048 particles (kmax 16) hold few cells, and one
// long fit among them can set the length of the whole EM phase: there the
// per-update latency of a single cell matters more than the bucket's
// throughput.  FP32 iterations run them with a lean build of more than 8
// waves (four waves per SIMD, the cell's CU to itself; in 3V the cells of
// 2049-4096 particles take the register-resident builds of the next rule
// instead).  On the Weibel-like batch one
// 2049-particle cell running 1000 sweeps made the warm phase 9.6-10.4 ms
// with it against 13.9-14.8 ms with the 8-wave builds, while a batch without
// such a fit cannot tell the builds apart, so the tuner keeps this choice.
constexpr int kChainMinN = 2048;
__host__ __device__ constexpr bool chain_bucket(int kt, bool fp64, int b)
{
    return !fp64 && kt == 16 && bucket_cfg(kt, b).max_n > kChainMinN;
}

// The cells of 1025-1792 particles (FP32, kmax 16) run as four waves,
// one per SIMD, with 5, 6 or 7 register-resident particles per thread
// instead of five to seven waves of 4: every update then waits for a SIMD
// with one of the cell's waves, not two.  On the Weibel-like batch the warm
// EM phase took 8.1 ms with them against 10.0-10.2 ms.
__host__ __device__ constexpr bool four_wave_bucket(int kt, bool fp64, int b)
{
    return kt == 16 && !fp64 && bucket_cfg(kt, b).max_n > 1024 && bucket_cfg(kt, b).max_n <= 1792;
}

// In 3V the cells of 2049-2560 and 2561-4096 particles (FP32, kmax 16) run
// as eight waves with 5 and up to 8 register-resident particles per thread (two
// waves per SIMD, the CU to the cell as with the 16-wave lean build): each
// update then evaluates one density per particle instead of recomputing the
// old one beside the new one, and a cell near 2049 particles computes 5
// particle slots per lane, not 8.  On the Weibel-like
// batch, where these cells hold the longest cold fits, with built-in plans:
// judged-fallback refit 20.7-20.9 ms against 26.7-29.3 ms with the lean
// build, headline step 30.6-31.0 ms against 35.5-38.9 ms.  The tuner may
// still pick a lean build there.
__host__ __device__ constexpr bool resident8_bucket(int D, int kt, bool fp64, int b)
{
    return D == 3 && kt == 16 && !fp64 && bucket_cfg(kt, b).max_n > 2048 && bucket_cfg(kt, b).max_n <= 4096;
}

template <int D>
__host__ __device__ constexpr EmDefault em_reported(int kt, bool fp64, int b)
{
    const Bucket& c = bucket_cfg(kt, b);
    if (resident8_bucket(D, kt, fp64, b)) return {c.max_n / (64 * 8), 8, kModeStoreE, true};
    if (chain_bucket(kt, fp64, b)) {
        // the lean builds recompute 4 or 8 particles per thread
        const int P = c.max_n <= kEmLeanThreads * 4 ? 4 : 8;
        return {P, (c.max_n + 64 * P - 1) / (64 * P), kModeLean, false};
    }
    if (four_wave_bucket(kt, fp64, b)) return {c.max_n / 256, 4, kModeStoreE, true};
    return {c.per_thread, c.waves, c.store_e ? kModeStoreE : 0, c.store_e && !fp64};
}

template <int D>
__host__ __device__ constexpr EmDefault em_default(int kt, bool fp64, int b)
{
    const Bucket& c = bucket_cfg(kt, b);
    // FP64 iterations: four particles per thread in 1V (two, on twice the
    // waves: 8.2 against 7.7 ms for 32 cells of 1000, most of an update being
    // what every wave computes alike); two up to 1024 particles in 3V, whose
    // four-particle build spills 196 B per lane (7.7-9.3 against 6.1-8.0 ms
    // for 512 cells of 256 on average).  Eight spill inside the update.
    // With sixteen slots, 40 replayed sweeps of one cell and of 512 cells, one
    // launch per bucket: 1V cells of 1000 1.07 and 1.5 ms with four particles per
    // thread, 1.00 and 2.1 with two; 3V cells of 1000 2.2 and 4.1 with four, 1.2
    // and 2.5 with two, of 500 1.6 and 2.5 against 0.8 and 1.4 (these launches,
    // whose build also holds four, 1.6 and 3.5, 1.0 and 1.7).  Against eight
    // particles per thread, 60 sweeps: 3V cells of 1000 7.2 -> 1.6 ms, of 2000 15.8
    // -> 4.9 ms, 1V cells of 2000 15.4 -> 2.3 ms.
    if (fp64 && c.max_n <= 2048) {
        const int most = D == 3 && c.max_n <= 1024 ? 2 : 4;
        const int P = c.max_n <= 64 * most ? c.max_n / 64 : most;
        return {P, D == 3 && c.max_n > 1024 ? 8 : (c.max_n + 64 * P - 1) / (64 * P), kModeStoreE, true};
    }
    return em_reported<D>(kt, fp64, b);
}

// k_em_span's workgroups only narrow on their way down the buckets
template <int D>
constexpr bool em_spans_narrow(int kt, bool fp64)
{
    int w = 0;
    for (int b = 0; b < kNumBuckets; ++b) {
        const EmDefault d = em_default<D>(kt, fp64, b);
        if (!d.span) continue;
        if (d.waves < w || d.waves > em_max_waves(false)) return false;
        w = d.waves;
    }
    return true;
}
static_assert(em_spans_narrow<1>(8, false) && em_spans_narrow<1>(16, false) && em_spans_narrow<1>(8, true) &&
                  em_spans_narrow<1>(16, true) && em_spans_narrow<3>(8, false) && em_spans_narrow<3>(16, false) &&
                  em_spans_narrow<3>(8, true) && em_spans_narrow<3>(16, true),
              "a bucket of larger cells runs on fewer waves");

// launch-plan code of a variant: per_thread * 1000 + waves * 10 + mode
__host__ __device__ constexpr int em_variant_code(int per_thread, int waves, int mode)
{
    return per_thread * 1000 + waves * 10 + mode;
}

// ---- reconstruct ---------------------------------------------------------
struct ReconArgs {
    const int32_t* K;
    const double* omega;
    const double* mu;
    const double* sigma;
    int32_t kmax;
    const int64_t* out_off;
    const double* target;
    int32_t D, dx;
    uint64_t seed;
    double* v_out;
    double* w_out;
    double* x_out;
    int32_t* status;
    int32_t tensor;  // 0: scalar projection (W, P, tr S); 1: full second moment (W, P, S)
};

int launch_reconstruct(const ReconArgs& a, int64_t n_cells, hipStream_t st);

// arguments of the projection of given particles
struct ProjArgs {
    const double* v;
    const double* w;
    const int64_t* off;
    const double* moments;
    int32_t D;
    int32_t tensor;
    double* v_out;
    int32_t* status;
};

int launch_project(const ProjArgs& a, int64_t n_cells, hipStream_t st);

}  // namespace gm
