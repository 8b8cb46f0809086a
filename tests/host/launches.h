// The launchers of fh_internal.h, for CPU tests: each notes what it was asked
// for and returns as the real ones do, with the stored error of the runtime.
#pragma once

#include <vector>

#include "../../paper_1407_8333_amd/csrc/fh_internal.h"

namespace fake {
struct Launch {
    const char *what;
    int64_t n_peaks;  // of the tiles: stripe edges' peaks
    int slots, parts;
    bool rank;  // windows from a rank table
};
inline thread_local std::vector<Launch> launches;
inline thread_local int64_t meta_total = 0, meta_most = 0;  // what a count reports
inline hipError_t launch(const Launch &l) {
    launches.push_back(l);
    return hipGetLastError();
}
inline void count(int64_t *meta) {
    if (!meta) return;
    meta[0] = meta_total;
    meta[1] = meta_most;
}
}  // namespace fake

namespace fh {
hipError_t launch_fill_i32(int32_t *, int64_t, int32_t, hipStream_t) { return fake::launch({"fill"}); }
hipError_t launch_set_sky(const SkyArg &, int, double *, hipStream_t) { return fake::launch({"set_sky"}); }
hipError_t launch_setup(const SetupArgs &, const int32_t *, int32_t, int32_t, uint2 *, hipStream_t) {
    return fake::launch({"setup"});
}
hipError_t launch_weight_stats(int32_t, const float *, int32_t, WeightStats *, int32_t *, hipStream_t) {
    return fake::launch({"weight_stats"});
}
hipError_t launch_prep(int32_t, int64_t n_peaks, const int64_t *, const int32_t *, const double *, const double *,
                       int32_t n_slots, int32_t, int64_t, int64_t *, const float *, int32_t, const WeightStats *,
                       int32_t, uint32_t *, uint32_t *, int32_t, double, hipStream_t) {
    return fake::launch({"prep", n_peaks, n_slots});
}
int front_ffts_per_block(int32_t max_per_fft) { return max_per_fft < 6000 ? 1 : 0; }
hipError_t launch_setup_front(const SetupArgs &, FrontArgs r, int32_t, hipStream_t) {
    return fake::launch({"front", r.n_peaks, r.n_slots});
}
int32_t rank_words(int32_t k_min, int32_t k_max) { return (k_max - k_min + 1) / 32 + 1; }
bool rank_front_fits(int32_t k_min, int32_t k_max, int32_t) { return rank_words(k_min, k_max) <= kRankMaxWords; }
hipError_t launch_front_rank(int32_t, int64_t n_peaks, const int64_t *, const int32_t *, const double *,
                             const double *, int32_t n_slots, int32_t, int64_t, const int64_t *, uint32_t *,
                             const float *, int32_t, const WeightStats *, int32_t, uint32_t *, int32_t, int32_t,
                             int32_t, int32_t, int32_t, const uint2 *, uint32_t *, int32_t, double, bool,
                             hipStream_t) {
    return fake::launch({"front", n_peaks, n_slots, 0, true});
}
hipError_t launch_sort_windows(int32_t, int32_t, int32_t, int32_t, const uint32_t *, const uint32_t *, int2 *,
                               const WeightArgs &, hipStream_t) {
    return fake::launch({"sort"});
}
hipError_t launch_windows(int32_t, const int64_t *, const int64_t *, int64_t, const int64_t *, int32_t, int32_t,
                          int32_t, int32_t, int32_t, uint32_t *, int, hipStream_t) {
    return fake::launch({"windows"});
}
hipError_t launch_tiles(const TileArgs &a, bool, bool, bool, int32_t, int32_t, hipStream_t) {
    return fake::launch({"tiles", a.n_peaks, a.n_slots, a.parts});
}
hipError_t launch_select(const unsigned long long *, int32_t, int32_t, const fh_select &, int32_t, int32_t,
                         const WeightStats *, int32_t, fh_candidate *, hipStream_t) {
    return fake::launch({"select"});
}
hipError_t launch_pm_rows(int32_t, int32_t, int64_t, const float *, const float *, int32_t, float, int32_t,
                          int32_t *, int32_t *, hipStream_t) {
    return fake::launch({"pm_rows"});
}
hipError_t launch_pm_scan(int32_t, const int32_t *, int64_t *, int64_t *meta, hipStream_t) {
    fake::count(meta);
    return fake::launch({"pm_scan"});
}
hipError_t launch_pm_pack(int32_t, int32_t, const int32_t *, const int64_t *, int32_t *, hipStream_t) {
    return fake::launch({"pm_pack"});
}
hipError_t launch_slice(int32_t, const int64_t *, const int32_t *, int32_t, int32_t, const double *, double *,
                        int64_t *, int32_t *, int64_t *, int32_t *, int64_t *meta, hipStream_t) {
    fake::count(meta);
    return fake::launch({"slice"});
}
int refine_cell_bytes(int kf, int nf, int ns) { return 4 * ns * (nf + kf - 1) <= 140000 ? 4 * ns * (nf + kf - 1) : 0; }
hipError_t launch_refine_cells(int32_t, const int64_t *, const int32_t *, const double *, const double *, int32_t,
                               int32_t, const double *, const RefineCand *, int2 *, int4 *, int32_t, int32_t, int32_t,
                               double, double, double, double, const float *, const WeightStats *, int32_t,
                               fh_candidate *, hipStream_t) {
    return fake::launch({"refine_cells"});
}
hipError_t launch_refine_pick(int32_t, int32_t, const fh_candidate *, const double *, const double *, fh_refined *,
                              hipStream_t) {
    return fake::launch({"refine_pick"});
}
hipError_t launch_gross_hist(int32_t, const int64_t *, const int32_t *, const double *, double, const fh_gross &,
                             int32_t *, hipStream_t) {
    return fake::launch({"gross_hist"});
}
hipError_t launch_filter(int32_t, const int64_t *, const int32_t *, const FilterSpec &, const double *, double *,
                         int32_t *, int64_t *, int32_t *, int phase, int64_t *meta, hipStream_t) {
    if (phase == 0) fake::count(meta);
    return fake::launch({"filter"});
}
hipError_t launch_bin_counts(int32_t, int64_t, const int64_t *, const int32_t *, int32_t, int32_t, int32_t *,
                             hipStream_t) {
    return fake::launch({"bin_counts"});
}
hipError_t launch_robust(const int32_t *, int32_t, int32_t, int32_t *, int64_t *, double *out, int32_t *, hipStream_t) {
    out[0] = out[1] = out[2] = 0.0;
    return fake::launch({"robust"});
}
hipError_t launch_colmax_decode(const unsigned long long *, int32_t, int32_t, const WeightStats *, int32_t, float *,
                                int32_t *, hipStream_t) {
    return fake::launch({"decode"});
}
hipError_t launch_colmax_values(const unsigned long long *, int32_t, int32_t *, hipStream_t) {
    return fake::launch({"values"});
}
int tile_lds_bytes(int W, int kf, int tail) {
    return (kTileRows * (W + kf - 1 + kDumpCols) + tail * (W + kf - 1 + kTailDump)) * 4;
}
int64_t part_words(int W, int kf, int tail) { return (tile_lds_bytes(W, kf, tail) / 4 + 3) / 4 * 4; }
int max_tile_bins(int kf, double, int rows) { return ((kLdsBytes - kLdsReserve) / 4 / rows - kf - 8) / 64 * 64; }
hipError_t init_kernel_attributes() { return hipSuccess; }
}  // namespace fh
