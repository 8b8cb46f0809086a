// HIP kernels of the frequency-Hough (FH) library for gfx950 (MI355X).
//
// Pipeline for one chunk of sky directions (Sec. "Frequency-Hough transform"):
//   k_setup        per (FFT, row block): the rows' shifts G_is in 2^-16 fine
//                  bins (Eqs. uno, sdstep) as compact tables, sky independent;
//                  per weight vector: sum w, sum w^2, fixed-point bits F
//   k_prep         per (sky, peak): Doppler-corrected stripe edge Y (Eq.
//                  fdopp, Eq. due) and per (sky, FFT) fixed-point weights.
//   k_windows      per (sky, row-block group, bin block, FFT): the contiguous
//                  range of that FFT's peaks whose stripes reach the tile.
//   k_tiles_*      per tile of 16 rows x W fine bins: LDS histogram of stripe
//                  starts (one ds_add_u32 per peak and row), then the
//                  differential +w/-w sum along each row as a width-K_f window
//                  (Eqs. ncount, ncountadap, freqres); writes the map and/or the
//                  per-bin maximum over rows.
//   k_select       per (sky, sub-band): first and second-order candidates
//                  (Sec. "Selection of first level candidates").
//
// All FP64 arithmetic is IEEE round-to-nearest-even with contraction off, so
// the integer stripe edges agree bit for bit with any other implementation of
// the same definition.
#include <hip/hip_runtime.h>
#include <math.h>
#include <stdint.h>

#include <algorithm>

#include "fh_internal.h"

#pragma clang fp contract(off)

namespace fh {

namespace {

// Fixed point of stripe edges: kQ = 2^kFrac steps per fine bin.
constexpr int kFrac = 16;
constexpr double kQd = 65536.0;
constexpr int64_t kQ = (int64_t)1 << kFrac;

__device__ __forceinline__ int64_t shrq(int64_t a) { return a >> kFrac; }  // floor(a / kQ)

// Stripe edge stored in the kYPad slots after each FFT's peaks (never inside
// a window; the slots keep every FFT's run of edges followed by readable
// memory).
constexpr int64_t kYSentinel = (int64_t)1 << 61;

// Tile-relative edges are 32-bit: with kFrac = 16 fractional bits a column is
// the upper half-word, inside +-2^15.  A peak of a window starts within 64
// rows' worth of spin-down steps of the tile (the window covers a group of
// 64 rows, the last group up to kTailRows more; the last row block may reach
// 16 rows past the grid), so max_tile_bins bounds W + K_f + 80 (step + 1) +
// 64 below 2^15.  kFarEdge
// (16384 bins) then stays in range and beyond the dump column for every row.
constexpr uint32_t kFarEdge = 16384u << kFrac;

// ----------------------------------------------------------------------------
// fills (graph-safe replacements for memset)

__global__ void k_fill_i32(int32_t *__restrict__ p, int64_t n, int32_t v) {
    for (int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; i < n;
         i += (int64_t)gridDim.x * blockDim.x)
        p[i] = v;
}

// ----------------------------------------------------------------------------
// spin-down shifts (Eqs. uno, sdstep): row s has the spin-down
// fdot_s = fdot0 + s dfdot, and FFT i's stripes in that row are shifted by
//   G_is = rint((fdot_s tau_i) S),  tau_i = t_i - t0,  S = (K_f T_FFT) kQ
// rounded once per row (rows past the grid, up to the end of the last row
// block, follow the same formula and never reach the output).

__device__ __forceinline__ int64_t row_shift(double tau, double S, double fdot0, double dfdot, int32_t s) {
    double fs = (double)s * dfdot;
    fs = fdot0 + fs;
    double a = fs * tau;
    a = a * S;
    return (int64_t)rint(a);
}

// The tiles need, for FFT i and the 16 rows s0 + j of a row block, the
// offsets G_{i,s0} - G_{i,s0+j}.  With q_i = rint(((dfdot tau_i) S) 2^16) the
// row step in 2^-32 fine bins, floor(j q_i / 2^16) is within (-1, 1] + 1e-3
// of j's exact step, and each G within 0.5 of its exact value, so
//   c_ij = G_{i,s0+j} - G_{i,s0} - floor(j q_i / 2^16)  lies in {-1, 0, 1, 2}.
// Tables (all sky independent):
//   step[i][j]  = low word of 1 - floor(j q_i / 2^16)              [N][16]
//   rec[rb][i]  = (low word of G_{i,s0}, sum_j (c_ij + 1) << 2j)   [nrb][N]
//   gwin[i][g]  = (G_is at the first and at the last grid row of row
//                 group g), for the peak windows                   [N][nrbg][2]
// A code outside {-1 .. 2} (impossible by the bound above) sets bit 2 of the
// error flag.
__device__ __forceinline__ void shift_tables(const SetupArgs &A, int64_t first, int64_t stride) {
    const int32_t n_fft = A.n_fft;
    // row groups of the row blocks the tiles run; the last one reaches the
    // grid's last row (the rows of a folded last block included)
    const int32_t nrbg = (A.nrb_run + kRowBlocksPerGroup - 1) / kRowBlocksPerGroup;
    const int64_t n = (int64_t)n_fft * A.nrb;
    for (int64_t x = first; x < n; x += stride) {
        const int32_t rb = (int32_t)(x / n_fft);
        const int32_t i = (int32_t)(x - (int64_t)rb * n_fft);
        if (rb == 0)  // run by run, as the window sort reads them
            A.base[(i % kTileWaves) * wave_ffts(n_fft) + i / kTileWaves] = (uint32_t)(A.offsets[i] + (int64_t)A.y_pad * i);
        const double tau = A.t[i] - A.t0;
        double sig = A.dfdot * tau;
        sig = sig * A.S;
        const int64_t q = (int64_t)rint(sig * 65536.0);
        const int32_t s0 = rb * kTileRows;
        const int64_t g0 = row_shift(tau, A.S, A.fdot0, A.dfdot, s0);
        uint32_t codes = 0;
        bool bad = false;
        for (int j = 0; j < kTileRows; ++j) {
            const int64_t lin = ((int64_t)j * q) >> 16;  // floor (arithmetic shift)
            const int64_t c = row_shift(tau, A.S, A.fdot0, A.dfdot, s0 + j) - g0 - lin;
            bad = bad || c < -1 || c > 2;
            codes |= (uint32_t)((c + 1) & 3) << (2 * j);
            if (rb == 0) A.step[(int64_t)i * kTileRows + j] = 1u - (uint32_t)(uint64_t)lin;
        }
        A.rec[(int64_t)rb * n_fft + i] = make_uint2((uint32_t)(uint64_t)g0, codes);
        if (bad) atomicOr(A.err, 2);
        if (rb < A.nrb_run && rb % kRowBlocksPerGroup == 0) {
            const int32_t g = rb / kRowBlocksPerGroup;
            const int32_t s_hi = g == nrbg - 1 ? A.ns - 1 : s0 + kRowBlocksPerGroup * kTileRows - 1;
            A.gwin[((int64_t)i * nrbg + g) * 2] = g0;
            A.gwin[((int64_t)i * nrbg + g) * 2 + 1] = row_shift(tau, A.S, A.fdot0, A.dfdot, s_hi);
        }
    }
}

// ----------------------------------------------------------------------------
// weight statistics and fixed-point scale (Eq. ncountadap) of one vector, by
// one workgroup of 256 threads

__device__ __forceinline__ void weight_stats(int32_t n, const float *__restrict__ wv, int32_t mult,
                                             WeightStats *__restrict__ ws, int32_t *__restrict__ err_flag) {
    double s1 = 0.0, s2 = 0.0;
    int bad = 0;
#pragma unroll 8
    for (int i = threadIdx.x; i < n; i += 256) {
        double x = (double)wv[i];
        if (!(x > 0.0 && x < 65536.0)) bad = 1;  // also catches NaN
        s1 += x;
        s2 += x * x;
    }
    __shared__ double r1[256], r2[256];
    __shared__ int rb[256];
    r1[threadIdx.x] = s1;
    r2[threadIdx.x] = s2;
    rb[threadIdx.x] = bad;
    __syncthreads();
    for (int o = 128; o > 0; o >>= 1) {
        if ((int)threadIdx.x < o) {
            r1[threadIdx.x] += r1[threadIdx.x + o];
            r2[threadIdx.x] += r2[threadIdx.x + o];
            rb[threadIdx.x] |= rb[threadIdx.x + o];
        }
        __syncthreads();
    }
    if (threadIdx.x == 0) {
        WeightStats st;
        st.sum_w = r1[0];
        st.sum_w2 = r2[0];
        st.bad = rb[0];
        // a cell holds at most mult * sum_i rint(w_i 2^F) <= mult (2^F sum w + N/2)
        double lim = (4294967295.0 / (double)mult - 0.5 * (double)n) / r1[0];
        int F = -1;
        if (!rb[0] && lim >= 1.0) {
            F = 0;
            while (F < 40 && ldexp(1.0, F + 1) <= lim) ++F;
        }
        if (F < 0) st.bad = 1;
        st.frac_bits = F < 0 ? 0 : F;
        *ws = st;
        if (st.bad) atomicOr(err_flag, 1);
    }
}

__global__ void __launch_bounds__(256) k_weight_stats(int32_t n, const float *__restrict__ w, int32_t mult,
                                                      WeightStats *__restrict__ ws,
                                                      int32_t *__restrict__ err_flag) {
    weight_stats(n, w, mult, ws, err_flag);
}

// Block b of the n_blocks that hold the shift tables, the cleared buffers and
// the directions.
__device__ __forceinline__ void setup_block(const SetupArgs &A, int b, int n_blocks) {
    const int64_t x = b * (int64_t)256 + threadIdx.x, stride = (int64_t)n_blocks * 256;
    shift_tables(A, x, stride);
    for (int64_t y = x; y < A.n_colmax; y += stride) A.colmax[y] = 0ull;
    if (b == 0) {
        if ((int)threadIdx.x < kXcds) A.qctr[threadIdx.x] = 0;
        if ((int)threadIdx.x < 3 * A.n_sky) A.sky[threadIdx.x] = A.sky_arg[threadIdx.x];
    }
}

// the directions of a small call (see SetupArgs::sky_arg)
__global__ void __launch_bounds__(128) k_set_sky(SkyArg s, int n, double *__restrict__ sky) {
    if ((int)threadIdx.x < 3 * n) sky[threadIdx.x] = s.v[threadIdx.x];
}

// A window before it is sorted: the places of its first peak and of the first
// peak past it within their FFT (an FFT holds fewer than 65536 peaks).
__device__ __forceinline__ uint32_t window(int lo, int hi) { return (uint32_t)lo | ((uint32_t)hi << 16); }

// ----------------------------------------------------------------------------
// per-peak stripe edge.  For peak (i, k) and sky n:
//   r = 1 / (1 + ((vx nx + vy ny) + vz nz))                     (Eq. fdopp)
//   X = floor(((double)(K_f k) r) kQ)
//   Y = X - b0 kQ - K_f kQ/2 + (kQ - 1)
// so that the first fine bin of the stripe in row s is
//   a_s = ceil((X - b0 kQ - K_f kQ/2 - G_is) / kQ)
//       = floor((Y - G_is) / kQ).
// One wave per FFT; grid.y = sky slot.

__global__ void __launch_bounds__(256) k_prep(
    int32_t n_fft, int64_t n_peaks, const int64_t *__restrict__ offsets,
    const int32_t *__restrict__ bins, const double *__restrict__ v,
    const double *__restrict__ sky, int32_t kf, int64_t b0,
    int64_t *__restrict__ Y, const float *__restrict__ w, int32_t w_stride,
    const WeightStats *__restrict__ ws, int32_t ws_stride, uint32_t *__restrict__ wq,
    uint32_t *__restrict__ Y32, int32_t shift_mode, double q) {
    const int lane = threadIdx.x & 63;
    const int i = blockIdx.x * (blockDim.x >> 6) + (threadIdx.x >> 6);
    const int slot = blockIdx.y;
    if (i >= n_fft) return;
    const double *n = sky + 3 * (int64_t)slot;
    const double *vi = v + 3 * (int64_t)i;
    double d = vi[0] * n[0];
    d = d + vi[1] * n[1];
    d = d + vi[2] * n[2];
    d = 1.0 + d;
    const double r = 1.0 / d;
    int64_t c = -b0 * kQ - (int64_t)kf * (kQ / 2) + (kQ - 1);
    if (shift_mode) c -= llrint((q * (1.0 - r)) * kQd);  // per-FFT shift at the reference
    // FFT i's edges start at offsets[i] + kYPad * i and are followed by kYPad
    // sentinels
    int64_t *Ys = Y + (int64_t)slot * y_stride(n_peaks, n_fft) + (int64_t)kYPad * i;
    uint32_t *Ys32 = Y32 + (int64_t)slot * y_stride(n_peaks, n_fft) + (int64_t)kYPad * i;
    const int64_t e = offsets[i + 1];
    for (int64_t p = offsets[i] + lane; p < e; p += 64) {
        int64_t y;
        if (shift_mode) {
            y = (int64_t)kf * (int64_t)bins[p] * kQ + c;
        } else {
            double x = (double)((int64_t)kf * (int64_t)bins[p]) * r;
            x = x * kQd;
            y = (int64_t)floor(x) + c;
        }
        Ys[p] = y;
        Ys32[p] = (uint32_t)y;
    }
    if (lane < kYPad) {
        Ys[e + lane] = kYSentinel;
        Ys32[e + lane] = (uint32_t)kYSentinel;
    }
    if (w != nullptr && lane == 0) {
        const WeightStats st = ws[(int64_t)slot * ws_stride];
        double wi = (double)w[(int64_t)slot * w_stride + i];
        wq[(int64_t)slot * n_fft + i] = st.bad ? 0u : (uint32_t)rint(ldexp(wi, st.frac_bits));
    }
}

// ----------------------------------------------------------------------------
// Fused front: for one direction slot and F consecutive FFTs f0 .. f0+F-1
// (grid.x over the padded FFT count, grid.y = slot), the stripe edges of
// their peaks (written out for the tiles and staged in LDS), their
// fixed-point weights, and every window entry (row group, bin block, FFT) by
// two binary searches over the staged edges.  The window of a tile is the run
// of peaks p with
//   max_s a_s(p) >= jb W - (K_f - 1)   and   min_s a_s(p) < (jb + 1) W
// over the group's rows s (a_s is monotone in Y, Y ascending within an FFT;
// G_is is monotone in s, so its extremes over the rows are those of the
// first and last row).  Consecutive threads write consecutive FFTs of a
// window row.

__device__ __forceinline__ void front_block(const SetupArgs &A, const FrontArgs &R, int block, int slot) {
    extern __shared__ int64_t ys[];
    __shared__ int64_t s_off[kFrontMaxF + 1];  // offsets of the block's FFTs
    __shared__ int32_t s_loc[kFrontMaxF + 1];  // the same, from the block's first peak
    __shared__ int64_t s_c[kFrontMaxF];        // per-FFT constant of the edge
    __shared__ double s_r[kFrontMaxF];         // per-FFT inverse Doppler factor
    const int32_t n_fft = A.n_fft, kf = R.kf, F = R.F, nrbg = R.nrbg, nbb = R.nbb, W = R.W;
    const int32_t search_top = R.search_top, shift_mode = R.shift_mode;
    const int64_t *__restrict__ offsets = A.offsets;
    const int32_t *__restrict__ bins = R.bins;
    const int f0 = block * F;
    const int fe = min(f0 + F, n_fft);
    const int nfl = fe - f0;  // FFTs of this block (<= 0 for padding blocks)
    const int32_t n_pad = win_stride(n_fft);
    uint32_t *Yslot = R.Y + (int64_t)slot * y_stride(R.n_peaks, n_fft);

    // per-FFT terms (r, constant), one thread per FFT; the directions of a
    // small call are read from the arguments (k_setup's copy may not be there)
    const double *n = slot < A.n_sky ? A.sky_arg + 3 * slot : R.sky + 3 * (int64_t)slot;
    if ((int)threadIdx.x <= nfl) {
        const int64_t o = offsets[f0 + threadIdx.x];
        s_off[threadIdx.x] = o;
        s_loc[threadIdx.x] = (int32_t)(o - offsets[f0]);
    }
    if ((int)threadIdx.x < nfl) {
        const int i = f0 + threadIdx.x;
        const double *vi = R.v + 3 * (int64_t)i;
        double d = vi[0] * n[0];
        d = d + vi[1] * n[1];
        d = d + vi[2] * n[2];
        d = 1.0 + d;
        const double r = 1.0 / d;
        s_r[threadIdx.x] = r;
        int64_t c = -R.b0 * kQ - (int64_t)kf * (kQ / 2) + (kQ - 1);
        if (shift_mode) c -= llrint((R.q * (1.0 - r)) * kQd);  // per-FFT shift at the reference
        s_c[threadIdx.x] = c;
    }
    __syncthreads();

    // stripe edges (as k_prep) of all the block's peaks: wave w takes FFTs w,
    // w + 4, ..., its lanes that FFT's consecutive peaks, so no lane searches
    // for its FFT and its Doppler factor and constant are read once per FFT
    if (nfl > 0) {
        const int64_t P0 = s_off[0];
        // peak indices local to the block (32-bit: a block holds at most
        // 48 KB of edges); K_f k < 2^28 (checked at upload), so the natural
        // frequency in fine bins converts to double from 32 bits exactly
        const int32_t *__restrict__ kbins = bins + P0;
        uint32_t *__restrict__ Yb = Yslot + P0 + (int64_t)kYPad * f0;
        const int lane = (int)threadIdx.x & 63, nw = (int)blockDim.x >> 6;
        constexpr int kU = 4;  // peaks per lane and round, their natural bins requested together
        for (int l = (int)threadIdx.x >> 6; l < nfl; l += nw) {
            const int pa = s_loc[l], pe = s_loc[l + 1];
            const double r = s_r[l];
            const int64_t c = s_c[l];
            for (int lb = pa + lane; lb < pe; lb += 64 * kU) {
                int32_t kb[kU];
#pragma unroll
                for (int u = 0; u < kU; ++u) {
                    const int lp = lb + 64 * u;
                    kb[u] = lp < pe ? kbins[lp] : 0;
                }
#pragma unroll
                for (int u = 0; u < kU; ++u) {
                    const int lp = lb + 64 * u;
                    if (lp >= pe) break;
                    int64_t y;
                    if (shift_mode) {
                        y = (int64_t)(kf * kb[u]) * kQ + c;
                    } else {
                        double x = (double)(kf * kb[u]) * r;
                        x = x * kQd;
                        y = (int64_t)floor(x) + c;
                    }
                    const int li = lp + kYPad * l;
                    Yb[li] = (uint32_t)y;  // the tiles use the low word
                    ys[li] = y;
                }
            }
        }
    }
    __syncthreads();

    // Window entries e = tid + k blockDim, e = (g nbb + jb) F + fl: F divides
    // blockDim, so a thread keeps one FFT fl, and its row index g nbb + jb
    // advances by blockDim / F per entry (no division per entry).  Each of
    // the two searches is a branchless binary lifting over the FFT's staged
    // edges: powers of two from search_top (the largest power of two up to
    // the longest FFT's peak count) down to 1, a step taken while the edge
    // it passes is below the bound.
    const int fl = (int)threadIdx.x & (F - 1);
    const int step_r = (int)blockDim.x / F;
    const int n_rows = nrbg * nbb;
    int rest = (int)threadIdx.x / F;
    int g = rest / nbb, jb = rest - g * nbb;
    const int dg = step_r / nbb, djb = step_r - dg * nbb;
    const int f = f0 + fl;
    const bool live = fl < nfl;
    int a0 = 0, end = 0;
    if (live) {
        a0 = s_loc[fl] + kYPad * fl;
        end = s_loc[fl + 1] + kYPad * fl;
    }
    const double tau = live ? A.t[f] - A.t0 : 0.0;
    uint32_t *__restrict__ wp = R.win + (int64_t)slot * n_rows * n_pad + f;
    int64_t q_lo = 0, q_hi = 0;  // shifts of the group's first and last grid rows
    for (int g_of = -1; rest < n_rows; rest += step_r) {
        uint32_t out = 0u;
        if (live) {
            if (g != g_of) {  // worked out here: the tables come from the same launch
                constexpr int kGroupRows = kTileRows * kRowBlocksPerGroup;
                q_lo = row_shift(tau, A.S, A.fdot0, A.dfdot, g * kGroupRows);
                q_hi = row_shift(tau, A.S, A.fdot0, A.dfdot, g == nrbg - 1 ? A.ns - 1 : (g + 1) * kGroupRows - 1);
                g_of = g;
            }
            // max_s a_s = floor((Y - min G) / kQ) >= t  <=>  Y >= t kQ + min G
            // min_s a_s = floor((Y - max G) / kQ) >= t  <=>  Y >= t kQ + max G
            const int64_t y_lo = ((int64_t)jb * W - (kf - 1)) * kQ + (q_lo < q_hi ? q_lo : q_hi);
            const int64_t y_hi = (int64_t)(jb + 1) * W * kQ + (q_lo < q_hi ? q_hi : q_lo);
            int lo = a0, hi = a0;  // first peaks with Y >= y_lo and with Y >= y_hi
            for (int stp = search_top; stp > 0; stp >>= 1) {
                const int t1 = lo + stp - 1, t2 = hi + stp - 1;
                const int64_t v1 = ys[t1 < end ? t1 : a0], v2 = ys[t2 < end ? t2 : a0];
                lo += (t1 < end && v1 < y_lo) ? stp : 0;
                hi += (t2 < end && v2 < y_hi) ? stp : 0;
            }
            out = window(lo - a0, hi - a0);
        }
        wp[(int64_t)rest * n_pad] = out;
        g += dg;
        jb += djb;
        if (jb >= nbb) {
            jb -= nbb;
            ++g;
        }
    }
}

// ----------------------------------------------------------------------------
// The front's table of an FFT's peaks (see k_front_rank):
// rank[i][w] = (bits of natural bins k_min + 32 w .. + 31, peaks of FFT i below
// them), nw words per FFT; one wave per FFT.
__device__ __forceinline__ void rank_block(int32_t n_fft, const int64_t *__restrict__ offsets,
                                           const int32_t *__restrict__ bins, int32_t k_min, int32_t nw,
                                           uint2 *__restrict__ rank, int block) {
    extern __shared__ uint32_t s_bits[];  // [4][nw]
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int i = block * 4 + wave;
    uint32_t *b = s_bits + wave * nw;
    for (int w = lane; w < nw; w += 64) b[w] = 0u;
    __syncthreads();
    if (i < n_fft) {
        const int64_t e = offsets[i + 1];
        for (int64_t p = offsets[i] + lane; p < e; p += 64) {
            const uint32_t x = (uint32_t)(bins[p] - k_min);
            atomicOr(&b[x >> 5], 1u << (x & 31));
        }
    }
    __syncthreads();
    if (i >= n_fft) return;
    uint32_t carry = 0;
    for (int w0 = 0; w0 < nw; w0 += 64) {
        const int w = w0 + lane;
        const uint32_t v = w < nw ? b[w] : 0u;
        const uint32_t c = __popc(v);
        uint32_t incl = c;
        for (int o = 1; o < 64; o <<= 1) {
            const uint32_t u = __shfl_up(incl, o);
            if (lane >= o) incl += u;
        }
        if (w < nw) rank[(int64_t)i * nw + w] = make_uint2(v, carry + incl - c);
        carry += __shfl(incl, 63);
    }
}

// ----------------------------------------------------------------------------
// Everything a search needs before its front (or beside it), in one launch: the
// weight statistics (one workgroup per vector), the shift tables, cleared
// column maxima and queue counters, and the directions of a small call, which
// come as kernel arguments.  All of it is latency: it replaces a copy, behind
// which the host waited for the stream, and four kernels.  A 0.1 Hz map of 200 FFTs
// went from 36 to 23 us, the column maxima of five directions (4096 s, own
// weights) from 153 to 126 us.
// With the rank table of launch_front_rank:
__global__ void __launch_bounds__(256) k_setup(SetupArgs A, RankArgs R) {
    int b = blockIdx.x;
    if (b < A.n_vec) {
        weight_stats(A.n_fft, A.w + (int64_t)b * A.w_stride, A.mult, A.ws + b, A.err);
        return;
    }
    b -= A.n_vec;
    if (b < R.n_blocks) {
        rank_block(A.n_fft, A.offsets, R.bins, R.k_min, R.nw, R.rank, b);
        return;
    }
    setup_block(A, b - R.n_blocks, (int)gridDim.x - A.n_vec - R.n_blocks);
}

// With the front of one or a few directions, which needs nothing of the rest
// (the window sort, the next launch, takes the fixed-point weights): 3 us less
// per call, 23 -> 20 us on a 0.1 Hz map of 200 FFTs.
__global__ void __launch_bounds__(256) k_setup_front(SetupArgs A, FrontArgs R) {
    int b = blockIdx.x;
    if (b < A.n_vec) {
        weight_stats(A.n_fft, A.w + (int64_t)b * A.w_stride, A.mult, A.ws + b, A.err);
        return;
    }
    b -= A.n_vec;
    const int per_slot = win_stride(A.n_fft) / R.F;
    if (b < per_slot * R.n_slots) {
        const int slot = b / per_slot;
        front_block(A, R, b - slot * per_slot, slot);
        return;
    }
    setup_block(A, b - per_slot * R.n_slots, (int)gridDim.x - A.n_vec - per_slot * R.n_slots);
}

// ----------------------------------------------------------------------------
// Front of many directions.  A window's ends are found without a search: the
// edge bound of an entry gives the least natural bin whose edge reaches it
// (an estimate and one exact test, since edges ascend with the bin), and a
// table of the FFT's peaks, 32 natural bins to a word with the number of peaks
// before it, gives that bin's place among them.  The table does not depend on
// the direction and is built once per call.

// For up to D direction slots and F consecutive FFTs f0 .. f0+F-1: the stripe
// edges of their peaks, their fixed-point weights and every window entry.  The
// FFTs' tables, offsets and natural bins are read once for all D directions: a
// workgroup of one direction is a chain of dependent loads around little work
// (as such this kernel, with a third of k_front's instructions, took the same
// time).  The edges go to memory only, so the LDS holds F tables, and up to 16
// FFTs share a workgroup: consecutive threads write whole lines of a window row.
// With Y(k) = floor(fl(fl(K_f k r) 2^16)) + c, Y(k) >= y is fl(K_f k r) >= z for
// z = (y - c) 2^-16, which a double holds exactly wherever an edge can lie; z
// d / K_f (d = 1 / r before rounding) is within 2^-23 of the real bound, so the
// least bin is the nearest whole number or the next one.
// With few row blocks the tiles compute the edges from the natural bins, and
// the front stores only each FFT's terms (terms_only): the multiplier fl(r)
// 2^16 and the low word of c, 16 B apart, where the slot's edges would begin.
// Bound by its stores (the edges, 4 B per peak, and 4 B per window entry).
// Against k_front: 112 directions of the 256 Hz band 1050 -> 464 us (3.2 TB/s
// written), 24 of the 10 Hz band at 1 kHz 1440 -> 900 us, 97 narrow ones at
// 1024 s 463 -> 334 us.
__global__ void __launch_bounds__(256) k_front_rank(
    int32_t n_fft, int64_t n_peaks, const int64_t *__restrict__ offsets, const int32_t *__restrict__ bins,
    const double *__restrict__ v, const double *__restrict__ sky, int32_t n_slots, int32_t kf, int64_t b0,
    const int64_t *__restrict__ gwin, uint32_t *__restrict__ Y, const float *__restrict__ w, int32_t w_stride,
    const WeightStats *__restrict__ ws, int32_t ws_stride, uint32_t *__restrict__ wq, int32_t nrbg, int32_t nbb,
    int32_t W, int32_t F, int32_t D, int32_t k_min, int32_t k_max, int32_t nw, const uint2 *__restrict__ rank,
    uint32_t *__restrict__ win, int32_t shift_mode, double q, bool terms_only) {
    extern __shared__ double s_dyn[];
    double *s_g = s_dyn;  // [nrbg][F][2]: least and largest shift of the group's rows, in fine bins
    const int ts = nw | 1;  // table stride (odd: the FFTs' words spread over the banks)
    uint2 *s_tab = reinterpret_cast<uint2 *>(s_dyn + 2 * nrbg * F);  // [F][ts]
    __shared__ int64_t s_off[kFrontMaxF + 1];
    __shared__ int64_t s_c[kRankDirs * kFrontMaxF];                  // [D][F], the edge's constant
    __shared__ double s_r[kRankDirs * kFrontMaxF], s_d[kRankDirs * kFrontMaxF];
    const int slot0 = blockIdx.y * D;
    const int nd = min(D, n_slots - slot0);
    const int f0 = blockIdx.x * F;
    const int nfl = min(f0 + F, n_fft) - f0;  // FFTs of this block (<= 0 for padding blocks)
    const int32_t n_pad = win_stride(n_fft);
    if ((int)threadIdx.x <= nfl) s_off[threadIdx.x] = offsets[f0 + threadIdx.x];
    // (F divides 256, so x & (F - 1) is the same FFT in every round)
    for (int x = threadIdx.x; x < nd * F; x += 256) {
        const int l = x & (F - 1), slot = slot0 + x / F;
        if (l >= nfl) continue;
        const int i = f0 + l;
        const double *n = sky + 3 * (int64_t)slot;
        const double *vi = v + 3 * (int64_t)i;
        double d = vi[0] * n[0];
        d = d + vi[1] * n[1];
        d = d + vi[2] * n[2];
        d = 1.0 + d;
        const double r = 1.0 / d;
        int64_t c = -b0 * kQ - (int64_t)kf * (kQ / 2) + (kQ - 1);
        if (shift_mode) c -= llrint((q * (1.0 - r)) * kQd);  // per-FFT shift at the reference
        s_r[x] = shift_mode ? 1.0 : r;
        s_d[x] = (shift_mode ? 1.0 : d) / (double)kf;
        s_c[x] = c;
        if (terms_only) {
            uint32_t *e = Y + (int64_t)slot * y_stride(n_peaks, n_fft) + 4 * (int64_t)i;
            const uint64_t rq = (uint64_t)__double_as_longlong(s_r[x] * kQd);
            e[0] = (uint32_t)rq;
            e[1] = (uint32_t)(rq >> 32);
            e[2] = (uint32_t)(uint64_t)c;
        }
        if (w != nullptr) {
            const WeightStats wst = ws[(int64_t)slot * ws_stride];
            double wi = (double)w[(int64_t)slot * w_stride + i];
            wq[(int64_t)slot * n_fft + i] = wst.bad ? 0u : (uint32_t)rint(ldexp(wi, wst.frac_bits));
        }
    }
    // the FFTs' tables are consecutive in memory
    for (int x = threadIdx.x; x < nfl * nw; x += 256) {
        const int l = x / nw;
        s_tab[l * ts + (x - l * nw)] = rank[(int64_t)f0 * nw + x];
    }
    for (int x = threadIdx.x; x < nrbg * F; x += 256) {
        const int g = x / F, l = x & (F - 1);
        if (l < nfl) {
            const int64_t *gq = gwin + ((int64_t)(f0 + l) * nrbg + g) * 2;
            const int64_t q0 = gq[0], q1 = gq[1];
            s_g[2 * x] = (double)(q0 < q1 ? q0 : q1) * (1.0 / kQd);
            s_g[2 * x + 1] = (double)(q0 < q1 ? q1 : q0) * (1.0 / kQd);
        }
    }
    __syncthreads();
    // stripe edges: wave w takes FFTs w, w + 4, ..., its lanes their
    // consecutive peaks; the entries between two FFTs' runs stay unwritten
    // (the tiles read past a window's end but do not use what they read)
    if (!terms_only) {
        const int64_t ys = y_stride(n_peaks, n_fft);
        const int lane = (int)threadIdx.x & 63;
        constexpr int kU = 4;  // peaks per lane and round, their natural bins requested together
        for (int l = (int)threadIdx.x >> 6; l < nfl; l += 4) {
            const int64_t p0 = s_off[l];
            const int cnt = (int)(s_off[l + 1] - p0);
            const int32_t *__restrict__ kb0 = bins + p0;
            uint32_t *__restrict__ Yb = Y + (int64_t)slot0 * ys + p0 + (int64_t)kYPad * (f0 + l);
            for (int lb = lane; lb < cnt; lb += 64 * kU) {
                double kb[kU];
#pragma unroll
                for (int u = 0; u < kU; ++u) {
                    const int lp = lb + 64 * u;
                    kb[u] = (double)(kf * (lp < cnt ? kb0[lp] : 0));
                }
                for (int d = 0; d < nd; ++d) {
                    const double r = s_r[d * F + l];
                    const int64_t c = s_c[d * F + l];
                    uint32_t *__restrict__ Yd = Yb + d * ys;
#pragma unroll
                    for (int u = 0; u < kU; ++u) {
                        const int lp = lb + 64 * u;
                        if (lp >= cnt) break;
                        // (r = 1 in shift mode, where the product is exact)
                        double x = kb[u] * r;
                        x = x * kQd;
                        Yd[lp] = (uint32_t)((int64_t)floor(x) + c);
                    }
                }
            }
        }
    }
    // window entries: a thread keeps one FFT and steps through the rows (row
    // group, bin block) of every direction
    const int fl = (int)threadIdx.x & (F - 1);
    const int step_r = 256 / F;
    const int n_rows = nrbg * nbb;
    const bool live = fl < nfl;
    const uint2 *__restrict__ tab = s_tab + fl * ts;
    const double e_lo = (double)k_min - 1.0, e_hi = (double)k_max + 2.0;
    int rest = (int)threadIdx.x / F, d = 0;
    int g = rest / nbb, jb = rest - g * nbb;
    const int dg = step_r / nbb, djb = step_r - dg * nbb;
    while (rest >= n_rows && d < nd) {
        rest -= n_rows;
        g -= nrbg;
        ++d;
    }
    while (d < nd) {
        uint32_t out = 0u;
        if (live) {
            const double r = s_r[d * F + fl], dk = s_d[d * F + fl];
            const double c = (double)s_c[d * F + fl] * (1.0 / kQd);
            // number of the FFT's peaks whose edge lies below bound z (fine bins)
            auto below = [&](double z) -> int32_t {
                const double e = fmin(fmax(z * dk, e_lo), e_hi);
                int32_t k = (int32_t)rint(e);
                k += (double)(kf * k) * r >= z ? 0 : 1;
                const uint32_t x = (uint32_t)(min(max(k, k_min), k_max + 1) - k_min);
                const uint2 t = tab[x >> 5];
                return (int32_t)(t.y + (uint32_t)__popc(t.x & ((1u << (x & 31)) - 1u)));
            };
            // max_s a_s = floor((Y - min G) / kQ) >= t  <=>  Y >= t kQ + min G
            // min_s a_s = floor((Y - max G) / kQ) >= t  <=>  Y >= t kQ + max G
            const double z_lo = (s_g[2 * (g * F + fl)] - c) + (double)(jb * W - (kf - 1));
            const double z_hi = (s_g[2 * (g * F + fl) + 1] - c) + (double)((jb + 1) * W);
            out = window(below(z_lo), below(z_hi));
        }
        win[((int64_t)(slot0 + d) * n_rows + rest) * n_pad + f0 + fl] = out;
        rest += step_r;
        g += dg;
        jb += djb;
        if (jb >= nbb) {
            jb -= nbb;
            ++g;
        }
        while (rest >= n_rows) {
            rest -= n_rows;
            g -= nrbg;
            ++d;
            if (d >= nd) break;
        }
    }
}

// ----------------------------------------------------------------------------
// peak windows.  A peak reaches tile (row group g, bin block jb) when its
// stripe start, over the group's rows, meets the tile's LDS columns
// [0, W + K_f - 1) measured from fine bin jb*W - (K_f - 1).  Stripe starts are
// monotone in Y, and Y is ascending within an FFT, so the peaks that reach a
// tile form one contiguous range, found by two binary searches.

__global__ void k_windows(int32_t n_fft, const int64_t *__restrict__ offsets,
                          const int64_t *__restrict__ Y, int64_t n_peaks,
                          const int64_t *__restrict__ gwin, int32_t nrbg,
                          int32_t nbb, int32_t W, int32_t kf, uint32_t *__restrict__ win) {
    const int32_t n_pad = win_stride(n_fft);
    const int64_t idx = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
    if (idx >= (int64_t)nbb * n_pad) return;
    const int32_t jb = (int32_t)(idx / n_pad);
    const int32_t i = (int32_t)(idx - (int64_t)jb * n_pad);
    const int32_t g = blockIdx.y, slot = blockIdx.z;
    uint32_t *out = win + (((int64_t)slot * nrbg + g) * nbb + jb) * n_pad + i;
    if (i >= n_fft) {  // padding: empty window
        *out = 0u;
        return;
    }
    const int64_t c0 = (int64_t)jb * W - (kf - 1);
    const int64_t wc = (int64_t)W + kf - 1;
    const int64_t q_lo = gwin[((int64_t)i * nrbg + g) * 2] + c0 * kQ;
    const int64_t q_hi = gwin[((int64_t)i * nrbg + g) * 2 + 1] + c0 * kQ;
    const int64_t *Ys = Y + (int64_t)slot * y_stride(n_peaks, n_fft);
    const int64_t p0 = offsets[i] + (int64_t)kYPad * i, p1 = offsets[i + 1] + (int64_t)kYPad * i;
    // lo: first peak whose larger column is >= 0
    int64_t a = p0, b = p1;
    while (a < b) {
        int64_t m = (a + b) >> 1;
        int64_t y = Ys[m];
        int64_t c1 = shrq(y - q_lo), c2 = shrq(y - q_hi);
        int64_t cmax = c1 > c2 ? c1 : c2;
        if (cmax >= 0) b = m; else a = m + 1;
    }
    const int64_t lo = a;
    // hi: first peak whose smaller column is >= W + K_f - 1
    b = p1;
    while (a < b) {
        int64_t m = (a + b) >> 1;
        int64_t y = Ys[m];
        int64_t c1 = shrq(y - q_lo), c2 = shrq(y - q_hi);
        int64_t cmin = c1 < c2 ? c1 : c2;
        if (cmin >= wc) b = m; else a = m + 1;
    }
    *out = window((int)(lo - p0), (int)(a - p0));
}

// Same windows by one sweep over each FFT's peaks (one wave per FFT, every
// row group): with jhi(p) / jlo(p) the last / first bin block that peak p
// reaches over a group's rows (non-decreasing in p),
//   lo[jb] = first p with jhi(p) >= jb,   hi[jb] = first p with jlo(p) > jb,
// and each lane writes the entries whose boundary falls on its peak.

__device__ __forceinline__ int floor_div_w(int64_t x, int W, float inv_w) {
    int q = (int)floorf((float)x * inv_w);
    if ((int64_t)q * W > x) --q;
    else if ((int64_t)(q + 1) * W <= x) ++q;
    return q;
}

__global__ void __launch_bounds__(256) k_windows_sweep(
    int32_t n_fft, const int64_t *__restrict__ offsets, const int64_t *__restrict__ Y,
    int64_t n_peaks, const int64_t *__restrict__ gwin, int32_t nrbg, int32_t nbb,
    int32_t W, int32_t kf, uint32_t *__restrict__ win) {
    const int lane = threadIdx.x & 63;
    const int i = blockIdx.x * (blockDim.x >> 6) + (threadIdx.x >> 6);
    const int slot = blockIdx.y;
    const int32_t n_pad = win_stride(n_fft);
    if (i >= n_pad) return;
    if (i >= n_fft) {  // padding: empty windows
        for (int e = lane; e < nrbg * nbb; e += 64)
            win[((int64_t)slot * nrbg * nbb + e) * n_pad + i] = 0u;
        return;
    }
    const int64_t *Ys = Y + (int64_t)slot * y_stride(n_peaks, n_fft);
    const int p0 = (int)(offsets[i] + (int64_t)kYPad * i);
    const int p1 = (int)(offsets[i + 1] + (int64_t)kYPad * i);
    const int64_t *gi = gwin + (int64_t)i * nrbg * 2;
    const float inv_w = 1.0f / (float)W;
    for (int g = 0; g < nrbg; ++g) {
        // the two halves of an entry, at stride 2 n_pad
        uint16_t *wg = reinterpret_cast<uint16_t *>(win + ((int64_t)slot * nrbg + g) * nbb * (int64_t)n_pad + i);
        const int64_t q_lo = gi[2 * g], q_hi = gi[2 * g + 1];
        int prev_hi = -1;  // jhi of the peak before this chunk
        int prev_lo = 0;   // jlo of the peak before this chunk
        for (int pb = p0; pb < p1; pb += 64) {
            const int p = pb + lane;
            int jhi = nbb - 1, jlo = nbb;  // past the segment end
            if (p < p1) {
                const int64_t y = Ys[p];
                const int64_t a1 = shrq(y - q_lo), a2 = shrq(y - q_hi);
                const int64_t amin = a1 < a2 ? a1 : a2, amax = a1 < a2 ? a2 : a1;
                jhi = max(-1, min(nbb - 1, floor_div_w(amax + kf - 1, W, inv_w)));
                jlo = max(0, min(nbb, floor_div_w(amin, W, inv_w)));
            }
            int before_hi = __shfl_up(jhi, 1);
            int before_lo = __shfl_up(jlo, 1);
            if (lane == 0) {
                before_hi = prev_hi;
                before_lo = prev_lo;
            }
            if (p < p1) {
                for (int jb = before_hi + 1; jb <= jhi; ++jb) wg[(int64_t)jb * n_pad * 2] = (uint16_t)(p - p0);
                for (int jb = before_lo; jb < jlo; ++jb) wg[(int64_t)jb * n_pad * 2 + 1] = (uint16_t)(p - p0);
            }
            const int last = min(63, p1 - 1 - pb);
            prev_hi = __shfl(jhi, last);
            prev_lo = __shfl(jlo, last);
        }
        // bin blocks past the last peak's reach end at the segment end
        for (int jb = prev_hi + 1 + lane; jb < nbb; jb += 64) wg[(int64_t)jb * n_pad * 2] = (uint16_t)(p1 - p0);
        for (int jb = prev_lo + lane; jb < nbb; jb += 64) wg[(int64_t)jb * n_pad * 2 + 1] = (uint16_t)(p1 - p0);
    }
}

// ----------------------------------------------------------------------------
// tiles

// Window rows ordered for the tiles.  Run w of a row holds every
// kTileWaves-th FFT, w, w + 16, w + 32, ... (so that every run spans the
// whole observation, whose windows widen with |t - t0|); its wave_ffts(N)
// FFTs are sorted by window size, largest first (a counting sort over sizes
// clipped to 127; the few windows of 127 peaks or more, which share the first
// bucket, are ranked exactly among themselves), so that the four FFTs of a
// tile block (four consecutive entries of a run) have nearly equal windows
// and the first holds the largest, which the tiles rely on.  An entry becomes
// (place of its first edge, m << 16 | count): FFT m * 16 + w of the row, whose
// edges start at base[w * wave_ffts(N) + m].  One workgroup per window row (grid.x = row group *
// bin blocks, grid.y = slot), one wave per run.
// Bound by the LDS atomics of the counts, many of which meet in the few buckets
// of the common sizes: there is one per entry, whose result is also the
// entry's rank in its bucket (a second pass of atomics that placed the entries
// made the sort half as long again).  The row is staged in LDS run by run, since
// its runs are strided (16 lanes to a bank), and the first edges lie in memory
// run by run too.  19 040 rows of 6336 entries: 517 -> 378 us.
constexpr int kSortBuckets = 128;
constexpr int kSortLdsBytes = kLdsBytes - kTileWaves * kSortBuckets * 4 - kLdsReserve;

// Place of a window of c >= 127 peaks (entry e of a run of `per`) among the
// run's windows of 127 peaks or more, which fill the run's first places:
// larger first, equal sizes in run order.  size(j) is that of entry j.
// Such windows are rare (dense peakmaps, K_f = 1), so a scan of the run is
// cheap enough.
template <typename Size>
__device__ __forceinline__ int big_window_rank(int c, int e, int per, Size size) {
    int pos = 0;
    for (int j = 0; j < per; ++j) {
        const int cj = size(j);
        pos += (cj > c || (cj == c && j < e)) ? 1 : 0;
    }
    return pos;
}

// A sorted entry as the tiles take it: the byte offset of the window's first
// stripe edge in the slot's edges, and FFT place in the run << 16 | peak
// count.  Entries past the last FFT (no peaks) name place 0, so that their
// table reads stay inside the tables.

// Words between the staged runs: 4 modulo 16, so that the four quarters of 16
// entries that a wave stores together lie in 64 banks.
__host__ __device__ inline int sort_run_stride(int per) { return per + ((4 - per) & 15); }

// The slot's fixed-point weights, when the front left them to the sort (its
// statistics came from the same launch); grid.x workgroups share them.
__device__ __forceinline__ void fixed_weights(int32_t n_fft, const WeightArgs &A) {
    if (A.w == nullptr) return;
    const int64_t slot = blockIdx.y;
    const WeightStats st = A.ws[slot * A.ws_stride];
    for (int i = blockIdx.x * blockDim.x + threadIdx.x; i < n_fft; i += gridDim.x * blockDim.x) {
        const double wi = (double)A.w[slot * A.w_stride + i];
        A.wq[slot * n_fft + i] = st.bad ? 0u : (uint32_t)rint(ldexp(wi, st.frac_bits));
    }
}

__device__ __forceinline__ int window_size(uint32_t w) { return (int)(w >> 16) - (int)(w & 0xFFFFu); }

// Exclusive prefix sums over a run's buckets (lane L holds buckets 2L, 2L+1).
__device__ __forceinline__ void scan_buckets(int *h, int lane) {
    const int a0 = h[2 * lane], a1 = h[2 * lane + 1];
    int incl = a0 + a1;
    for (int o = 1; o < 64; o <<= 1) {
        const int t = __shfl_up(incl, o);
        if (lane >= o) incl += t;
    }
    const int excl = incl - (a0 + a1);
    __syncthreads();
    h[2 * lane] = excl;
    h[2 * lane + 1] = excl + a0;
    __syncthreads();
}

__global__ void __launch_bounds__(kTileThreads) k_sort_windows(int32_t n_fft, int32_t nrows,
                                                               const uint32_t *__restrict__ win,
                                                               const uint32_t *__restrict__ base,
                                                               int2 *__restrict__ wsorted, WeightArgs wa) {
    fixed_weights(n_fft, wa);
    extern __shared__ uint32_t s_run[];  // the row, run by run, then the entries' ranks in their buckets (16-bit)
    __shared__ int hist[kTileWaves][kSortBuckets];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int per = wave_ffts(n_fft);
    const int n_pad = win_stride(n_fft);  // a multiple of 64 entries
    const int rs = sort_run_stride(per);
    const int64_t row = (int64_t)blockIdx.y * nrows + blockIdx.x;
    // FFT m * kTileWaves + w of the row is entry m of run w
    {
        const uint4 *g4 = reinterpret_cast<const uint4 *>(win + row * n_pad);
        for (int i = threadIdx.x; i < n_pad / 4; i += blockDim.x) {
            const uint4 q = g4[i];
            uint32_t *d = s_run + (i & 3) * 4 * rs + (i >> 2);
            d[0] = q.x;
            d[rs] = q.y;
            d[2 * rs] = q.z;
            d[3 * rs] = q.w;
        }
    }
    const uint32_t *src = s_run + wave * rs;
    uint16_t *rk = reinterpret_cast<uint16_t *>(s_run + kTileWaves * rs) + wave * per;
    int2 *dst = wsorted + row * n_pad + (int64_t)wave * per;
    int *h = hist[wave];
    for (int b = lane; b < kSortBuckets; b += 64) h[b] = 0;
    __syncthreads();
    constexpr int kU = 4;  // entries per lane and round, their LDS accesses issued together
    for (int e0 = lane; e0 < per; e0 += kU * 64) {
        int c[kU], r[kU];
#pragma unroll
        for (int u = 0; u < kU; ++u) c[u] = e0 + 64 * u < per ? window_size(src[e0 + 64 * u]) : -1;
#pragma unroll
        for (int u = 0; u < kU; ++u)
            r[u] = c[u] >= 0 ? atomicAdd(&h[kSortBuckets - 1 - min(c[u], kSortBuckets - 1)], 1) : 0;
#pragma unroll
        for (int u = 0; u < kU; ++u)
            if (c[u] >= 0) rk[e0 + 64 * u] = (uint16_t)r[u];
    }
    __syncthreads();
    scan_buckets(h, lane);
    for (int e0 = lane; e0 < per; e0 += kU * 64) {
        uint32_t w[kU], b[kU];
#pragma unroll
        for (int u = 0; u < kU; ++u) {
            const int e = e0 + 64 * u, i = e * kTileWaves + wave;
            b[u] = e < per && i < n_fft ? base[wave * per + e] : 0u;
            w[u] = e < per ? src[e] : 0u;
        }
#pragma unroll
        for (int u = 0; u < kU; ++u) {
            const int e = e0 + 64 * u;
            if (e >= per) break;
            const int c = window_size(w[u]);
            const int pos = c >= kSortBuckets - 1
                                ? big_window_rank(c, e, per, [&](int j) { return window_size(src[j]); })
                                : h[kSortBuckets - 1 - c] + rk[e];
            const int place = e * kTileWaves + wave < n_fft ? e : 0;
            dst[pos] = make_int2((int)((b[u] + (w[u] & 0xFFFFu)) << 2), (place << 16) | c);
        }
    }
}

// Rows whose entries and ranks do not fit the LDS (more than 25 728 FFTs): the same sort, the
// row copied into LDS in pieces of kSortPiece entries (128 KB), once per pass,
// and the entries written where they belong.
constexpr int kSortPiece = 32768;

__global__ void __launch_bounds__(kTileThreads) k_sort_windows_long(int32_t n_fft, int32_t nrows,
                                                                    const uint32_t *__restrict__ win,
                                                                    const uint32_t *__restrict__ base,
                                                                    int2 *__restrict__ wsorted, WeightArgs wa) {
    fixed_weights(n_fft, wa);
    extern __shared__ uint4 s_row4[];
    __shared__ int hist[kTileWaves][kSortBuckets];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int per = wave_ffts(n_fft);
    const int n_pad = win_stride(n_fft);  // a multiple of 64 entries
    const int64_t row = (int64_t)blockIdx.y * nrows + blockIdx.x;
    const uint32_t *rowp = win + row * n_pad;
    const uint32_t *s_row = reinterpret_cast<const uint32_t *>(s_row4);
    int2 *dst = wsorted + row * n_pad + (int64_t)wave * per;
    int *h = hist[wave];
    for (int b = lane; b < kSortBuckets; b += 64) h[b] = 0;
    // entry e of run `wave` is row entry e * kTileWaves + wave; a piece
    // starting at p0 holds the run's entries [p0 / 16, (p0 + piece) / 16)
    for (int pass = 0; pass < 2; ++pass) {
        for (int p0 = 0; p0 < n_pad; p0 += kSortPiece) {
            __syncthreads();
            const uint4 *g4 = reinterpret_cast<const uint4 *>(rowp + p0);
            for (int i = threadIdx.x; i < min(kSortPiece, n_pad - p0) / 4; i += blockDim.x) s_row4[i] = g4[i];
            __syncthreads();
            const int e_lo = p0 / kTileWaves, e_hi = min(per, (p0 + kSortPiece) / kTileWaves);
            for (int e = e_lo + lane; e < e_hi; e += 64) {
                const uint32_t w = s_row[(e - e_lo) * kTileWaves + wave];
                const int c = window_size(w);
                if (pass == 0) {
                    atomicAdd(&h[kSortBuckets - 1 - min(c, kSortBuckets - 1)], 1);
                    continue;
                }
                int pos;
                if (c >= kSortBuckets - 1)  // the run's other pieces are not staged: read the row in memory
                    pos = big_window_rank(c, e, per, [&](int j) { return window_size(rowp[(int64_t)j * kTileWaves + wave]); });
                else
                    pos = atomicAdd(&h[kSortBuckets - 1 - c], 1);
                const int i = e * kTileWaves + wave;
                const uint32_t b = i < n_fft ? base[wave * per + e] : 0u;
                dst[pos] = make_int2((int)((b + (w & 0xFFFFu)) << 2), ((i < n_fft ? e : 0) << 16) | c);
            }
        }
        __syncthreads();
        if (pass == 0) scan_buckets(h, lane);
    }
}

// Raw buffer access with unsigned 32-bit byte offsets (no 64-bit address
// arithmetic per load), unlimited: a direction's stripe edges may fill 4 GiB.
__device__ __forceinline__ __amdgpu_buffer_rsrc_t buf(const void *p) {
    return __builtin_amdgcn_make_buffer_rsrc(const_cast<void *>(p), 0, (int)0xFFFFFFFFu, 0x00020000);
}
__device__ __forceinline__ uint32_t ld_u32(__amdgpu_buffer_rsrc_t r, uint32_t byte_off) {
    return __builtin_amdgcn_raw_buffer_load_b32(r, byte_off, 0, 0);
}

// s_waitcnt operand that waits for every vector-memory access of the wave
// (vmcnt 0) and leaves the export and LDS/scalar counters alone.
constexpr int kWaitVmcnt0 = (0x7 << 4) | (0xF << 8);

// Workgroup barrier that orders LDS accesses only: global stores and atomics
// still in flight are not waited for.
__device__ __forceinline__ void lds_barrier() {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup", "local");
    __builtin_amdgcn_s_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup", "local");
}

// LDS tile: word (c, j) = c * 16 + j holds the stripe starts of column c
// (fine bin jb*W - (K_f-1) + c) in row s0 + j; column W + K_f - 1 is a dump
// column for updates that fall outside the tile.  The 16 lanes of a group
// address 16 consecutive words, so a group's part of an LDS atomic never
// conflicts with itself (the four groups of a wave can still collide on the
// bank halves that their columns map to).
// One step of the accumulation.  Lane (group g, row j) adds the stripe of the
// peak held by lane (g, U): its edge v = Y reaches the group's 16 lanes
// through DPP row_newbcast:U fused into the add of the lane's row term
// t = -c0 kQ - G_{i,s0+j} (the sum is exact in 32 bits for every peak of a
// window).  The upper half-word of the sum is the tile column of the stripe
// start in row s0 + j; columns outside [0, W + K_f - 1) (negative ones read
// as 2^15 and more) go to the group's dump column.
//
// stripe_steps runs steps n-1 .. 0 of up to 32 peaks of each group's FFT:
// lane j of a group holds the edges of its peaks j (v0) and 16 + j (v1).  The
// steps are one straight sequence, entered by a computed jump n steps before
// its end, so a block of four FFTs takes one jump.  With the peaks in
// patterns of 8, 4, 2, 1 and 1 lanes and a scalar test before each run a block
// issued 14 branches, 36 scalar and 98 vector instructions for its ~20 steps;
// now 3, about 30 and 80.  The step itself was never the limit (alone, its
// three vector instructions and its LDS update take 4.13 clocks per CU, the
// update's own 4.1): the branches were, each one a gap in its wave's issue,
// and with four waves per SIMD the gaps reached the LDS.  Tile kernel, 112
// directions of the 256 Hz batch: 21.7 -> 18.7 ms, 69 -> 80 % of the LDS
// rate; 13 directions of a 1162-row grid 5.36 -> 4.48 ms; 24 of a 10 Hz band
// 11.6 -> 10.7 ms.  The LDS updates are outside the compiler's count: who
// waits for them says so.
#define FH_STEP(U, V)                                                                       \
    "v_add_u32_dpp %[a], " V ", %[t] row_newbcast:" #U " row_mask:0xf bank_mask:0xf\n"      \
    "v_min_u32_sdwa %[a], %[a], %[dump] dst_sel:DWORD dst_unused:UNUSED_PAD src0_sel:WORD_1 src1_sel:DWORD\n" \
    "v_lshl_add_u32 %[a], %[a], 6, %[lane]\n"                                               \
    "ds_add_u32 %[a], %[val]\n"
#define FH_STEPS16(V)                                                                       \
    FH_STEP(15, V) FH_STEP(14, V) FH_STEP(13, V) FH_STEP(12, V) FH_STEP(11, V) FH_STEP(10, V) \
    FH_STEP(9, V) FH_STEP(8, V) FH_STEP(7, V) FH_STEP(6, V) FH_STEP(5, V) FH_STEP(4, V)      \
    FH_STEP(3, V) FH_STEP(2, V) FH_STEP(1, V) FH_STEP(0, V)
__device__ __forceinline__ void stripe_steps(int n, uint32_t v0, uint32_t v1, uint32_t t, uint32_t dump,
                                             uint32_t lane_addr, uint32_t val) {
    const int skip = 12 + (32 - n) * 32;  // bytes from the instruction after s_getpc; 0 <= n <= 32
    uint32_t a;
    asm volatile(
        "s_getpc_b64 s[98:99]\n"
        "s_add_u32 s98, s98, %[skip]\n"
        "s_addc_u32 s99, s99, 0\n"
        "s_setpc_b64 s[98:99]\n"
        ".Lsteps%=:\n" FH_STEPS16("%[v1]") FH_STEPS16("%[v0]")
        ".if (. - .Lsteps%=) != 1024\n.error \"a step is not 32 bytes\"\n.endif\n"
        : [a] "=&v"(a)
        : [skip] "s"(skip), [v0] "v"(v0), [v1] "v"(v1), [t] "v"(t), [dump] "v"(dump), [lane] "v"(lane_addr),
          [val] "v"(val)
        : "memory", "scc", "s98", "s99");
}

// Tail rows (rows 16 .. 16 + A.tail - 1 of the tiles of the last run row
// block): every lane adds its own peak's stripe start in each tail row, one
// atomic per peak and row, in the row-major tail region `lt` (row stride
// `stride` words).  Lane r of a group holds the group's tail row term of row
// 16 + r, broadcast to the group by DPP row_newbcast:r fused into the add;
// lanes past the window (whose edge lies far away) and starts outside the
// tile go to the lane's own dump word, so that no two lanes of an atomic
// update one word.
template <int R>
__device__ __forceinline__ void tail_row(uint32_t v, uint32_t tt, uint32_t dump, uint32_t val,
                                         uint32_t *__restrict__ lt) {
    const uint32_t b = __builtin_amdgcn_update_dpp(0u, tt, 0x150 + R, 0xF, 0xF, true);
    const uint16_t col = (uint16_t)((v + b) >> kFrac);
    const uint32_t cu = col < (uint16_t)dump ? col : (uint16_t)dump;
    atomicAdd(lt + cu, val);
}

__device__ __forceinline__ void tail_steps(int rows, uint32_t v, uint32_t tt, uint32_t dump, uint32_t stride,
                                           uint32_t val, uint32_t *__restrict__ lt) {
    static_assert(kTailRows == 3, "tail_steps unrolls kTailRows rows");
    tail_row<0>(v, tt, dump, val, lt);
    if (rows > 1) tail_row<1>(v, tt, dump, val, lt + stride);
    if (rows > 2) tail_row<2>(v, tt, dump, val, lt + 2 * stride);
}

// One block: four consecutive FFTs of a sorted run, entry 4 b + g in lane
// group g.  Lane (g, j) holds its group's window, row term and weight, and
// the stripe edges of peaks j and 16 + j.
struct Quad {
    int g, run;          // block id claimed from the tile's counter; its run g % 16
    uint32_t lo;         // byte offset of the window's first stripe edge
    uint32_t pk;         // FFT place in the run << 16 | peak count
    uint32_t gb, codes;  // G_{i,s0} of the group's FFT i (mod 2^32); residual codes of its rows
    uint32_t step;       // 1 - floor(j q_i / 2^16) (mod 2^32)
    uint32_t gb2, codes2;  // record of the tail rows (tiles with tail rows)
    uint32_t wq;         // fixed-point weight
    int cnt;             // peaks in the window
    uint32_t y0, y1;     // low words of the stripe edges of peaks j and 16 + j, or their natural bins
    uint32_t rl, rh, c;  // (natural bins) the FFT's edge terms
    int cmax;            // largest window of the four groups
};

__device__ __forceinline__ void decode_tile(const TileArgs &A, int t, int &slot, int &rb, int &jb) {
    jb = t % A.nbb;
    const int r = t / A.nbb;
    rb = r % A.nrb;
    slot = r / A.nrb;
}
// Tile t as its slot, row block and bin block; slot -1: none.
__device__ __forceinline__ int4 tile_place(const TileArgs &A, int t) {
    if (t < 0) return make_int4(-1, 0, 0, 0);
    int slot, rb, jb;
    decode_tile(A, t, slot, rb, jb);
    return make_int4(slot, rb, jb, 0);
}

// Persistent form.  Tile groups (sky, bin block) are dealt round-robin to
// kXcds queues (workgroups are dispatched round-robin over the XCDs, so
// workgroup w serves queue w % 8 and the tiles of one group, which read the
// same stripe edges, stay in one XCD's L2); a queue holds its groups in order,
// each with all its row blocks.  Position pos of queue qi is therefore
// group qi + 8 (pos / nrb), row block pos % nrb.
__device__ __forceinline__ int queue_len(const TileArgs &A, int qi) {
    const int groups = A.n_slots * A.nbb;
    return qi < groups ? A.nrb * ((groups - qi + kXcds - 1) / kXcds) : 0;
}

__device__ __forceinline__ int queue_tile(const TileArgs &A, int qi, int pos) {
    const int k = pos / A.nrb, rb = pos - k * A.nrb;
    const int grp = qi + kXcds * k;
    const int sl = grp / A.nbb, jb = grp - sl * A.nbb;
    return (sl * A.nrb + rb) * A.nbb + jb;
}

// A tile from the first queue, starting at `home`, that is not exhausted; -1
// when all are.  *at: its position in the home queue, kNotHome elsewhere.
constexpr int kNotHome = 0x3fffffff;

__device__ int steal_tile(const TileArgs &A, int home, int *at) {
    for (int k = 0; k < kXcds; ++k) {
        const int qi = (home + k) % kXcds;
        const int len = queue_len(A, qi);
        if (__hip_atomic_load(A.queue_ctr + qi, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) >= len)
            continue;
        const int pos = atomicAdd(A.queue_ctr + qi, 1);
        if (pos < len) {
            *at = k == 0 ? pos : kNotHome;
            return queue_tile(A, qi, pos);
        }
    }
    return -1;
}

// LDS words of a tile: W + K_f - 1 columns plus the dump columns, 16 rows
// (column-major), then A.tail rows of W + K_f - 1 + kTailDump words
// (row-major).
__device__ __forceinline__ int tile_words(const TileArgs &A) {
    return kTileRows * (A.W + A.kf - 1 + kDumpCols) + A.tail * (A.W + A.kf - 1 + kTailDump);
}

__device__ __forceinline__ void tile_zero(const TileArgs &A, uint32_t *__restrict__ lds) {
    const int nwords = tile_words(A);
    for (int x = threadIdx.x * 4; x < nwords; x += blockDim.x * 4) {
        if (x + 3 < nwords) {
            *reinterpret_cast<uint4 *>(lds + x) = make_uint4(0, 0, 0, 0);
        } else {
            for (int y = x; y < nwords; ++y) lds[y] = 0;
        }
    }
}

// Output phase of tile (slot, rb, jb) for K_f > kHold + 1: per-row window sums
// of the start histogram, written as a map or reduced to per-bin column maxima.
// Column maxima: a lane group owns a segment [x0, x1) of columns.  Its first
// K_f - 1 columns are still read by the previous group's window sums, so
// their maxima are reduced across the group's 16 lanes at once (DPP); every
// later column is read by its own group only, and its window sums replace
// its start counts in place.  After a barrier one thread per such column
// reduces the 16 rows in registers and updates the global maximum.
template <bool WEIGHTED, bool MAP>
__device__ __forceinline__ void tile_output(const TileArgs &A, int slot, int rb, int jb,
                                            uint32_t *__restrict__ lds) {
    constexpr bool COLMAX = !MAP;
    const int tid = threadIdx.x;
    const int j = tid & 15;
    const int W = A.W, kf = A.kf;
    const int s0 = rb * kTileRows;
    // Row sums: H(x) = sum_{c = x}^{x + K_f - 1} P(c), x in [0, W): the +w at
    // the stripe start and the -w K_f bins later, prefix-summed along the row.
    const int nseg = blockDim.x / kTileRows;
    const int seg = tid >> 4;
    const int len = (W + nseg - 1) / nseg;
    const int64_t bbase = (int64_t)jb * W;
    const int xend = (int)min((int64_t)W, (int64_t)A.nf - bbase);  // columns of the map
    const int x0 = seg * len;
    const int x1 = min(x0 + len, xend);
    const int xs = x0 + kf - 1;  // first column rewritten in place
    const int s = s0 + j;
    const bool row_ok = s < A.ns;
    uint32_t *__restrict__ P = lds + j;
    unsigned long long *__restrict__ cm = A.colmax + (int64_t)slot * A.nf + bbase;
    float scale = 1.0f;
    if (WEIGHTED) scale = ldexpf(1.0f, -A.ws[(int64_t)slot * A.ws_stride].frac_bits);
    uint32_t acc = 0;
    if (x0 < x1)
        for (int c = x0; c < x0 + kf - 1; ++c) acc += P[c * kTileRows];
    for (int x = x0; x < x1; ++x) {
        acc += P[(x + kf - 1) * kTileRows];
        const int64_t b = bbase + x;
        if (MAP && row_ok) {
            if (WEIGHTED) A.map_f32[(int64_t)s * A.nf + b] = (float)acc * scale;
            else A.map_i32[(int64_t)s * A.nf + b] = (int32_t)acc;
        }
        const uint32_t trail = P[x * kTileRows];
        if (COLMAX && x < xs) {
            // largest value over the 16 rows (DPP row_shr prefix max: lane 15
            // ends with it), then the smallest row holding it (prefix min)
            const uint32_t a = row_ok ? acc : 0u;
            uint32_t mx = a;
            mx = max(mx, (uint32_t)__builtin_amdgcn_update_dpp(0, (int)mx, 0x111, 0xF, 0xF, false));
            mx = max(mx, (uint32_t)__builtin_amdgcn_update_dpp(0, (int)mx, 0x112, 0xF, 0xF, false));
            mx = max(mx, (uint32_t)__builtin_amdgcn_update_dpp(0, (int)mx, 0x114, 0xF, 0xF, false));
            mx = max(mx, (uint32_t)__builtin_amdgcn_update_dpp(0, (int)mx, 0x118, 0xF, 0xF, false));
            const uint32_t top = (uint32_t)__builtin_amdgcn_update_dpp(0, (int)mx, 0x15F, 0xF, 0xF, true);
            int r = row_ok && a == top ? j : kTileRows;
            r = min(r, __builtin_amdgcn_update_dpp(r, r, 0x111, 0xF, 0xF, false));
            r = min(r, __builtin_amdgcn_update_dpp(r, r, 0x112, 0xF, 0xF, false));
            r = min(r, __builtin_amdgcn_update_dpp(r, r, 0x114, 0xF, 0xF, false));
            r = min(r, __builtin_amdgcn_update_dpp(r, r, 0x118, 0xF, 0xF, false));
            if (j == kTileRows - 1)
                atomicMax(cm + x, ((unsigned long long)top << 32) | (0xFFFFFFFFull - (unsigned)(s0 + r)));
        } else if (COLMAX) {
            P[x * kTileRows] = row_ok ? acc : 0u;
        }
        acc -= trail;
    }
    if (!COLMAX) return;
    lds_barrier();
    // columns rewritten in place: x in [x0 + K_f - 1, x1) of each segment
    for (int x = tid; x < xend; x += blockDim.x) {
        const int sx = x / len;
        if (x < sx * len + kf - 1) continue;
        const uint4 *q = reinterpret_cast<const uint4 *>(lds + x * kTileRows);
        const uint4 h0 = q[0], h1 = q[1], h2 = q[2], h3 = q[3];
        const uint32_t h[16] = {h0.x, h0.y, h0.z, h0.w, h1.x, h1.y, h1.z, h1.w,
                                h2.x, h2.y, h2.z, h2.w, h3.x, h3.y, h3.z, h3.w};
        uint32_t top = h[0];
#pragma unroll
        for (int k = 1; k < kTileRows; ++k) top = max(top, h[k]);
        // smallest row holding the maximum (rows past the grid hold 0, and
        // row 0 always exists, so a row past the grid is never chosen)
        int r = kTileRows - 1;
#pragma unroll
        for (int k = kTileRows - 2; k >= 0; --k) r = h[k] == top ? k : r;
        atomicMax(cm + x, ((unsigned long long)top << 32) | (0xFFFFFFFFull - (unsigned)(s0 + r)));
    }
}

// Output of tile (slot, rb, jb) for K_f <= kHold + 1: column maxima (the
// candidate search), or the map.
// Phase 1, lane group = segment of columns, lane = row: the window sums H(x)
// along each row.  The first K_f - 1 columns of a segment are still read by
// the previous segment, so their sums wait in registers; the later ones are
// rewritten in place, eight columns per round with every LDS read of a round
// issued before the first is used.  After a barrier the held sums go back in
// place, and after another one, phase 2: one thread per column either reduces
// its 16 rows and updates the global maximum, or writes them to the map,
// where consecutive lanes then write consecutive bins of a row (stores by the
// lanes of phase 1, one row each, went to 64 lines per instruction: the tile
// kernel of the 100 Hz map of 3140 FFTs and 118 rows took 140 us, now 89 us,
// also through an even cut of the band).  A persistent
// kernel also clears the column for its next tile (dump columns and columns
// past the map are only cleared).  `mid` runs between the
// phases (the caller's prefetch of the next tile); the caller's barrier then
// separates the clearing from the next tile's updates.
constexpr int kHold = 9;  // held columns per lane: K_f - 1 <= kHold
constexpr int kRound = 8;  // columns per round of the first output phase

// The whole rounds of the first phase from column x of a segment ending at
// x1: window sums written in place, with no test per column; MASK writes
// zeros for a row past the grid (only the last row block has such rows).
// Returns the first column not done (fewer than kRound remain).
template <bool MASK>
__device__ __forceinline__ int colmax_rounds(uint32_t *__restrict__ P, int x, int x1, int kf,
                                             uint32_t &acc, bool row_ok) {
    for (; x + kRound <= x1; x += kRound) {
        const uint32_t *ph = P + (x + kf - 1) * kTileRows;
        uint32_t *pt = P + x * kTileRows;
        uint32_t h[kRound], t[kRound], o[kRound];
#pragma unroll
        for (int c = 0; c < kRound; ++c) {
            h[c] = ph[c * kTileRows];
            t[c] = pt[c * kTileRows];
        }
#pragma unroll
        for (int c = 0; c < kRound; ++c) {
            acc += h[c];
            o[c] = MASK && !row_ok ? 0u : acc;
            acc -= t[c];
        }
        // a round's writes follow all of its reads: column x + c is read as a
        // head by earlier rounds only, and as a trail by this round
#pragma unroll
        for (int c = 0; c < kRound; ++c) pt[c * kTileRows] = o[c];
    }
    return x;
}

template <bool WEIGHTED, bool MAP, bool CLEAR, typename Mid>
__device__ __forceinline__ void tile_windows(const TileArgs &A, int slot, int rb, int jb,
                                             uint32_t *__restrict__ lds, Mid mid) {
    const int tid = threadIdx.x;
    const int j = tid & 15;
    const int W = A.W, kf = A.kf;
    const int s0 = rb * kTileRows;
    const int nseg = blockDim.x / kTileRows;
    const int seg = tid >> 4;
    const int len = (W + nseg - 1) / nseg;
    const int64_t bbase = (int64_t)jb * W;
    const int xend = (int)min((int64_t)W, (int64_t)A.nf - bbase);  // columns of the map
    const int x0 = seg * len;
    const int x1 = min(x0 + len, xend);
    const int nh = max(0, min(kf - 1, x1 - x0));  // held columns [x0, x0 + nh)
    const bool row_ok = s0 + j < A.ns;
    uint32_t *__restrict__ P = lds + j;
    unsigned long long *__restrict__ cm = A.colmax + (int64_t)slot * A.nf + bbase;

    // Phase 1.  Reads past a segment's end are clamped to its last column
    // (their values are not used); W is a multiple of 64, so a segment starts
    // at column 63 len <= W even past the map, and no read passes column
    // W + K_f - 1 (the first dump column).
    uint32_t acc = 0;
    if (x0 < x1)
        for (int c = x0; c < x0 + kf - 1; ++c) acc += P[c * kTileRows];
    uint32_t hold[kHold];
    {
        uint32_t h[kHold], t[kHold];
#pragma unroll
        for (int c = 0; c < kHold; ++c) {
            const int xc = x0 + min(c, max(nh - 1, 0));
            h[c] = P[(xc + kf - 1) * kTileRows];
            t[c] = P[xc * kTileRows];
        }
#pragma unroll
        for (int c = 0; c < kHold; ++c) {
            const uint32_t v = acc + h[c];
            hold[c] = row_ok ? v : 0u;
            if (c < nh) acc = v - t[c];
        }
    }
    int x = x0 + nh;
    if (s0 + kTileRows <= A.ns) x = colmax_rounds<false>(P, x, x1, kf, acc, true);
    else x = colmax_rounds<true>(P, x, x1, kf, acc, row_ok);
    if (x < x1) {  // the segment's last, partial round
        uint32_t h[kRound], t[kRound], o[kRound];
#pragma unroll
        for (int c = 0; c < kRound; ++c) {
            const int xc = min(x + c, x1 - 1);
            h[c] = P[(xc + kf - 1) * kTileRows];
            t[c] = P[xc * kTileRows];
        }
#pragma unroll
        for (int c = 0; c < kRound; ++c) {
            acc += h[c];
            o[c] = row_ok ? acc : 0u;
            acc -= t[c];
        }
#pragma unroll
        for (int c = 0; c < kRound; ++c)
            if (x + c < x1) P[(x + c) * kTileRows] = o[c];
    }
    mid();
    lds_barrier();
#pragma unroll
    for (int c = 0; c < kHold; ++c)
        if (c < nh) P[(x0 + c) * kTileRows] = hold[c];
    lds_barrier();

    // Phase 2.  Lane l reads the four 16-byte quarters of its column starting
    // at quarter (l >> 1) & 3: with columns 64 bytes apart, every eight lanes
    // then cover the 32 banks once.
    const int ncols = CLEAR ? W + kf - 1 + kDumpCols : xend;
    const int st = ((tid & 63) >> 1) & 3;
    int qo[4];
#pragma unroll
    for (int k = 0; k < 4; ++k) qo[k] = (k + st) & 3;
    const uint4 z = make_uint4(0u, 0u, 0u, 0u);
    float scale = 1.0f;
    if (MAP && WEIGHTED) scale = ldexpf(1.0f, -A.ws[(int64_t)slot * A.ws_stride].frac_bits);
    for (int c = tid; c < ncols; c += blockDim.x) {
        uint4 *q = reinterpret_cast<uint4 *>(lds + c * kTileRows);
        if (MAP && c < xend) {
            uint4 v[4];
#pragma unroll
            for (int k = 0; k < 4; ++k) v[k] = q[qo[k]];
#pragma unroll
            for (int k = 0; k < 4; ++k) {
                const uint32_t h[4] = {v[k].x, v[k].y, v[k].z, v[k].w};
#pragma unroll
                for (int r = 0; r < 4; ++r) {
                    const int s = s0 + 4 * qo[k] + r;
                    if (s < A.ns) {
                        const int64_t at = (int64_t)s * A.nf + bbase + c;
                        if (WEIGHTED) A.map_f32[at] = (float)h[r] * scale;
                        else A.map_i32[at] = (int32_t)h[r];
                    }
                }
            }
        } else if (c < xend) {
            uint4 v[4];
#pragma unroll
            for (int k = 0; k < 4; ++k) v[k] = q[qo[k]];
            uint32_t top = 0;
#pragma unroll
            for (int k = 0; k < 4; ++k) top = max(max(top, max(v[k].x, v[k].y)), max(v[k].z, v[k].w));
            // smallest row holding the maximum (rows past the grid hold 0,
            // and row 0 always exists, so a row past the grid is never chosen)
            int r = kTileRows;
#pragma unroll
            for (int k = 0; k < 4; ++k) {
                const int rk = v[k].x == top ? 0 : v[k].y == top ? 1 : v[k].z == top ? 2 : v[k].w == top ? 3 : 4;
                r = min(r, rk < 4 ? 4 * qo[k] + rk : kTileRows);
            }
            atomicMax(cm + c, ((unsigned long long)top << 32) | (0xFFFFFFFFull - (unsigned)(s0 + r)));
        }
        if (CLEAR) {
#pragma unroll
            for (int k = 0; k < 4; ++k) q[qo[k]] = z;
        }
    }
}

// Column maxima of an unweighted tile at K_f = kColKf, in registers: a lane
// holds one 16-byte quarter (four rows) of kColSeg consecutive columns, the
// four lanes of a quad one segment (kColSeg is odd, so that the segments of a
// wave start in different banks).  Prefix sums along the segment carry
// 16 count + 15 - row, so that one maximum finds the largest count and its
// smallest row; lane q of the quad keeps columns q, q + 4 and q + 8.  (Counts
// are at most two per FFT and the FFTs fewer than 2^20, so nothing overflows.)
// The general output below rewrites the tile in LDS and reads it again.
// Weighted sums fill their 32 bits, the row then costs as much again in
// vector instructions, and the general output is as fast (256 Hz batch within
// 0.5 %, 10 Hz band 1 % faster).  Tile kernel, 1162 rows, 13 directions: 4.49
// -> 4.29 ms, half of it from the next tile being decoded by the thread that
// claims it (weighted, 256 Hz batch: 18.46 -> 18.29 ms).
constexpr int kColKf = 10;
constexpr int kColSeg = 11;
constexpr int kWaveCols = 16 * kColSeg;  // columns of a wave's segments

template <bool MASK>
__device__ __forceinline__ void colmax_keys(const uint32_t *__restrict__ lds, int x0, int q, int rows,
                                            uint32_t (&key)[3]) {
    constexpr int kReads = kColSeg + kColKf - 1;
    const uint4 *__restrict__ p = reinterpret_cast<const uint4 *>(lds + x0 * kTileRows + 4 * q);
    const uint32_t code = 15u - 4u * (uint32_t)q;  // of the quarter's first row
    uint32_t keep[4];
#pragma unroll
    for (int k = 0; k < 4; ++k) keep[k] = !MASK || 4 * q + k < rows ? ~0u : 0u;
    uint32_t a[kReads][4];  // 16 x sums of columns [x0, x0 + i], and the code once per kColKf columns
    uint32_t acc[4] = {0u, 0u, 0u, 0u};
#pragma unroll
    for (int i = 0; i < kReads; ++i) {
        const uint4 h4 = p[i * 4];
        const uint32_t h[4] = {h4.x, h4.y, h4.z, h4.w};
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            acc[k] = (h[k] << 4) + acc[k];
            if (i % kColKf == kColKf - 1) acc[k] += code - (uint32_t)k;
            a[i][k] = acc[k];
        }
        const int c = i - (kColKf - 1);  // the column that is complete now
        if (c < 0) continue;
        uint32_t v[4];
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            v[k] = c == 0 ? acc[k] : acc[k] - a[c - 1][k];
            if (MASK) v[k] &= keep[k];
        }
        uint32_t best = max(max(v[0], v[1]), max(v[2], v[3]));
        best = max(best, (uint32_t)__builtin_amdgcn_update_dpp(0, (int)best, 0xB1, 0xF, 0xF, true));
        best = max(best, (uint32_t)__builtin_amdgcn_update_dpp(0, (int)best, 0x4E, 0xF, 0xF, true));
        if (q == (c & 3)) key[c >> 2] = best;
    }
}

template <bool CLEAR, typename Mid>
__device__ __forceinline__ void tile_colmax(const TileArgs &A, int slot, int rb, int jb,
                                            uint32_t *__restrict__ lds, Mid mid) {
    const int tid = threadIdx.x;
    const int W = A.W;
    const int q = tid & 3;
    const int s0 = rb * kTileRows;
    const int64_t bbase = (int64_t)jb * W;
    const int xend = (int)min((int64_t)W, (int64_t)A.nf - bbase);  // columns of the map
    // the last segment starts early enough to end with the tile: the columns
    // it shares with the one before are raised twice, to the same values (W is
    // a multiple of 64, so the last wave with columns has at least 16 and both
    // segments are its own)
    static_assert(kWaveCols % 16 == 0 && kColSeg < 16 && kTileWaves * kWaveCols * kTileRows * 4 > kLdsBytes,
                  "segments of a tile");
    const int xs = (tid >> 2) * kColSeg;
    const int x0 = min(xs, W - kColSeg);
    const bool act = xs < xend;
    uint32_t key[3] = {0u, 0u, 0u};
    if (act) {
        const int rows = A.ns - s0;
        if (rows >= kTileRows) colmax_keys<false>(lds, x0, q, rows, key);
        else colmax_keys<true>(lds, x0, q, rows, key);
    }
    // Clearing: a wave reads the kWaveCols columns of its segments and the
    // kColKf - 1 after them, so the columns past its first kColKf - 1 are its
    // own (W % 64 == 0, see launch_tiles_t), and its LDS accesses are in order:
    // it clears them as soon as it has read them.  A lane clears what others
    // have read, so the order is stated for the compiler.  The columns that two
    // waves read, and those after the tile, wait for the barrier.
    constexpr int kQ = kTileRows / 4;  // 16-byte quarters of a column
    uint4 *q4 = reinterpret_cast<uint4 *>(lds);
    const uint4 z = make_uint4(0u, 0u, 0u, 0u);
    const int lane = tid & 63, wave = tid >> 6;
    if (CLEAR) {
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront", "local");
        __builtin_amdgcn_wave_barrier();
        const int c1 = min((wave + 1) * kWaveCols, W);
        for (int x = (wave * kWaveCols + kColKf - 1) * kQ + lane; x < c1 * kQ; x += 64) q4[x] = z;
    }
    mid();
    if (CLEAR) {
        lds_barrier();
        if (lane < (kColKf - 1) * kQ && wave * kWaveCols < W) q4[wave * kWaveCols * kQ + lane] = z;
        const int x = W * kQ + tid;
        if (tid < (kColKf - 1 + kDumpCols) * kQ) q4[x] = z;
    }
    if (act) {
        unsigned long long *__restrict__ cm = A.colmax + (int64_t)slot * A.nf + bbase;
#pragma unroll
        for (int m = 0; m < 3; ++m) {
            const int c = 4 * m + q;
            if (c < kColSeg && x0 + c < xend)
                atomicMax(cm + x0 + c,
                          ((unsigned long long)(key[m] >> 4) << 32) |
                              (0xFFFFFFFFull - ((unsigned)s0 + 15u - (key[m] & 15u))));
        }
    }
}

// Output of the tail rows of a tile (rows (rb + 1) 16 + r, r < A.tail): their
// window sums, one thread per column summing K_f start counts per row, as a
// map or raised into the column maxima; then, after a barrier, the tail
// region is cleared for the next tile.  Reads only the tail region, so it
// may follow either output phase of the 16 rows without a barrier between.
template <bool WEIGHTED, bool MAP>
__device__ __forceinline__ void tail_output(const TileArgs &A, int slot, int rb, int jb,
                                            uint32_t *__restrict__ lt) {
    constexpr bool COLMAX = !MAP;
    const int W = A.W, kf = A.kf;
    const int stride = W + kf - 1 + kTailDump;
    const int s_t = (rb + 1) * kTileRows;  // first tail row
    const int64_t bbase = (int64_t)jb * W;
    const int xend = (int)min((int64_t)W, (int64_t)A.nf - bbase);
    unsigned long long *__restrict__ cm = A.colmax + (int64_t)slot * A.nf + bbase;
    float scale = 1.0f;
    if (WEIGHTED) scale = ldexpf(1.0f, -A.ws[(int64_t)slot * A.ws_stride].frac_bits);
    for (int x = threadIdx.x; x < xend; x += blockDim.x) {
        uint32_t top = 0;
        int brow = 0;
        for (int r = 0; r < A.tail; ++r) {
            const uint32_t *P = lt + r * stride + x;
            uint32_t acc = 0;
            for (int c = 0; c < kf; ++c) acc += P[c];
            if (MAP) {
                const int64_t idx = (int64_t)(s_t + r) * A.nf + bbase + x;
                if (WEIGHTED) A.map_f32[idx] = (float)acc * scale;
                else A.map_i32[idx] = (int32_t)acc;
            }
            if (acc > top) {  // the smallest row holding the maximum
                top = acc;
                brow = r;
            }
        }
        if (COLMAX) atomicMax(cm + x, ((unsigned long long)top << 32) | (0xFFFFFFFFull - (unsigned)(s_t + brow)));
    }
    lds_barrier();
    const int nwords = A.tail * stride;
    for (int x = threadIdx.x; x < nwords; x += blockDim.x) lt[x] = 0;
}

// The tiles of one workgroup.  The waves take the tile's blocks (four FFTs
// of a sorted run, one per lane group; windows past the last FFT are empty)
// from a counter in LDS, so that each wave takes as many as it can process.
// A block's window data are loaded two blocks ahead and its stripe edges one
// block ahead (a ring of kRing blocks), so that the accumulation of a block
// never waits for memory; the first two blocks of the next tile are loaded
// during the output phase of the current one.  Every load of the ring is
// issued on every path so that the wait counts stay exact.  Rings of four and
// five blocks, with the edges one or two blocks ahead, ran 0.5 to 2 % slower
// (256 Hz batch, 1162 rows) and no faster on a 10 Hz band, whose edges miss
// the L2 most.  Dealing the first 60 % of the blocks in turn instead of from
// the counter was no faster either.  PERSISTENT: tiles come from the
// XCD queues until all are exhausted; otherwise the workgroup runs tile
// tile_base + blockIdx.x only.  BINS: the lanes hold natural bins and compute
// the edges.  OUT says what becomes of the tile: a map,
// column maxima, or (kOutPart, not persistent) one of A.parts partial tiles:
// workgroup u takes every A.parts-th block of tile u / A.parts, starting at
// block u % A.parts, and copies its LDS tile to A.part for k_tiles_merge.
enum { kOutColmax = 0, kOutMap = 1, kOutPart = 2 };

constexpr int kRing = 3;
constexpr int kEdge = 1;  // blocks ahead of a block that the stripe edges are requested

template <bool WEIGHTED, int OUT, bool PERSISTENT, bool TAIL, bool BINS>
__device__ __forceinline__ void run_tiles(const TileArgs &A, uint32_t *__restrict__ lds, int4 *s_next,
                                          int *s_cnt) {
    const int tid = threadIdx.x;
    const int lane = tid & 63;
    const int j = lane & 15;
    const int grp = lane >> 4;
    const int W = A.W, kf = A.kf;
    const int wc = W + kf - 1;
    // LDS column c holds fine bin c0 + c, c in [0, wc); columns wc + g are
    // the dumps of the four lane groups.
    const uint32_t dump = (uint32_t)(wc + grp);
    // LDS byte address of column 0 in this lane's row
    const uint32_t lane_addr =
        (uint32_t)(uintptr_t)(__attribute__((address_space(3))) uint32_t *)(lds + j);
    const int32_t n_pad = win_stride(A.n_fft);
    const int per = wave_ffts(A.n_fft);
    const int nblk = per >> 2;
    const int total = kTileWaves * nblk;  // blocks of a tile
    const int i_last = A.n_fft - 1;
    const int home = blockIdx.x % kXcds;
    const int parts = OUT == kOutPart ? A.parts : 1;
    const int part = OUT == kOutPart ? (int)blockIdx.x % parts : 0;
    const __amdgpu_buffer_rsrc_t r_rec = buf(A.rec), r_step = buf(A.step);
    // natural bins: reads past the last peak return 0 (the records end there)
    const __amdgpu_buffer_rsrc_t r_bins =
        __builtin_amdgcn_make_buffer_rsrc(const_cast<int32_t *>(A.bins), 0, BINS ? (int)(4 * A.n_peaks) : 0, 0x00020000);
    const double kf_d = (double)kf;
    const uint32_t lane_code = 2u * (uint32_t)j;  // bit offset of this row's residual code
    const uint32_t lane_byte = 4u * (uint32_t)j;
    // tail rows after the 16-row tile (row-major, rows of wc + kTailDump
    // words; every lane of a wave has its own dump word in each row)
    const uint32_t t_stride = (uint32_t)(wc + kTailDump);
    const uint32_t t_dump = (uint32_t)(wc + lane);
    uint32_t *__restrict__ const ltail = lds + kTileRows * (wc + kDumpCols);

    // a tile's place, and its buffers: window row, stripe edges and weights of
    // the slot
    struct Bufs {
        __amdgpu_buffer_rsrc_t win, y, wq;
        int slot, rb, jb;  // (slot -1: no tile)
    };
    auto tile_bufs = [&](const int4 &p) {
        Bufs b;
        b.slot = __builtin_amdgcn_readfirstlane(p.x);
        b.rb = __builtin_amdgcn_readfirstlane(p.y);
        b.jb = __builtin_amdgcn_readfirstlane(p.z);
        const int slot = max(b.slot, 0);
        const int g = b.rb / kRowBlocksPerGroup;
        b.win = buf(A.win + (((int64_t)slot * A.nrbg + g) * A.nbb + b.jb) * n_pad);
        // low 32 bits of the stripe edges (all the tile needs: see stripe_steps)
        b.y = buf(A.Y + (int64_t)slot * y_stride(A.n_peaks, A.n_fft));
        b.wq = buf(WEIGHTED ? (const void *)(A.wq + (int64_t)slot * A.n_fft) : (const void *)A.step);
        return b;
    };
    // Blocks are handed out dynamically: block g of a tile is block g / 16 of
    // run g % 16 (four consecutive entries of that run), so the counter walks
    // the runs' largest windows first, and a wave that the SIMD arbiter
    // serves less simply takes fewer blocks.  `claim` takes n blocks and
    // returns the first in lane 0; it is read (and waited for) only when the
    // blocks are staged.
    auto claim = [&](int par, int n) {
        int g = 0;
        if (lane == 0) g = atomicAdd(s_cnt + par, n);
        return g;
    };
    // window data of block g (stage 1).  Blocks past the last one (claims
    // after the counter ran out) read the row's last entries and are not run.
    // All but the lane group's part of the offset is scalar.
    auto stage_w = [&](Quad &Q, int g, const Bufs &B) {
        Q.g = g;
        if (OUT == kOutPart) Q.g = Q.g * parts + part;
        Q.run = Q.g & (kTileWaves - 1);
        const int e = Q.g < total ? Q.run * per + 4 * (Q.g >> 4) : n_pad - 4;
        const auto w2 = __builtin_amdgcn_raw_buffer_load_b64(B.win, (uint32_t)grp * 8u, e * 8, 0);
        Q.lo = w2[0];
        Q.pk = w2[1];
    };
    // stripe edges, row terms and weights of a block (stage 2): the number of
    // steps follows the largest window of the four groups, group 0's (the runs
    // are sorted by window size, exactly).  The row term of row s0 + j,
    // G_{i,s0} - G_{i,s0+j} = step[i][j] - code_j (mod 2^32) comes from the
    // FFT's step table and the row block's record (the host keeps N nrb below
    // 2^28, so the byte offsets fit 31 bits).  FFT i = place * 16 + run: the
    // run's part of an offset is scalar; windows past the last FFT name place
    // 0, whose run is clamped where N < 16.
    auto stage_y = [&](Quad &Q, const Bufs &B) {
        Q.cnt = (int)(Q.pk & 0xFFFFu);
        const uint32_t place = Q.pk >> 16;
        const int run = min(Q.run, i_last);
        const auto r = __builtin_amdgcn_raw_buffer_load_b64(r_rec, place << 7, (B.rb * A.n_fft + run) * 8, 0);
        Q.gb = r[0];
        Q.codes = r[1];
        Q.step = __builtin_amdgcn_raw_buffer_load_b32(r_step, (place << 10) | lane_byte, run * (kTileRows * 4), 0);
        // tiles with tail rows: the next row block's record, whose rows share
        // this block's linear steps (other row blocks read their own record
        // and leave the term unused; no branch, so that nothing here waits
        // for the loads)
        if (TAIL) {
            const int rb2 = B.rb + (B.rb == A.nrb - 1 ? 1 : 0);
            const auto r2 = __builtin_amdgcn_raw_buffer_load_b64(r_rec, place << 7, (rb2 * A.n_fft + run) * 8, 0);
            Q.gb2 = r2[0];
            Q.codes2 = r2[1];
        }
        Q.wq = WEIGHTED ? __builtin_amdgcn_raw_buffer_load_b32(B.wq, place << 6, run * 4, 0) : 1u;
        Q.cmax = __builtin_amdgcn_readlane(Q.cnt, 0);
        if (BINS) {
            const auto e = __builtin_amdgcn_raw_buffer_load_b96(B.y, place << 8, run * 16, 0);
            Q.rl = e[0];
            Q.rh = e[1];
            Q.c = e[2];
        }
        Q.y0 = ld_u32(BINS ? r_bins : B.y, Q.lo + lane_byte);
        Q.y1 = ld_u32(BINS ? r_bins : B.y, Q.lo + lane_byte + 64u);
    };

    // (thread 0) position of the current tile in the home queue
    int at = kNotHome;
    if (PERSISTENT) {
        if (tid == 0) s_next[0] = tile_place(A, steal_tile(A, home, &at));
    }
    if (tid < 2) s_cnt[tid] = 0;
    tile_zero(A, lds);
    lds_barrier();
    Bufs cur = tile_bufs(PERSISTENT ? s_next[0]
                                    : tile_place(A, OUT == kOutPart ? (int)blockIdx.x / parts
                                                                    : A.tile_base + (int)blockIdx.x));
    if (cur.slot < 0 || nblk == 0) return;  // nblk > 0 whenever there is an FFT
    Quad q[kRing];
    {
        const int g0 = __builtin_amdgcn_readfirstlane(claim(0, kRing - 1));
#pragma unroll
        for (int u = 0; u < kRing - 1; ++u) stage_w(q[u], g0 + u, cur);
#pragma unroll
        for (int u = 0; u < kEdge; ++u) stage_y(q[u], cur);
    }
    for (int it = 0;; ++it) {
        const int par = it & 1;  // block counter of this tile; the other is the next tile's
        // The next tile is claimed ahead while the home queue holds two more
        // rounds of its workgroups; the last ones are claimed when they are
        // needed, so that no workgroup holds a tile that an idle one could run
        // (703 tiles on 256 CUs took four rounds of tiles instead of three).
        int pos = kNotHome;
        if (PERSISTENT && tid == 0 && at + 2 * (int)(gridDim.x / kXcds) < queue_len(A, home))
            pos = atomicAdd(A.queue_ctr + home, 1);
        // the next tile's counter was last used by the previous tile, whose
        // claims all came before the barrier that ended its accumulation
        if (tid == 0) s_cnt[par ^ 1] = 0;
        const int slot = cur.slot, rb = cur.rb, jb = cur.jb;
        const uint32_t c0q = (uint32_t)(jb * W - (kf - 1)) << kFrac;
        const bool tailed = TAIL && rb == A.nrb - 1;  // this tile also does the tail rows
        auto consume = [&](const Quad &Q) {
            // the edges stay as loaded: the tile's origin and G_{i,s0} go into
            // the row term, and lanes past the window hold an edge far from it
            const uint32_t base = c0q + Q.gb - (BINS ? Q.c : 0u);
            // BINS: the edge without its constant, floor(fl(K_f k r) 2^16), whose
            // low word is that of its sum with 2^52 (0 <= edge < 2^45)
            auto edge = [&](uint32_t k) -> uint32_t {
                if (!BINS) return k;
                const double r = __hiloint2double((int)Q.rh, (int)Q.rl);
                return (uint32_t)__double2loint(floor((double)k * kf_d * r) + 4503599627370496.0);
            };
            const uint32_t code = __builtin_amdgcn_ubfe(Q.codes, lane_code, 2u);
            const uint32_t t = Q.step - code - base;
            const uint32_t far = base + kFarEdge;
            uint32_t tt = 0;
            if (TAIL)
                tt = t + code - __builtin_amdgcn_ubfe(Q.codes2, lane_code, 2u) + (Q.gb - Q.gb2);
            uint32_t val = Q.wq;
            asm volatile("" : "+v"(val));
            const uint32_t v0 = j < Q.cnt ? edge(Q.y0) : far;
            const uint32_t v1 = j + 16 < Q.cnt ? edge(Q.y1) : far;
            stripe_steps(min(Q.cmax, 32), v0, v1, t, dump, lane_addr, val);
            if (tailed) {
                tail_steps(A.tail, v0, tt, t_dump, t_stride, val, ltail);
                if (Q.cmax > 16) tail_steps(A.tail, v1, tt, t_dump, t_stride, val, ltail);
            }
            // windows longer than 32 peaks: further chunks, loaded here
            for (int off = 32; off < Q.cmax; off += 16) {
                uint32_t v = far;
                if (off + j < Q.cnt)
                    v = edge(ld_u32(BINS ? r_bins : cur.y, Q.lo + lane_byte + 4u * (uint32_t)off));
                stripe_steps(min(Q.cmax - off, 16), v, far, t, dump, lane_addr, val);
                if (tailed) tail_steps(A.tail, v, tt, t_dump, t_stride, val, ltail);
            }
        };
        // Blocks are claimed kRing at a time, one round ahead, so a wave
        // drains its LDS queue to read a claim once per round.  A wave's
        // claims grow, so once one block is past the end, so are the blocks
        // staged after it; it is left before it stages more (staging first
        // made the last wave of a tile wait for loads nobody uses: 1 %).
        int gv = claim(par, kRing);
        for (bool more = true; more;) {
            const int g3 = __builtin_amdgcn_readfirstlane(gv);
            gv = claim(par, kRing);
#pragma unroll
            for (int u = 0; u < kRing; ++u) {
                if (q[u].g >= total) {
                    more = false;
                    break;
                }
                stage_w(q[(u + kRing - 1) % kRing], g3 + u, cur);
                stage_y(q[(u + kEdge) % kRing], cur);
                consume(q[u]);
            }
        }
        if (PERSISTENT) {
            if (tid == 0) {
                if (pos < queue_len(A, home)) {
                    at = pos;
                    s_next[(it + 1) & 1] = tile_place(A, queue_tile(A, home, pos));
                } else {
                    s_next[(it + 1) & 1] = tile_place(A, steal_tile(A, home, &at));
                }
            }
        }
        // Drain this wave's vector-memory queue here, where the workgroup
        // waits anyway: otherwise the compiler cannot tell that the tile
        // claim above has returned on every path, and the output phase would
        // open with a full wait that also covers the next tile's prefetch.
        // The LDS updates of stripe_steps are waited for by name, too: the
        // compiler does not count them.
        __builtin_amdgcn_s_waitcnt(kWaitVmcnt0);
        asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
        lds_barrier();
        Bufs nxt = cur;
        if (PERSISTENT) nxt = tile_bufs(s_next[(it + 1) & 1]);
        const bool go_on = PERSISTENT && nxt.slot >= 0;
        if (go_on) {
            const int g0 = __builtin_amdgcn_readfirstlane(claim(par ^ 1, kRing - 1));
#pragma unroll
            for (int u = 0; u < kRing - 1; ++u) stage_w(q[u], g0 + u, nxt);
        }
        if (OUT == kOutPart) {
            uint32_t *__restrict__ dst = A.part + (int64_t)blockIdx.x * A.part_stride;
            const int nwords = tile_words(A);
            for (int x = tid * 4; x < nwords; x += blockDim.x * 4) {
                if (x + 3 < nwords) {
                    *reinterpret_cast<uint4 *>(dst + x) = *reinterpret_cast<const uint4 *>(lds + x);
                } else {
                    for (int y = x; y < nwords; ++y) dst[y] = lds[y];
                }
            }
            break;
        }
        // K_f <= kHold + 1: clearing fused into the output, and the next
        // tile's stripe edges requested while the output still runs
        const bool fused = kf <= kHold + 1;
        auto first_edges = [&] {
            if (!go_on) return;
#pragma unroll
            for (int u = 0; u < kEdge; ++u) stage_y(q[u], nxt);
        };
        if (!WEIGHTED && OUT == kOutColmax && kf == kColKf) {
            tile_colmax<PERSISTENT>(A, slot, rb, jb, lds, first_edges);
        } else if (fused) {
            tile_windows<WEIGHTED, OUT == kOutMap, PERSISTENT>(A, slot, rb, jb, lds, first_edges);
        } else {
            tile_output<WEIGHTED, OUT == kOutMap>(A, slot, rb, jb, lds);
        }
        if (TAIL && tailed) tail_output<WEIGHTED, OUT == kOutMap>(A, slot, rb, jb, ltail);
        if (!go_on) break;
        if (!fused) first_edges();
        lds_barrier();
        if (!fused) {
            tile_zero(A, lds);
            lds_barrier();
        }
        cur = nxt;
    }
}

template <bool WEIGHTED, int OUT, bool TAIL>
__global__ void __launch_bounds__(kTileThreads) k_tiles_plain(TileArgs A) {
    extern __shared__ __align__(16) uint32_t lds[];
    __shared__ int s_cnt[2];
    run_tiles<WEIGHTED, OUT, false, TAIL, false>(A, lds, nullptr, s_cnt);
}

// One workgroup per CU.  The next tile of the home queue is claimed when a
// tile starts (its counter update overlaps the tile's work) and used when it
// ends; an exhausted home queue sends the workgroup to the others.  Every
// workgroup leaves the loop once all queues are exhausted.
template <bool WEIGHTED, bool TAIL, bool BINS>
__global__ void __launch_bounds__(kTileThreads) k_tiles_persistent(TileArgs A) {
    extern __shared__ __align__(16) uint32_t lds[];
    __shared__ int4 s_next[2];
    __shared__ int s_cnt[2];
    run_tiles<WEIGHTED, kOutColmax, true, TAIL, BINS>(A, lds, s_next, s_cnt);
}

// Sums of the partial tiles and their output: grid (column chunks of a tile,
// tiles), kMergeCols columns per workgroup.  The A.parts partial tiles of the
// chunk (and the K_f - 1 columns past it) are read with 16 bytes per lane,
// added in registers and laid out row-major in LDS, where every output is
// the sum of K_f consecutive words: one wave writes 64 consecutive bins of a
// row of the map, or raises the column maxima (two threads per column, eight
// rows each).  Bound by reading the partial tiles.
constexpr int kMergeCols = 128;
constexpr int kMergeThreads = 256;
// words per row: kMergeCols + 63 (K_f = 64) and 4 modulo 16, so that the four
// quarters of 16 columns that a wave stores together lie in 64 banks
constexpr int kMergeStride = 196;

template <bool WEIGHTED, bool MAP>
__global__ void __launch_bounds__(kMergeThreads) k_tiles_merge(TileArgs A) {
    __shared__ uint32_t h[(kTileRows + kTailRows) * kMergeStride];
    const int tid = threadIdx.x;
    const int t = blockIdx.y;
    int slot, rb, jb;
    decode_tile(A, t, slot, rb, jb);
    const int W = A.W, kf = A.kf;
    const int64_t bbase = (int64_t)jb * W;
    const int xend = (int)min((int64_t)W, (int64_t)A.nf - bbase);
    const int c0 = (int)blockIdx.x * kMergeCols;
    if (c0 >= xend) return;  // (the whole workgroup)
    const int ncol = min(kMergeCols, xend - c0);
    const int nin = ncol + kf - 1;
    const uint32_t *__restrict__ src = A.part + (int64_t)t * A.parts * A.part_stride;
    for (int e = tid; e < nin * 4; e += kMergeThreads) {
        const uint32_t *__restrict__ q = src + (int64_t)c0 * kTileRows + 4 * e;
        uint4 sum = make_uint4(0u, 0u, 0u, 0u);
#pragma unroll 4
        for (int p = 0; p < A.parts; ++p) {
            const uint4 v = *reinterpret_cast<const uint4 *>(q + p * A.part_stride);
            sum.x += v.x;
            sum.y += v.y;
            sum.z += v.z;
            sum.w += v.w;
        }
        uint32_t *d = h + (e & 3) * 4 * kMergeStride + (e >> 2);
        d[0] = sum.x;
        d[kMergeStride] = sum.y;
        d[2 * kMergeStride] = sum.z;
        d[3 * kMergeStride] = sum.w;
    }
    const int tail = rb == A.nrb - 1 ? A.tail : 0;
    const int wc = W + kf - 1;
    for (int e = tid; e < tail * nin; e += kMergeThreads) {
        const int r = e / nin, c = e - r * nin;
        const uint32_t *__restrict__ q = src + kTileRows * (wc + kDumpCols) + r * (wc + kTailDump) + c0 + c;
        uint32_t sum = 0;
        for (int p = 0; p < A.parts; ++p) sum += q[p * A.part_stride];
        h[(kTileRows + r) * kMergeStride + c] = sum;
    }
    __syncthreads();
    const int s0 = rb * kTileRows;
    const int rows = min(kTileRows, A.ns - s0) + tail;
    const int c = tid & (kMergeCols - 1), half = tid / kMergeCols;
    if (c >= ncol) return;
    if (MAP) {
        float scale = 1.0f;
        if (WEIGHTED) scale = ldexpf(1.0f, -A.ws[(int64_t)slot * A.ws_stride].frac_bits);
        for (int r = half; r < rows; r += kMergeThreads / kMergeCols) {
            const uint32_t *P = h + r * kMergeStride + c;
            uint32_t acc = 0;
            for (int k = 0; k < kf; ++k) acc += P[k];
            const int64_t at = (int64_t)(s0 + r) * A.nf + bbase + c0 + c;
            if (WEIGHTED) A.map_f32[at] = (float)acc * scale;
            else A.map_i32[at] = (int32_t)acc;
        }
    } else {
        // rows 0-7, and 8 to the last (tail rows follow the 16 in the grid too)
        const int r0 = half * 8, r1 = half == 0 ? min(rows, 8) : rows;
        if (r0 >= r1) return;
        uint32_t top = 0;
        int at = r0;
        for (int r = r0; r < r1; ++r) {
            const uint32_t *P = h + r * kMergeStride + c;
            uint32_t acc = 0;
            for (int k = 0; k < kf; ++k) acc += P[k];
            if (acc > top) {  // the smallest row holding the maximum
                top = acc;
                at = r;
            }
        }
        atomicMax(A.colmax + (int64_t)slot * A.nf + bbase + c0 + c,
                  ((unsigned long long)top << 32) | (0xFFFFFFFFull - (unsigned)(s0 + at)));
    }
}

// ----------------------------------------------------------------------------
// candidates per (sky, sub-band)

// A column as a key: larger value first, then smaller bin (its row is the
// smallest holding the value already); 0 is no column.
__device__ __forceinline__ unsigned long long column_key(uint32_t val, int bin) {
    return ((unsigned long long)val << 32) | (0xFFFFFFFFull - (unsigned)bin);
}
__device__ __forceinline__ int key_bin(unsigned long long k) { return (int)(0xFFFFFFFFu - (uint32_t)k); }

__device__ unsigned long long block_best(unsigned long long m, unsigned long long *red) {
#pragma unroll
    for (int o = 32; o >= 1; o >>= 1) {
        const unsigned long long o2 = __shfl_xor(m, o);
        m = o2 > m ? o2 : m;
    }
    const int wave = threadIdx.x >> 6, nw = blockDim.x >> 6;
    if ((threadIdx.x & 63) == 0) red[wave] = m;
    __syncthreads();
    unsigned long long r = red[0];
    for (int k = 1; k < nw; ++k) r = red[k] > r ? red[k] : r;
    return r;
}

// Mean and deviation of a cell's noise value, and the value's scale: a count,
// or a fixed-point weighted sum when ws is given.
struct CellStats {
    double mu, sd;
    float scale;
};
__device__ __forceinline__ CellStats cell_stats(int32_t n_fft, double theta, const WeightStats *__restrict__ ws) {
    const double p0 = exp(-theta) - exp(-2.0 * theta) + exp(-3.0 * theta) / 3.0;
    CellStats c;
    if (ws != nullptr) {
        const WeightStats st = *ws;
        c.scale = (float)ldexp(1.0, -st.frac_bits);
        c.mu = p0 * st.sum_w;
        c.sd = sqrt(p0 * (1.0 - p0) * st.sum_w2);
    } else {
        c.scale = 1.0f;
        c.mu = (double)n_fft * p0;
        c.sd = sqrt((double)n_fft * p0 * (1.0 - p0));
    }
    return c;
}

// Value and critical ratio of a cell holding `val`.
__device__ __forceinline__ void cell_value(uint32_t val, const CellStats &c, bool weighted, float *value, float *cr) {
    const double v = weighted ? (double)((float)val * c.scale) : (double)val;
    *value = (float)v;
    *cr = (float)((v - c.mu) / c.sd);
}

// One workgroup per (sub-band, direction).  Every column is read once: a thread
// holds up to kHeld of them for the second search, all requested before the
// first is used; only sub-bands of more than kHeld columns per thread read the
// rest again.  Bound by latency: with 256 threads reading each column twice, one
// at a time, the ten sub-bands of 8192 columns of a 1 Hz band took 24 us, now
// launch_select.
constexpr int kHeld = 8;

__global__ void __launch_bounds__(1024) k_select(const unsigned long long *__restrict__ colmax,
                                                 int32_t nf, fh_select sel, int32_t sky_base,
                                                 int32_t n_fft, const WeightStats *__restrict__ ws,
                                                 int32_t ws_stride, fh_candidate *__restrict__ out) {
    __shared__ unsigned long long red[2][16];
    const int sb = blockIdx.x, slot = blockIdx.y;
    const int n_sb = gridDim.x;
    const int lo = sb * sel.width;
    const int hi = lo + sel.width < nf ? lo + sel.width : nf;
    const unsigned long long *cm = colmax + (int64_t)slot * nf;
    const int step = blockDim.x;
    unsigned long long held[kHeld];
#pragma unroll
    for (int u = 0; u < kHeld; ++u) {
        const int b = lo + (int)threadIdx.x + u * step;
        held[u] = b < hi ? cm[b] : 0ull;
    }
    // (two threads write the two candidates; their cells' statistics are
    // worked out while the columns are on their way)
    CellStats stats{};
    if (threadIdx.x < 2)
        stats = cell_stats(n_fft, sel.theta, ws != nullptr ? ws + (int64_t)slot * ws_stride : nullptr);
    unsigned long long m = 0ull;
#pragma unroll
    for (int u = 0; u < kHeld; ++u) {
        const int b = lo + (int)threadIdx.x + u * step;
        const unsigned long long k = column_key((uint32_t)(held[u] >> 32), b);
        m = b < hi && k > m ? k : m;
    }
    for (int b = lo + (int)threadIdx.x + kHeld * step; b < hi; b += step) {
        const unsigned long long k = column_key((uint32_t)(cm[b] >> 32), b);
        m = k > m ? k : m;
    }
    const unsigned long long b1 = block_best(m, red[0]);
    unsigned long long b2 = 0ull;
    if (sel.sep >= 0) {
        const int first = key_bin(b1);
        m = 0ull;
#pragma unroll
        for (int u = 0; u < kHeld; ++u) {
            const int b = lo + (int)threadIdx.x + u * step;
            const int d = b > first ? b - first : first - b;
            const unsigned long long k = column_key((uint32_t)(held[u] >> 32), b);
            m = b < hi && d > sel.excl && k > m ? k : m;
        }
        for (int b = lo + (int)threadIdx.x + kHeld * step; b < hi; b += step) {
            const int d = b > first ? b - first : first - b;
            if (d <= sel.excl) continue;
            const unsigned long long k = column_key((uint32_t)(cm[b] >> 32), b);
            m = k > m ? k : m;
        }
        b2 = block_best(m, red[1]);
    }
    if (threadIdx.x < 2) {
        const int r = threadIdx.x;
        const unsigned long long best = r == 0 ? b1 : b2;
        fh_candidate c;
        c.sky = sky_base + slot;
        c.subband = sb;
        c.rank = r;
        bool valid = best != 0ull;
        if (r == 1 && valid) {
            const int d = key_bin(b2) > key_bin(b1) ? key_bin(b2) - key_bin(b1) : key_bin(b1) - key_bin(b2);
            valid = d >= sel.sep;
        }
        c.valid = valid ? 1 : 0;
        if (valid) {
            c.bin = key_bin(best);
            c.row = (int32_t)(0xFFFFFFFFu - (uint32_t)cm[c.bin]);
            cell_value((uint32_t)(best >> 32), stats, ws != nullptr, &c.value, &c.cr);
        } else {
            c.bin = -1;
            c.row = -1;
            c.value = 0.0f;
            c.cr = 0.0f;
        }
        out[((int64_t)(sky_base + slot) * n_sb + sb) * 2 + r] = c;
    }
}

// ----------------------------------------------------------------------------
// peakmap construction (Sec. "Peakmap", Eq. pm): R = S_P / S_AR bin by bin; a
// peak is a bin above theta that is strictly larger than both neighbours.
// One workgroup per FFT writes its peaks compactly into a per-FFT scratch run
// (at most one peak in every two bins) and its count; after a scan of the
// counts a second kernel packs the runs into the CSR.

// Bound by HBM (each spectrum value once).  A wave takes 512 consecutive bins:
// its lanes request them, and the two bins past them, in nine coalesced loads
// per array before the first is used, every ratio is divided once, and the
// neighbours come from the next lanes.  With one bin per thread and round,
// each reading and dividing its neighbours' values too, 6286 FFTs x 4650 bins
// (234 MB) took 70 us; now 45 us, 5.2 TB/s, the rate of a large copy.
constexpr int kRowRun = 8;  // bins per lane and round

__global__ void __launch_bounds__(256) k_pm_rows(int32_t n_bins, int64_t ld,
                                                 const float *__restrict__ sp,
                                                 const float *__restrict__ sar, int32_t k0,
                                                 float theta, int32_t cap,
                                                 int32_t *__restrict__ scratch,
                                                 int32_t *__restrict__ counts) {
    __shared__ int wsum[2][4];
    const int i = blockIdx.x;
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const float *P = sp + (int64_t)i * ld;
    const float *A = sar ? sar + (int64_t)i * ld : nullptr;
    int32_t *out = scratch + (int64_t)i * cap;
    const uint64_t below = (1ull << lane) - 1ull;
    const int n1 = (lane + 1) & 63, n2 = (lane + 2) & 63;
    int base = 0, par = 0;
    for (int r0 = 0; r0 < n_bins - 2; r0 += 4 * 64 * kRowRun, par ^= 1) {
        // lane l, step u: left neighbour j = j0 + 64 u + l, the bin itself j + 1
        const int j0 = r0 + wave * 64 * kRowRun;
        float x[kRowRun + 1], a[kRowRun + 1];
#pragma unroll
        for (int u = 0; u <= kRowRun; ++u) {
            const int j = j0 + 64 * u + lane;
            const bool in = j < n_bins && (u < kRowRun || lane < 2);
            x[u] = in ? P[j] : 0.0f;
            a[u] = in && A ? A[j] : 1.0f;
        }
        if (A) {
#pragma unroll
            for (int u = 0; u <= kRowRun; ++u) x[u] = x[u] / a[u];
        }
        uint64_t m[kRowRun];
        int total = 0;
        float c0 = __shfl(x[0], n1), r1 = __shfl(x[0], n2);
#pragma unroll
        for (int u = 0; u < kRowRun; ++u) {
            const float c1 = __shfl(x[u + 1], n1), r2 = __shfl(x[u + 1], n2);
            const float c = lane < 63 ? c0 : c1, r = lane < 62 ? r1 : r2;
            const bool in = j0 + 64 * u + lane + 2 < n_bins;
            m[u] = __ballot(in && c > theta && c > x[u] && c > r);
            total += __popcll(m[u]);
            c0 = c1;
            r1 = r2;
        }
        if (lane == 0) wsum[par][wave] = total;
        __syncthreads();  // one per round: the next round writes the other half
        int pos = base;
#pragma unroll
        for (int w = 0; w < 4; ++w) {
            const int n = wsum[par][w];
            pos += w < wave ? n : 0;
            base += n;
        }
#pragma unroll
        for (int u = 0; u < kRowRun; ++u) {
            if ((m[u] >> lane) & 1ull) out[pos + __popcll(m[u] & below)] = k0 + j0 + 64 * u + lane + 1;
            pos += __popcll(m[u]);
        }
    }
    if (threadIdx.x == 0) counts[i] = base;
}

// exclusive scan of per-FFT counts into CSR offsets (one workgroup, eight
// counts per thread and round); meta (optional) receives the total and the
// largest count.  With one count per thread and a scan of twenty barriers in
// LDS, 6286 counts took 18 us; now 5 us.
__global__ void __launch_bounds__(1024) k_pm_scan(int32_t n, const int32_t *__restrict__ counts,
                                                  int64_t *__restrict__ offsets, int64_t *__restrict__ meta) {
    constexpr int kU = 8;
    __shared__ int64_t part[2][16];
    __shared__ int32_t s_max[16];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    int64_t carry = 0;
    int32_t most = 0;
    int par = 0;
    for (int b = 0; b < n; b += 1024 * kU, par ^= 1) {
        const int i = b + (int)threadIdx.x * kU;
        int32_t v[kU];
        int64_t sum = 0;
        if (i + kU <= n) {
            const int4 lo = reinterpret_cast<const int4 *>(counts + i)[0];
            const int4 hi = reinterpret_cast<const int4 *>(counts + i)[1];
            v[0] = lo.x; v[1] = lo.y; v[2] = lo.z; v[3] = lo.w;
            v[4] = hi.x; v[5] = hi.y; v[6] = hi.z; v[7] = hi.w;
        } else {
#pragma unroll
            for (int u = 0; u < kU; ++u) v[u] = i + u < n ? counts[i + u] : 0;
        }
#pragma unroll
        for (int u = 0; u < kU; ++u) {
            sum += v[u];
            most = max(most, v[u]);
        }
        int64_t incl = sum;
        for (int o = 1; o < 64; o <<= 1) {
            const int64_t t = __shfl_up(incl, o);
            if (lane >= o) incl += t;
        }
        if (lane == 63) part[par][wave] = incl;
        __syncthreads();  // one per round: the next round writes the other half
        int64_t at = carry + incl - sum;
#pragma unroll
        for (int k = 0; k < 16; ++k) {
            const int64_t t = part[par][k];
            at += k < wave ? t : 0;
            carry += t;
        }
#pragma unroll
        for (int u = 0; u < kU; ++u) {
            if (i + u < n) offsets[i + u] = at;
            at += v[u];
        }
    }
    if (threadIdx.x == 0) offsets[n] = carry;
    if (meta != nullptr) {
        for (int o = 32; o >= 1; o >>= 1) most = max(most, __shfl_xor(most, o));
        if (lane == 0) s_max[wave] = most;
        __syncthreads();
        if (threadIdx.x == 0) {
            for (int k = 1; k < 16; ++k) most = max(most, s_max[k]);
            meta[0] = carry;
            meta[1] = most;
        }
    }
}

__global__ void __launch_bounds__(256) k_pm_pack(int32_t cap, const int32_t *__restrict__ scratch,
                                                 const int64_t *__restrict__ offsets,
                                                 int32_t *__restrict__ bins) {
    const int i = blockIdx.x;
    const int64_t o = offsets[i];
    const int c = (int)(offsets[i + 1] - o);
    const int32_t *src = scratch + (int64_t)i * cap;
    for (int t = threadIdx.x; t < c; t += blockDim.x) bins[o + t] = src[t];
}

inline unsigned grid_for(int64_t n, int block) {
    int64_t g = (n + block - 1) / block;
    if (g > 65535 * 16) g = 65535 * 16;
    return (unsigned)(g < 1 ? 1 : g);
}

}  // namespace

int tile_lds_bytes(int W, int kf, int tail) {
    return (kTileRows * (W + kf - 1 + kDumpCols) + tail * (W + kf - 1 + kTailDump)) * 4;
}

int64_t part_words(int W, int kf, int tail) { return (tile_lds_bytes(W, kf, tail) / 4 + 3) / 4 * 4; }

int max_tile_bins(int kf, double step_bins, int rows) {
    // rows past 16 are tail rows, with kTailDump dump words each
    const int words = (kLdsBytes - kLdsReserve) / 4 - kDumpCols * kTileRows - kTailDump * (rows - kTileRows);
    int w = words / rows - kf + 1;  // rows (W + kf - 1) + dump words <= words
    // supported row steps: below 128 fine bins
    if (step_bins * kQd + 1.0 >= 8388608.0) return 0;
    // 32-bit tile-relative edges (see kFarEdge)
    const double m = ceil(step_bins) + 1.0;
    const double wr = (double)(1 << (31 - kFrac)) - 64.0 - kf - 80.0 * m;
    if (wr < (double)w) w = wr < 0.0 ? 0 : (int)wr;
    return (w / 64) * 64;
}

hipError_t launch_fill_i32(int32_t *p, int64_t n, int32_t v, hipStream_t st) {
    if (n <= 0) return hipSuccess;
    k_fill_i32<<<grid_for(n, 256) > 4096 ? 4096 : grid_for(n, 256), 256, 0, st>>>(p, n, v);
    return hipGetLastError();
}

// workgroups for the shift tables and the cleared buffers; 0: invalid
static int setup_blocks(const SetupArgs &a) {
    if (a.n_fft < 1 || a.nrb < 1 || a.nrb_run < 1 || a.nrb_run > a.nrb || a.n_sky > kArgSky) return 0;
    const int64_t work = std::max((int64_t)a.n_fft * a.nrb, a.n_colmax / 4);
    return (int)std::min<int64_t>((work + 255) / 256, 8192);
}

hipError_t launch_setup(const SetupArgs &a, const int32_t *bins, int32_t k_min, int32_t k_max, uint2 *rank,
                        hipStream_t st) {
    const int blocks = setup_blocks(a);
    if (blocks == 0) return hipErrorInvalidValue;
    RankArgs r{};
    if (rank != nullptr) {
        r.bins = bins;
        r.k_min = k_min;
        r.nw = rank_words(k_min, k_max);
        r.rank = rank;
        r.n_blocks = (a.n_fft + 3) / 4;
        if (r.nw == 0) return hipErrorInvalidValue;
    }
    k_setup<<<a.n_vec + r.n_blocks + blocks, 256, (size_t)16 * r.nw, st>>>(a, r);
    return hipGetLastError();
}

hipError_t launch_set_sky(const SkyArg &s, int n, double *sky, hipStream_t st) {
    if (n > kArgSky) return hipErrorInvalidValue;
    k_set_sky<<<1, 128, 0, st>>>(s, n, sky);
    return hipGetLastError();
}

hipError_t launch_weight_stats(int32_t n_fft, const float *w, int32_t mult, WeightStats *ws, int32_t *err_flag,
                               hipStream_t st) {
    k_weight_stats<<<1, 256, 0, st>>>(n_fft, w, mult, ws, err_flag);
    return hipGetLastError();
}

hipError_t launch_prep(int32_t n_fft, int64_t n_peaks, const int64_t *offsets, const int32_t *bins,
                       const double *v, const double *sky, int32_t n_slots, int32_t kf, int64_t b0,
                       int64_t *Y, const float *w, int32_t w_stride,
                       const WeightStats *ws, int32_t ws_stride, uint32_t *wq, uint32_t *Y32,
                       int32_t shift_mode, double q, hipStream_t st) {
    dim3 grid((n_fft + 3) / 4, n_slots);
    k_prep<<<grid, 256, 0, st>>>(n_fft, n_peaks, offsets, bins, v, sky, kf, b0, Y, w, w_stride,
                                 ws, ws_stride, wq, Y32, shift_mode, q);
    return hipGetLastError();
}

int front_ffts_per_block(int32_t max_per_fft) {
    for (int F = max_per_fft >= kFrontBigFft ? 4 : kFrontMaxF; F >= 1; F >>= 1)
        if ((int64_t)F * (max_per_fft + kYPad) * 8 <= kFrontLdsBytes) return F;
    return 0;
}

hipError_t launch_setup_front(const SetupArgs &a, FrontArgs r, int32_t max_per_fft, hipStream_t st) {
    const int blocks = setup_blocks(a);
    if (blocks == 0 || r.F < 1 || r.F > kFrontMaxF || win_stride(a.n_fft) % r.F != 0) return hipErrorInvalidValue;
    const size_t lds = ((size_t)r.F * (max_per_fft + kYPad) * 8 + 255) / 256 * 256;
    if (lds > (size_t)kFrontLdsBytes) return hipErrorInvalidValue;
    r.search_top = 0;  // largest power of two up to max_per_fft (0 when no FFT has a peak)
    while (r.search_top * 2 <= max_per_fft && r.search_top < (1 << 30)) r.search_top = r.search_top ? 2 * r.search_top : 1;
    // a launch holds fewer than 2^32 threads: fronts past that follow the setup
    // in launches of their own, as many directions at a time as fit
    constexpr int64_t kMaxBlocks = (((int64_t)1 << 32) - 1) / 256;
    const int64_t per_slot = win_stride(a.n_fft) / r.F;
    if (per_slot * r.n_slots + a.n_vec + blocks <= kMaxBlocks) {
        k_setup_front<<<(unsigned)(a.n_vec + per_slot * r.n_slots + blocks), 256, lds, st>>>(a, r);
        return hipGetLastError();
    }
    hipError_t e = launch_setup(a, nullptr, 0, 0, nullptr, st);
    SetupArgs b = a;
    b.n_vec = 0;
    b.n_sky = 0;  // (the setup has written the directions)
    FrontArgs p = r;
    for (int s0 = 0; s0 < r.n_slots && e == hipSuccess; s0 += p.n_slots) {
        p.n_slots = (int32_t)std::min<int64_t>(r.n_slots - s0, kMaxBlocks / per_slot);
        p.sky = r.sky + 3 * (int64_t)s0;
        p.Y = r.Y + (int64_t)s0 * y_stride(r.n_peaks, a.n_fft);
        p.win = r.win + (int64_t)s0 * r.nrbg * r.nbb * win_stride(a.n_fft);
        k_setup_front<<<(unsigned)(per_slot * p.n_slots), 256, lds, st>>>(b, p);
        e = hipGetLastError();
    }
    return e;
}

// Words of an FFT's rank table.
int32_t rank_words(int32_t k_min, int32_t k_max) {
    const int64_t w = ((int64_t)k_max - k_min + 1) / 32 + 1;
    return w <= kRankMaxWords ? (int32_t)w : 0;
}

// FFTs per workgroup: as many as fit kRankLdsBytes (eight workgroups per CU),
// up to a whole line of a window row; at least one, in up to kFrontLdsBytes.
static int rank_ffts_per_block(int32_t nw, int32_t nrbg) {
    const int64_t one = (int64_t)(nw | 1) * 8 + (int64_t)nrbg * 16;
    for (int F = kFrontMaxF; F >= 1; F >>= 1)
        if (F * one <= kRankLdsBytes) return F;
    return one <= kFrontLdsBytes ? 1 : 0;
}

bool rank_front_fits(int32_t k_min, int32_t k_max, int32_t nrbg) {
    const int32_t nw = rank_words(k_min, k_max);
    return nw > 0 && rank_ffts_per_block(nw, nrbg) > 0;
}

hipError_t launch_front_rank(int32_t n_fft, int64_t n_peaks, const int64_t *offsets, const int32_t *bins,
                             const double *v, const double *sky, int32_t n_slots, int32_t kf, int64_t b0,
                             const int64_t *gwin, uint32_t *Y, const float *w, int32_t w_stride,
                             const WeightStats *ws, int32_t ws_stride, uint32_t *wq, int32_t nrbg, int32_t nbb,
                             int32_t W, int32_t k_min, int32_t k_max, const uint2 *rank, uint32_t *win,
                             int32_t shift_mode, double q, bool terms_only, hipStream_t st) {
    const int32_t nw = rank_words(k_min, k_max);
    const int F = nw ? rank_ffts_per_block(nw, nrbg) : 0;
    if (F < 1 || win_stride(n_fft) % F != 0) return hipErrorInvalidValue;
    const size_t lds = (size_t)F * ((size_t)(nw | 1) * 8 + (size_t)nrbg * 16);
    // directions per workgroup: up to kRankDirs while that leaves four rounds
    // of workgroups (eight per CU)
    const int64_t blocks = (int64_t)(win_stride(n_fft) / F) * n_slots;
    const int D = (int)std::max<int64_t>(1, std::min<int64_t>(kRankDirs, blocks / (4 * 8 * 256)));
    k_front_rank<<<dim3(win_stride(n_fft) / F, (n_slots + D - 1) / D), 256, lds, st>>>(
        n_fft, n_peaks, offsets, bins, v, sky, n_slots, kf, b0, gwin, Y, w, w_stride, ws, ws_stride, wq, nrbg, nbb, W, F,
        D, k_min, k_max, nw, rank, win, shift_mode, q, terms_only);
    return hipGetLastError();
}

hipError_t launch_sort_windows(int32_t n_fft, int32_t nrbg, int32_t nbb, int32_t n_slots, const uint32_t *win,
                               const uint32_t *base, int2 *wsorted, const WeightArgs &wa, hipStream_t st) {
    dim3 grid(nrbg * nbb, n_slots);
    const size_t lds = (size_t)kTileWaves * (4 * (size_t)sort_run_stride(wave_ffts(n_fft)) + 2 * (size_t)wave_ffts(n_fft));
    if (lds <= (size_t)kSortLdsBytes)
        k_sort_windows<<<grid, kTileThreads, lds, st>>>(n_fft, nrbg * nbb, win, base, wsorted, wa);
    else
        k_sort_windows_long<<<grid, kTileThreads, (size_t)kSortPiece * sizeof(uint32_t), st>>>(n_fft, nrbg * nbb, win,
                                                                                              base, wsorted, wa);
    return hipGetLastError();
}

hipError_t launch_windows(int32_t n_fft, const int64_t *offsets, const int64_t *Y, int64_t n_peaks,
                          const int64_t *gwin, int32_t nrbg, int32_t nbb, int32_t W,
                          int32_t kf, int32_t n_slots, uint32_t *win, int method, hipStream_t st) {
    if (method == 0) {
        dim3 grid(grid_for((int64_t)nbb * win_stride(n_fft), 256), nrbg, n_slots);
        k_windows<<<grid, 256, 0, st>>>(n_fft, offsets, Y, n_peaks, gwin, nrbg, nbb, W, kf, win);
    } else {
        dim3 grid((win_stride(n_fft) + 3) / 4, n_slots);
        k_windows_sweep<<<grid, 256, 0, st>>>(n_fft, offsets, Y, n_peaks, gwin, nrbg, nbb, W, kf, win);
    }
    return hipGetLastError();
}

template <bool Wt, bool T>
static hipError_t set_tile_attrs() {
    const int lds = kLdsBytes - kLdsReserve;
    for (const void *f : {(const void *)k_tiles_persistent<Wt, T, false>, (const void *)k_tiles_persistent<Wt, T, true>,
                          (const void *)k_tiles_plain<Wt, kOutColmax, T>,
                          (const void *)k_tiles_plain<Wt, kOutMap, T>, (const void *)k_tiles_plain<Wt, kOutPart, T>}) {
        const hipError_t e = hipFuncSetAttribute(f, hipFuncAttributeMaxDynamicSharedMemorySize, lds);
        if (e != hipSuccess) return e;
    }
    return hipSuccess;
}

// Tiles with tail rows run the TAIL form of the kernels; without, the plain
// form has no trace of them.
template <bool Wt, bool T>
static hipError_t launch_tiles_t(const TileArgs &a, bool map, bool persistent, int32_t n_tiles,
                                 int32_t grid_blocks, hipStream_t st) {
    if (a.tail < 0 || a.tail > kTailRows || a.W < 64 || a.W % 64 != 0) return hipErrorInvalidValue;
    const int lds = tile_lds_bytes(a.W, a.kf, a.tail);
    if (lds > kLdsBytes - kLdsReserve) return hipErrorInvalidValue;
    if (a.bins && (map || !persistent || a.parts > 1)) return hipErrorInvalidValue;
    if (a.parts > 1) {
        // (the launch grid below holds 65535 tiles)
        if (a.part == nullptr || a.part_stride < part_words(a.W, a.kf, a.tail) || n_tiles > 65535)
            return hipErrorInvalidValue;
        k_tiles_plain<Wt, kOutPart, T><<<n_tiles * a.parts, kTileThreads, lds, st>>>(a);
        const hipError_t e = hipGetLastError();
        if (e != hipSuccess) return e;
        const dim3 grid((a.W + kMergeCols - 1) / kMergeCols, n_tiles);
        if (map) k_tiles_merge<Wt, true><<<grid, kMergeThreads, 0, st>>>(a);
        else k_tiles_merge<Wt, false><<<grid, kMergeThreads, 0, st>>>(a);
        return hipGetLastError();
    }
    if (map) k_tiles_plain<Wt, kOutMap, T><<<n_tiles, kTileThreads, lds, st>>>(a);
    else if (persistent && a.bins) k_tiles_persistent<Wt, T, true><<<grid_blocks, kTileThreads, lds, st>>>(a);
    else if (persistent) k_tiles_persistent<Wt, T, false><<<grid_blocks, kTileThreads, lds, st>>>(a);
    else k_tiles_plain<Wt, kOutColmax, T><<<n_tiles, kTileThreads, lds, st>>>(a);
    return hipGetLastError();
}

static hipError_t set_refine_attributes();
static hipError_t set_cleaning_attributes();

hipError_t init_kernel_attributes() {
    hipError_t e;
    if ((e = set_refine_attributes()) != hipSuccess) return e;
    if ((e = set_cleaning_attributes()) != hipSuccess) return e;
    if ((e = set_tile_attrs<true, true>()) != hipSuccess) return e;
    if ((e = set_tile_attrs<true, false>()) != hipSuccess) return e;
    if ((e = set_tile_attrs<false, true>()) != hipSuccess) return e;
    if ((e = set_tile_attrs<false, false>()) != hipSuccess) return e;
    if ((e = hipFuncSetAttribute((const void *)k_sort_windows, hipFuncAttributeMaxDynamicSharedMemorySize,
                                 kSortLdsBytes)) != hipSuccess)
        return e;
    return hipFuncSetAttribute((const void *)k_sort_windows_long, hipFuncAttributeMaxDynamicSharedMemorySize,
                               kSortPiece * (int)sizeof(uint32_t));
}

hipError_t launch_tiles(const TileArgs &a, bool weighted, bool map, bool persistent, int32_t n_tiles,
                        int32_t grid_blocks, hipStream_t st) {
    if (n_tiles <= 0) return hipSuccess;
    if (weighted)
        return a.tail > 0 ? launch_tiles_t<true, true>(a, map, persistent, n_tiles, grid_blocks, st)
                          : launch_tiles_t<true, false>(a, map, persistent, n_tiles, grid_blocks, st);
    return a.tail > 0 ? launch_tiles_t<false, true>(a, map, persistent, n_tiles, grid_blocks, st)
                      : launch_tiles_t<false, false>(a, map, persistent, n_tiles, grid_blocks, st);
}

hipError_t launch_select(const unsigned long long *colmax, int32_t nf, int32_t n_slots,
                         const fh_select &sel, int32_t sky_base, int32_t n_fft,
                         const WeightStats *ws, int32_t ws_stride, fh_candidate *out,
                         hipStream_t st) {
    const int n_sb = (nf + sel.width - 1) / sel.width;
    dim3 grid(n_sb, n_slots);
    // threads for four columns each where the launch leaves CUs idle, else for
    // the eight that a thread holds (1120 sub-bands of 4096 columns: 25 and
    // 11 us); a wider sub-band gets them all
    const int held = (int64_t)n_sb * n_slots <= 256 ? kHeld / 2 : kHeld;
    const int threads = std::min(1024, std::max(64, (std::min(sel.width, nf) + held * 64 - 1) / (held * 64) * 64));
    k_select<<<grid, threads, 0, st>>>(colmax, nf, sel, sky_base, n_fft, ws, ws_stride, out);
    return hipGetLastError();
}

hipError_t launch_pm_rows(int32_t n_fft, int32_t n_bins, int64_t ld, const float *sp, const float *sar,
                          int32_t k0, float theta, int32_t cap, int32_t *scratch, int32_t *counts,
                          hipStream_t st) {
    k_pm_rows<<<n_fft, 256, 0, st>>>(n_bins, ld, sp, sar, k0, theta, cap, scratch, counts);
    return hipGetLastError();
}

namespace {

// ----------------------------------------------------------------------------
// peakmap slice: the peaks of each FFT with natural bin in [k_lo, k_hi)

__global__ void k_slice_count(int32_t n_fft, const int64_t *__restrict__ offsets,
                              const int32_t *__restrict__ bins, int32_t k_lo, int32_t k_hi,
                              const double *__restrict__ tv, double *__restrict__ tv_out,
                              int64_t *__restrict__ first, int32_t *__restrict__ counts) {
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n_fft) return;
    if (tv_out != nullptr)  // the head's times [N] and velocities [N][3]
        for (int c = 0; c < 4; ++c) tv_out[(int64_t)c * n_fft + i] = tv[(int64_t)c * n_fft + i];
    const int64_t p0 = offsets[i], p1 = offsets[i + 1];
    int64_t a = p0, b = p1;
    while (a < b) {  // first bin >= k_lo
        const int64_t m = (a + b) >> 1;
        if (bins[m] >= k_lo) b = m; else a = m + 1;
    }
    const int64_t lo = a;
    b = p1;
    while (a < b) {  // first bin >= k_hi
        const int64_t m = (a + b) >> 1;
        if (bins[m] >= k_hi) b = m; else a = m + 1;
    }
    first[i] = lo;
    counts[i] = (int32_t)(a - lo);
}

__global__ void k_slice_pack(const int64_t *__restrict__ first, const int32_t *__restrict__ counts,
                             const int64_t *__restrict__ offsets, const int32_t *__restrict__ bins,
                             int32_t *__restrict__ out) {
    const int i = blockIdx.x;
    const int64_t src = first[i], dst = offsets[i];
    for (int k = threadIdx.x; k < counts[i]; k += blockDim.x) out[dst + k] = bins[src + k];
}

// ----------------------------------------------------------------------------
// refinement of many coarse candidates.  A refined volume is small (2 K_f + 1
// bins x 4 K_fdot rows), so per (candidate, direction) only a few peaks of
// each FFT can reach it: the tiles' machinery (stripe edges of a sliced
// peakmap, sorted windows, tiles) costs eleven launches per candidate, each
// far too small for the GPU.  Here all candidates run in two launches.

// Per (candidate, FFT): the run of peaks that can meet the volume in any of the
// candidate's directions (its place in the FFT: the peakmap, of which the volume
// needs a few bins, may hold more peaks than 32 bits count), and its first four
// natural bins.  The directions lie
// within `spread` of the middle one, so their Doppler factors within |v| spread
// of its: a run is a few natural bins (0.3-1 peaks on average), and the cells
// kernel, which reads it once per direction, needs no search.  grid.y =
// candidate.
__global__ void __launch_bounds__(256) k_refine_runs(
    int32_t n_fft, const int64_t *__restrict__ offsets, const int32_t *__restrict__ bins, const double *__restrict__ t,
    const double *__restrict__ v, const double *__restrict__ sky, const RefineCand *__restrict__ rc, int32_t n_dir,
    int32_t kf, int32_t nf, int32_t ns, double dfdot, double t0, double S, int32_t shift_mode, int2 *__restrict__ runs,
    int4 *__restrict__ firsts) {
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n_fft) return;
    const RefineCand q = rc[blockIdx.y];
    const double *n = sky + 3 * ((int64_t)blockIdx.y * n_dir + n_dir / 2);
    const double *vi = v + 3 * (int64_t)i;
    const double d = 1.0 + (vi[0] * n[0] + vi[1] * n[1] + vi[2] * n[2]);
    // largest change of the Doppler factor (and of its inverse) over the
    // directions; the factor 1.1 covers 1 / D and every rounding
    const double dd = 1.1 * q.spread * sqrt(vi[0] * vi[0] + vi[1] * vi[1] + vi[2] * vi[2]) + 1e-14;
    const double tau = t[i] - t0;
    const double ga = rint(((q.fdot0 + 0.0 * dfdot) * tau) * S), gb = rint(((q.fdot0 + (double)(ns - 1) * dfdot) * tau) * S);
    // edges (without their Doppler term) of the volume's ends, in fine bins
    const double off = (double)q.b0 + 0.5 * (double)kf;
    const double z_lo = off + (double)(1 - kf) + fmin(ga, gb) * (1.0 / kQd) - 2.0;
    const double z_hi = off + (double)nf + fmax(ga, gb) * (1.0 / kQd) + 2.0;
    double lo, hi;
    if (shift_mode) {
        const double sh = q.q * (1.0 - 1.0 / d), m = fabs(q.q) * dd + 1.0;
        lo = z_lo + sh - m;
        hi = z_hi + sh + m;
    } else {
        lo = fmin(z_lo * (d - dd), z_lo * (d + dd));
        hi = fmax(z_hi * (d - dd), z_hi * (d + dd));
    }
    const int32_t k1 = max(q.k_lo, (int32_t)fmin(fmax(floor(lo / (double)kf) - 1.0, -2e9), 2e9));
    const int32_t k2 = min(q.k_hi, (int32_t)fmin(fmax(ceil(hi / (double)kf) + 2.0, -2e9), 2e9));
    const int32_t *__restrict__ k = bins + offsets[i];
    const uint32_t n_i = (uint32_t)(offsets[i + 1] - offsets[i]);  // < 2^31
    // first peaks with natural bin >= k1 and >= k2, in lockstep
    uint32_t a = 0, b = 0;
    uint32_t top = 1;
    while (top <= n_i >> 1) top <<= 1;
    for (uint32_t st = top; st > 0; st >>= 1) {
        const uint32_t ta = a + st - 1, tb = b + st - 1;
        const int32_t va = ta < n_i ? k[ta] : 0x7fffffff, vb = tb < n_i ? k[tb] : 0x7fffffff;
        if (va < k1) a += st;
        if (vb < k2) b += st;
    }
    const int32_t c = b > a ? (int32_t)(b - a) : 0;
    const int64_t at = (int64_t)blockIdx.y * n_fft + i;
    runs[at] = make_int2((int32_t)a, c);
    firsts[at] = make_int4(c > 0 ? k[a] : 0, c > 1 ? k[a + 1] : 0, c > 2 ? k[a + 2] : 0, c > 3 ? k[a + 3] : 0);
}

// One workgroup per (direction, candidate): grid (n_dir, n_cand).  Threads
// own FFTs and test the peaks of their runs against the volume's bounds (the
// shifts' extremes over the rows are those of the first and last row).  The
// peaks that meet it are compacted into an LDS list, so that the (peak, row)
// pairs then spread evenly over the threads, one LDS atomic each; a thread
// keeps its row and its row's spin-down.  Window sums and the maximum follow in
// LDS.  Edges and shifts stay doubles: they are whole numbers below 2^53
// wherever a start can lie in the volume, so their difference is exact.
// Measured on 22 candidates x 25 directions (3140 FFTs of 8192 s at 100 Hz, 20
// rows): the whole call 2290 us with a slice and a tile search per candidate;
// 133 us while every direction searched runs as wide as the year's Doppler
// shift (their scattered lines, fetched at every step of the searches, bound
// it); lanes in groups of 16 over such runs, without a search, 143 us; 66 us with
// runs narrowed to the candidate's directions.
constexpr int kRefineThreads = 512;
constexpr int kRefineList = 1024;  // listed peaks per pass

struct RefinePeak {
    double y;     // stripe edge, from column 0 (fine bin 1 - K_f)
    double tau;   // t_i - t0
};

__global__ void __launch_bounds__(kRefineThreads) k_refine_cells(
    int32_t n_fft, const int64_t *__restrict__ offsets, const int32_t *__restrict__ bins,
    const double *__restrict__ t, const double *__restrict__ v, const double *__restrict__ sky,
    const RefineCand *__restrict__ rc, const int2 *__restrict__ runs,
    const int4 *__restrict__ firsts, int32_t kf, int32_t nf, int32_t ns, double dfdot, double t0, double S,
    double theta, const float *__restrict__ w, const WeightStats *__restrict__ ws, int32_t shift_mode,
    fh_candidate *__restrict__ out) {
    extern __shared__ uint32_t cells[];  // [ns][nf + kf - 1] stripe starts
    __shared__ RefinePeak s_peak[kRefineList];
    __shared__ uint32_t s_w[kRefineList];
    __shared__ int s_wave[kRefineThreads / 64];
    __shared__ unsigned long long s_best;
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int cand = blockIdx.y, dir = blockIdx.x, n_dir = gridDim.x;
    const RefineCand q = rc[cand];
    const double *n = sky + 3 * ((int64_t)cand * n_dir + dir);
    const double n0 = n[0], n1 = n[1], n2 = n[2];
    const int wc = nf + kf - 1;
    const int n_cells = ns * wc;
    for (int x = tid; x < n_cells; x += kRefineThreads) cells[x] = 0u;
    if (tid == 0) s_best = 0ull;
    bool bad = false;
    int frac = 0;
    if (w != nullptr) {
        bad = ws->bad != 0;
        frac = ws->frac_bits;
    }
    const int64_t ybase = -q.b0 * kQ - (int64_t)kf * (kQ / 2) + (kQ - 1);
    // the pairs of this thread: rows s0, s0 + n_rows, ... of peaks p0, p0 + step, ...
    const int n_rows = min(ns, kRefineThreads);
    const int step = kRefineThreads / n_rows;
    const int p_first = tid / n_rows, s_first = tid - p_first * n_rows;
    // spin-downs of the first and last row (row_shift's steps)
    const double fd_first = q.fdot0 + 0.0 * dfdot, fd_last = q.fdot0 + (double)(ns - 1) * dfdot;
    for (int i0 = 0; i0 < n_fft; i0 += kRefineThreads) {
        const int i = i0 + tid;
        int cnt = 0, most = 0;  // peaks that meet the volume; peaks of the run
        int2 run = make_int2(0, 0);
        int4 fk = make_int4(0, 0, 0, 0);
        double r = 1.0, tau = 0.0, c = 0.0, y_lo = 0.0, y_hi = 0.0;
        // edge of the run's u-th peak, and whether it meets the volume
        auto edge = [&](int u, double *y) {
            const int32_t k = u == 0 ? fk.x : u == 1 ? fk.y : u == 2 ? fk.z : u == 3 ? fk.w : bins[offsets[i] + run.x + u];
            double x = (double)(kf * k) * r;
            x = x * kQd;
            *y = floor(x) + c;
            return u < most && *y >= y_lo && *y < y_hi;
        };
        if (i < n_fft) {
            run = runs[(int64_t)cand * n_fft + i];
            fk = firsts[(int64_t)cand * n_fft + i];
            most = run.y;
            const double *vi = v + 3 * (int64_t)i;
            double d = vi[0] * n0;
            d = d + vi[1] * n1;
            d = d + vi[2] * n2;
            d = 1.0 + d;
            r = 1.0 / d;
            int64_t ci = ybase;
            if (shift_mode) {
                ci -= llrint((q.q * (1.0 - r)) * kQd);
                r = 1.0;  // (the product above is then exact)
            }
            c = (double)ci;
            tau = t[i] - t0;
            const double ga = rint((fd_first * tau) * S), gb = rint((fd_last * tau) * S);
            // some row's start lies in columns [0, wc), column = start + K_f - 1
            y_lo = (double)(1 - kf) * kQd + fmin(ga, gb);
            y_hi = (double)nf * kQd + fmax(ga, gb);
        }
        double y;
        for (int u = 0; u < most; ++u) cnt += edge(u, &y) ? 1 : 0;
        // places of the thread's peaks in the list: exclusive scan of the counts
        int incl = cnt;
        for (int o = 1; o < 64; o <<= 1) {
            const int u = __shfl_up(incl, o);
            if (lane >= o) incl += u;
        }
        if (lane == 63) s_wave[wave] = incl;
        __syncthreads();
        int first = incl - cnt, total = 0;
        for (int k = 0; k < kRefineThreads / 64; ++k) {
            const int u = s_wave[k];
            first += k < wave ? u : 0;
            total += u;
        }
        uint32_t wq = 1u;
        if (w != nullptr && cnt > 0) wq = bad ? 0u : (uint32_t)rint(ldexp((double)w[i], frac));
        for (int base = 0; base < total; base += kRefineList) {
            int at = first - base;
            for (int u = 0; cnt > 0 && u < most; ++u) {
                if (!edge(u, &y)) continue;
                if (at >= 0 && at < kRefineList) {
                    s_peak[at] = {y + (double)(kf - 1) * kQd, tau};
                    s_w[at] = wq;
                }
                ++at;
            }
            __syncthreads();
            const int n_list = min(total - base, kRefineList);
            if (p_first < step) {
                for (int s = s_first; s < ns; s += n_rows) {
                    const double fs = q.fdot0 + (double)s * dfdot;
                    for (int p = p_first; p < n_list; p += step) {
                        const RefinePeak pk = s_peak[p];
                        const double g = rint((fs * pk.tau) * S);
                        const double col = floor((pk.y - g) * (1.0 / kQd));
                        if (col >= 0.0 && col < (double)wc) atomicAdd(&cells[s * wc + (int)col], s_w[p]);
                    }
                }
            }
            __syncthreads();
        }
        if (total == 0) __syncthreads();  // s_wave is rewritten by the next round
    }
    __syncthreads();
    // window sums and their maximum (larger value, smaller bin, smaller row)
    unsigned long long best = 0ull;
    for (int e = tid; e < nf * ns; e += kRefineThreads) {
        const int s = e / nf, b = e - s * nf;
        const uint32_t *P = cells + s * wc + b;
        uint32_t h = 0;
        for (int k = 0; k < kf; ++k) h += P[k];
        const unsigned long long key = ((unsigned long long)h << 32) | (0xFFFFFFFFull - (unsigned)(b * ns + s));
        best = key > best ? key : best;
    }
    for (int o = 32; o >= 1; o >>= 1) {
        const unsigned long long u = __shfl_xor(best, o);
        best = u > best ? u : best;
    }
    if (lane == 0) atomicMax(&s_best, best);
    __syncthreads();
    if (tid == 0) {
        const unsigned long long k = s_best;
        const uint32_t at = 0xFFFFFFFFu - (uint32_t)k;
        fh_candidate x;
        x.sky = dir;
        x.subband = 0;
        x.rank = 0;
        x.bin = (int32_t)(at / (uint32_t)ns);
        x.row = (int32_t)(at % (uint32_t)ns);
        cell_value((uint32_t)(k >> 32), cell_stats(n_fft, theta, ws), ws != nullptr, &x.value, &x.cr);
        x.valid = 1;
        out[2 * ((int64_t)cand * n_dir + dir)] = x;
    }
}

// ----------------------------------------------------------------------------
// refined candidates: the best of the k_sky^2 directions' first candidates

// one wave per candidate (larger value, then smaller direction)
__global__ void __launch_bounds__(64) k_refine_pick(int32_t n_cand, int32_t n_dir,
                                                    const fh_candidate *__restrict__ cands,
                                                    const double *__restrict__ params, const double *__restrict__ lamb,
                                                    fh_refined *__restrict__ out) {
    const int c = blockIdx.x, lane = threadIdx.x;
    const fh_candidate *cc = cands + (int64_t)c * n_dir * 2;
    int best = -1;
    float val = 0.0f;
    for (int s = lane; s < n_dir; s += 64) {
        const fh_candidate &x = cc[2 * s];
        if (x.valid && (best < 0 || x.value > val)) {
            best = s;
            val = x.value;
        }
    }
    for (int o = 32; o >= 1; o >>= 1) {
        const int b2 = __shfl_xor(best, o);
        const float v2 = __shfl_xor(val, o);
        if (b2 >= 0 && (best < 0 || v2 > val || (v2 == val && b2 < best))) {
            best = b2;
            val = v2;
        }
    }
    if (lane != 0) return;
    fh_refined r{};
    r.cand = c;
    if (best >= 0) {
        const fh_candidate &x = cc[2 * best];
        const double *pr = params + 4 * (int64_t)c;  // f0 of bin 0, bin width, fdot of row 0, row step
        r.sky = best;
        r.bin = x.bin;
        r.row = x.row;
        r.value = x.value;
        r.cr = x.cr;
        r.valid = 1;
        r.f0 = pr[0] + x.bin * pr[1];
        r.fdot = pr[2] + x.row * pr[3];
        r.lambda = lamb[2 * ((int64_t)c * n_dir + best)];
        r.beta = lamb[2 * ((int64_t)c * n_dir + best) + 1];
    } else {
        r.sky = r.bin = r.row = -1;
    }
    out[c] = r;
}

// ----------------------------------------------------------------------------
// peakmap cleaning

// Filters on the peaks of a peakmap: mode 0 drops the peaks of gross cells
// holding more than thr peaks; mode 1 drops the peaks of natural bins k in
// [k_lo, k_hi) whose statistic x[step (k - k_lo) + offset] exceeds thr.
struct PeakFilter {
    int mode;
    // mode 0
    const double *t;
    double t_origin, dt_h, B;  // B = df_h T_FFT
    int64_t c0;
    int32_t n_t, n_f;
    const int32_t *hist;
    // mode 1
    int32_t k_lo, k_hi, step;
    int64_t offset, n_x;
    const int32_t *x;
    double thr;
};

__device__ __forceinline__ int gross_time_cell(const PeakFilter &f, int i) {
    return (int)floor((f.t[i] - f.t_origin) / f.dt_h);
}

// frequency cell of natural bin k, -1 when outside [0, n_f)
__device__ __forceinline__ int64_t gross_freq_cell(const PeakFilter &f, int32_t k) {
    const int64_t c = (int64_t)floor((double)k / f.B) - f.c0;
    return c >= 0 && c < f.n_f ? c : -1;
}

__device__ __forceinline__ bool filter_drop(const PeakFilter &f, int ct, int32_t k) {
    if (f.mode == 0) {
        if (ct < 0 || ct >= f.n_t) return false;
        const int64_t cf = gross_freq_cell(f, k);
        return cf >= 0 && (double)f.hist[(int64_t)ct * f.n_f + cf] > f.thr;
    }
    if (k < f.k_lo || k >= f.k_hi) return false;
    const int64_t idx = (int64_t)f.step * (k - f.k_lo) + f.offset;
    return idx >= 0 && idx < f.n_x && (double)f.x[idx] > f.thr;
}

// one wave per FFT: cells of its peaks counted into the gross histogram
__global__ void __launch_bounds__(256) k_gross_hist(int32_t n_fft, const int64_t *__restrict__ offsets,
                                                    const int32_t *__restrict__ bins, PeakFilter f,
                                                    int32_t *__restrict__ hist) {
    const int lane = threadIdx.x & 63;
    const int i = blockIdx.x * 4 + (threadIdx.x >> 6);
    if (i >= n_fft) return;
    const int ct = gross_time_cell(f, i);
    if (ct < 0 || ct >= f.n_t) return;
    for (int64_t p = offsets[i] + lane; p < offsets[i + 1]; p += 64) {
        const int64_t cf = gross_freq_cell(f, bins[p]);
        if (cf >= 0) atomicAdd(hist + (int64_t)ct * f.n_f + cf, 1);
    }
}

// The same through LDS: a workgroup counts kGrossFfts consecutive FFTs (one
// wave each at a time), whose time cells are nearly always the same (12 h hold
// 21 FFTs of 4096 s), in one row of cells, and adds the row to the histogram
// when the time cell changes.  Global atomics of single peaks, three or four
// to a cell and FFT, took 100 us for 2.1 M peaks (6286 FFTs, 120 cells); row
// by row, with consecutive lanes on consecutive cells, see launch_gross_hist.
constexpr int kGrossFfts = 16;
constexpr int kGrossCells = 8192;  // frequency cells of a row in LDS (32 KB)

__global__ void __launch_bounds__(1024) k_gross_rows(int32_t n_fft, const int64_t *__restrict__ offsets,
                                                    const int32_t *__restrict__ bins, PeakFilter f,
                                                    int32_t *__restrict__ hist) {
    extern __shared__ int32_t s_cells[];  // [n_f]
    __shared__ int s_ct[kGrossFfts];
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int f0 = blockIdx.x * kGrossFfts;
    const int nl = min(kGrossFfts, n_fft - f0);
    if (tid < nl) s_ct[tid] = gross_time_cell(f, f0 + tid);
    for (int x = tid; x < f.n_f; x += 1024) s_cells[x] = 0;
    __syncthreads();
    for (int a = 0; a < nl;) {
        const int ct = s_ct[a];
        int e = a + 1;
        while (e < nl && s_ct[e] == ct) ++e;
        if (ct >= 0 && ct < f.n_t) {
            for (int l = a + wave; l < e; l += 16) {
                const int64_t pe = offsets[f0 + l + 1];
                for (int64_t p = offsets[f0 + l] + lane; p < pe; p += 64) {
                    const int64_t cf = gross_freq_cell(f, bins[p]);
                    if (cf >= 0) atomicAdd(&s_cells[cf], 1);
                }
            }
            __syncthreads();
            int32_t *row = hist + (int64_t)ct * f.n_f;
            for (int x = tid; x < f.n_f; x += 1024) {
                const int32_t c = s_cells[x];
                if (c) atomicAdd(row + x, c);
                s_cells[x] = 0;
            }
            __syncthreads();
        }
        a = e;
    }
}

// one wave per FFT: surviving peaks counted
__global__ void __launch_bounds__(256) k_filter_count(int32_t n_fft, const int64_t *__restrict__ offsets,
                                                      const int32_t *__restrict__ bins, PeakFilter f,
                                                      const double *__restrict__ tv, double *__restrict__ tv_out,
                                                      int32_t *__restrict__ counts) {
    const int lane = threadIdx.x & 63;
    const int i = blockIdx.x * 4 + (threadIdx.x >> 6);
    if (i >= n_fft) return;
    // the head's times [N] and velocities [N][3]
    if (lane < 4) tv_out[(int64_t)lane * n_fft + i] = tv[(int64_t)lane * n_fft + i];
    const int ct = f.mode == 0 ? gross_time_cell(f, i) : 0;
    int kept = 0;
    for (int64_t p = offsets[i] + lane; p < offsets[i + 1]; p += 64) kept += filter_drop(f, ct, bins[p]) ? 0 : 1;
    for (int o = 32; o >= 1; o >>= 1) kept += __shfl_xor(kept, o);
    if (lane == 0) counts[i] = kept;
}

// one wave per FFT: surviving peaks packed in order
__global__ void __launch_bounds__(256) k_filter_pack(int32_t n_fft, const int64_t *__restrict__ offsets,
                                                     const int32_t *__restrict__ bins, PeakFilter f,
                                                     const int64_t *__restrict__ out_offsets,
                                                     int32_t *__restrict__ out_bins) {
    const int lane = threadIdx.x & 63;
    const int i = blockIdx.x * 4 + (threadIdx.x >> 6);
    if (i >= n_fft) return;
    const int ct = f.mode == 0 ? gross_time_cell(f, i) : 0;
    int64_t dst = out_offsets[i];
    const uint64_t below = (1ull << lane) - 1ull;
    for (int64_t pb = offsets[i]; pb < offsets[i + 1]; pb += 64) {
        const int64_t p = pb + lane;
        const bool in = p < offsets[i + 1];
        const int32_t k = in ? bins[p] : 0;
        const bool keep = in && !filter_drop(f, ct, k);
        const uint64_t m = __ballot(keep);
        if (keep) out_bins[dst + __popcll(m & below)] = k;
        dst += __popcll(m);
    }
}

// one wave per FFT: peaks per natural bin in [k_lo, k_hi)
__global__ void __launch_bounds__(256) k_bin_counts(int32_t n_fft, const int64_t *__restrict__ offsets,
                                                    const int32_t *__restrict__ bins, int32_t k_lo,
                                                    int32_t k_hi, int32_t *__restrict__ counts) {
    const int lane = threadIdx.x & 63;
    const int i = blockIdx.x * 4 + (threadIdx.x >> 6);
    if (i >= n_fft) return;
    for (int64_t p = offsets[i] + lane; p < offsets[i + 1]; p += 64) {
        const int32_t k = bins[p];
        if (k >= k_lo && k < k_hi) atomicAdd(counts + (k - k_lo), 1);
    }
}

// The same through LDS: workgroup (x, y) counts the x-th share of all peaks
// (the FFT does not matter) in the y-th segment of at most kCountBins bins and
// adds its counts with consecutive lanes on consecutive bins, so that one
// request carries 16 of them.  The global atomics of single peaks are bound by
// the requests to the few lines that all FFTs share: 172 us for 2.1 M peaks
// over 4600 bins, against 7 us here.
constexpr int kCountBins = 32768;   // bins of a segment (128 KB of LDS)
constexpr int kCountShare = 16384;  // peaks per workgroup: 16 per thread

__global__ void __launch_bounds__(1024) k_bin_hist(int64_t n_peaks, const int32_t *__restrict__ bins, int32_t k_lo,
                                                   int32_t k_hi, int32_t *__restrict__ counts) {
    extern __shared__ int32_t s_count[];  // [min(kCountBins, k_hi - k_lo)]
    const int32_t lo = k_lo + (int32_t)blockIdx.y * kCountBins;
    const uint32_t width = (uint32_t)min(kCountBins, k_hi - lo);
    for (uint32_t x = threadIdx.x; x < width; x += 1024) s_count[x] = 0;
    __syncthreads();
    // shares are multiples of 4 peaks, so that whole groups are 16-byte aligned
    const int64_t share = ((n_peaks + gridDim.x - 1) / gridDim.x + 3) / 4 * 4;
    const int64_t p0 = share * blockIdx.x, p1 = min(p0 + share, n_peaks);
    auto add = [&](int32_t k) {
        const uint32_t x = (uint32_t)(k - lo);
        if (k >= lo && x < width) atomicAdd(&s_count[x], 1);
    };
    for (int64_t p = p0 + 4 * (int64_t)threadIdx.x; p < p1; p += 4 * 1024) {
        if (p + 4 <= p1) {
            const int4 k = *reinterpret_cast<const int4 *>(bins + p);
            add(k.x);
            add(k.y);
            add(k.z);
            add(k.w);
        } else {
            for (int64_t u = p; u < p1; ++u) add(bins[u]);
        }
    }
    __syncthreads();
    int32_t *out = counts + (lo - k_lo);
    for (uint32_t x = threadIdx.x; x < width; x += 1024) {
        const int32_t c = s_count[x];
        if (c) atomicAdd(out + x, c);
    }
}

// value histograms for the robust statistic: pass 0 counts x, pass 1 counts
// |2 x - s| (s = twice the median, an integer)
__global__ void k_value_hist(const int32_t *__restrict__ x, int32_t n, int32_t x_max, int pass,
                             const int64_t *__restrict__ s2, int32_t *__restrict__ hist,
                             int32_t *__restrict__ err) {
    const int64_t e = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
    if (e >= n) return;
    const int32_t v = x[e];
    if (v < 0 || v > x_max) {
        atomicOr(err, 1);
        return;
    }
    if (pass == 0) {
        atomicAdd(hist + v, 1);
    } else {
        int64_t d = 2 * (int64_t)v - s2[0];
        d = d < 0 ? -d : d;
        if (d <= 2 * (int64_t)x_max) atomicAdd(hist + d, 1);
    }
}

// One block: the values at 1-based ranks ra and rb of a value histogram of
// m bins; writes their sum to s2[0] and, for pass 0, m1 = sum / 2 to out[0],
// for pass 1, m2 = sum / 4 / 0.6745 to out[1].
__global__ void __launch_bounds__(1024) k_rank_pick(const int32_t *__restrict__ hist, int32_t m, int64_t ra,
                                                    int64_t rb, int pass, int64_t *__restrict__ s2,
                                                    double *__restrict__ out, const int32_t *__restrict__ err) {
    __shared__ int64_t part[1024];
    __shared__ int32_t val[2];
    const int tid = threadIdx.x;
    if (tid < 2) val[tid] = 0;  // stays 0 for a rank past the total (invalid data)
    const int chunk = (m + 1023) / 1024;
    const int v0 = tid * chunk, v1 = min(v0 + chunk, m);
    int64_t sum = 0;
    for (int v = v0; v < v1; ++v) sum += hist[v];
    part[tid] = sum;
    __syncthreads();
    for (int o = 1; o < 1024; o <<= 1) {  // inclusive scan
        const int64_t a = tid >= o ? part[tid - o] : 0;
        __syncthreads();
        part[tid] += a;
        __syncthreads();
    }
    const int64_t before = part[tid] - sum;
    for (int q = 0; q < 2; ++q) {
        const int64_t r = q == 0 ? ra : rb;
        if (r > before && r <= before + sum) {
            int64_t c = before;
            for (int v = v0; v < v1; ++v) {
                c += hist[v];
                if (c >= r) {
                    val[q] = v;
                    break;
                }
            }
        }
    }
    __syncthreads();
    if (tid == 0) {
        const int64_t t = (int64_t)val[0] + (int64_t)val[1];
        if (pass == 0) {
            s2[0] = t;
            out[0] = 0.5 * (double)t;
        } else {
            // median of |x - m1| = (t / 2) / 2: both halves exact
            out[1] = 0.5 * (0.5 * (double)val[0] + 0.5 * (double)val[1]) / 0.6745;
            out[2] = (double)*err;  // a value outside [0, x_max]
        }
    }
}

// The whole statistic in one workgroup, when the values' histogram fits the
// LDS: counts, their prefix sums, the median's two ranks s = a + b, and the
// ranks of |2 x - s| from the same prefix sums (values at most d away are those
// in [ceil((s - d) / 2), floor((s + d) / 2)]), found by bisection.  It replaces
// two fills, two histograms and two rank searches, 40 us of launches on 4600
// counts of 6286 FFTs.  out[2] (as a number) and *err report a value outside
// [0, x_max].
constexpr int kRobustBins = 36 * 1024;  // 144 KB of LDS

__global__ void __launch_bounds__(1024) k_robust_lds(const int32_t *__restrict__ x, int32_t n, int32_t x_max,
                                                     int64_t ra, int64_t rb, double *__restrict__ out,
                                                     int32_t *__restrict__ err) {
    extern __shared__ int32_t s_cum[];  // [x_max + 1]
    __shared__ int32_t s_part[16];
    __shared__ int32_t s_bad;
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int m = x_max + 1;
    if (tid == 0) s_bad = 0;
    for (int v = tid; v < m; v += 1024) s_cum[v] = 0;
    __syncthreads();
    for (int e = tid; e < n; e += 1024) {
        const int32_t v = x[e];
        if (v < 0 || v > x_max) s_bad = 1;
        else atomicAdd(&s_cum[v], 1);
    }
    __syncthreads();
    // inclusive prefix sums: every thread a run of values
    const int chunk = (m + 1023) / 1024;
    const int v0 = min(tid * chunk, m), v1 = min(v0 + chunk, m);
    int32_t sum = 0;
    for (int v = v0; v < v1; ++v) sum += s_cum[v];
    int32_t incl = sum;
    for (int o = 1; o < 64; o <<= 1) {
        const int32_t u = __shfl_up(incl, o);
        if (lane >= o) incl += u;
    }
    if (lane == 63) s_part[wave] = incl;
    __syncthreads();
    int32_t before = incl - sum;
    for (int k = 0; k < wave; ++k) before += s_part[k];
    for (int v = v0; v < v1; ++v) {
        before += s_cum[v];
        s_cum[v] = before;
    }
    __syncthreads();
    if (tid != 0) return;
    // smallest v with at least r values up to it (0 when there are fewer)
    auto value_at = [&](int64_t r) {
        int a = 0, b = m;
        while (a < b) {
            const int c = (a + b) >> 1;
            if (s_cum[c] >= r) b = c; else a = c + 1;
        }
        return (int64_t)(a < m ? a : 0);
    };
    const int64_t s = value_at(ra) + value_at(rb);
    // smallest d with at least r values at |2 v - s| <= d (0 when there are fewer)
    auto deviation_at = [&](int64_t r) {
        int64_t a = 0, b = 2 * (int64_t)x_max + 1;
        while (a < b) {
            const int64_t d = (a + b) >> 1;
            const int64_t hi = min((s + d) >> 1, (int64_t)x_max), lo = (s - d + 1) >> 1;
            const int64_t c = s_cum[hi] - (lo > 0 ? s_cum[lo - 1] : 0);
            if (c >= r) b = d; else a = d + 1;
        }
        return a <= 2 * (int64_t)x_max ? a : (int64_t)0;
    };
    out[0] = 0.5 * (double)s;
    // median of |x - m1| = (t / 2) / 2: both halves exact
    out[1] = 0.5 * (0.5 * (double)deviation_at(ra) + 0.5 * (double)deviation_at(rb)) / 0.6745;
    out[2] = (double)s_bad;
    *err = s_bad;
}

// fine-bin counts of a column-maximum buffer (value << 32 | ~row)
__global__ void k_colmax_values(const unsigned long long *__restrict__ colmax, int32_t nf,
                                int32_t *__restrict__ out) {
    const int b = blockIdx.x * blockDim.x + threadIdx.x;
    if (b < nf) out[b] = (int32_t)(colmax[b] >> 32);
}

// Column maxima of n_slots directions decoded: value (the count, or the
// weighted sum as k_select forms it from the fixed point) and smallest row.
__global__ void k_colmax_decode(const unsigned long long *__restrict__ colmax, int32_t nf, int32_t n_slots,
                                const WeightStats *__restrict__ ws, int32_t ws_stride,
                                float *__restrict__ value, int32_t *__restrict__ row) {
    const int64_t n = (int64_t)n_slots * nf;
    for (int64_t x = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; x < n; x += (int64_t)gridDim.x * blockDim.x) {
        const unsigned long long k = colmax[x];
        const uint32_t v = (uint32_t)(k >> 32);
        float f = (float)v;
        if (ws != nullptr) {
            const int64_t slot = x / nf;
            f = f * (float)ldexp(1.0, -ws[slot * ws_stride].frac_bits);
        }
        value[x] = f;
        row[x] = (int32_t)(0xFFFFFFFFu - (uint32_t)k);
    }
}

}  // namespace

hipError_t launch_colmax_decode(const unsigned long long *colmax, int32_t nf, int32_t n_slots, const WeightStats *ws,
                                int32_t ws_stride, float *value, int32_t *row, hipStream_t st) {
    const int64_t n = (int64_t)n_slots * nf;
    if (n <= 0) return hipSuccess;
    k_colmax_decode<<<grid_for(n, 256) > 8192 ? 8192 : grid_for(n, 256), 256, 0, st>>>(colmax, nf, n_slots, ws,
                                                                                       ws_stride, value, row);
    return hipGetLastError();
}

hipError_t launch_slice(int32_t n_fft, const int64_t *offsets, const int32_t *bins, int32_t k_lo, int32_t k_hi,
                        const double *tv, double *tv_out, int64_t *first, int32_t *counts, int64_t *out_offsets, int32_t *out_bins,
                        int64_t *meta, hipStream_t st) {
    k_slice_count<<<grid_for(n_fft, 256), 256, 0, st>>>(n_fft, offsets, bins, k_lo, k_hi, tv, tv_out, first, counts);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    k_pm_scan<<<1, 1024, 0, st>>>(n_fft, counts, out_offsets, meta);
    if ((e = hipGetLastError()) != hipSuccess) return e;
    k_slice_pack<<<n_fft, 256, 0, st>>>(first, counts, out_offsets, bins, out_bins);
    return hipGetLastError();
}

static hipError_t set_refine_attributes() {
    const int fixed = (int)sizeof(RefinePeak) * kRefineList + 4 * kRefineList + 1024;
    return hipFuncSetAttribute((const void *)k_refine_cells, hipFuncAttributeMaxDynamicSharedMemorySize,
                               kLdsBytes - fixed);
}

// The line lies where the volume and the peak list fill the LDS of a CU (up to
// 4 x 46 rows at K_f = 64, 4 x 296 at K_f = 10); beyond it the cells have no
// place and the volume is searched with the tiles, candidate by candidate.
int refine_cell_bytes(int kf, int nf, int ns) {
    const int64_t n = 4ll * ns * (nf + kf - 1);
    const int64_t fixed = (int64_t)sizeof(RefinePeak) * kRefineList + 4 * kRefineList + 1024;
    return n + fixed <= kLdsBytes ? (int)n : 0;
}

hipError_t launch_refine_cells(int32_t n_fft, const int64_t *offsets, const int32_t *bins, const double *t,
                               const double *v, int32_t n_cand, int32_t n_dir, const double *sky,
                               const RefineCand *rc, int2 *runs, int4 *firsts, int32_t kf, int32_t nf, int32_t ns,
                               double dfdot, double t0, double t_fft, double theta, const float *w,
                               const WeightStats *ws, int32_t shift_mode, fh_candidate *out, hipStream_t st) {
    const int lds = refine_cell_bytes(kf, nf, ns);
    if (lds == 0 || n_cand > 65535) return hipErrorInvalidValue;
    const double S = ((double)kf * t_fft) * kQd;
    k_refine_runs<<<dim3(grid_for(n_fft, 256), n_cand), 256, 0, st>>>(n_fft, offsets, bins, t, v, sky, rc, n_dir, kf, nf,
                                                                      ns, dfdot, t0, S, shift_mode, runs, firsts);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    k_refine_cells<<<dim3(n_dir, n_cand), kRefineThreads, lds, st>>>(n_fft, offsets, bins, t, v, sky, rc, runs, firsts,
                                                                     kf, nf, ns, dfdot, t0, S, theta, w, ws, shift_mode,
                                                                     out);
    return hipGetLastError();
}

hipError_t launch_refine_pick(int32_t n_cand, int32_t n_dir, const fh_candidate *cands, const double *params,
                              const double *lamb, fh_refined *out, hipStream_t st) {
    if (n_cand <= 0) return hipSuccess;
    k_refine_pick<<<n_cand, 64, 0, st>>>(n_cand, n_dir, cands, params, lamb, out);
    return hipGetLastError();
}

static hipError_t set_cleaning_attributes() {
    hipError_t e = hipFuncSetAttribute((const void *)k_bin_hist, hipFuncAttributeMaxDynamicSharedMemorySize,
                                       4 * kCountBins);
    if (e != hipSuccess) return e;
    return hipFuncSetAttribute((const void *)k_robust_lds, hipFuncAttributeMaxDynamicSharedMemorySize,
                               4 * kRobustBins);
}

hipError_t launch_gross_hist(int32_t n_fft, const int64_t *offsets, const int32_t *bins, const double *t,
                             double t_fft, const fh_gross &geo, int32_t *hist, hipStream_t st) {
    hipError_t e = launch_fill_i32(hist, (int64_t)geo.n_t * geo.n_f, 0, st);
    if (e != hipSuccess || n_fft == 0) return e;
    PeakFilter f{};
    f.mode = 0;
    f.t = t;
    f.t_origin = geo.t_origin;
    f.dt_h = geo.dt_h;
    f.B = geo.df_h * t_fft;
    f.c0 = geo.c0;
    f.n_t = geo.n_t;
    f.n_f = geo.n_f;
    // a row of cells that fits a quarter of the LDS (the 0.01 Hz cells of 80 Hz)
    // is counted there: 100 -> 12 us at 6286 FFTs x 120 cells
    if (f.n_f <= kGrossCells)
        k_gross_rows<<<(n_fft + kGrossFfts - 1) / kGrossFfts, 1024, 4 * f.n_f, st>>>(n_fft, offsets, bins, f, hist);
    else
        k_gross_hist<<<(n_fft + 3) / 4, 256, 0, st>>>(n_fft, offsets, bins, f, hist);
    return hipGetLastError();
}

hipError_t launch_filter(int32_t n_fft, const int64_t *offsets, const int32_t *bins, const FilterSpec &spec,
                         const double *tv, double *tv_out, int32_t *counts, int64_t *out_offsets, int32_t *out_bins, int phase, int64_t *meta,
                         hipStream_t st) {
    PeakFilter f{};
    f.mode = spec.mode;
    f.t = spec.t;
    f.t_origin = spec.geo.t_origin;
    f.dt_h = spec.geo.dt_h;
    f.B = spec.geo.df_h * spec.t_fft;
    f.c0 = spec.geo.c0;
    f.n_t = spec.geo.n_t;
    f.n_f = spec.geo.n_f;
    f.hist = spec.hist;
    f.k_lo = spec.k_lo;
    f.k_hi = spec.k_hi;
    f.step = spec.step;
    f.offset = spec.offset;
    f.n_x = spec.n_x;
    f.x = spec.x;
    f.thr = spec.thr;
    if (n_fft == 0) return hipSuccess;
    if (phase == 0) {
        k_filter_count<<<(n_fft + 3) / 4, 256, 0, st>>>(n_fft, offsets, bins, f, tv, tv_out, counts);
        hipError_t e = hipGetLastError();
        if (e != hipSuccess) return e;
        k_pm_scan<<<1, 1024, 0, st>>>(n_fft, counts, out_offsets, meta);
    } else {
        k_filter_pack<<<(n_fft + 3) / 4, 256, 0, st>>>(n_fft, offsets, bins, f, out_offsets, out_bins);
    }
    return hipGetLastError();
}

hipError_t launch_bin_counts(int32_t n_fft, int64_t n_peaks, const int64_t *offsets, const int32_t *bins,
                             int32_t k_lo, int32_t k_hi, int32_t *counts, hipStream_t st) {
    hipError_t e = launch_fill_i32(counts, (int64_t)k_hi - k_lo, 0, st);
    if (e != hipSuccess || n_fft == 0 || n_peaks == 0) return e;
    // up to four LDS segments (each reads every peak once): 172 -> 7 us at
    // 2.1 M peaks over 4600 bins.  Wider ranges spread the single atomics over
    // enough lines, and more segments would read the peaks more often.
    const int64_t width = (int64_t)k_hi - k_lo;
    if (width <= 4 * kCountBins) {
        const int share = (int)std::min<int64_t>(128, (n_peaks + kCountShare - 1) / kCountShare);
        const size_t lds = 4 * (size_t)std::min<int64_t>(width, kCountBins);
        k_bin_hist<<<dim3(share, (unsigned)((width + kCountBins - 1) / kCountBins)), 1024, lds, st>>>(
            n_peaks, bins, k_lo, k_hi, counts);
        return hipGetLastError();
    }
    k_bin_counts<<<(n_fft + 3) / 4, 256, 0, st>>>(n_fft, offsets, bins, k_lo, k_hi, counts);
    return hipGetLastError();
}

hipError_t launch_robust(const int32_t *x, int32_t n, int32_t x_max, int32_t *hist, int64_t *s2, double *out,
                         int32_t *err, hipStream_t st) {
    const int64_t ra = (int64_t)(n + 1) / 2, rb = (int64_t)n / 2 + 1;  // odd n: both the middle
    // one workgroup while its histogram fits the LDS and its 64 rounds of
    // values stay below the launches it saves: 40 -> 11 us at 4600 values
    if (x_max < kRobustBins && n <= 65536) {
        k_robust_lds<<<1, 1024, 4 * ((size_t)x_max + 1), st>>>(x, n, x_max, ra, rb, out, err);
        return hipGetLastError();
    }
    hipError_t e = launch_fill_i32(err, 1, 0, st);
    if (e != hipSuccess) return e;
    for (int pass = 0; pass < 2; ++pass) {
        const int32_t m = pass == 0 ? x_max + 1 : 2 * x_max + 1;
        e = launch_fill_i32(hist, m, 0, st);
        if (e != hipSuccess) return e;
        k_value_hist<<<grid_for(n, 256), 256, 0, st>>>(x, n, x_max, pass, s2, hist, err);
        if ((e = hipGetLastError()) != hipSuccess) return e;
        k_rank_pick<<<1, 1024, 0, st>>>(hist, m, ra, rb, pass, s2, out, err);
        if ((e = hipGetLastError()) != hipSuccess) return e;
    }
    return hipSuccess;
}

hipError_t launch_colmax_values(const unsigned long long *colmax, int32_t nf, int32_t *out, hipStream_t st) {
    k_colmax_values<<<grid_for(nf, 256), 256, 0, st>>>(colmax, nf, out);
    return hipGetLastError();
}

hipError_t launch_pm_scan(int32_t n_fft, const int32_t *counts, int64_t *offsets, int64_t *meta, hipStream_t st) {
    k_pm_scan<<<1, 1024, 0, st>>>(n_fft, counts, offsets, meta);
    return hipGetLastError();
}

hipError_t launch_pm_pack(int32_t n_fft, int32_t cap, const int32_t *scratch, const int64_t *offsets,
                          int32_t *bins, hipStream_t st) {
    k_pm_pack<<<n_fft, 256, 0, st>>>(cap, scratch, offsets, bins);
    return hipGetLastError();
}

}  // namespace fh
