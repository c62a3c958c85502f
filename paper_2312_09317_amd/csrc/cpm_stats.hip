// Cell-level summary statistics of batched runs: per-cell samples (volume,
// surface, centroid) taken every few MCS, reduced per lattice to the means
// and variances of volume, surface, speed and persistence time.  FP64, with
// floating-point contraction off so that every per-cell quantity is
// rounded exactly as written.
//
// Speed and directional persistence are the motility read-outs of the paper
// (Results, Fig. 5B: directional autocorrelation; the tissue-model sections:
// cell speeds); the paper gives no formula, the definitions follow.
//   speed:       |d_k| / interval, d_k the minimum-image centroid
//                displacement between consecutive samples (cell alive at both)
//   persistence: first lag where A(tau) = mean_k u_k . u_{k+tau} of the unit
//                displacements drops below 1/e, linearly interpolated between
//                the lags, in MCS; the longest defined lag if it never does
#include <algorithm>

#include "cpm_internal.hpp"

#pragma clang fp contract(off)

namespace cpm {
namespace {

constexpr int kRec = 5;  // V, S, x, y, z

__device__ __forceinline__ int find_lattice(const int64_t *off, int n, int64_t j)
{
    int lo = 0, hi = n;  // off[lo] <= j < off[hi]
    while (hi - lo > 1) {
        const int mid = (lo + hi) / 2;
        if (off[mid] <= j) lo = mid;
        else hi = mid;
    }
    return lo;
}

// One record per label: (V, S, centroid position in [0, L) per axis).
__global__ void sample_kernel(const StatsTables t, const int32_t *vol, const int32_t *surf, const int64_t *csum,
                              double *samples, int k, int n_samples)
{
    const int64_t j = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (j >= t.label_off[t.n]) return;
    const int i = find_lattice(t.label_off, t.n, j);
    const int64_t c = j - t.label_off[i];
    const int64_t labels = t.label_off[i + 1] - t.label_off[i];
    double *rec = samples + (t.label_off[i] * n_samples + (int64_t)k * labels + c) * kRec;
    const int32_t v = vol[j];
    rec[0] = (double)v;
    rec[1] = (double)surf[j];
    for (int d = 0; d < 3; ++d) {
        double x = 0.0;
        if (d < t.ndim && v > 0) {
            const double L = (double)t.dims[3 * i + d];
            x = fmod((double)csum[j * t.ndim + d] / (double)v, L);
            if (x < 0.0) x += L;
        }
        rec[2 + d] = x;
    }
}

__device__ double block_sum(double v, double *red)
{
    const int tid = threadIdx.x;
    red[tid] = v;
    __syncthreads();
    for (int w = blockDim.x / 2; w > 0; w >>= 1) {
        if (tid < w) red[tid] += red[tid + w];
        __syncthreads();
    }
    const double r = red[0];
    __syncthreads();
    return r;
}

// Displacement of cell c between samples k and k+1 (minimum image); false if
// the cell is dead at either sample.
__device__ __forceinline__ bool displacement(const double *base, int64_t labels, int ndim, const double *L, int k,
                                             int64_t c, double *d)
{
    const double *a = base + ((int64_t)k * labels + c) * kRec;
    const double *b = base + ((int64_t)(k + 1) * labels + c) * kRec;
    if (!(a[0] > 0.0) || !(b[0] > 0.0)) return false;
    for (int e = 0; e < ndim; ++e) {
        const double x = b[2 + e] - a[2 + e];
        d[e] = x - L[e] * rint(x / L[e]);
    }
    return true;
}

// The eight statistics from the eleven sums (count, sum and sum of squares,
// volume and surface sharing a count).
__device__ __forceinline__ void write_moments(const double *r, double *o)
{
    auto moments = [](double n, double s1, double s2, double *mv) {
        if (n > 0) {
            // variance (n s2 - s1^2) / n^2, both products with their rounding
            // errors: s2 / n - mean^2 lost the digits that cancel.  What is
            // left is the rounding of the sums (of a single value, that of
            // its square): the variance of one value is 0, and none is negative
            const double p = s1 * s1, pe = fma(s1, s1, -p), q = n * s2, qe = fma(n, s2, -q);
            const double var = ((q - p) + (qe - pe)) / (n * n);
            mv[0] = s1 / n;
            mv[1] = n > 1.0 && !(var < 0.0) ? var : 0.0;
        } else {
            mv[0] = 0.0;
            mv[1] = 0.0;
        }
    };
    moments(r[0], r[1], r[2], o);
    moments(r[0], r[3], r[4], o + 2);
    moments(r[5], r[6], r[7], o + 4);
    moments(r[8], r[9], r[10], o + 6);
}

// The general form, for sample series whose steps do not fit the LDS: one
// workgroup per lattice, every step computed where it is used.
__global__ void __launch_bounds__(256) summary_kernel(const StatsTables t, const double *samples, int n_samples,
                                                      double interval, double *out)
{
    __shared__ double red[256];
    const int i = blockIdx.x;
    const int tid = threadIdx.x;
    const int64_t labels = t.label_off[i + 1] - t.label_off[i];
    const double *base = samples + t.label_off[i] * n_samples * kRec;
    const int ndim = t.ndim;
    double L[3];
    for (int d = 0; d < 3; ++d) L[d] = (double)t.dims[3 * i + d];
    const int K = n_samples;
    const double inv_e = exp(-1.0);

    double n_vs = 0, sv = 0, svv = 0, ss = 0, sss = 0;
    double n_sp = 0, ssp = 0, sspp = 0;
    double n_pe = 0, spe = 0, spee = 0;
    for (int64_t c = 1 + tid; c < labels; c += blockDim.x) {
        for (int k = 0; k < K; ++k) {
            const double *r = base + ((int64_t)k * labels + c) * kRec;
            if (r[0] > 0.0) {
                n_vs += 1.0;
                sv += r[0];
                svv += r[0] * r[0];
                ss += r[1];
                sss += r[1] * r[1];
            }
        }
        // speeds and persistence of cell c
        bool any_lag = false, done = false;
        double a_prev = 1.0, p = 0.0;
        int last = 0;
        for (int k = 0; k + 1 < K; ++k) {
            double d[3] = {0, 0, 0};
            if (displacement(base, labels, ndim, L, k, c, d)) {
                double n2 = 0.0;
                for (int e = 0; e < ndim; ++e) n2 = n2 + d[e] * d[e];
                const double sp = sqrt(n2) / interval;
                n_sp += 1.0;
                ssp += sp;
                sspp += sp * sp;
            }
        }
        const int m = K - 1;  // displacement steps
        for (int tau = 1; tau < m && !done; ++tau) {
            double acc = 0.0;
            int cnt = 0;
            for (int k = 0; k + tau < m; ++k) {
                double u[3] = {0, 0, 0}, w[3] = {0, 0, 0};
                if (!displacement(base, labels, ndim, L, k, c, u)) continue;
                if (!displacement(base, labels, ndim, L, k + tau, c, w)) continue;
                double nu = 0.0, nw = 0.0;
                for (int e = 0; e < ndim; ++e) {
                    nu = nu + u[e] * u[e];
                    nw = nw + w[e] * w[e];
                }
                nu = sqrt(nu);
                nw = sqrt(nw);
                if (!(nu > 0.0) || !(nw > 0.0)) continue;
                double dot = 0.0;
                for (int e = 0; e < ndim; ++e) dot = dot + (u[e] / nu) * (w[e] / nw);
                acc = acc + dot;
                ++cnt;
            }
            if (cnt == 0) continue;
            any_lag = true;
            const double a = acc / (double)cnt;
            if (a < inv_e) {
                // linear between the last defined lag and this one
                p = (double)last + (double)(tau - last) * (a_prev - inv_e) / (a_prev - a);
                done = true;
            } else {
                a_prev = a;
                last = tau;
            }
        }
        if (any_lag) {
            if (!done) p = (double)last;
            const double pm = p * interval;
            n_pe += 1.0;
            spe += pm;
            spee += pm * pm;
        }
    }
    const double tot[11] = {n_vs, sv, svv, ss, sss, n_sp, ssp, sspp, n_pe, spe, spee};
    double r[11];
    for (int q = 0; q < 11; ++q) r[q] = block_sum(tot[q], red);
    if (tid == 0) write_moments(r, out + 8 * (int64_t)i);
}

// Unit displacement of cell c over step k (false when undefined: the cell is
// dead at either sample or did not move).
__device__ __forceinline__ bool unit_step(const double *base, int64_t labels, int ndim, const double *L, int k,
                                          int64_t c, double *u)
{
    if (!displacement(base, labels, ndim, L, k, c, u)) return false;
    double n = 0.0;
    for (int e = 0; e < ndim; ++e) n = n + u[e] * u[e];
    n = sqrt(n);
    if (!(n > 0.0)) return false;
    for (int e = 0; e < ndim; ++e) u[e] = u[e] / n;
    return true;
}

// Directional autocorrelation of lattice blockIdx.x: per lag tau, the sum of
// u_k . u_{k+tau} over cells and steps with both unit steps defined, and the
// number of such pairs.  One workgroup per lattice, cells strided over its
// threads; lags one after another.  The general form, as summary_kernel.
__global__ void __launch_bounds__(256) autocorr_kernel(const StatsTables t, const double *samples, int n_samples,
                                                       double *out)
{
    __shared__ double red[256];
    const int i = blockIdx.x;
    const int tid = threadIdx.x;
    const int64_t labels = t.label_off[i + 1] - t.label_off[i];
    const double *base = samples + t.label_off[i] * n_samples * kRec;
    const int ndim = t.ndim;
    double L[3];
    for (int d = 0; d < 3; ++d) L[d] = (double)t.dims[3 * i + d];
    const int m = n_samples - 1;  // steps
    for (int tau = 0; tau < m; ++tau) {
        double acc = 0.0, cnt = 0.0;
        for (int64_t c = 1 + tid; c < labels; c += blockDim.x) {
            for (int k = 0; k + tau < m; ++k) {
                double u[3] = {0, 0, 0}, w[3] = {0, 0, 0};
                if (!unit_step(base, labels, ndim, L, k, c, u)) continue;
                if (!unit_step(base, labels, ndim, L, k + tau, c, w)) continue;
                double dot = 0.0;
                for (int e = 0; e < ndim; ++e) dot = dot + u[e] * w[e];
                acc = acc + dot;
                cnt = cnt + 1.0;
            }
        }
        const double sa = block_sum(acc, red), sc = block_sum(cnt, red);
        if (tid == 0) {
            out[2 * ((int64_t)i * m + tau)] = sa;
            out[2 * ((int64_t)i * m + tau) + 1] = sc;
        }
    }
}

// ---------------------------------------------------------------- staged forms
//
// The two reductions with each cell's steps computed once and kept in LDS.
// Per (cell, lag) the general kernels above recompute both steps of every
// pair from five loads each, a division and a square root, on one workgroup
// per lattice: 6.7 ms (autocorrelation) and 5.4 ms (summary) on 256 lattices
// of 64^2 to 512^2 (about 300 cells each) with 41 samples.  Here a workgroup takes
// a chunk of 2^lc cells: its threads first compute the unit steps (one per
// cell and sample) into LDS, cells fastest, then take (cell, kLags lags)
// items each, in which a window of kLags steps slides along k, so one step
// read from LDS serves kLags pairs.  Lags go in increasing order over the
// waves, the long sums first.  Chunks of one lattice are dealt to `splits`
// workgroups (a lattice on one workgroup left the largest of uneven lattices
// running alone), whose partial sums finish_kernel adds in a fixed order, so
// the result does not depend on timing.  Both together on that workload: 0.25
// ms, bound by FP64 issue and LDS reads of the pairs.
constexpr int kStatThreads = 512;
constexpr int kLags = 4;
constexpr int kSums = 11;               // partial sums of the summary
constexpr size_t kStatLds = 144 * 1024;  // LDS a workgroup may take (160 KiB on gfx950)

// LDS bytes per cell for m steps: unit steps, flags and, for the summary,
// the mean and count of every lag.
__host__ __device__ constexpr size_t stat_cell_bytes(bool autoc, int ndim, int m)
{
    return (size_t)m * ((size_t)ndim * 8 + 1 + (autoc ? 0 : 12));
}

// Workgroups of a lattice of `labels` labels: one per chunk, but no more
// than its share of the partial buffer (3 doubles per label) holds.
__host__ __device__ inline int stat_splits(int64_t labels, int lc, int values)
{
    const int64_t chunks = (labels - 1 + (1 << lc) - 1) >> lc, room = labels * 3 / values;
    const int64_t s = chunks < room ? chunks : room;
    return s < 1 ? 1 : s > 1024 ? 1024 : (int)s;
}

// Sum over the 2^lc lanes of this lane's aligned group.
__device__ __forceinline__ double lane_sum(double v, int lc)
{
    for (int o = (1 << lc) >> 1; o > 0; o >>= 1) v = v + __shfl_xor(v, o, 64);
    return v;
}

// The persistence time of a cell in sample intervals from its lags' means
// (first lag below 1/e, interpolated; the last defined lag if none is);
// false without a defined lag.
__device__ __forceinline__ bool persistence_lag(const double *mean, const int *cnt, int m, int pitch, double inv_e,
                                                double &p)
{
    bool any_lag = false;
    double a_prev = 1.0;
    int last = 0;
    for (int tau = 1; tau < m; ++tau) {
        if (cnt[tau * pitch] == 0) continue;
        any_lag = true;
        const double a = mean[tau * pitch];
        if (a < inv_e) {
            p = (double)last + (double)(tau - last) * (a_prev - inv_e) / (a_prev - a);
            return true;
        }
        a_prev = a;
        last = tau;
    }
    p = (double)last;
    return any_lag;
}

template <int D, bool AUTO>
__global__ void __launch_bounds__(kStatThreads) staged_stats_kernel(const StatsTables t, const double *samples,
                                                                    int n_samples, double interval, int lc, int max_splits, double *part,
                                                                    double *out)
{
    extern __shared__ __align__(16) unsigned char lds[];
    // blocks of a lattice next to each other (all lattices' first blocks first
    // left the large lattices' others to the end: 0.28 against 0.25 ms)
    const int i = (int)(blockIdx.x / (unsigned)max_splits), split = (int)(blockIdx.x % (unsigned)max_splits);
    const int tid = threadIdx.x;
    const int64_t labels = t.label_off[i + 1] - t.label_off[i];
    const int K = n_samples, m = K - 1, C = 1 << lc;
    const int values = AUTO ? 2 * m : kSums;
    const int splits = stat_splits(labels, lc, values);
    if (split >= splits) return;  // uniform over the block
    const double *base = samples + t.label_off[i] * n_samples * kRec;
    double L[D];
    for (int d = 0; d < D; ++d) L[d] = (double)t.dims[3 * i + d];
    // [k][axis][cell] unit steps; [lag][cell] means and counts; [k][cell]
    // flags (the unit step is defined); AUTO: the running sums per lag
    double *U = reinterpret_cast<double *>(lds);
    double *mean = U + (size_t)m * D * C;
    int *count = reinterpret_cast<int *>(mean + (AUTO ? 0 : (size_t)m * C));
    uint8_t *ok = reinterpret_cast<uint8_t *>(count + (AUTO ? 0 : (size_t)m * C));
    double *lag_sums = reinterpret_cast<double *>(lds + (((size_t)(ok - lds) + (size_t)m * C + 15) & ~(size_t)15));
    if (AUTO)
        for (int q = tid; q < 2 * m; q += kStatThreads) lag_sums[q] = 0.0;

    double sums[kSums];
#pragma unroll
    for (int q = 0; q < kSums; ++q) sums[q] = 0.0;
    const double inv_e = exp(-1.0);
    for (int64_t c0 = 1 + ((int64_t)split << lc); c0 < labels; c0 += (int64_t)splits << lc) {
        __syncthreads();  // the previous chunk's readers are done
        for (int q = tid; q < K * C; q += kStatThreads) {
            const int k = q >> lc, cl = q & (C - 1);
            const int64_t c = c0 + cl;
            if (!AUTO && c < labels) {
                const double *r = base + ((int64_t)k * labels + c) * kRec;
                if (r[0] > 0.0) {
                    sums[0] += 1.0;
                    sums[1] += r[0];
                    sums[2] += r[0] * r[0];
                    sums[3] += r[1];
                    sums[4] += r[1] * r[1];
                }
            }
            if (k == m) continue;
            double u[3] = {0, 0, 0};
            bool def = false;
            if (c < labels && displacement(base, labels, D, L, k, c, u)) {
                double n = 0.0;
#pragma unroll
                for (int e = 0; e < D; ++e) n = n + u[e] * u[e];
                n = sqrt(n);
                if (!AUTO) {
                    const double sp = n / interval;
                    sums[5] += 1.0;
                    sums[6] += sp;
                    sums[7] += sp * sp;
                }
                def = n > 0.0;
                if (def) {
#pragma unroll
                    for (int e = 0; e < D; ++e) u[e] = u[e] / n;
                }
            }
#pragma unroll
            for (int e = 0; e < D; ++e) U[(size_t)(k * D + e) * C + cl] = u[e];
            ok[k * C + cl] = def;
        }
        __syncthreads();
        for (int q = tid; q < (((m + kLags - 1) / kLags) << lc); q += kStatThreads) {
            const int cl = q & (C - 1), tau0 = (q >> lc) * kLags;
            double acc[kLags], w[kLags][D];
            int cnt[kLags];
            bool wok[kLags];
            auto window = [&](int slot, int k) {
                wok[slot] = k < m && ok[k * C + cl];
#pragma unroll
                for (int e = 0; e < D; ++e) w[slot][e] = k < m ? U[(size_t)(k * D + e) * C + cl] : 0.0;
            };
#pragma unroll
            for (int j = 0; j < kLags; ++j) {
                acc[j] = 0.0;
                cnt[j] = 0;
                if (j + 1 < kLags) window(j, tau0 + j);
            }
            for (int k0 = 0; k0 + tau0 < m; k0 += kLags) {
#pragma unroll
                for (int r = 0; r < kLags; ++r) {
                    // slot (r + j) mod kLags holds step k + tau0 + j
                    const int k = k0 + r;
                    window((r + kLags - 1) % kLags, k + tau0 + kLags - 1);
                    const bool mine = k < m && ok[k * C + cl];
                    double u[D];
#pragma unroll
                    for (int e = 0; e < D; ++e) u[e] = k < m ? U[(size_t)(k * D + e) * C + cl] : 0.0;
#pragma unroll
                    for (int j = 0; j < kLags; ++j) {
                        const int sl = (r + j) % kLags;
                        double dot = 0.0;
#pragma unroll
                        for (int e = 0; e < D; ++e) dot = dot + u[e] * w[sl][e];
                        const bool both = mine && wok[sl];
                        acc[j] = acc[j] + (both ? dot : 0.0);
                        cnt[j] += both;
                    }
                }
            }
#pragma unroll
            for (int j = 0; j < kLags; ++j) {
                if (AUTO) {
                    // one group of lanes owns a lag in every chunk
                    const double a = lane_sum(acc[j], lc), n = lane_sum((double)cnt[j], lc);
                    if (cl == 0 && tau0 + j < m) {
                        lag_sums[2 * (tau0 + j)] += a;
                        lag_sums[2 * (tau0 + j) + 1] += n;
                    }
                } else if (tau0 + j < m) {
                    mean[(tau0 + j) * C + cl] = acc[j] / (double)cnt[j];
                    count[(tau0 + j) * C + cl] = cnt[j];
                }
            }
        }
        if (!AUTO) {
            __syncthreads();
            double p;
            if (tid < C && persistence_lag(mean + tid, count + tid, m, C, inv_e, p)) {
                const double pm = p * interval;
                sums[8] += 1.0;
                sums[9] += pm;
                sums[10] += pm * pm;
            }
        }
    }
    // the workgroup's sums: straight to the output when it is the lattice's
    // only one, else `values` doubles of the lattice's part of the buffer
    double *mine = part + t.label_off[i] * 3 + (int64_t)split * values;
    __syncthreads();
    if (AUTO) {
        double *to = splits == 1 ? out + (int64_t)i * values : mine;
        for (int q = tid; q < values; q += kStatThreads) to[q] = lag_sums[q];
    } else {
        constexpr int kWaves = kStatThreads / 64;
        double *red = reinterpret_cast<double *>(lds);
#pragma unroll
        for (int q = 0; q < kSums; ++q) {
            const double v = lane_sum(sums[q], 6);
            if ((tid & 63) == 0) red[q * kWaves + (tid >> 6)] = v;
        }
        __syncthreads();
        if (tid < kSums) {
            double v = 0.0;
            for (int w = 0; w < kWaves; ++w) v = v + red[tid * kWaves + w];
            red[tid * kWaves] = v;
            if (splits > 1) mine[tid] = v;
        }
        __syncthreads();
        if (tid == 0 && splits == 1) {
            double r[kSums];
            for (int q = 0; q < kSums; ++q) r[q] = red[q * kWaves];
            write_moments(r, out + 8 * (int64_t)i);
        }
    }
}

// The sums of lattices that took several workgroups, added in their order.
template <bool AUTO>
__global__ void __launch_bounds__(256) finish_stats_kernel(const StatsTables t, int m, int lc, const double *part, double *out)
{
    const int i = blockIdx.x, tid = threadIdx.x;
    const int values = AUTO ? 2 * m : kSums;
    const int splits = stat_splits(t.label_off[i + 1] - t.label_off[i], lc, values);
    if (splits == 1) return;
    const double *p = part + t.label_off[i] * 3;
    if (AUTO) {
        for (int q = tid; q < values; q += 256) {
            double v = 0.0;
            for (int w = 0; w < splits; ++w) v = v + p[(int64_t)w * values + q];
            out[(int64_t)i * values + q] = v;
        }
    } else {
        __shared__ double r[kSums];
        if (tid < kSums) {
            double v = 0.0;
            for (int w = 0; w < splits; ++w) v = v + p[(int64_t)w * values + tid];
            r[tid] = v;
        }
        __syncthreads();
        if (tid == 0) write_moments(r, out + 8 * (int64_t)i);
    }
}

// Cells per chunk (log2) and LDS bytes of the staged kernel, lc < 0 when one
// cell's steps do not fit the LDS (over 4,000 samples): the general kernel
// then.  Chunks of 64 cells (a wave per lag group) as long as two workgroups
// share a CU, else the largest that fits.
template <bool AUTO>
int stat_chunk(int ndim, int m, size_t &bytes)
{
    for (int pass = 0; pass < 2; ++pass)
        for (int lc = 6; lc >= (pass == 0 ? 4 : 0); --lc) {
            bytes = std::max<size_t>((stat_cell_bytes(AUTO, ndim, m) << lc) + 16 + (AUTO ? (size_t)m * 16 : 0),
                                     kSums * (kStatThreads / 64) * sizeof(double));
            if (bytes <= (pass == 0 ? kStatLds / 2 + 6144 : kStatLds)) return lc;
        }
    return -1;
}

template <int D, bool AUTO>
hipError_t launch_staged(const StatsTables &t, const double *samples, int n_samples, double interval, int lc, size_t lds,
                         double *out, hipStream_t stream)
{
    const int m = n_samples - 1;
    const int splits = stat_splits(t.max_labels, lc, AUTO ? 2 * m : kSums);
    if (lds > 65536) {  // (always the same value: other threads may launch with other sizes)
        const hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void *>(&staged_stats_kernel<D, AUTO>),
                                                 hipFuncAttributeMaxDynamicSharedMemorySize, (int)kStatLds);
        if (e != hipSuccess) return e;
    }
    staged_stats_kernel<D, AUTO><<<(unsigned)t.n * (unsigned)splits, kStatThreads, lds, stream>>>(
        t, samples, n_samples, interval, lc, splits, t.part, out);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess || splits == 1) return e;
    finish_stats_kernel<AUTO><<<t.n, 256, 0, stream>>>(t, m, lc, t.part, out);
    return hipGetLastError();
}

}  // namespace

hipError_t launch_autocorrelation(const StatsTables &t, const double *samples, int n_samples, double *out,
                                  hipStream_t stream)
{
    size_t lds = 0;
    const int lc = stat_chunk<true>(t.ndim, n_samples - 1, lds);
    if (lc >= 0)
        return t.ndim == 2 ? launch_staged<2, true>(t, samples, n_samples, 1.0, lc, lds, out, stream)
                           : launch_staged<3, true>(t, samples, n_samples, 1.0, lc, lds, out, stream);
    autocorr_kernel<<<t.n, 256, 0, stream>>>(t, samples, n_samples, out);
    return hipGetLastError();
}

hipError_t launch_sample(const StatsTables &t, const int32_t *vol, const int32_t *surf, const int64_t *csum,
                         double *samples, int k, int n_samples, hipStream_t stream)
{
    const int64_t total = t.total_labels;
    sample_kernel<<<(unsigned)((total + 255) / 256), 256, 0, stream>>>(t, vol, surf, csum, samples, k, n_samples);
    return hipGetLastError();
}

hipError_t launch_summary(const StatsTables &t, const double *samples, int n_samples, double interval, double *out,
                          hipStream_t stream)
{
    size_t lds = 0;
    const int lc = stat_chunk<false>(t.ndim, n_samples - 1, lds);
    if (lc >= 0)
        return t.ndim == 2 ? launch_staged<2, false>(t, samples, n_samples, interval, lc, lds, out, stream)
                           : launch_staged<3, false>(t, samples, n_samples, interval, lc, lds, out, stream);
    summary_kernel<<<t.n, 256, 0, stream>>>(t, samples, n_samples, interval, out);
    return hipGetLastError();
}

}  // namespace cpm
