// HIP kernels around the sweep: counting volumes / surfaces from the lattice,
// centroid sums, activity decay, fills and counter copies.
#include <algorithm>
#include <type_traits>

#include "cpm_device.hpp"

namespace cpm {
namespace {

// Reductions over the cells of a lattice.  A workgroup takes a brick of it, a
// thread kRun consecutive sites of one row, and adds once per run of one label
// to a label map in LDS, which is flushed with one global atomic per label
// and sum.  A label that finds no free slot within kProbe probes goes straight
// to global memory.  Bricks rather than row strips keep the workgroups that
// see one cell, and so the global atomics per cell, few.
//
//   kCount     volumes and surfaces, from the int32 labels; with `ref` also
//              each cell's lowest site index
//   kRef       the lowest site index alone
//   kCentroid  coordinate sums, each site as its periodic image nearest to
//              the cell's site of lowest index
//
// The counts are bound by instruction issue (two per compared pair, 27 pairs a
// site in 3D).  With a map access per site, the neighbours' indices wrapped
// one by one and a pass of its own for the lowest sites, 256^3 took 143 + 27
// us and its centroids 59; now 82 and 35.  512 2D lattices of 51.6 million
// sites in all: 517 + 118 + 252 us, now 192 + 116.
constexpr int kMapSize = 512;
constexpr int kProbe = 32;
constexpr int kRun = 16;

// Threads of a brick: kTX along x (kRun sites each), kY rows, kZ planes.
template <int D>
struct ReduceBrick {
    static constexpr int kTX = D == 3 ? 1 : 4;
    static constexpr int kY = D == 3 ? 16 : 64;
    static constexpr int kZ = D == 3 ? 16 : 1;
    static constexpr int kX = kTX * kRun;
    static_assert(kTX * kY * kZ == kBlock, "one thread per brick row segment");
};

template <int D>
__host__ __device__ inline int64_t reduce_bricks(const int *L)
{
    using B = ReduceBrick<D>;
    return (int64_t)((L[0] + B::kX - 1) / B::kX) * ((L[1] + B::kY - 1) / B::kY) * ((L[2] + B::kZ - 1) / B::kZ);
}

enum ReduceMode { kCount = 0, kRef = 1, kCentroid = 2 };

template <int MODE>
struct LabelMap {
    int32_t key[kMapSize];
    int32_t v[MODE == kCount ? kMapSize : 1], s[MODE == kCount ? kMapSize : 1];
    int32_t low[MODE == kCentroid ? 1 : kMapSize];                        // lowest site index
    unsigned long long c[MODE == kCentroid ? 3 : 1][MODE == kCentroid ? kMapSize : 1];
};

template <int MODE>
__device__ __forceinline__ int map_slot(LabelMap<MODE> &m, int label)
{
    uint32_t h = ((uint32_t)label * 2654435761u) >> 23;
    static_assert(kMapSize == 1 << 9, "the hash is the product's upper 9 bits");
    for (int p = 0; p < kProbe; ++p) {
        const int k = atomicCAS(&m.key[h], -1, label);
        if (k == -1 || k == label) return (int)h;
        h = (h + 1) & (kMapSize - 1);
    }
    return -1;
}

// A label from an int32 lattice word: the label itself, or a packed word.
template <int WORDS>
__device__ __forceinline__ int word_label(int32_t v)
{
    if (WORDS == kWordsPacked) return label_of((uint32_t)v);
    if (WORDS == kWordsPackedAct) return label_of((char32_t)(uint32_t)v);
    return v;
}

// The labels of the kRun consecutive sites from site i0 (n of them valid),
// vector loads where the run is whole and 16-byte aligned.
template <int WORDS>
__device__ __forceinline__ void load_run_labels(const SweepArgs &a, int64_t i0, int n, int *lab)
{
    static_assert(kRun == 16, "vector loads below assume 16 sites per thread");
    if (WORDS == kWords16) {
        const uint16_t *src = reinterpret_cast<const uint16_t *>(a.cells) + i0;
        if (n == kRun && (reinterpret_cast<uintptr_t>(src) & 15) == 0) {
            const uint4 v[2] = {reinterpret_cast<const uint4 *>(src)[0], reinterpret_cast<const uint4 *>(src)[1]};
#pragma unroll
            for (int k = 0; k < 8; ++k) {
                const uint32_t w = (&v[k >> 2].x)[k & 3];
                lab[2 * k] = label_of((uint16_t)(w & 0xFFFFu));
                lab[2 * k + 1] = label_of((uint16_t)(w >> 16));
            }
        } else {
#pragma unroll
            for (int k = 0; k < kRun; ++k) lab[k] = k < n ? label_of(src[k]) : 0;
        }
    } else {
        const int32_t *src = a.lat + i0;
        if (n == kRun && (reinterpret_cast<uintptr_t>(src) & 15) == 0) {
#pragma unroll
            for (int k = 0; k < 4; ++k) {
                const int4 v = reinterpret_cast<const int4 *>(src)[k];
                lab[4 * k] = word_label<WORDS>(v.x);
                lab[4 * k + 1] = word_label<WORDS>(v.y);
                lab[4 * k + 2] = word_label<WORDS>(v.z);
                lab[4 * k + 3] = word_label<WORDS>(v.w);
            }
        } else {
#pragma unroll
            for (int k = 0; k < kRun; ++k) lab[k] = k < n ? word_label<WORDS>(src[k]) : 0;
        }
    }
}

// floor(n / d) for 0 <= n < 2^31 by the reciprocal of d in FP64, off by at
// most one before the correction.
__device__ __forceinline__ int div_index(int n, int d, double inv)
{
    const int q = (int)((double)n * inv), r = n - q * d;
    return r < 0 ? q - 1 : r >= d ? q + 1 : q;
}

// p - r as the nearest periodic image on an axis of length L.
__device__ __forceinline__ int nearest_image(int diff, int L)
{
    if (diff > L / 2) diff -= L;
    if (diff < -(L - 1) / 2) diff += L;
    return diff;
}

// One workgroup's share of a reduction over lattice a: brick `block`, read
// from its int32 labels, its 16-bit working copy or its packed words (WORDS).
template <int D, int MODE, int WORDS = kWords32>
__device__ __forceinline__ void reduce_block(const SweepArgs &a, int64_t block, int32_t *v_out, int32_t *s_out,
                                             int stride, int32_t *ref, int64_t *cent)
{
    __shared__ LabelMap<MODE> m;
    const int tid = threadIdx.x;
    for (int i = tid; i < kMapSize; i += kBlock) {
        m.key[i] = -1;
        if (MODE == kCount) m.v[i] = m.s[i] = 0;
        if (MODE != kCentroid) m.low[i] = INT32_MAX;
        else m.c[0][i] = m.c[1][i] = m.c[2][i] = 0;
    }
    __syncthreads();
    const int L0 = a.L[0], L1 = a.L[1], L2 = a.L[2];
    using B = ReduceBrick<D>;
    const int nbx = (L0 + B::kX - 1) / B::kX, nby = (L1 + B::kY - 1) / B::kY;
    const int bx = (int)(block % nbx), by = (int)((block / nbx) % nby), bz = (int)(block / ((int64_t)nbx * nby));
    const int tx = tid % B::kTX, ty = (tid / B::kTX) % B::kY, tz = tid / (B::kTX * B::kY);
    const int x = bx * B::kX + tx * kRun, y = by * B::kY + ty, z = bz * B::kZ + tz;
    // 3D counts: the brick's labels with their neighbours, in LDS.  A row's
    // 16 labels straight from global memory cost a lane a cache line of its
    // own for each of nine rows: 241 us for 256^3.
    constexpr int kBoxX = kRun + 2, kBoxY = B::kY + 2, kBoxZ = B::kZ + 2;
    constexpr bool BOX = D == 3 && MODE == kCount;
    __shared__ int32_t box[BOX ? kBoxX * kBoxY * kBoxZ : 1];
    __shared__ struct {
        int32_t lab[BOX ? 1 : kRun][kBlock];
        uint16_t unlike[MODE == kCount ? kRun : 1][kBlock];
    } runs;
    if (BOX) {
        const int x0 = bx * B::kX, y0 = by * B::kY - 1, z0 = bz * B::kZ - 1;
        const bool vec = x0 + kRun <= L0 && L0 % 4 == 0 && (reinterpret_cast<uintptr_t>(a.lat) & 15) == 0;
        auto row_of = [&](int r) {  // rows past the lattice's end are never used
            const int ry = r % kBoxY, rz = r / kBoxY;
            const int gy = y0 + ry < 0 ? L1 - 1 : (y0 + ry) % L1, gz = z0 + rz < 0 ? L2 - 1 : (z0 + rz) % L2;
            return (gz * L1 + gy) * L0;
        };
        if (vec) {
            // per row four vectors and the two labels beside them
            for (int i = tid; i < 6 * kBoxY * kBoxZ; i += kBlock) {
                const int r = i / 6, k = i - 6 * r, row = row_of(r);
                int32_t *d = box + r * kBoxX;
                if (k < 4) {
                    const int4 v = *reinterpret_cast<const int4 *>(a.lat + row + x0 + 4 * k);
                    d[4 * k + 1] = v.x;
                    d[4 * k + 2] = v.y;
                    d[4 * k + 3] = v.z;
                    d[4 * k + 4] = v.w;
                } else if (k == 4) {
                    d[0] = a.lat[row + (x0 > 0 ? x0 - 1 : L0 - 1)];
                } else {
                    d[kRun + 1] = a.lat[row + (x0 + kRun < L0 ? x0 + kRun : 0)];
                }
            }
        } else {
            for (int i = tid; i < kBoxX * kBoxY * kBoxZ; i += kBlock) {
                const int r = i / kBoxX, gx = x0 - 1 + i - r * kBoxX;
                box[i] = a.lat[row_of(r) + (gx < 0 ? L0 - 1 : gx % L0)];
            }
        }
        __syncthreads();
    }
    if (x < L0 && y < L1 && z < L2) {
        const int n = min(kRun, L0 - x);
        const int first = (z * L1 + y) * L0 + x;  // lattices hold fewer than 2^31 sites
        int lab[kRun];
        if (BOX) {
#pragma unroll
            for (int j = 0; j < kRun; ++j) lab[j] = box[((tz + 1) * kBoxY + ty + 1) * kBoxX + 1 + j];
        } else {
            load_run_labels<WORDS>(a, first, n, lab);
        }
        if (n < kRun) {
#pragma unroll
            for (int j = 0; j < kRun; ++j)
                if (j >= n) lab[j] = 0;  // past the row's end: medium
        }
        bool any = false;
#pragma unroll
        for (int j = 0; j < kRun; ++j) any |= lab[j] > 0;
        int cnt[kRun];  // kCount: unlike neighbours
        if (MODE == kCount && any) {
#pragma unroll
            for (int j = 0; j < kRun; ++j) cnt[j] = 0;
            const int xm = x > 0 ? x - 1 : L0 - 1, xp = x + n < L0 ? x + n : 0;
            auto compare = [&](const int *u) {  // (a site never differs from itself)
#pragma unroll
                for (int j = 0; j < kRun; ++j) cnt[j] += (u[j] != lab[j]) + (u[j + 1] != lab[j]) + (u[j + 2] != lab[j]);
            };
            if (D == 3) {
#pragma unroll 1
                for (int dz = 0; dz < 3; ++dz)
#pragma unroll
                    for (int dy = 0; dy < 3; ++dy) compare(box + ((tz + dz) * kBoxY + ty + dy) * kBoxX);
            } else {
                int u[3][kRun + 2];
#pragma unroll
                for (int r = 0; r < 3; ++r) {  // all loads before the first use
                    const int row = wrap_once(y + r - 1, L1) * L0;
                    load_run_labels<WORDS>(a, (int64_t)row + x, n, u[r] + 1);
                    u[r][0] = a.lat[row + xm];
                    u[r][kRun + 1] = a.lat[row + xp];
                }
#pragma unroll
                for (int r = 0; r < 3; ++r) {
                    if (n < kRun) {
#pragma unroll
                        for (int j = 0; j < kRun; ++j)
                            if (j == n) u[r][j + 1] = u[r][kRun + 1];
                    }
                    compare(u[r]);
                }
            }
        }
        if (any) {
            // the runs, one after another: as many rounds per wave as its
            // busiest thread has runs, their labels and sums by index from LDS
            uint32_t starts = 0, ends = 0;
            int sum = 0;
#pragma unroll
            for (int j = 0; j < kRun; ++j) {
                if (!BOX) runs.lab[j][tid] = lab[j];
                if (MODE == kCount) {
                    sum += cnt[j];
                    runs.unlike[j][tid] = (uint16_t)sum;  // of the run's sites up to j, and before it
                }
                starts |= (uint32_t)(lab[j] > 0 && (j == 0 || lab[j] != lab[j > 0 ? j - 1 : 0])) << j;
                ends |= (uint32_t)(lab[j] > 0 && (j == kRun - 1 || lab[j] != lab[j < kRun - 1 ? j + 1 : j])) << j;
            }
            const double inv0 = 1.0 / (double)L0, inv1 = 1.0 / (double)L1;
            while (ends) {
                const int s = __ffs(starts) - 1, e = __ffs(ends) - 1, len = e - s + 1;
                starts &= starts - 1;
                ends &= ends - 1;
                const int c = BOX ? box[((tz + 1) * kBoxY + ty + 1) * kBoxX + 1 + e] : runs.lab[e][tid];
                const int slot = map_slot(m, c);
                if (MODE == kCount) {
                    const int unlike = runs.unlike[e][tid] - (s > 0 ? (int)runs.unlike[s > 0 ? s - 1 : 0][tid] : 0);
                    if (slot >= 0) {
                        atomicAdd(&m.v[slot], len);
                        atomicAdd(&m.s[slot], unlike);
                    } else {
                        atomicAdd(&v_out[(size_t)c * stride], len);
                        atomicAdd(&s_out[(size_t)c * stride], unlike);
                    }
                }
                if (MODE == kRef || (MODE == kCount && ref)) {
                    if (slot >= 0) atomicMin(&m.low[slot], first + s);
                    else atomicMin(&ref[c], first + s);
                }
                if (MODE == kCentroid) {
                    const int r0 = ref[c], q = div_index(r0, L0, inv0), rx = r0 - q * L0;
                    const int rz = D == 3 ? div_index(q, L1, inv1) : 0, ry = q - rz * L1;
                    // the images along the run are consecutive, unless the far
                    // side of the lattice lies within it
                    const int i0 = nearest_image(x + s - rx, L0), i1 = nearest_image(x + e - rx, L0);
                    int64_t sx = (int64_t)len * i0 + len * (len - 1) / 2;
                    if (i1 != i0 + len - 1) {
                        sx = 0;
                        for (int j = s; j <= e; ++j) sx += nearest_image(x + j - rx, L0);
                    }
                    const int64_t d[3] = {(int64_t)len * rx + sx, (int64_t)len * (ry + nearest_image(y - ry, L1)),
                                          (int64_t)len * (rz + nearest_image(z - rz, L2))};
#pragma unroll
                    for (int k = 0; k < D; ++k) {
                        if (slot >= 0) atomicAdd(&m.c[k][slot], (unsigned long long)d[k]);
                        else atomicAdd(reinterpret_cast<unsigned long long *>(&cent[(size_t)c * D + k]), (unsigned long long)d[k]);
                    }
                }
            }
        }
    }
    __syncthreads();
    for (int h = tid; h < kMapSize; h += kBlock) {
        const int c = m.key[h];
        if (c < 0) continue;
        if (MODE == kCount) {
            atomicAdd(&v_out[(size_t)c * stride], m.v[h]);
            atomicAdd(&s_out[(size_t)c * stride], m.s[h]);
        }
        if (MODE == kRef || (MODE == kCount && ref)) atomicMin(&ref[c], m.low[h]);
        if (MODE == kCentroid) {
#pragma unroll
            for (int d = 0; d < D; ++d)
                atomicAdd(reinterpret_cast<unsigned long long *>(&cent[(size_t)c * D + d]), m.c[d][h]);
        }
    }
}

template <int D, int MODE, int WORDS = kWords32>
__global__ void __launch_bounds__(kBlock) reduce_kernel(SweepArgs a, int32_t *v_out, int32_t *s_out, int stride,
                                                        int32_t *ref, int64_t *cent)
{
    static_assert(WORDS == kWords32 || MODE != kCount, "counts read the int32 labels");
    reduce_block<D, MODE, WORDS>(a, blockIdx.x, v_out, s_out, stride, ref, cent);
}

// Every lattice of a batch in one launch: blockIdx.y is the lattice, outputs
// are packed per label (label_off) as in the batch's per-cell arrays.
template <int D, int MODE>
__global__ void __launch_bounds__(kBlock) batch_reduce_kernel(const SweepArgs *args, const int64_t *label_off,
                                                              int32_t *v_out, int32_t *s_out, int32_t *ref,
                                                              int64_t *cent)
{
    const SweepArgs &a = args[blockIdx.y];
    if (blockIdx.x >= reduce_bricks<D>(a.L)) return;  // uniform over the block
    const int64_t o = label_off[blockIdx.y];
    reduce_block<D, MODE>(a, blockIdx.x, v_out ? v_out + o : nullptr, s_out ? s_out + o : nullptr, 1,
                          ref ? ref + o : nullptr, cent ? cent + o * D : nullptr);
}

// The reductions' outputs before they are added to: sums 0 (volumes and
// surfaces, n labels each; n_cent words of centroid sums), lowest sites none.
__global__ void clear_stats_kernel(int32_t *v, int32_t *s, int32_t *ref, size_t n, int64_t *cent, size_t n_cent)
{
    const size_t i = (size_t)blockIdx.x * kBlock + threadIdx.x;
    if (i < n) {
        if (v) v[i] = 0;
        if (s) s[i] = 0;
        if (ref) ref[i] = INT32_MAX;
    }
    if (cent && i < n_cent) cent[i] = 0;
}

// Ordered Moore pairs (x, y) of different labels, neither an obstacle, counted
// by (type of x, type of y); the medium is type 0.  Each unordered pair is met
// once, from the site whose neighbour lies ahead in x, y or z, and counted
// both ways at the end.  A thread compares the kRun sites of its brick row
// with the rows ahead; the few pairs that differ go to a queue of the wave,
// which looks up their types 64 at a time: looked up where found, one lane
// in twenty at a time, they took 69 us at 2048^2, now 25.
template <int D>
__global__ void __launch_bounds__(kBlock) contact_kernel(SweepArgs a, unsigned long long *out, int n_types)
{
    constexpr int kBins = kMaxTypes * kMaxTypes, kCopies = 16, kQueued = 128;
    __shared__ uint32_t hist[kCopies][kBins];  // by lane, to spread the updates of one bin
    __shared__ int2 queue[kBlock / 64][kQueued];
    const int tid = threadIdx.x, lane = tid & 63;
    for (int i = tid; i < kCopies * kBins; i += kBlock) (&hist[0][0])[i] = 0;
    __syncthreads();
    using B = ReduceBrick<D>;
    const int L0 = a.L[0], L1 = a.L[1], L2 = a.L[2];
    const int nbx = (L0 + B::kX - 1) / B::kX, nby = (L1 + B::kY - 1) / B::kY;
    const int bx = (int)(blockIdx.x % nbx), by = (int)((blockIdx.x / nbx) % nby), bz = (int)(blockIdx.x / ((int64_t)nbx * nby));
    const int x = bx * B::kX + tid % B::kTX * kRun, y = by * B::kY + (tid / B::kTX) % B::kY, z = bz * B::kZ + tid / (B::kTX * B::kY);
    const bool in = x < L0 && y < L1 && z < L2;
    const int n = in ? min(kRun, L0 - x) : 0;
    const int xm = x > 0 ? x - 1 : L0 - 1, xp = x + n < L0 ? x + n : 0;
    int2 *q = queue[tid >> 6];
    int queued = 0;  // of the wave
    auto count = [&](int first, int entries) {
        if (lane < entries) {
            const int2 e = q[first + lane];
            const int tx = e.x == 0 ? 0 : a.cell_type[e.x], ty = e.y == 0 ? 0 : a.cell_type[e.y];
            atomicAdd(&hist[lane % kCopies][tx * kMaxTypes + ty], 1u);
        }
    };
    auto pair = [&](bool valid, int c, int u) {
        const bool differ = valid && c != u && c >= 0 && u >= 0;
        const uint64_t mask = __ballot(differ);
        if (mask == 0) return;
        if (differ)
            q[queued + (int)__builtin_amdgcn_mbcnt_hi((uint32_t)(mask >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)mask, 0u))] =
                make_int2(c, u);
        queued += (int)__popcll(mask);
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
        if (queued >= 64) {
            queued -= 64;
            count(queued, 64);
            __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
        }
    };
    int lab[kRun + 1];
    auto load_row = [&](int row, int *u) {  // n labels from x, and the one beyond them
        load_run_labels<kWords32>(a, (int64_t)row + x, n, u);
        u[kRun] = a.lat[row + xp];
        if (n < kRun) {
#pragma unroll
            for (int j = 0; j < kRun; ++j)
                if (j == n) u[j] = u[kRun];
        }
    };
    if (in) load_row((z * L1 + y) * L0, lab);
#pragma unroll
    for (int j = 0; j < kRun; ++j) pair(j < n, lab[j], lab[j + 1]);
    // the rows ahead: y + 1, and in 3D the three rows of z + 1
#pragma unroll 1
    for (int r = 0; r < (D == 3 ? 4 : 1); ++r) {
        int u[kRun + 1], before = 0;
        if (in) {
            const int gy = wrap_once(r == 0 ? y + 1 : y + r - 2, L1), gz = r == 0 ? z : wrap_once(z + 1, L2);
            const int row = (gz * L1 + gy) * L0;
            before = a.lat[row + xm];
            load_row(row, u);
        }
#pragma unroll
        for (int j = 0; j < kRun; ++j) {
            pair(j < n, lab[j], j > 0 ? u[j > 0 ? j - 1 : 0] : before);
            pair(j < n, lab[j], u[j]);
            pair(j < n, lab[j], u[j + 1]);
        }
    }
    count(0, queued);
    __syncthreads();
    for (int b = tid; b < kBins; b += kBlock) {
        const int ta = b / kMaxTypes, tb = b % kMaxTypes;
        if (ta >= n_types || tb >= n_types) continue;
        unsigned long long v = 0;
        for (int w = 0; w < kCopies; ++w) v += (unsigned long long)hist[w][b] + hist[w][tb * kMaxTypes + ta];
        if (v) atomicAdd(&out[ta * n_types + tb], v);
    }
}

// floor(sqrt(n)) for 0 <= n < 2^62; the FP64 root is only a first guess
__device__ __forceinline__ int64_t isqrt_floor(int64_t n)
{
    if (n <= 0) return 0;
    int64_t r = (int64_t)sqrt((double)n);
    while (r > 0 && r * r > n) --r;
    while ((r + 1) * (r + 1) <= n) ++r;
    return r;
}

__device__ __forceinline__ int64_t div_floor(int64_t a, int64_t b)  // b > 0
{
    const int64_t q = a / b;
    return (a % b != 0 && a < 0) ? q - 1 : q;
}

// One thread per label (label 0 untouched).  t == 0: initialise; t >= 1:
// update number t, writing history slot t mod slots and reading slot
// (t + 1) mod slots (the centroid of update t - dt, or the initial one).
__global__ void persist_kernel(PersistArgs p, int64_t t)
{
    const int c = blockIdx.x * blockDim.x + threadIdx.x;
    if (c < 1 || c >= p.n_labels) return;
    const int64_t v = p.pairs[2 * c];
    int64_t X[3] = {0, 0, 0};
    for (int d = 0; d < p.ndim; ++d)
        if (v > 0) X[d] = div_floor(p.csum[(int64_t)c * p.ndim + d] * 65536, v);
    int64_t *h = p.hist + (int64_t)c * p.slots * 3;
    // the sweeps unwrap an accepted copy's site to the image nearest this
    // point (the centroid rounded to a site), in the frame of the sums
    if (v > 0) {
        int r[3] = {0, 0, 0};
        for (int d = 0; d < p.ndim; ++d) r[d] = (int)div_floor(X[d] + 32768, 65536);
        p.cpos[c] = make_int4(r[0], r[1], r[2], 0);
    }
    if (t == 0) {
        for (int k = 0; k < p.slots; ++k)
            for (int d = 0; d < 3; ++d) h[3 * k + d] = X[d];
        p.pdir[c] = make_int4(0, 0, 0, 0);
        return;
    }
    if (v == 0) {
        p.pdir[c] = make_int4(0, 0, 0, 0);
        return;
    }
    const int64_t *old = h + 3 * ((t + 1) % p.slots);
    int64_t D[3];
    for (int d = 0; d < 3; ++d) {
        const int64_t W = (int64_t)p.L[d] * 65536;
        int64_t w = (X[d] - old[d]) % W;
        if (w < 0) w += W;
        if (w >= W / 2) w -= W;
        D[d] = d < p.ndim ? w : 0;
    }
    int64_t *slot = h + 3 * (t % p.slots);
    for (int d = 0; d < 3; ++d) slot[d] = X[d];
    const int64_t nd = isqrt_floor(D[0] * D[0] + D[1] * D[1] + D[2] * D[2]);
    const int4 prev = p.pdir[c];
    const int64_t pp[3] = {prev.x, prev.y, prev.z};
    const int64_t mu = p.model->mu_p[p.cell_type[c]];
    int64_t q[3];
    for (int d = 0; d < 3; ++d) {
        const int64_t u = nd > 0 ? (D[d] * 16384) / nd : 0;
        q[d] = (16384 - mu) * u + mu * pp[d];
    }
    const int64_t np = isqrt_floor(q[0] * q[0] + q[1] * q[1] + q[2] * q[2]);
    p.pdir[c] = np > 0 ? make_int4((int)((q[0] * 16384) / np), (int)((q[1] * 16384) / np),
                                   (int)((q[2] * 16384) / np), 0)
                       : make_int4(0, 0, 0, 0);
}

__global__ void fill_i32_kernel(int32_t *p, int32_t value, size_t n)
{
    const size_t i = (size_t)blockIdx.x * kBlock + threadIdx.x;
    if (i < n) p[i] = value;
}

__global__ void act_decay_kernel(uint8_t *act, size_t n)
{
    const size_t i = ((size_t)blockIdx.x * kBlock + threadIdx.x) * 16;
    if (i + 16 <= n && (reinterpret_cast<uintptr_t>(act) & 15) == 0) {
        uint4 v = *reinterpret_cast<const uint4 *>(act + i);
        uint32_t w[4] = {v.x, v.y, v.z, v.w};
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            // per-byte saturating decrement
            uint32_t x = w[e];
            uint32_t nz = ((x & 0x7F7F7F7Fu) + 0x7F7F7F7Fu | x) & 0x80808080u;  // 0x80 where byte != 0
            w[e] = x - (nz >> 7);
        }
        *reinterpret_cast<uint4 *>(act + i) = make_uint4(w[0], w[1], w[2], w[3]);
    } else {
        for (size_t j = i; j < i + 16 && j < n; ++j)
            if (act[j] > 0) act[j] = (uint8_t)(act[j] - 1);
    }
}

__global__ void copy_counters_kernel(const int32_t *pairs, int32_t n_labels, int32_t *v_out, int32_t *s_out)
{
    const int i = blockIdx.x * kBlock + threadIdx.x;
    if (i >= n_labels) return;
    v_out[i] = i == 0 ? 0 : pairs[2 * i];
    s_out[i] = i == 0 ? 0 : pairs[2 * i + 1];
}

// The same for every lattice of a batch (blockIdx.x), outputs packed per
// label: one launch (one per lattice cost 1.7 us each, 0.4 ms for 250).
__global__ void __launch_bounds__(kBlock) batch_copy_counters_kernel(const SweepArgs *args, const int64_t *label_off,
                                                                     int parity, int32_t *v_out, int32_t *s_out)
{
    const int64_t o = label_off[blockIdx.x], n = label_off[blockIdx.x + 1] - o;
    const int32_t *pairs = args[blockIdx.x].counters[parity];
    for (int64_t i = (int64_t)blockIdx.y * kBlock + threadIdx.x; i < n; i += (int64_t)gridDim.y * kBlock) {
        v_out[o + i] = i == 0 ? 0 : pairs[2 * i];
        s_out[o + i] = i == 0 ? 0 : pairs[2 * i + 1];
    }
}

// Sites whose label lies outside [-1, n_cells], or is an obstacle (-1) in a
// model without an obstacle type: counted into *bad (one atomic per wave).
__global__ void __launch_bounds__(kBlock) bad_label_kernel(const int32_t *lat, size_t n, int32_t n_cells,
                                                           int allow_obstacle, int32_t *bad)
{
    const int lo = allow_obstacle ? -1 : 0;
    int cnt = 0;
    for (size_t i = (size_t)blockIdx.x * kBlock + threadIdx.x; i < n; i += (size_t)gridDim.x * kBlock) {
        const int v = lat[i];
        cnt += v < lo || v > n_cells;
    }
    for (int off = 32; off > 0; off >>= 1) cnt += __shfl_xor(cnt, off);
    if ((threadIdx.x & 63) == 0 && cnt) atomicAdd(bad, cnt);
}

// Labels 1..n_labels-1 whose tracked (V, S) pair differs from the recount
// (v, s): counted into *bad.
__global__ void compare_counters_kernel(const int32_t *pairs, const int32_t *v, const int32_t *s, int32_t n_labels,
                                        int32_t *bad)
{
    const int i = blockIdx.x * kBlock + threadIdx.x;
    if (i < 1 || i >= n_labels) return;
    if (pairs[2 * i] != v[i] || pairs[2 * i + 1] != s[i]) atomicAdd(bad, 1);
}

__global__ void set_u32_kernel(uint32_t *p, uint32_t v) { *p = v; }
__global__ void add_u32_kernel(uint32_t *p, uint32_t v) { *p += v; }

inline unsigned blocks_for(size_t n) { return (unsigned)((n + kBlock - 1) / kBlock); }

}  // namespace

hipError_t launch_fill_i32(int32_t *p, int32_t value, size_t n, hipStream_t stream)
{
    if (n == 0) return hipSuccess;
    fill_i32_kernel<<<blocks_for(n), kBlock, 0, stream>>>(p, value, n);
    return hipGetLastError();
}

hipError_t launch_clear_stats(int32_t *v, int32_t *s, int32_t *ref, size_t n, int64_t *cent, int ndim, hipStream_t stream)
{
    clear_stats_kernel<<<blocks_for(cent ? n * ndim : n), kBlock, 0, stream>>>(v, s, ref, n, cent, n * ndim);
    return hipGetLastError();
}

hipError_t launch_count(const SweepArgs &a, int ndim, int32_t *v_out, int32_t *s_out, int stride, hipStream_t stream,
                        int32_t *ref)
{
    const unsigned grid = (unsigned)reduce_brick_count(a.L, ndim);
    if (ndim == 2)
        reduce_kernel<2, kCount><<<grid, kBlock, 0, stream>>>(a, v_out, s_out, stride, ref, nullptr);
    else
        reduce_kernel<3, kCount><<<grid, kBlock, 0, stream>>>(a, v_out, s_out, stride, ref, nullptr);
    return hipGetLastError();
}

hipError_t launch_contacts(const SweepArgs &a, int ndim, int n_types, int64_t *out, hipStream_t stream)
{
    hipError_t e = launch_fill_i32(reinterpret_cast<int32_t *>(out), 0, (size_t)n_types * n_types * 2, stream);
    if (e != hipSuccess) return e;
    const unsigned grid = (unsigned)reduce_brick_count(a.L, ndim);
    auto *o = reinterpret_cast<unsigned long long *>(out);
    if (ndim == 2) contact_kernel<2><<<grid, kBlock, 0, stream>>>(a, o, n_types);
    else contact_kernel<3><<<grid, kBlock, 0, stream>>>(a, o, n_types);
    return hipGetLastError();
}

hipError_t launch_persist(const PersistArgs &p, int64_t t, hipStream_t stream)
{
    persist_kernel<<<blocks_for((size_t)p.n_labels), kBlock, 0, stream>>>(p, t);
    return hipGetLastError();
}

hipError_t launch_act_decay(uint8_t *act, size_t n, hipStream_t stream)
{
    const size_t threads = (n + 15) / 16;
    act_decay_kernel<<<blocks_for(threads), kBlock, 0, stream>>>(act, n);
    return hipGetLastError();
}

hipError_t launch_centroids(const SweepArgs &a, int ndim, int32_t n_cells, int32_t *ref, int64_t *out,
                            hipStream_t stream, int words, bool have_ref)
{
    const unsigned grid = (unsigned)reduce_brick_count(a.L, ndim);
    if (!have_ref) {
        const hipError_t e = launch_clear_stats(nullptr, nullptr, ref, (size_t)n_cells + 1, out, ndim, stream);
        if (e != hipSuccess) return e;
    }
    auto run = [&](auto d_tag, auto w_tag) {
        constexpr int D = decltype(d_tag)::value, W = decltype(w_tag)::value;
        if (!have_ref) reduce_kernel<D, kRef, W><<<grid, kBlock, 0, stream>>>(a, nullptr, nullptr, 0, ref, nullptr);
        reduce_kernel<D, kCentroid, W><<<grid, kBlock, 0, stream>>>(a, nullptr, nullptr, 0, ref, out);
    };
    using D2 = std::integral_constant<int, 2>;
    using D3 = std::integral_constant<int, 3>;
    using W32 = std::integral_constant<int, kWords32>;
    using W16 = std::integral_constant<int, kWords16>;
    using WP = std::integral_constant<int, kWordsPacked>;
    using WPA = std::integral_constant<int, kWordsPackedAct>;
    if (ndim == 2) {
        if (words == kWords16) run(D2{}, W16{});
        else if (words == kWordsPacked) run(D2{}, WP{});
        else if (words == kWordsPackedAct) run(D2{}, WPA{});
        else run(D2{}, W32{});
    } else {
        if (words == kWords16) run(D3{}, W16{});
        else if (words == kWordsPacked) run(D3{}, WP{});
        else if (words == kWordsPackedAct) run(D3{}, WPA{});
        else run(D3{}, W32{});
    }
    return hipGetLastError();
}

namespace {
__global__ void copy_dirs_kernel(const int4 *pdir, int32_t n_labels, int32_t *out)
{
    const int i = blockIdx.x * kBlock + threadIdx.x;
    if (i >= n_labels) return;
    const int4 v = i == 0 ? make_int4(0, 0, 0, 0) : pdir[i];
    out[3 * i] = v.x;
    out[3 * i + 1] = v.y;
    out[3 * i + 2] = v.z;
}
}  // namespace

namespace {
// Four sites per thread, kOccLattices lattices per workgroup row: a thread per
// site over all lattices left most of the GPU idle (62 us for 250 lattices of
// 256^2, now 14).  Up to kOccOneRow lattices one row takes them all, and no
// launch clears the counts first (48 of 256^2 3.9 us against 4.0 in rows, 64
// 4.6 against 4.1, but the call's host side 9 us against 11.5).
constexpr int kOccLattices = 16;
constexpr int kOccOneRow = 64;
template <bool VEC>
__global__ void __launch_bounds__(kBlock) occupancy_kernel(const int32_t *lat, int n_lattices, int per_row, size_t n_sites,
                                                           int32_t *counts)
{
    const size_t i = ((size_t)blockIdx.x * kBlock + threadIdx.x) * 4;
    if (i >= n_sites) return;
    const int l0 = (int)blockIdx.y * per_row, l1 = min(n_lattices, l0 + per_row);
    int c[4] = {0, 0, 0, 0};
#pragma unroll 8
    for (int l = l0; l < l1; ++l) {
        const int32_t *p = lat + (size_t)l * n_sites + i;
        int4 v;
        if (VEC) v = *reinterpret_cast<const int4 *>(p);
        else v = make_int4(p[0], p[1], p[2], p[3]);
        c[0] += v.x > 0;
        c[1] += v.y > 0;
        c[2] += v.z > 0;
        c[3] += v.w > 0;
    }
    for (int k = 0; k < 4; ++k) {
        if (gridDim.y == 1) counts[i + k] = c[k];
        else if (c[k]) atomicAdd(&counts[i + k], c[k]);
    }
}
}  // namespace

hipError_t launch_occupancy(const int32_t *lattices, int n_lattices, size_t n_sites, int32_t *counts,
                            hipStream_t st)
{
    const int per_row = n_lattices <= kOccOneRow ? n_lattices : kOccLattices;
    const unsigned rows = (unsigned)((n_lattices + per_row - 1) / per_row);
    if (rows > 1) {  // rows add to the counts
        const hipError_t e = launch_fill_i32(counts, 0, n_sites, st);
        if (e != hipSuccess) return e;
    }
    // sides are even, so a lattice holds a multiple of four sites
    const dim3 grid(blocks_for(n_sites / 4), rows);
    if ((reinterpret_cast<uintptr_t>(lattices) & 15) == 0)
        occupancy_kernel<true><<<grid, kBlock, 0, st>>>(lattices, n_lattices, per_row, n_sites, counts);
    else
        occupancy_kernel<false><<<grid, kBlock, 0, st>>>(lattices, n_lattices, per_row, n_sites, counts);
    return hipGetLastError();
}

int64_t reduce_brick_count(const int *L, int ndim) { return ndim == 2 ? reduce_bricks<2>(L) : reduce_bricks<3>(L); }

hipError_t launch_copy_dirs(const int4 *pdir, int32_t n_labels, int32_t *out, hipStream_t stream)
{
    copy_dirs_kernel<<<blocks_for((size_t)n_labels), kBlock, 0, stream>>>(pdir, n_labels, out);
    return hipGetLastError();
}

hipError_t launch_batch_cell_stats(const SweepArgs *d_args, const int64_t *d_label_off, int n_lattices, int ndim,
                                   int64_t max_bricks, size_t total_labels, int32_t *v_out, int32_t *s_out, int32_t *ref,
                                   int64_t *cent, hipStream_t stream)
{
    const dim3 grid((unsigned)max_bricks, (unsigned)n_lattices);
    if (!cent) ref = nullptr;  // the lowest sites are the centroids' references
    const hipError_t e = launch_clear_stats(v_out, s_out, ref, total_labels, cent, ndim, stream);
    if (e != hipSuccess) return e;
    if (ndim == 2) {
        batch_reduce_kernel<2, kCount><<<grid, kBlock, 0, stream>>>(d_args, d_label_off, v_out, s_out, ref, nullptr);
        if (cent) batch_reduce_kernel<2, kCentroid><<<grid, kBlock, 0, stream>>>(d_args, d_label_off, nullptr, nullptr, ref, cent);
    } else {
        batch_reduce_kernel<3, kCount><<<grid, kBlock, 0, stream>>>(d_args, d_label_off, v_out, s_out, ref, nullptr);
        if (cent) batch_reduce_kernel<3, kCentroid><<<grid, kBlock, 0, stream>>>(d_args, d_label_off, nullptr, nullptr, ref, cent);
    }
    return hipGetLastError();
}

hipError_t launch_copy_counters(const int32_t *pairs, int32_t n_labels, int32_t *v_out, int32_t *s_out,
                                hipStream_t stream)
{
    copy_counters_kernel<<<blocks_for((size_t)n_labels), kBlock, 0, stream>>>(pairs, n_labels, v_out, s_out);
    return hipGetLastError();
}

hipError_t launch_batch_copy_counters(const SweepArgs *d_args, const int64_t *d_label_off, int n_lattices,
                                      int64_t max_labels, int parity, int32_t *v_out, int32_t *s_out, hipStream_t stream)
{
    const unsigned per = (unsigned)std::min<int64_t>((max_labels + kBlock - 1) / kBlock, 64);
    batch_copy_counters_kernel<<<dim3((unsigned)n_lattices, per), kBlock, 0, stream>>>(d_args, d_label_off, parity, v_out,
                                                                                       s_out);
    return hipGetLastError();
}

hipError_t launch_bad_labels(const int32_t *lat, size_t n, int32_t n_cells, bool allow_obstacle, int32_t *bad,
                             hipStream_t stream)
{
    if (n == 0) return hipSuccess;
    const unsigned grid = std::min<unsigned>(blocks_for(n), 4096u);
    bad_label_kernel<<<grid, kBlock, 0, stream>>>(lat, n, n_cells, allow_obstacle ? 1 : 0, bad);
    return hipGetLastError();
}

hipError_t launch_compare_counters(const int32_t *pairs, const int32_t *v, const int32_t *s, int32_t n_labels,
                                   int32_t *bad, hipStream_t stream)
{
    compare_counters_kernel<<<blocks_for((size_t)n_labels), kBlock, 0, stream>>>(pairs, v, s, n_labels, bad);
    return hipGetLastError();
}

hipError_t launch_set_u32(uint32_t *p, uint32_t value, hipStream_t stream)
{
    set_u32_kernel<<<1, 1, 0, stream>>>(p, value);
    return hipGetLastError();
}

hipError_t launch_add_u32(uint32_t *p, uint32_t value, hipStream_t stream)
{
    add_u32_kernel<<<1, 1, 0, stream>>>(p, value);
    return hipGetLastError();
}

}  // namespace cpm
