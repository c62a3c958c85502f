// The serial CPM on the GPU (Methods, first paragraph): per MCS, N copy
// attempts at uniformly drawn targets, each seeing the lattice and the
// per-cell counters exactly as the attempt before it left them.  It is the
// reference the parallel scheme is compared with (Fig. 5, Fig. 6E), run for
// every lattice of a batch at once: one workgroup per lattice, attempts
// evaluated one after another.
//
// The workgroup's four waves draw kDraws attempts per lane at once
// (kRound in all) and read both labels of each: most attempts find two like
// labels (99% and more of those of single-cell and chemotaxis ensembles) and
// change nothing.  The others are taken in attempt order, wave after wave,
// found by ballot within a wave; an accepted one corrects, in registers, the
// labels of the drawn attempts that touch its target (those of later waves
// through a list in LDS), so each attempt sees exactly the lattice the one
// before it left.  The next round is drawn while this one's labels load.
// What bounds it is the latency of each attempt that is evaluated (its loads
// and table look-ups, the tables in LDS): 250 single-cell lattices of 200^2
// with the Act term took 23.6 ms per MCS one attempt at a time, 0.54 ms with
// one wave per lattice and the tables in global memory, 0.44 ms this way.
//
// Within an evaluated attempt the wave's lanes load in parallel: lanes 0..31
// the target's neighbourhood (lane l < |NB|: Moore neighbour l; lane 31: the
// target), lanes 32..63 the source's (lane 32 + l: its neighbour l; lane 63:
// the source).  Counts over neighbours are ballots, the sum of the Act term
// runs within a half-wave.  Every load of data the kernel writes (labels,
// activity, counters) has a lane-dependent address, so it is a vector load
// that sees the wave's earlier stores; lane 0 commits.
#include <algorithm>
#include <type_traits>

#include "cpm_device.hpp"

namespace cpm {
namespace {

constexpr int kDraws = 4;                   // attempts drawn per lane at once
constexpr int kWaves = 4;                   // waves per lattice: one per SIMD of a CU
constexpr int kRound = 64 * kDraws * kWaves;  // attempts of a round

// Sums of v over lanes 0..31 (into lane 31) and 32..63 (into lane 63): row
// prefix sums, then the lower row's total added to the upper one.
template <int CTRL, int ROWS>
__device__ __forceinline__ uint32_t add_dpp(uint32_t v)
{
    return v + (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, CTRL, ROWS, 0xF, false);
}
__device__ __forceinline__ uint32_t half_sums(uint32_t v)
{
    v = add_dpp<0x111, 0xF>(v);  // row_shr:1
    v = add_dpp<0x112, 0xF>(v);  // row_shr:2
    v = add_dpp<0x114, 0xF>(v);  // row_shr:4
    v = add_dpp<0x118, 0xF>(v);  // row_shr:8
    return add_dpp<0x142, 0xA>(v);  // row_bcast:15 into rows 1 and 3
}

__device__ __forceinline__ int lane_value(int v, int lane) { return __builtin_amdgcn_readlane(v, lane); }

// floor(n / d) for n < 2^31 by the reciprocal of d in FP64, off by at most
// one before the correction.
__device__ __forceinline__ int div_site(int n, int d, double inv)
{
    int q = (int)((double)n * inv);
    const int r = n - q * d;
    return r < 0 ? q - 1 : r >= d ? q + 1 : q;
}

// The tables an evaluated attempt reads, in LDS: acceptance, and the Act
// term's logarithms and exponentials.
struct AttemptTables {
    uint32_t ti[kMaxTI], tm[256], tl[256];
};
struct ActTables {
    uint32_t lg[256];  // ln(255) 2^24 < 2^27
    uint64_t eh[2048], em[256], el[256];
};

// The Metropolis decision of metropolis32, reading only the table entries
// it needs, after the branches on q: attempts here run one at a time and
// most decisions need no table, so an unconditional round of loads per
// attempt would add up.
__device__ __forceinline__ bool metropolis32_lazy(const AttemptTables &tb, int n_ti, int64_t q, uint32_t u)
{
    if (q <= 0) return true;
    const uint64_t h = (uint64_t)q >> 16;
    if (h >= (uint64_t)n_ti) return false;
    const uint64_t two32 = (uint64_t)1 << 32;
    const uint64_t ti = h == 0 ? two32 : (uint64_t)tb.ti[h];
    if ((q & 0xFFFF) == 0) return (uint64_t)u < ti;
    const int mm = (int)((q >> 8) & 255), ll = (int)(q & 255);
    const uint64_t tm = mm ? (uint64_t)tb.tm[mm] : two32, tl = ll ? (uint64_t)tb.tl[ll] : two32;
    return (uint64_t)u < __umul64hi(ti, tm * tl);  // tm * tl < 2^64 since (mm, ll) != (0, 0)
}

// exp_log24 from the tables in LDS.
__device__ __forceinline__ int64_t exp_log24(const ActTables &t, uint32_t ell)
{
    const uint64_t p1 = (t.eh[ell >> 16] * t.em[(ell >> 8) & 255]) >> 31;
    const uint64_t p2 = (p1 * t.el[ell & 255]) >> 30;
    return (int64_t)(p2 >> 8);
}

template <int D>
__device__ __forceinline__ int site_at(const int *L, int x, int y, int z)
{
    return wrap_once(x, L[0]) + L[0] * (wrap_once(y, L[1]) + L[1] * (D == 3 ? wrap_once(z, L[2]) : 0));
}

// One MCS of the serial CPM on lattice blockIdx.x (without the Act decay that
// ends it).  Counters are the exact (V, S) pairs of buffer `parity`.
template <typename Cell, int D, bool ACT>
__global__ void __launch_bounds__(64 * kWaves) serial_mcs_kernel(const SweepArgs *args, uint32_t mcs, int parity)
{
    constexpr int NNB = D == 2 ? 8 : 26;
    constexpr uint64_t kLow = 0xFFFFFFFFull;
    __shared__ AttemptTables tb;
    __shared__ typename std::conditional<ACT, ActTables, int>::type act_tables;
    // commits of the round: target site and label
    __shared__ int2 committed[kRound];
    __shared__ int n_committed;
    const SweepArgs &a = args[blockIdx.x];
    const DeviceModel *m = a.model;
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int half = lane >> 5, hl = lane & 31;
    const bool own = hl == 31, nb = hl < NNB, used = own || nb;
    const int L[3] = {a.L[0], a.L[1], a.L[2]};
    const uint32_t N = (uint32_t)L[0] * (uint32_t)L[1] * (uint32_t)L[2];
    const double inv0 = 1.0 / L[0], inv1 = 1.0 / L[1];
    // int32 labels: the caller's lattice itself (a batch may keep other words
    // for its parallel sweeps in a.cells)
    Cell *cells = std::is_same<Cell, int32_t>::value ? reinterpret_cast<Cell *>(a.lat) : reinterpret_cast<Cell *>(a.cells);
    int32_t *cnt = a.counters[parity];
    const int n_ti = m->n_ti;
    for (int i = threadIdx.x; i < n_ti; i += 64 * kWaves) tb.ti[i] = m->TI32[i];
    for (int i = threadIdx.x; i < 256; i += 64 * kWaves) {
        tb.tm[i] = m->TM32[i];
        tb.tl[i] = m->TL32[i];
    }
    if constexpr (ACT) {
        for (int i = threadIdx.x; i < 2048; i += 64 * kWaves) act_tables.eh[i] = m->EH[i];
        for (int i = threadIdx.x; i < 256; i += 64 * kWaves) {
            act_tables.lg[i] = (uint32_t)m->LG[i];
            act_tables.em[i] = m->EM[i];
            act_tables.el[i] = m->EL[i];
        }
    }
    if (threadIdx.x == 0) n_committed = 0;
    const int n_types = a.n_types, single = a.single_type, obstacle = a.obstacle_type;
    uint32_t n_nontrivial = 0, n_accepted = 0;
    // this lane's offset from the target (half 0) or the source
    const int n_of = nb ? hl : 0;
    const int ox = own ? 0 : nb_dx<D>(n_of), oy = own ? 0 : nb_dy<D>(n_of), oz = own ? 0 : nb_dz<D>(n_of);

    // one round's draws: attempt base + 256 wave + 64 d + lane
    struct Draws {
        int tx[kDraws], ty[kDraws], tz[kDraws], sel[kDraws], t[kDraws], src[kDraws];
        uint32_t u2[kDraws];
    };
    auto draw = [&](uint32_t base, Draws &r) {
#pragma unroll
        for (int d = 0; d < kDraws; ++d) {
            const uint32_t i = base + 64 * (kDraws * wave + d) + lane;
            const uint4 u = philox4x32_10(make_uint4(i, mcs, 0xFFFFFF00u, a.lattice_id), a.key0, a.key1);
            r.t[d] = (int)(((uint64_t)u.x * N) >> 32);
            const int q = div_site(r.t[d], L[0], inv0);
            r.tx[d] = r.t[d] - q * L[0];
            r.tz[d] = D == 3 ? div_site(q, L[1], inv1) : 0;
            r.ty[d] = q - r.tz[d] * L[1];
            r.sel[d] = (int)(((uint64_t)u.y * (uint32_t)NNB) >> 32);
            r.src[d] = site_at<D>(L, r.tx[d] + nb_dx<D>(r.sel[d]), r.ty[d] + nb_dy<D>(r.sel[d]), r.tz[d] + nb_dz<D>(r.sel[d]));
            r.u2[d] = u.z;
        }
    };
    Draws cur, next;
    draw(0, next);
    for (uint32_t base = 0; base < N; base += kRound) {
        cur = next;
        int (&tx)[kDraws] = cur.tx, (&ty)[kDraws] = cur.ty, (&tz)[kDraws] = cur.tz, (&sel)[kDraws] = cur.sel;
        int (&t)[kDraws] = cur.t, (&src)[kDraws] = cur.src;
        uint32_t (&u2)[kDraws] = cur.u2;
        int lt[kDraws], ls[kDraws];
        __syncthreads();  // the last round's commits are visible, its list read
#pragma unroll
        for (int d = 0; d < kDraws; ++d) {
            lt[d] = label_of(cells[t[d]]);
            ls[d] = label_of(cells[src[d]]);
        }
        if (base + kRound < N) draw(base + kRound, next);
#pragma unroll
        for (int d = 0; d < kDraws; ++d) {
            // past the last attempt: two like labels, at no site
            const bool in = base + 64 * (kDraws * wave + d) + lane < N;
            lt[d] = in ? lt[d] : 0;
            ls[d] = in ? ls[d] : 0;
            t[d] = in ? t[d] : -1;
            src[d] = in ? src[d] : -1;
        }
        // the waves' turns
        for (int turn = 0; turn < kWaves; ++turn) {
            // every wave has its labels; the turn before has committed
            __syncthreads();
            if (turn != wave) continue;
            int n_list = n_committed;
            for (int e = 0; e < n_list; ++e) {
                const int2 c = committed[e];
#pragma unroll
                for (int d = 0; d < kDraws; ++d) {
                    lt[d] = t[d] == c.x ? c.y : lt[d];
                    ls[d] = src[d] == c.x ? c.y : ls[d];
                }
            }
#pragma unroll
            for (int d = 0; d < kDraws; ++d) {
                uint64_t todo = __ballot(lt[d] != ls[d] && lt[d] >= 0 && ls[d] >= 0);
                while (todo) {
                    const int f = __ffsll((unsigned long long)todo) - 1;
                    ++n_nontrivial;
                    const int ct = lane_value(lt[d], f), cs = lane_value(ls[d], f);
                    const int px = lane_value(tx[d], f), py = lane_value(ty[d], f), pz = lane_value(tz[d], f);
                    const int nsel = lane_value(sel[d], f), tsite = lane_value(t[d], f), ssite = lane_value(src[d], f);
                    const int dx = nb_dx<D>(nsel), dy = nb_dy<D>(nsel), dz = nb_dz<D>(nsel);
                    // this lane's site: a neighbour of the target (half 0) or of
                    // the source; its label and activity, and both cells'
                    // counters (even lanes the target's), in one round of loads
                    const int site = site_at<D>(L, px + (half ? dx : 0) + ox, py + (half ? dy : 0) + oy,
                                                pz + (half ? dz : 0) + oz);
                    const int c_of = lane & 1 ? cs : ct;
                    const int lab = label_of(cells[site]);
                    const int2 pair = reinterpret_cast<const int2 *>(cnt)[c_of];
                    const uint32_t av = ACT ? a.act[site] : 0u;
                    int tu = lab == 0 ? 0 : lab < 0 ? obstacle : single;
                    int tt = ct == 0 ? 0 : single, ts = cs == 0 ? 0 : single;
                    if (single < 0) {
                        tu = lab > 0 ? a.cell_type[lab] : tu;
                        tt = ct == 0 ? 0 : a.cell_type[ct];
                        ts = cs == 0 ? 0 : a.cell_type[cs];
                    }
                    // neighbours of the target by label and type
                    const uint64_t b_old = __ballot(nb && lab == ct) & kLow, b_new = __ballot(nb && lab == cs) & kLow;
                    const uint64_t b_nb = (1ull << NNB) - 1;
                    int64_t q = 0;
                    for (int ty_ = 0; ty_ < n_types; ++ty_) {
                        const uint64_t b = __ballot(tu == ty_) & b_nb;
                        q += m->J[ts * kMaxTypes + ty_] * __popcll(b & ~b_new) - m->J[tt * kMaxTypes + ty_] * __popcll(b & ~b_old);
                    }
                    const int64_t k_old = __popcll(b_old), k_new = __popcll(b_new);
                    const int64_t dso = 2 * k_old - NNB, dsn = NNB - 2 * k_new;
                    const int vt = lane_value(pair.x, 0), st_ = lane_value(pair.y, 0);
                    const int vs = lane_value(pair.x, 1), ss = lane_value(pair.y, 1);
                    if (ct >= 1) {
                        q += m->lam_v[tt] * (1 - 2 * ((int64_t)vt - m->v_target[tt]));
                        q += m->lam_s[tt] * (2 * dso * ((int64_t)st_ - m->s_target[tt]) + dso * dso);
                    }
                    if (cs >= 1) {
                        q += m->lam_v[ts] * (2 * ((int64_t)vs - m->v_target[ts]) + 1);
                        q += m->lam_s[ts] * (2 * dsn * ((int64_t)ss - m->s_target[ts]) + dsn * dsn);
                    }
                    if constexpr (ACT) {
                        // geometric means over each half's own site and its
                        // neighbours of the same cell
                        const bool mine = used && lab == (half ? cs : ct);
                        const uint32_t sums = half_sums(mine ? act_tables.lg[av] : 0u);
                        const uint64_t b_mine = __ballot(mine), b_dead = __ballot(mine && av == 0);
                        const uint32_t sum_t = (uint32_t)lane_value((int)sums, 31), sum_s = (uint32_t)lane_value((int)sums, 63);
                        int64_t gt = 0, gs = 0;
                        if (ct > 0 && m->max_act[tt] > 0 && !(b_dead & kLow))
                            gt = exp_log24(act_tables, sum_t / (uint32_t)__popcll(b_mine & kLow));
                        if (cs > 0 && m->max_act[ts] > 0 && !(b_dead >> 32))
                            gs = exp_log24(act_tables, sum_s / (uint32_t)__popcll(b_mine >> 32));
                        const int64_t rt = ct >= 1 ? m->r_act[tt] : 0, rs = cs >= 1 ? m->r_act[ts] : 0;
                        q += (rt * gt - rs * gs) >> 16;
                    }
                    if (a.chem && cs >= 1) {
                        // offset target - source = -(dx, dy, dz)
                        const int o = (1 - dx) + 3 * (1 - dy) + 9 * (D == 3 ? 1 - dz : 1);
                        const int16_t *c = a.chem + (size_t)D * ssite;
                        int64_t dot = (int64_t)m->unit[o][0] * c[0] + (int64_t)m->unit[o][1] * c[1];
                        if (D == 3) dot += (int64_t)m->unit[o][2] * c[2];
                        q -= (m->lam_c[ts] * dot) >> 28;
                    }
                    if (metropolis32_lazy(tb, n_ti, q, (uint32_t)lane_value((int)u2[d], f))) {
                        ++n_accepted;
                        if (lane == 0) {
                            committed[n_list] = make_int2(tsite, cs);
                            cells[tsite] = stored_label<Cell>(cs);
                            if (ACT)
                                a.act[tsite] = (cs >= 1 && m->max_act[ts] > 0) ? (uint8_t)m->max_act[ts] : (uint8_t)0;
                            if (ct >= 1) reinterpret_cast<int2 *>(cnt)[ct] = make_int2(vt - 1, st_ + (int)dso);
                            if (cs >= 1) reinterpret_cast<int2 *>(cnt)[cs] = make_int2(vs + 1, ss + (int)dsn);
                        }
                        ++n_list;
                        // later loads see this commit, drawn attempts its label
                        __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "workgroup");
#pragma unroll
                        for (int e = 0; e < kDraws; ++e) {
                            if (e < d) continue;
                            lt[e] = t[e] == tsite ? cs : lt[e];
                            ls[e] = src[e] == tsite ? cs : ls[e];
                        }
                    }
                    const uint64_t later = f == 63 ? 0ull : ~0ull << (f + 1);
                    todo = __ballot(lt[d] != ls[d] && lt[d] >= 0 && ls[d] >= 0) & later;
                }
            }
            // the last wave empties the list for the next round
            if (lane == 0) n_committed = turn == kWaves - 1 ? 0 : n_list;
        }
    }
    if (lane == 0) {
        atomicAdd(reinterpret_cast<unsigned long long *>(&a.stats[0]), (unsigned long long)n_nontrivial);
        atomicAdd(reinterpret_cast<unsigned long long *>(&a.stats[1]), (unsigned long long)n_accepted);
    }
}

// After serial MCS, for every lattice of a batch: the other counter buffer
// and the pending delta lists as the next parallel activation expects them
// (exact counters, no deltas to re-add).
__global__ void __launch_bounds__(kBlock) after_serial_kernel(const SweepArgs *args, const int64_t *label_off, int parity)
{
    const SweepArgs &a = args[blockIdx.x];
    const int64_t n = 2 * (label_off[blockIdx.x + 1] - label_off[blockIdx.x]);
    const int32_t *from = a.counters[parity];
    int32_t *to = a.counters[parity ^ 1], *listed = a.dcount[parity ^ 1];
    const int64_t i0 = (int64_t)blockIdx.y * kBlock + threadIdx.x, step = (int64_t)gridDim.y * kBlock;
    for (int64_t i = i0; i < n; i += step) to[i] = from[i];
    for (int64_t i = i0; i < a.tg.n_tiles; i += step) listed[i] = 0;
}

}  // namespace

hipError_t launch_serial_mcs(const SweepArgs *d_args, int n_lattices, int ndim, bool act, bool mirror, uint32_t mcs,
                             int parity, hipStream_t st)
{
    const dim3 grid((unsigned)n_lattices), block(64 * kWaves);
    if (mirror) {
        if (ndim == 2) {
            if (act) serial_mcs_kernel<uint16_t, 2, true><<<grid, block, 0, st>>>(d_args, mcs, parity);
            else serial_mcs_kernel<uint16_t, 2, false><<<grid, block, 0, st>>>(d_args, mcs, parity);
        } else {
            if (act) serial_mcs_kernel<uint16_t, 3, true><<<grid, block, 0, st>>>(d_args, mcs, parity);
            else serial_mcs_kernel<uint16_t, 3, false><<<grid, block, 0, st>>>(d_args, mcs, parity);
        }
    } else {
        if (ndim == 2) {
            if (act) serial_mcs_kernel<int32_t, 2, true><<<grid, block, 0, st>>>(d_args, mcs, parity);
            else serial_mcs_kernel<int32_t, 2, false><<<grid, block, 0, st>>>(d_args, mcs, parity);
        } else {
            if (act) serial_mcs_kernel<int32_t, 3, true><<<grid, block, 0, st>>>(d_args, mcs, parity);
            else serial_mcs_kernel<int32_t, 3, false><<<grid, block, 0, st>>>(d_args, mcs, parity);
        }
    }
    return hipGetLastError();
}

hipError_t launch_after_serial(const SweepArgs *d_args, const int64_t *d_label_off, int n_lattices, int64_t max_labels,
                               int parity, hipStream_t st)
{
    const unsigned per = (unsigned)std::min<int64_t>((2 * max_labels + kBlock - 1) / kBlock, 64);
    after_serial_kernel<<<dim3((unsigned)n_lattices, per), kBlock, 0, st>>>(d_args, d_label_off, parity);
    return hipGetLastError();
}

}  // namespace cpm
