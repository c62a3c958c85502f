// Sweeps of lattices that stay in LDS from the first activation of a call to
// its last, compiled once per stored-word type and dimension
// (CPM_RESIDENT_PART = 0..4), and the sweep of a lattice whose parts do not
// come together (5).
//
// An activation launched by itself (cpm_sweep_kernels.hpp) waits for its
// launch, for a chain of dependent loads of labels and counters, and for the
// slowest workgroup, and reads the lattice through the caches every time.
// Here a workgroup takes one part of a lattice (all of it, where that fits)
// into LDS as 16- or 32-bit words and runs every activation of the call on
// it; a barrier of the workgroup takes the place of the launch.
//
// A 2D lattice of several parts is cut across y, whole rows along x (3D
// lattices are swept here uncut or not at all).  Its parts meet after every activation: each writes accepted copies
// within reach of a cut through to the words in global memory and reads the
// rows next to its own back from there; cell counters are in global memory.
// All of that, and the meeting, goes through agent-scope atomic operations,
// which act where every XCD sees them, so no cache is flushed.  A colour
// reads across a cut on one side only (the sub-areas of colour bit 0 start
// at the cut, those of bit 1 end at it): one set of R rows serves both sides,
// and the box's y wraps at its extent plus R.
//
// The random draws of an activation depend on its number alone: a thread
// makes those of the next activation while other waves evaluate this one,
// or while the parts meet.
//
// What bounds it is the chain of each activation (a barrier, the labels, the
// evaluation of an attempt by one wave, its commit: 1.6 to 2 us where few
// areas are hot) and, in large lattices, instruction issue (about 90 VALU
// instructions per 64 draws, 500 per 64 attempts evaluated with the Act
// term).  Against one launch per activation: 100^2 with 20 cells 5.5 -> 2.0 us
// per activation; 250 lattices of 256^2 with 8 attempts per activation
// 129 -> 20 us; 512 Act lattices of 64..512 per side, 10 MCS 12.0 -> 6.2 ms.
#include "cpm_sweep_kernels.hpp"

#ifndef CPM_RESIDENT_PART
#error "compile with -DCPM_RESIDENT_PART=<0..5>"
#endif

namespace cpm {
namespace {

// MCS between two searches for hot areas.
constexpr int kFindHot = 4;
// An entry of a list of hot areas that has not been written yet.
constexpr uint16_t kNoArea = 0xFFFF;

// LDS of a workgroup beside its box, its counters and the tables sized by the
// host (resident_tables).
struct ResidentShared {
    uint2 queue[kResidentQueue];
    // accepted copies of an activation (its number modulo 3: this one's, the
    // last one's and the next one's):
    // label << 6 | surface delta of the target's and of the source's cell;
    // and the area's accepted copy before it (k > 1)
    int2 list[3][kResidentList];
    uint16_t list_next[3][kResidentList];
    TypeParams tp;
    int32_t J[kMaxTypes * kMaxTypes];
    uint32_t tm[256], tl[256];
    unsigned long long stats[2];
    int32_t unit[27][3], lam_p[kMaxTypes], lam_c[kMaxTypes];
    int queue_n[2], list_n[3], go;
    int hot_n[4];
};
static_assert(sizeof(ResidentShared) <= kResidentStaticLds && kResidentStaticLds % 16 == 0, "the host reserves as much");

template <typename T>
__device__ __forceinline__ T agent_load(const T *p)
{
    return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
template <typename T>
__device__ __forceinline__ void agent_store(T *p, T v)
{
    __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// A word of LDS that other waves may be writing.
template <typename T>
__device__ __forceinline__ T lds_load(const T *p)
{
    return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
}
template <typename T>
__device__ __forceinline__ void lds_store(T *p, T v)
{
    __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
}

// The word of a site as the sweep stores it.
template <typename Cell, typename A>
__device__ __forceinline__ Cell resident_word(const A &a, int label, uint32_t act)
{
    if constexpr (std::is_same<Cell, uint16_t>::value) return stored_label<uint16_t>(label);
    else if constexpr (std::is_same<Cell, char16_t>::value) return (Cell)((uint32_t)(label + 1) | (act << 11));
    else return act_word(label, type_of_label(a, label), act);
}

// A (V, S) pair of the global counters, where other parts update it.
__device__ __forceinline__ int2 agent_pair(const int32_t *pairs, int c)
{
    const uint64_t v = agent_load(reinterpret_cast<const uint64_t *>(pairs) + c);
    return make_int2((int)(uint32_t)v, (int)(uint32_t)(v >> 32));
}

// Tables of the Act term in LDS: LG, and EH, EM and EL of exp_log24, whose
// entries for logarithms of up to ln(255) fit 32 bits.
struct ActLds {
    const uint32_t *lg, *eh, *em, *el;
};

// Adds (dv, ds) to label c's (V, S) pair in one atomic: the pair as one
// 64-bit number V + 2^32 S, modulo 2^64.
__device__ __forceinline__ void add_pair(int2 *pairs, int c, int dv, int ds)
{
    atomicAdd(reinterpret_cast<unsigned long long *>(pairs) + c, (unsigned long long)(((int64_t)ds << 32) + dv));
}
// An accepted copy (labels of target and source, their surface deltas).
__device__ __forceinline__ void add_copy(int2 *pairs, int4 r)
{
    if (r.x >= 1) add_pair(pairs, r.x, -1, r.z);
    if (r.y >= 1) add_pair(pairs, r.y, 1, r.w);
}

// exp_log24 of a mean logarithm ell <= ln(255), 2^16 fixed point.
__device__ __forceinline__ uint32_t exp_act(const ActLds &t, uint32_t ell)
{
    const uint32_t p1 = (uint32_t)(((uint64_t)t.eh[ell >> 16] * t.em[(ell >> 8) & 255u]) >> 31);
    return (uint32_t)(((uint64_t)p1 * t.el[ell & 255u]) >> 38);
}

template <typename Cell, int D, bool ACT, bool SINGLE, bool K1, bool EXT, bool LONE, typename A>
__device__ __forceinline__ void sweep_resident(const A &a, const ResidentPart &pt, const ResidentLaunch &rl)
{
    static_assert(!ACT || WordAct<Cell>::kIn, "the Act term reads activities from the words");
    extern __shared__ __align__(16) unsigned char smem[];
    ResidentShared &sh = *reinterpret_cast<ResidentShared *>(smem);
    constexpr int R = ACT ? 2 : 1;
    constexpr int NNB = D == 2 ? 8 : 26;
    constexpr int kPer = 4 / (int)sizeof(Cell);  // words per 32 bits
    // attempts a thread draws ahead
    constexpr int kGroup = D == 2 ? 4 : 2;
    // skip areas whose attempts cannot change anything (below)
    constexpr bool HOT = D == 2 && LONE;
    constexpr bool lone = LONE;
    static_assert(D == 2 || LONE, "only 2D lattices are cut into parts");

    const int tid = threadIdx.x, block = blockDim.x;
    const int s = a.s, L0 = a.L[0], L1 = a.L[1], L2 = a.L[2], na0 = a.na[0], na1 = a.na[1];
    const DeviceModel *model = plain(a.model);
    const int y0 = LONE ? 0 : 2 * s * pt.a1, N1 = LONE ? L1 : 2 * s * pt.n1;  // own rows
    const int P1 = N1 + (LONE ? 0 : R), P2 = L2;                              // with those across the cut
    const LdsMap<kResident> map{L0, P1, L0, P1, P2};
    const int n1 = LONE ? na1 : pt.n1, areas = na0 * n1 * (D == 3 ? a.na[2] : 1);
    Cell *lab = reinterpret_cast<Cell *>(smem + kResidentStaticLds);
    unsigned char *sp = smem + kResidentStaticLds + align16(L0 * P1 * P2 * (int)sizeof(Cell));
    // an uncut lattice: both counter buffers in LDS
    int2 *pairs_lds = reinterpret_cast<int2 *>(sp);
    uint32_t *ti_lds = reinterpret_cast<uint32_t *>(pairs_lds + (lone ? 2 * pt.n_labels : 0));
    const int n_ti = model->n_ti;
    constexpr int kEh = resident_eh(sizeof(Cell));
    uint32_t *lg_lds = ti_lds + n_ti, *eh_lds = lg_lds + (ACT ? 256 : 0), *em_lds = eh_lds + (ACT ? kEh : 0),
             *el_lds = em_lds + (ACT ? 256 : 0);
    // the hot areas of each colour, a bit per area and their list
    const int hot_words = HOT ? (areas + 63) / 64 * 2 : 0, hot_cap = HOT ? pt.hot_cap : 0;
    uint32_t *hot_bits = el_lds + (ACT ? 256 : 0);
    uint16_t *hot = reinterpret_cast<uint16_t *>(hot_bits + 4 * hot_words);
    uint16_t *head = hot + 4 * hot_cap;  // k > 1: an area's last accepted copy
    Cell *words = static_cast<Cell *>(plain(a.cells));
    int32_t *lat = plain(a.lat);
    uint8_t *act = plain(a.act);
    int32_t *counters[2] = {plain(a.counters[0]), plain(a.counters[1])};
    const FastDiv by_L0((uint32_t)L0), by_P1((uint32_t)P1), by_N1((uint32_t)N1);

    if (tid < 3) sh.list_n[tid] = 0;
    if (tid < 2) {
        sh.queue_n[tid] = 0;
        sh.stats[tid] = 0;
    }
    for (int i = tid; i < (SINGLE ? 0 : kMaxTypes * kMaxTypes); i += block) sh.J[i] = (int32_t)model->J[i];
    if (ACT) {
        for (int i = tid; i < 256; i += block) {
            lg_lds[i] = (uint32_t)model->LG[i];
            em_lds[i] = (uint32_t)model->EM[i];
            el_lds[i] = (uint32_t)model->EL[i];
        }
        for (int i = tid; i < kEh; i += block) eh_lds[i] = (uint32_t)model->EH[i];
    }
    for (int i = tid; i < (int)(sizeof(TypeParams) / sizeof(int4)); i += block)
        reinterpret_cast<int4 *>(&sh.tp)[i] = reinterpret_cast<const int4 *>(model->lam_v)[i];
    for (int i = tid; EXT && i < 27; i += block)
        for (int d = 0; d < 3; ++d) sh.unit[i][d] = model->unit[i][d];
    for (int i = tid; EXT && i < kMaxTypes; i += block) {
        sh.lam_p[i] = (int32_t)model->lam_p[i];
        sh.lam_c[i] = (int32_t)model->lam_c[i];
    }
    for (int i = tid; i < 256; i += block) {
        sh.tm[i] = model->TM32[i];
        sh.tl[i] = model->TL32[i];
    }
    for (int i = tid; i < n_ti; i += block) ti_lds[i] = model->TI32[i];
    if (lone)
        for (int i = tid; i < pt.n_labels; i += block)
            pairs_lds[i] = pairs_lds[pt.n_labels + i] = reinterpret_cast<const int2 *>(counters[rl.parity])[i];

    // own rows: global site index of the row's start, from its number
    auto own_row = [&](int r, int &ry, int &rz) {
        rz = D == 3 ? (int)by_N1.div((uint32_t)r) : 0;
        ry = r - rz * N1;
    };
    const bool vec = (L0 & 3) == 0 && (reinterpret_cast<uintptr_t>(lat) & 15) == 0 &&
                     (!ACT || (reinterpret_cast<uintptr_t>(act) & 3) == 0);
    auto site = [&](int y, int z) { return ((size_t)z * L1 + (size_t)(y0 + y)) * L0; };
    bool over = false;
    {
        const int per = vec ? L0 / 4 : L0;
        const FastDiv by_per((uint32_t)per);
        for (int c = tid; c < per * N1 * P2; c += block) {
            int ry, rz;
            const int r = (int)by_per.div((uint32_t)c), x = c - r * per;
            own_row(r, ry, rz);
            const size_t g = site(ry, rz) + (size_t)x * (vec ? 4 : 1);
            Cell *d = lab + (ry + P1 * rz) * L0 + x * (vec ? 4 : 1);
            if (vec) {
                const int4 v = *reinterpret_cast<const int4 *>(lat + g);
                const uchar4 w = ACT ? *reinterpret_cast<const uchar4 *>(act + g) : make_uchar4(0, 0, 0, 0);
                d[0] = resident_word<Cell>(a, v.x, w.x);
                d[1] = resident_word<Cell>(a, v.y, w.y);
                d[2] = resident_word<Cell>(a, v.z, w.z);
                d[3] = resident_word<Cell>(a, v.w, w.w);
                if (ACT) over |= w.x > 31 || w.y > 31 || w.z > 31 || w.w > 31;
            } else {
                const uint32_t w = ACT ? act[g] : 0u;
                d[0] = resident_word<Cell>(a, lat[g], w);
                if (ACT) over |= w > 31;
            }
        }
    }
    if (std::is_same<Cell, char16_t>::value && over) atomicOr(reinterpret_cast<int32_t *>(&rl.bar->act_overflow), 1);

    // rows within R of a cut, as the neighbouring parts read them: from LDS
    // to the words in global memory
    const int pitch32 = L0 / kPer;  // 32-bit words per row (L0 is even)
    const FastDiv by_pitch((uint32_t)pitch32);
    auto publish_edges = [&]() {
        for (int c = tid; c < 2 * R * pitch32; c += block) {
            const int q = (int)by_pitch.div((uint32_t)c), x = c - q * pitch32, y = q < R ? q : N1 - 2 * R + q;
            agent_store(reinterpret_cast<uint32_t *>(words + site(y, 0)) + x,
                        reinterpret_cast<const uint32_t *>(lab + y * L0)[x]);
        }
    };
    // the rows across the cut that a colour reads, from global memory
    auto refresh = [&](int cy) {
        for (int c = tid; c < R * pitch32; c += block) {
            const int q = (int)by_pitch.div((uint32_t)c), x = c - q * pitch32;
            const size_t g = (size_t)wrap_once(y0 + (cy ? N1 + q : q - R), L1) * L0;
            reinterpret_cast<uint32_t *>(lab + (N1 + q) * L0)[x] = agent_load(reinterpret_cast<const uint32_t *>(words + g) + x);
        }
    };
    // Meeting of a lattice's parts: every wave's stores and atomics complete,
    // then one arrival per part; the count only grows.  The wait is bounded.
    uint32_t meeting = 0;
    uint32_t *arrivals = rl.arrivals + (size_t)pt.lattice * kResidentArrivalStride;
    auto arrive = [&]() {
        asm volatile("s_waitcnt vmcnt(0) lgkmcnt(0)" ::: "memory");
        __syncthreads();
        ++meeting;
        if (tid == 0) __hip_atomic_fetch_add(arrivals, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    };
    auto wait = [&]() {  // false: a part gave up waiting
        if (tid == 0) {
            const uint32_t target = meeting * (uint32_t)pt.n_parts;
            uint32_t polls = 0;
            int go = 1;
            while ((int32_t)(agent_load(arrivals) - target) < 0) {
                ++polls;
                if (polls >= rl.spin_limit || ((polls & 63u) == 0 && agent_load(&rl.bar->abort) != 0u)) {
                    agent_store(&rl.bar->abort, 1u);
                    go = 0;
                    break;
                }
                __builtin_amdgcn_s_sleep(1);
            }
            sh.go = go;
        }
        __syncthreads();
        return sh.go != 0;
    };

    // Draws.  What depends on the area alone is kept per thread: its corner
    // and, of the first Philox round, the product of the area's number.
    const uint32_t sd = D == 2 ? (uint32_t)(s * s) : (uint32_t)(s * s * s);
    const uint32_t by_s = 65536u / (uint32_t)s + 1u;  // floor(o / s) = o by_s >> 16 for o < s^D, s <= 15
    const FastDiv by_na0((uint32_t)na0), by_n1((uint32_t)n1), by_2s(2u * (uint32_t)s), by_s32((uint32_t)s);
    struct Area {
        uint32_t xy, z, c2, c3;  // corner in the box: x | y << 16, z
    };
    auto area_of = [&](int i) {
        Area r{0, 0, 0, 0};
        const int q0 = (int)by_na0.div((uint32_t)i), ax = i - q0 * na0;
        const int az = D == 3 ? (int)by_n1.div((uint32_t)q0) : 0, ay = q0 - az * n1;
        const uint32_t id = (uint32_t)ax + (uint32_t)na0 * ((uint32_t)((LONE ? 0 : pt.a1) + ay) + (uint32_t)na1 * (uint32_t)az);
        const uint64_t p0 = (uint64_t)0xD2511F53u * id;
        r.xy = (uint32_t)(2 * s * ax) | ((uint32_t)(2 * s * ay) << 16);
        r.z = (uint32_t)(2 * s * az);
        r.c2 = (uint32_t)(p0 >> 32) ^ a.lattice_id ^ a.key1;
        r.c3 = (uint32_t)p0;
        return r;
    };
    struct Draw {
        uint32_t t;    // target: x | y << 16 (2D) or its LDS index (3D)
        uint32_t src;  // source: LDS index | Moore offset << 17
        uint32_t u2;   // acceptance draw
    };
    auto target = [&](const Draw &d) {  // LDS index
        return D == 2 ? (int)((d.t & 0xFFFFu) + __umul24((uint32_t)L0, d.t >> 16)) : (int)d.t;
    };
    auto draw = [&](const Area &ar, uint32_t mcs, uint32_t alpha, int j) {
        const uint64_t p1 = (uint64_t)0xCD9E8D57u * ((alpha << 8) | (uint32_t)j);
        const uint4 u = philox4x32_10<9>(make_uint4((uint32_t)(p1 >> 32) ^ mcs ^ a.key0, (uint32_t)p1, ar.c2, ar.c3), a.key0, a.key1);
        const uint32_t o = __umulhi(u.x, sd);
        const uint32_t q1 = __umul24(o, by_s) >> 16, ox = o - __umul24(q1, (uint32_t)s);
        const uint32_t oz = D == 3 ? __umul24(q1, by_s) >> 16 : 0, oy = D == 3 ? q1 - __umul24(oz, (uint32_t)s) : q1;
        const uint32_t corner = (uint32_t)s * ((alpha & 1) | (((alpha >> 1) & 1) << 16));
        const uint32_t xy = ar.xy + corner + (ox | (oy << 16));
        const int x = (int)(xy & 0xFFFFu), y = (int)(xy >> 16);
        const int z = D == 3 ? (int)(ar.z + (uint32_t)s * ((alpha >> 2) & 1) + oz) : 0;
        const uint32_t nsel = D == 2 ? u.y >> 29 : __umulhi(u.y, (uint32_t)NNB);
        const uint32_t msel = nsel < NNB / 2 ? nsel : nsel + 1;
        const uint32_t m3 = (msel * 11u) >> 5, dx = msel - 3u * m3;  // floor(msel / 3), msel < 27
        const uint32_t m9 = D == 3 ? (m3 * 11u) >> 5 : 0, dy = m3 - 3u * m9;
        Draw d;
        d.t = D == 2 ? xy : (uint32_t)(x + (int)__umul24((uint32_t)L0, (uint32_t)y + __umul24((uint32_t)P1, (uint32_t)z)));
        d.src = (uint32_t)map.at(x + (int)dx - 1, y + (int)dy - 1, D == 3 ? z + (int)m9 - 1 : 0) | (msel << 17);
        d.u2 = u.z;
        return d;
    };
    const ThrTables tb{sh.tm, sh.tl, ti_lds, n_ti};
    const ActLds act_lds{lg_lds, eh_lds, em_lds, el_lds};
    // the single type's rows of J (each entry fits 32 bits)
    int32_t j_cc = 0, j_cm = 0, j_co = 0, j_mm = 0, j_mo = 0;
    if (SINGLE) {
        const int64_t *J = model->J;
        const int tc = a.single_type, to = a.obstacle_type;
        j_cc = (int32_t)J[tc * kMaxTypes + tc];
        j_cm = (int32_t)J[tc * kMaxTypes];
        j_co = (int32_t)J[tc * kMaxTypes + to];
        j_mm = (int32_t)J[0];
        j_mo = (int32_t)J[to];
    }
    // the energy parameters of a type (of the single type, in registers)
    struct Terms {
        int32_t lam_v, v_t, lam_s, s_t, max_act, r_act;
    };
    const int one = SINGLE ? a.single_type : 0;
    const Terms single_terms{(int32_t)model->lam_v[one], model->v_target[one], (int32_t)model->lam_s[one],
                             model->s_target[one], model->max_act[one], (int32_t)model->r_act[one]};
    auto terms = [&](int type) {
        if (SINGLE) return single_terms;  // of the medium, never used
        return Terms{(int32_t)sh.tp.lam_v[type], sh.tp.v_target[type], (int32_t)sh.tp.lam_s[type],
                     sh.tp.s_target[type], ACT ? sh.tp.max_act[type] : 0, ACT ? (int32_t)sh.tp.r_act[type] : 0};
    };
    uint32_t my_nontrivial = 0, my_accepted = 0;
    int4 *list_spill[2];
    {
        const size_t off = LONE ? 0 : (size_t)na0 * pt.a1 * (size_t)a.k;
        list_spill[0] = plain(a.dlist[0]) + off;
        list_spill[1] = plain(a.dlist[1]) + off;
    }

    // The last activation's accepted copies have to reach the counter buffer
    // that this one writes: a thread keeps its first one (k = 1), the others
    // go to a list.
    int4 last_copy = make_int4(-1, 0, 0, 0);
    auto pairs_of = [&](int p) { return lone ? pairs_lds + p * pt.n_labels : reinterpret_cast<int2 *>(counters[p]); };
    bool marking = false;
    // Accepted copy `slot` of list li (of an activation of parity p); next: the area's one before it.
    auto record = [&](int li, int p, int slot, int &next) {
        if (slot < kResidentList) {
            const int2 e = sh.list[li][slot];
            next = K1 ? 0 : sh.list_next[li][slot];
            return make_int4(e.x >> 6, e.y >> 6, (e.x << 26) >> 26, (e.y << 26) >> 26);
        }
        const int4 r = list_spill[p][slot - kResidentList];
        next = (int)((uint32_t)r.z >> 16);
        return make_int4(r.x, r.y, (int)(int8_t)r.z, (int)(int8_t)(r.z >> 8));
    };

    // LDS index offsets of a site's neighbours along each axis, wrapping at
    // the box.
    struct Offsets {
        int x[2], y[2], z[2];
        __device__ __forceinline__ int of(int dx, int dy, int dz) const
        {
            return (dx < 0 ? x[0] : dx > 0 ? x[1] : 0) + (dy < 0 ? y[0] : dy > 0 ? y[1] : 0) +
                   (D == 3 ? (dz < 0 ? z[0] : dz > 0 ? z[1] : 0) : 0);
        }
    };
    const int plane = L0 * P1, round_y = plane - L0, round_z = plane * (P2 - 1);
    auto offsets = [&](int x, int y, int z) {
        Offsets o;
        o.x[0] = x == 0 ? L0 - 1 : -1, o.x[1] = x == L0 - 1 ? 1 - L0 : 1;
        o.y[0] = y == 0 ? round_y : -L0, o.y[1] = y == P1 - 1 ? -round_y : L0;
        o.z[0] = z == 0 ? round_z : -plane, o.z[1] = z == P2 - 1 ? -round_z : plane;
        return o;
    };

    // Hot areas (2D).  An attempt whose sub-area, with the ring around it,
    // holds one label is a copy of a label onto itself, whatever is drawn: it
    // is not drawn.  `mark` adds the sub-areas that see site (x, y), whose
    // label has just changed; `find_hot` lists all anew.  A list that has
    // grown past its room stands for all areas.  Uncut lattices only.
    //
    // `mark` counts an entry before it writes it, and other waves draw ahead
    // meanwhile: every entry past the count of `find_hot` holds kNoArea until
    // it is written, and a thread that reads kNoArea makes no draw from it.
    // After the barrier of the step all counted entries are written.
    auto mark = [&](int x, int y) {
        const int gx[3] = {(int)by_s32.div((uint32_t)wrap_min(x - 1, L0)), (int)by_s32.div((uint32_t)wrap_min(x + 1, L0)), x};
        const int gy[3] = {(int)by_s32.div((uint32_t)wrap_min(y - 1, L1)), (int)by_s32.div((uint32_t)wrap_min(y + 1, L1)), y};
        auto add = [&](int i, int j, uint32_t old) {
            const int c = (gx[i] & 1) | ((gy[j] & 1) << 1), area = (gx[i] >> 1) + na0 * (gy[j] >> 1);
            const uint32_t bit = 1u << (area & 31);
            if (!(old & bit) && !(atomicOr(hot_bits + c * hot_words + (area >> 5), bit) & bit)) {
                const int slot = atomicAdd(&sh.hot_n[c], 1);
                if (slot < hot_cap) lds_store(&hot[c * hot_cap + slot], (uint16_t)area);
            }
        };
        auto word = [&](int i, int j) {
            return lds_load(&hot_bits[((gx[i] & 1) | ((gy[j] & 1) << 1)) * hot_words + (((gx[i] >> 1) + na0 * (gy[j] >> 1)) >> 5)]);
        };
        // s >= 2: of x - 1, x, x + 1 the outer two lie in every sub-area that sees x
        const uint32_t w0 = word(0, 0), w1 = word(1, 0), w2 = word(0, 1), w3 = word(1, 1);
        add(0, 0, w0);
        add(1, 0, w1);
        add(0, 1, w2);
        add(1, 1, w3);
        if (s == 1)
            for (int i = 0; i < 3; ++i) {
                add(i, 2, 0);
                if (i < 2) add(2, i, 0);
            }
    };
    auto find_hot = [&]() {
        if (!HOT) return;
        if (tid < 4) sh.hot_n[tid] = 0;
        __syncthreads();
        for (int a0 = 0; a0 < areas; a0 += block) {  // every lane of a wave, for the ballots
            const int area = a0 + tid;
            const int ay = (int)by_na0.div((uint32_t)min(area, areas - 1)), ax = min(area, areas - 1) - ay * na0;
#pragma unroll
            for (int c = 0; c < 4; ++c) {
                const int cx = c & 1, cy = c >> 1;
                const int x = 2 * s * ax + s * cx - 1, y = 2 * s * ay + s * cy - 1;
                bool is = false;
                {
                    const int first = label_of(lab[map.at(x, y, 0)]);
                    for (int j = 0; j < s + 2; ++j)
                        for (int i = 0; i < s + 2; ++i) is |= label_of(lab[map.at(x + i, y + j, 0)]) != first;
                }
                is = is && area < areas;
                const uint64_t mask = __ballot(is);
                if ((tid & 63) < 2 && area - (tid & 63) < areas)
                    hot_bits[c * hot_words + ((area - (tid & 63)) >> 5) + (tid & 63)] = (uint32_t)(mask >> (32 * (tid & 63)));
                int base = 0;
                if ((tid & 63) == 0 && mask) base = atomicAdd(&sh.hot_n[c], (int)__popcll(mask));
                base = __builtin_amdgcn_readfirstlane(base);
                const int slot = base + (int)__builtin_amdgcn_mbcnt_hi((uint32_t)(mask >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)mask, 0u));
                if (is && slot < hot_cap) hot[c * hot_cap + slot] = (uint16_t)area;
            }
        }
        __syncthreads();
        for (int i = tid; i < 4 * hot_cap; i += block)
            if (i % hot_cap >= sh.hot_n[i / hot_cap]) hot[i] = kNoArea;
        __syncthreads();
    };

    // f(word) of a site (LDS index c) and its neighbours, plane by plane.
    auto around = [&](int c, const Offsets &o, auto &&f) {
#pragma unroll 1
        for (int pz = 0; pz < (D == 3 ? 3 : 1); ++pz) {
            const int cz = c + (D == 3 ? (pz == 0 ? o.z[0] : pz == 2 ? o.z[1] : 0) : 0);
#pragma unroll
            for (int n = 0; n < 9; ++n) f(lab[cz + o.of(n % 3 - 1, n / 3 - 1, 0)]);
        }
    };

    // Evaluates an attempt (of an activation whose list is li and that reads
    // counter buffer p; first_of_area: j = 0) and commits it if accepted: the
    // energy change of the copy (eq. 1, 3, 7) and the Metropolis test (eq. 2).  The lattice's size and the targets
    // (checked by the host) leave every factor below 2^31, so that each
    // product is one 32-bit multiply.
    auto attempt = [&](const Draw &d, int li, int p, bool first_of_area) {
        const int t = target(d), src = (int)(d.src & 0x1FFFFu), msel = (int)(d.src >> 17);
        int x, y, z = 0;
        if (D == 2) {
            x = (int)(d.t & 0xFFFFu);
            y = (int)(d.t >> 16);
        } else {
            const int q0 = (int)by_L0.div((uint32_t)t);
            x = t - (int)__umul24((uint32_t)q0, (uint32_t)L0);
            z = (int)by_P1.div((uint32_t)q0);
            y = q0 - (int)__umul24((uint32_t)z, (uint32_t)P1);
        }
        const Offsets to = offsets(x, y, z);
        const int m3 = (msel * 11) >> 5, m9 = D == 3 ? (m3 * 11) >> 5 : 0, sdx = msel - 3 * m3 - 1, sdy = m3 - 3 * m9 - 1,
                  sdz = D == 3 ? m9 - 1 : 0;
        const Cell wt = lab[t], ws = lab[src];
        const int lt = label_of(wt), ls = label_of(ws);
        int2 ct = make_int2(0, 0), cs = ct;
        if (lone) {
            ct = pairs_lds[p * pt.n_labels + lt];
            cs = pairs_lds[p * pt.n_labels + ls];
        } else {
            const int32_t *rd = counters[p];
            ct = agent_pair(rd, lt);
            cs = agent_pair(rd, ls);
        }
        int area = 0;
        if (!K1) {
            // own accepted copies earlier in this activation
            const int ax = (int)by_2s.div((uint32_t)x), ay = (int)by_2s.div((uint32_t)y), az = D == 3 ? (int)by_2s.div((uint32_t)z) : 0;
            area = ax + na0 * (ay + n1 * az);
            for (int i = first_of_area ? 0xFFFF : head[area], next; i != 0xFFFF; i = next) {
                const int4 r = record(li, p, i, next);
                if (r.x == lt) { ct.x -= 1; ct.y += r.z; }
                if (r.y == lt) { ct.x += 1; ct.y += r.w; }
                if (r.x == ls) { cs.x -= 1; cs.y += r.z; }
                if (r.y == ls) { cs.x += 1; cs.y += r.w; }
            }
        }
        const int tt = lt == 0 ? 0 : (SINGLE ? a.single_type : type_of_word(a, wt, lt));
        const int ts = ls == 0 ? 0 : (SINGLE ? a.single_type : type_of_word(a, ws, ls));
        // read early: from global memory
        int c[3] = {0, 0, 0};
        int32_t u[3] = {0, 0, 0};
        int4 pd = make_int4(0, 0, 0, 0);
        if (EXT) {
            const int o = (1 - sdx) + 3 * (1 - sdy) + 9 * (D == 3 ? 1 - sdz : 1);
#pragma unroll
            for (int d = 0; d < D; ++d) u[d] = sh.unit[o][d];
            if (a.pdir) pd = plain(a.pdir)[ls];
            if (a.chem) {
                const int gx = wrap_once(x + sdx, L0), gy = wrap_once(y0 + y + sdy, L1), gz = D == 3 ? wrap_once(z + sdz, L2) : 0;
                const int16_t *f = plain(a.chem) + D * (((size_t)gz * L1 + gy) * L0 + gx);
#pragma unroll
                for (int d = 0; d < D; ++d) c[d] = f[d];
            }
        }
        // the target and its neighbours, of which the target itself is then
        // taken out again (all but of its own mean activity)
        int k_old = -1, k_new = 0, n_cell = -(lt > 0), n_med = -(lt == 0);
        int64_t adh = 0;
        uint32_t sum = 0;
        bool dead = false;
        around(t, to, [&](Cell word) {
            const int lu = label_of(word);
            const bool same = lu == lt;
            k_old += same;
            k_new += lu == ls;
            if (SINGLE) {
                n_cell += lu > 0;
                n_med += lu == 0;
            } else {
                const int tu = type_of_word(a, word, lu);
                const int32_t js = sh.J[ts * kMaxTypes + tu], jt = sh.J[tt * kMaxTypes + tu];
                adh += (int64_t)(lu != ls ? js : 0) - (int64_t)(same ? 0 : jt);
            }
            if (ACT) {
                const uint32_t act = (uint32_t)word >> WordAct<Cell>::kShift, v = lg_lds[act];
                dead |= same && act == 0;
                sum += same ? v : 0u;  // at most 27 ln(255) 2^24 < 2^32
            }
        });
        if (!SINGLE) adh -= sh.J[ts * kMaxTypes + tt];
        if (SINGLE) {
            // neighbours unlike the label, weighted by J(label type, their type)
            const int n_obs = NNB - n_cell - n_med;
            const int cs_ = n_cell - (ls > 0 ? k_new : 0), ms = n_med - (ls == 0 ? k_new : 0);
            const int ct_ = n_cell - (lt > 0 ? k_old : 0), mt = n_med - (lt == 0 ? k_old : 0);
            adh = mul32(ls > 0 ? j_cc : j_cm, cs_) + mul32(ls > 0 ? j_cm : j_mm, ms) - mul32(lt > 0 ? j_cc : j_cm, ct_) -
                  mul32(lt > 0 ? j_cm : j_mm, mt) +
                  mul32(n_obs, (ls > 0 ? j_co : j_mo)) - mul32(n_obs, (lt > 0 ? j_co : j_mo));
        }
        const int dso = 2 * k_old - NNB, dsn = NNB - 2 * k_new;
        const Terms et = terms(tt), es = terms(ts);
        const int64_t old = mul32(et.lam_v, 1 - 2 * (ct.x - et.v_t)) + mul32(et.lam_s, dso * (2 * (ct.y - et.s_t) + dso));
        const int64_t now = mul32(es.lam_v, 2 * (cs.x - es.v_t) + 1) + mul32(es.lam_s, dsn * (2 * (cs.y - es.s_t) + dsn));
        int64_t q = adh + (lt >= 1 ? old : 0) + (ls >= 1 ? now : 0);
        if (ACT) {
            const bool mot_t = lt > 0 && et.max_act > 0, mot_s = ls > 0 && es.max_act > 0;
            int32_t gt = 0, gs = 0;
            if (mot_t && !dead) gt = (int32_t)exp_act(act_lds, sum / (uint32_t)(k_old + 1));
            if (mot_s) {
                uint32_t cnt = 0;
                sum = 0;
                dead = false;
                around(src, offsets(wrap_min(x + sdx, L0), wrap_min(y + sdy, P1), D == 3 ? wrap_min(z + sdz, P2) : 0),
                       [&](Cell word) {
                           const bool same = label_of(word) == ls;
                           const uint32_t act = (uint32_t)word >> WordAct<Cell>::kShift, v = lg_lds[act];
                           dead |= same && act == 0;
                           sum += same ? v : 0u;
                           cnt += same;
                       });
                if (!dead) gs = (int32_t)exp_act(act_lds, sum / cnt);
            }
            q += (mul32(et.r_act, gt) - mul32(es.r_act, gs)) >> 16;
        }
        if (EXT && ls >= 1) {
            // copies along the cell's direction / up the field are favoured
            // (|U . P| <= 3 2^28, |U . C| < 3 2^29)
            if (a.pdir)
                q -= mul32(sh.lam_p[ts], u[0] * pd.x + u[1] * pd.y + (D == 3 ? u[2] * pd.z : 0)) >> 28;
            if (a.chem) q -= mul32(sh.lam_c[ts], u[0] * c[0] + u[1] * c[1] + (D == 3 ? u[2] * c[2] : 0)) >> 28;
        }
        if (!metropolis32(tb, q, d.u2)) return;
        ++my_accepted;
        uint32_t na = 0;
        if (ACT && ls >= 1 && es.max_act > 0) na = (uint32_t)es.max_act & 255u;
        const Cell nw = WordAct<Cell>::kIn ? (Cell)(((uint32_t)ws & WordAct<Cell>::kKeep) | (na << WordAct<Cell>::kShift)) : ws;
        lab[t] = nw;
        if (HOT && marking) mark(x, y);
        if (EXT && a.csum) move_centroids<D>(a, (int)(site(y, z) + (size_t)x), lt, ls);
        const int4 rec = make_int4(lt, ls, dso, dsn);
        if (!lone && (y < R || y >= N1 - R)) agent_store(words + site(y, 0) + x, nw);
        add_copy(pairs_of(p ^ 1), rec);
        if (K1 && last_copy.x < 0) {
            last_copy = rec;
            return;
        }
        const int slot = atomicAdd(&sh.list_n[li], 1);
        const int next = K1 || first_of_area ? 0xFFFF : head[area];
        if (slot < kResidentList) {
            sh.list[li][slot] = make_int2((lt << 6) | (dso & 63), (ls << 6) | (dsn & 63));
            if (!K1) sh.list_next[li][slot] = (uint16_t)next;
        } else {
            list_spill[p][slot - kResidentList] = make_int4(lt, ls, (dso & 255) | ((dsn & 255) << 8) | (int)((uint32_t)next << 16), 0);
        }
        if (!K1) head[area] = (uint16_t)slot;
    };
    // the last activation's accepted copies (list li, buffer p), into the
    // buffer that does not hold them yet: on the last lanes, which evaluate
    // first, and last, of all
    auto readd = [&](int li, int p) {
        if (K1 && last_copy.x >= 0) {
            add_copy(pairs_of(p), last_copy);
            last_copy.x = -1;
        }
        const int n = sh.list_n[li];
        for (int i = block - 1 - tid; i < n; i += block) {
            int next;
            add_copy(pairs_of(p), record(li, p, i, next));
        }
    };

    // How the attempts of a step (an activation's j-th attempts) are taken:
    // attempt i is that of hot area i of the colour, or of area i.  Few
    // attempts (most of them nontrivial: the areas are hot) are evaluated
    // where drawn, by the two halves of the workgroup in turn, the other half
    // drawing the next step's meanwhile; many pass through the queue.
    const int half = HOT ? block / 128 * 64 : 0;
    struct Step {
        int n, tag;  // attempts; number of the step and how it is taken
        bool listed, few;
    };
    auto step_of = [&](int seq, uint32_t alpha) {
        Step st{areas, seq * 4, false, false};
        if (HOT) {
            const int n = lds_load(&sh.hot_n[alpha & 3]);
            st.listed = n <= hot_cap;
            if (st.listed) st.n = n;
            st.few = st.listed && n <= half;
            st.tag += (st.listed ? 1 : 0) + (st.few ? 2 : 0);
        }
        return st;
    };
    auto area_number = [&](uint32_t alpha, bool listed, int i) {
        return HOT && listed ? (int)lds_load(&hot[__umul24(alpha & 3u, (uint32_t)hot_cap) + (uint32_t)i]) : i;
    };
    // This thread's first attempts of the next step, drawn ahead; they stand
    // if the step is then taken as its tag says: entries below ahead_n had
    // been written when they were drawn from, and stay until the next search.
    Draw ahead[kGroup];
    int ahead_tag = -1, ahead_n = 0;
    auto draw_ahead = [&](int seq, uint32_t mcs, uint32_t alpha, int j) {
        const Step st = step_of(seq, alpha);
        ahead_tag = st.tag;
        ahead_n = st.n;
        if (st.few) {
            const int i = tid - (seq & 1) * half;
            if (i >= 0 && i < st.n) {
                const int area = area_number(alpha, true, i);
                if (area == kNoArea) ahead_n = i;
                else ahead[0] = draw(area_of(area), mcs, alpha, j);
            }
            return;
        }
#pragma unroll
        for (int r = 0; r < kGroup; ++r) {
            const int i = tid + r * block;
            if (i >= st.n) continue;
            const int area = area_number(alpha, st.listed, i);
            if (HOT && area == kNoArea) ahead_n = min(ahead_n, i);
            else ahead[r] = draw(area_of(area), mcs, alpha, j);
        }
    };
    __syncthreads();
    if (!lone) {
        publish_edges();
        arrive();
    }
    if (!lone && !wait()) return;

    int qi = 0, parity = rl.parity, li = 0, last_li = 2, seq = 0;
    for (int m = 0; m < rl.n_mcs; ++m) {
        const uint32_t mcs = rl.mcs0 + (uint32_t)m;
        if (HOT && m % kFindHot == 0) {
            find_hot();
            ahead_tag = -1;
            marking = sh.hot_n[0] <= hot_cap || sh.hot_n[1] <= hot_cap || sh.hot_n[2] <= hot_cap || sh.hot_n[3] <= hot_cap;
        }
        for (uint32_t alpha = 0; alpha < rl.n_act; ++alpha, parity ^= 1, last_li = li, li = li == 2 ? 0 : li + 1) {
            if (!lone) refresh((int)((alpha >> 1) & 1));
            readd(last_li, parity ^ 1);
            if (!lone) __syncthreads();
            if (tid == 0) sh.list_n[li == 2 ? 0 : li + 1] = 0;
            for (int j = 0; j < (K1 ? 1 : a.k); ++j, ++seq) {
                const bool end_act = K1 || j + 1 == a.k, end_mcs = end_act && alpha + 1 == rl.n_act;
                const uint32_t next_mcs = end_mcs ? mcs + 1 : mcs, next_alpha = end_mcs ? 0u : end_act ? alpha + 1 : alpha;
                const int next_j = end_act ? 0 : j + 1;
                const Step st = step_of(seq, alpha);
                if (st.few) {
                    const int i = tid - (seq & 1) * half;
                    if (i >= 0 && i < half) {
                        if (i < st.n) {
                            if (ahead_tag != st.tag || i >= ahead_n)
                                ahead[0] = draw(area_of(area_number(alpha, true, i)), mcs, alpha, j);
                            const int lt = label_of(lab[target(ahead[0])]), ls = label_of(lab[ahead[0].src & 0x1FFFFu]);
                            if (!K1 && j == 0) head[area_number(alpha, true, i)] = 0xFFFF;
                            if (lt != ls && lt >= 0 && ls >= 0) {
                                ++my_nontrivial;
                                __builtin_amdgcn_s_setprio(3);
                                attempt(ahead[0], li, parity, j == 0);
                                __builtin_amdgcn_s_setprio(0);
                            }
                        }
                        ahead_tag = -1;
                    } else {
                        draw_ahead(seq + 1, next_mcs, next_alpha, next_j);
                    }
                    __syncthreads();
                    continue;
                }
                // the nontrivial attempts go to a queue, which the last lanes
                // work off: the energy change, which most attempts skip, runs
                // on as few waves as it fills; those that find it full are
                // pushed again after it has been worked off
                uint32_t open = 0xFFFFFFFFu;
                for (bool first = true;; first = false) {
                    // kGroup attempts: one slot request per wave for all of them
                    auto push = [&](const Draw *d, int r0) {
                        bool todo[kGroup];
                        uint64_t mask[kGroup];
                        int n = 0, pre[kGroup];
#pragma unroll
                        for (int r = 0; r < kGroup; ++r) {
                            const int lt = label_of(lab[target(d[r])]), ls = label_of(lab[d[r].src & 0x1FFFFu]);
                            todo[r] = tid + (r0 + r) * block < st.n && lt != ls && lt >= 0 && ls >= 0 && ((open >> (r0 + r)) & 1u);
                            if (first) my_nontrivial += todo[r];
                            mask[r] = __ballot(todo[r]);
                            pre[r] = n;
                            n += (int)__popcll(mask[r]);
                        }
                        if (n == 0) return;
                        int base = 0;
                        if ((tid & 63) == 0) base = atomicAdd(&sh.queue_n[qi], n);
                        base = __builtin_amdgcn_readfirstlane(base);
#pragma unroll
                        for (int r = 0; r < kGroup; ++r) {
                            const int slot = base + pre[r] +
                                             (int)__builtin_amdgcn_mbcnt_hi((uint32_t)(mask[r] >> 32),
                                                                            __builtin_amdgcn_mbcnt_lo((uint32_t)mask[r], 0u));
                            if (todo[r] && slot < kResidentQueue) {
                                sh.queue[slot] = make_uint2((uint32_t)target(d[r]) | (d[r].src & ~0x1FFFFu), d[r].u2);
                                open &= ~(1u << (r0 + r));
                            }
                        }
                    };
                    for (int r0 = 0; tid - (tid & 63) + r0 * block < st.n; r0 += kGroup) {  // uniform over a wave
                        Draw d[kGroup];
#pragma unroll
                        for (int r = 0; r < kGroup; ++r) {
                            const int i = tid + (r0 + r) * block;
                            d[r].t = d[r].src = 0;
                            if (i < st.n) {
                                if (r0 == 0 && first && ahead_tag == st.tag && i < ahead_n) d[r] = ahead[r];
                                else d[r] = draw(area_of(area_number(alpha, st.listed, i)), mcs, alpha, j);
                                if (!K1 && j == 0 && first) head[area_number(alpha, st.listed, i)] = 0xFFFF;
                            }
                        }
                        push(d, r0);
                    }
                    __syncthreads();
                    const int qn = sh.queue_n[qi];
                    if (tid == 0) sh.queue_n[qi ^ 1] = 0;
                    // ahead of the waves that draw meanwhile
                    __builtin_amdgcn_s_setprio(3);
                    for (int i = block - 1 - tid; i < min(qn, kResidentQueue); i += block) {
                        const uint2 e = sh.queue[i];
                        Draw d;
                        d.t = e.x & 0x1FFFFu;
                        d.u2 = e.y;
                        const int q0 = (int)by_L0.div(d.t), x = (int)d.t - (int)__umul24((uint32_t)q0, (uint32_t)L0);
                        const int z = D == 3 ? (int)by_P1.div((uint32_t)q0) : 0, y = D == 3 ? q0 - (int)__umul24((uint32_t)z, (uint32_t)P1) : q0;
                        const Offsets to = offsets(x, y, z);
                        const int msel = (int)(e.x >> 17), m3 = (msel * 11) >> 5, m9 = D == 3 ? (m3 * 11) >> 5 : 0;
                        d.src = (d.t + (uint32_t)to.of(msel - 3 * m3 - 1, m3 - 3 * m9 - 1, D == 3 ? m9 - 1 : 0)) | ((uint32_t)msel << 17);
                        if (D == 2) d.t = (uint32_t)x | ((uint32_t)y << 16);
                        attempt(d, li, parity, j == 0);
                    }
                    __builtin_amdgcn_s_setprio(0);
                    qi ^= 1;
                    if (qn <= kResidentQueue) break;
                    __syncthreads();
                }
                if (!lone && end_act) arrive();
                draw_ahead(seq + 1, next_mcs, next_alpha, next_j);
                if (lone || !end_act) __syncthreads();
                else if (!wait()) return;
            }
        }
        if (ACT) {
            // the Act decay, in the words; other parts read this part's edges
            // until they have met once more
            uint32_t *w32 = reinterpret_cast<uint32_t *>(lab);
            const int n32 = L0 * P1 * P2 / kPer;
            for (int i = tid; i < n32; i += block) {
                uint32_t v = w32[i];
                if (sizeof(Cell) == 2) {
                    v -= (v & 0xF800u) ? 1u << 11 : 0u;
                    v -= (v & 0xF8000000u) ? 1u << 27 : 0u;
                } else {
                    v -= (v >> 24) ? 1u << 24 : 0u;
                }
                w32[i] = v;
            }
            __syncthreads();
            if (!lone && m + 1 < rl.n_mcs) {
                publish_edges();
                arrive();
                if (!wait()) return;
            }
        }
    }

    // own rows back to the caller's lattice
    {
        const int per = vec ? L0 / 4 : L0;
        const FastDiv by_per((uint32_t)per);
        for (int c = tid; c < per * N1 * P2; c += block) {
            int ry, rz;
            const int r = (int)by_per.div((uint32_t)c), x = c - r * per;
            own_row(r, ry, rz);
            const size_t g = site(ry, rz) + (size_t)x * (vec ? 4 : 1);
            const Cell *w = lab + (ry + P1 * rz) * L0 + x * (vec ? 4 : 1);
            if (vec) {
                *reinterpret_cast<int4 *>(lat + g) = make_int4(label_of(w[0]), label_of(w[1]), label_of(w[2]), label_of(w[3]));
                if (ACT)
                    *reinterpret_cast<uchar4 *>(act + g) =
                        make_uchar4((uint32_t)w[0] >> WordAct<Cell>::kShift, (uint32_t)w[1] >> WordAct<Cell>::kShift,
                                    (uint32_t)w[2] >> WordAct<Cell>::kShift, (uint32_t)w[3] >> WordAct<Cell>::kShift);
            } else {
                lat[g] = label_of(w[0]);
                if (ACT) act[g] = (uint8_t)((uint32_t)w[0] >> WordAct<Cell>::kShift);
            }
        }
    }
    // both counter buffers hold the exact state, and no list is pending
    if (lone) {
        for (int i = tid; i < pt.n_labels; i += block) {
            const int2 v = pairs_lds[parity * pt.n_labels + i];
            reinterpret_cast<int2 *>(counters[0])[i] = v;
            reinterpret_cast<int2 *>(counters[1])[i] = v;
        }
    } else {
        readd(last_li, parity ^ 1);
    }
    for (int off = 32; off > 0; off >>= 1) {
        my_nontrivial += __shfl_xor(my_nontrivial, off);
        my_accepted += __shfl_xor(my_accepted, off);
    }
    if ((tid & 63) == 0) {
        atomicAdd(&sh.stats[0], (unsigned long long)my_nontrivial);
        atomicAdd(&sh.stats[1], (unsigned long long)my_accepted);
    }
    __syncthreads();
    if (tid < 2) atomicAdd(reinterpret_cast<unsigned long long *>(plain(a.stats)) + tid, sh.stats[tid]);
}

// One uncut lattice, one workgroup.
template <typename Cell, int D, bool ACT, bool SINGLE, bool K1, bool EXT>
__global__ void __launch_bounds__(kResidentMaxThreads) resident_kernel(SweepArgs a, ResidentPart pt, ResidentLaunch rl)
{
    sweep_resident<Cell, D, ACT, SINGLE, K1, EXT, true>(a, pt, rl);
}

// A batch: workgroups take the parts in order (a ticket each), so that the
// parts a workgroup waits for have been taken or are taken next, whatever
// the order of dispatch.
//
// Parts of one lattice meet only once all of them run, which takes as many
// free CUs as it has parts: kernels of other streams may hold them for any
// time.  The parts come together first, before anything is written; if they
// do not within gather_limit polls (kCrowdedPolls once it has happened in
// this launch), one of them marks the lattice, all leave it as it is, and
// alone_kernel sweeps it after this launch.  Either all parts find the count
// complete or all find the mark: it is set by compare-and-swap on an
// incomplete count only.
constexpr uint32_t kCrowdedPolls = 4096;
constexpr uint32_t kNoPart = 0xFFFFFFFFu;
__device__ __forceinline__ uint32_t take_part(const ResidentPart *parts, const ResidentLaunch &rl)
{
    const uint32_t ticket = atomicAdd(&rl.bar->ticket, 1u);
    if (ticket >= gridDim.x) return kNoPart;
    const uint32_t n_parts = (uint32_t)parts[ticket].n_parts;
    if (n_parts == 1) return ticket;
    uint32_t *here = rl.arrivals + (size_t)parts[ticket].lattice * kResidentArrivalStride + 1;
    if (rl.gather_limit == 0) {  // no wait at all: every lattice in parts is marked
        __hip_atomic_fetch_or(here, kResidentAlone, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        return kNoPart;
    }
    __hip_atomic_fetch_add(here, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    for (uint32_t polls = 0;;) {
        uint32_t v = agent_load(here);
        if (v & kResidentAlone) return kNoPart;
        if (v == n_parts) return ticket;
        if (polls < rl.gather_limit && (polls < kCrowdedPolls || (polls & 63u) != 0 || agent_load(&rl.bar->crowded) == 0u)) {
            ++polls;
            __builtin_amdgcn_s_sleep(1);
        } else if (__hip_atomic_compare_exchange_strong(here, &v, v | kResidentAlone, __ATOMIC_RELAXED, __ATOMIC_RELAXED,
                                                        __HIP_MEMORY_SCOPE_AGENT)) {
            agent_store(&rl.bar->crowded, 1u);
            return kNoPart;
        }
    }
}

template <typename Cell, int D, bool ACT, bool SINGLE, bool K1, bool EXT>
__global__ void __launch_bounds__(kResidentMaxThreads) batch_resident_kernel(const SweepArgsG *args,
                                                                             const ResidentPart *parts, ResidentLaunch rl)
{
    extern __shared__ __align__(16) unsigned char smem[];
    int &s_ticket = reinterpret_cast<ResidentShared *>(smem)->go;
    if (threadIdx.x == 0) s_ticket = (int)(rl.meet ? take_part(parts, rl) : blockIdx.x);
    __syncthreads();
    const uint32_t ticket = (uint32_t)__builtin_amdgcn_readfirstlane(s_ticket);
    if (ticket >= gridDim.x) return;
    // both tables as constant memory: nothing writes them while the kernel
    // runs, so the compiler reads a value again rather than hold or spill it
    using ConstArgs = const SweepArgsG __attribute__((address_space(4)));
    using ConstPart = const ResidentPart __attribute__((address_space(4)));
    const ConstPart &cp = ((ConstPart *)parts)[ticket];
    const ResidentPart pt{cp.lattice, cp.n_parts, cp.a1, cp.n1, cp.n_labels, cp.hot_cap};
    ConstArgs &a = ((ConstArgs *)args)[pt.lattice];
    // lattices in parts: see resident_pays
    if constexpr (D == 2 && !(K1 && std::is_same<Cell, char32_t>::value)) {
        if (pt.n_parts > 1) {
            sweep_resident<Cell, D, ACT, SINGLE, K1, EXT, false>(a, pt, rl);
            return;
        }
    }
    sweep_resident<Cell, D, ACT, SINGLE, K1, EXT, true>(a, pt, rl);
}

// One activation after another of a lattice whose parts did not come
// together, on one workgroup, from the caller's labels and activities in
// global memory.  It runs only where the GPU is crowded, and is written to be
// short: an accepted copy is a record of its area, added to the counters
// after the activation.
template <bool ACT>
__global__ void __launch_bounds__(kBlock) alone_kernel(const SweepArgs *args, const int64_t *label_off, ResidentLaunch rl)
{
    __shared__ int32_t j_lds[kMaxTypes * kMaxTypes];
    const SweepArgs &a = args[blockIdx.x];
    const int tid = threadIdx.x;
    uint32_t *line = rl.arrivals + (size_t)blockIdx.x * kResidentArrivalStride;
    const bool alone = (line[1] & kResidentAlone) != 0;
    __syncthreads();
    if (tid < 2) line[tid] = 0;
    if (blockIdx.x == 0 && tid == 0) rl.bar->ticket = rl.bar->crowded = 0;
    if (!alone) return;
    if (tid == 0) atomicAdd(&rl.bar->alone, 1u);

    const DeviceModel *m = a.model;
    j_lds[tid] = (int32_t)m->J[tid];
    static_assert(kMaxTypes * kMaxTypes == kBlock, "one entry of J per thread");
    const SharedTables tables{j_lds, m->LG, reinterpret_cast<const TypeParams *>(m->lam_v)};
    const ThrTables tb{m->TM32, m->TL32, m->TI32, m->n_ti};
    const int L0 = a.L[0], L1 = a.L[1], s = a.s, areas = a.na[0] * a.na[1];
    const LdsMap<kDirect> map{L0, L1, L0, L1, 1};
    const uint32_t sd = (uint32_t)(s * s);
    int32_t *cnt = a.counters[0];  // both buffers hold the exact state
    int4 *records = a.dlist[0];    // k per area
    int32_t *n_records = reinterpret_cast<int32_t *>(a.dlist[1]);
    uint32_t nontrivial = 0, accepted = 0;
    auto barrier = [] {
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "agent");
        __syncthreads();
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "agent");
    };
    barrier();
    for (int i_mcs = 0; i_mcs < rl.n_mcs; ++i_mcs) {
        const uint32_t mcs = rl.mcs0 + (uint32_t)i_mcs;
        for (uint32_t alpha = 0; alpha < rl.n_act; ++alpha) {
            const int cx = (int)(alpha & 1), cy = (int)((alpha >> 1) & 1);
            for (int i = tid; i < areas; i += kBlock) {
                const int ax = i % a.na[0], ay = i / a.na[0];
                int4 *own = records + (size_t)i * a.k;
                int n_own = 0;
                for (int j = 0; j < a.k; ++j) {
                    const uint4 u = philox4x32_10(make_uint4((uint32_t)i, mcs, (alpha << 8) | (uint32_t)j, a.lattice_id), a.key0, a.key1);
                    const int o = (int)__umulhi(u.x, sd);
                    const int tx = s * (2 * ax + cx) + o % s, ty = s * (2 * ay + cy) + o / s;
                    const int nsel = (int)(u.y >> 29);
                    const int sx = tx + nb_dx<2>(nsel), sy = ty + nb_dy<2>(nsel);
                    const int t = map.at(tx, ty, 0), src = map.at(sx, sy, 0);
                    const int lt = a.lat[t], ls = a.lat[src];
                    if (lt == ls || lt < 0 || ls < 0) continue;
                    ++nontrivial;
                    const int tt = lt == 0 ? 0 : a.cell_type[lt], ts = ls == 0 ? 0 : a.cell_type[ls];
                    int64_t dso, dsn;
                    if (!evaluate<int32_t, 2, ACT, false, kDirect, true>(
                            a, tb, JRows{}, tables, a.lat, a.act, map, tx, ty, 0, sx, sy, 0, src, lt, ls, tt, ts,
                            seen_counters(cnt, lt, own, n_own, own + kOwnInRegs),
                            seen_counters(cnt, ls, own, n_own, own + kOwnInRegs), u.z, dso, dsn))
                        continue;
                    ++accepted;
                    a.lat[t] = ls;
                    if (ACT) a.act[t] = (uint8_t)(ls >= 1 ? max(m->max_act[ts], 0) : 0);
                    own[n_own++] = make_int4(lt, ls, (int)dso, (int)dsn);
                }
                n_records[i] = n_own;
            }
            barrier();
            for (int i = tid; i < areas; i += kBlock)
                for (int j = 0; j < n_records[i]; ++j) add_deltas(cnt, records[(size_t)i * a.k + j]);
            barrier();
        }
        if (ACT) {
            for (int i = tid; i < L0 * L1; i += kBlock) a.act[i] = (uint8_t)max((int)a.act[i] - 1, 0);
            barrier();
        }
    }
    const int64_t n_labels = label_off[blockIdx.x + 1] - label_off[blockIdx.x];
    for (int64_t i = tid; i < 2 * n_labels; i += kBlock) a.counters[1][i] = cnt[i];
    atomicAdd(reinterpret_cast<unsigned long long *>(a.stats), (unsigned long long)nontrivial);
    atomicAdd(reinterpret_cast<unsigned long long *>(a.stats) + 1, (unsigned long long)accepted);
}

// The attribute belongs to the kernel, which other threads may launch with
// other sizes: always the same value.
template <typename F>
hipError_t allow_lds(F *kernel, size_t lds)
{
    return lds <= 65536 ? hipSuccess
                        : hipFuncSetAttribute(reinterpret_cast<const void *>(kernel),
                                              hipFuncAttributeMaxDynamicSharedMemorySize, 160 * 1024);
}

template <typename Cell, int D, bool ACT, bool SINGLE, bool K1, bool EXT>
hipError_t launch_one(const ResidentCall &c, hipStream_t st)
{
    hipError_t e;
    if (std::is_same<Cell, char16_t>::value && !c.args) return hipErrorInvalidValue;  // batches only
    if (c.args) {
        auto k = batch_resident_kernel<Cell, D, ACT, SINGLE, K1, EXT>;
        if ((e = allow_lds(k, c.lds)) != hipSuccess) return e;
        k<<<c.grid, c.threads, c.lds, st>>>(reinterpret_cast<const SweepArgsG *>(c.args), c.parts, c.launch);
    } else if constexpr (!std::is_same<Cell, char16_t>::value) {
        auto k = resident_kernel<Cell, D, ACT, SINGLE, K1, EXT>;
        if ((e = allow_lds(k, c.lds)) != hipSuccess) return e;
        k<<<1, c.threads, c.lds, st>>>(*c.one, c.whole, c.launch);
    }
    return hipGetLastError();
}

template <typename Cell, int D, bool ACT, bool SINGLE>
hipError_t launch_k(const ResidentCall &c, hipStream_t st)
{
    if (c.k1) return c.ext ? launch_one<Cell, D, ACT, SINGLE, true, true>(c, st)
                           : launch_one<Cell, D, ACT, SINGLE, true, false>(c, st);
    return c.ext ? launch_one<Cell, D, ACT, SINGLE, false, true>(c, st)
                 : launch_one<Cell, D, ACT, SINGLE, false, false>(c, st);
}

}  // namespace

#define CPM_RESIDENT(NAME, CELL, D, ACT)                                        \
    hipError_t NAME(const ResidentCall &c, hipStream_t st)                      \
    {                                                                           \
        return c.single ? launch_k<CELL, D, ACT, true>(c, st)                   \
                        : launch_k<CELL, D, ACT, false>(c, st);                 \
    }
#if CPM_RESIDENT_PART == 0
CPM_RESIDENT(launch_resident_u16_2d, uint16_t, 2, false)
#elif CPM_RESIDENT_PART == 1
CPM_RESIDENT(launch_resident_u16_3d, uint16_t, 3, false)
#elif CPM_RESIDENT_PART == 2
CPM_RESIDENT(launch_resident_act32_2d, char32_t, 2, true)
#elif CPM_RESIDENT_PART == 3
CPM_RESIDENT(launch_resident_act32_3d, char32_t, 3, true)
#elif CPM_RESIDENT_PART == 4
// one cell type, no further terms, batches only
hipError_t launch_resident_act16(const ResidentCall &c, hipStream_t st)
{
    if (c.ndim == 2)
        return c.k1 ? launch_one<char16_t, 2, true, true, true, false>(c, st)
                    : launch_one<char16_t, 2, true, true, false, false>(c, st);
    return c.k1 ? launch_one<char16_t, 3, true, true, true, false>(c, st)
                : launch_one<char16_t, 3, true, true, false, false>(c, st);
}
#elif CPM_RESIDENT_PART == 5
hipError_t launch_resident_alone(const SweepArgs *args, const int64_t *label_off, int n_lattices, bool act,
                                 const ResidentLaunch &rl, hipStream_t st)
{
    if (act) alone_kernel<true><<<n_lattices, kBlock, 0, st>>>(args, label_off, rl);
    else alone_kernel<false><<<n_lattices, kBlock, 0, st>>>(args, label_off, rl);
    return hipGetLastError();
}
#endif

}  // namespace cpm
