// Neighbour search and SPH density on the tree: the paper's Discussion notes
// that its tree serves neighbour search and makes smoothed particle
// hydrodynamics straightforward.  Definitions taken (gather form):
//   * the neighbours of particle i are the j (i included) with
//     d2 <= r_i * r_i, d = x_j - x_i, d2 = (dx*dx + dy*dy) + dz*dz, every
//     operation float32 and rounded (no contraction), so that any
//     implementation decides every pair alike;
//   * rho_i = sum over the neighbours within r_i = 2 h_i of m_j W(|d|, h_i),
//     W the cubic spline of Monaghan & Lattanzio (1985).
//
// One wave64 per group, persistent waves on the walk's per-XCD group queues, and
// eight for a group with many candidates (unless most have as many) or where
// groups are few.  The
// traversal opens a cell when the gap between the group's bounding box and
// the cell's particle box (both float32, from the multipole pass) is within
// the group's largest radius, with a relative margin of 1e-5 on the squared
// radius: the float32 gap can differ from the exact one by a few ulps, and the
// margin makes the test a superset of the pairs the exact predicate admits.
// Opened leaves put their particles on a candidate list in LDS; tiles of 64
// candidates (one per lane) are tested against the group's particles one after
// the other, taken from LDS, or for densities broadcast from their lanes into
// scalar registers, 8 at a time.  Counts go to the lane of their particle by a
// select (no lane-dependent branch inside a loop that holds cross-lane
// operations); list entries are placed by ballot ranks; densities are summed per
// lane, reduced across the wave by three transposed stages and three
// butterflies, moved to their particle's lane, and added up over the waves in
// their order (float64): every run gives the same bits.
#include "mibh_device.h"

namespace mibh {

namespace {

constexpr unsigned NGB_LSTACK = 512;   // LDS part of the cell stack (spills to the global stack)
constexpr unsigned NGB_LIST = 1536;    // candidate list of a group's wave
constexpr unsigned NGB_WAVES = 8;      // waves of a group with more candidates
// Heavy groups up to which they are taken in parts, and beyond which each takes one
// wave after all: a workgroup per part or group costs several times the work of a
// wave, so it is for the groups that would outlast the others.  Densities with 512
// neighbours, us: 131072 particles 678 (parts of every group 2605, one wave for every
// group 3750), 500000 particles 1300 (10244, 2050); up to 8192 heavy groups on eight
// waves 816 at 131072.
constexpr unsigned NGB_FEW = 512;
constexpr unsigned NGB_MANY = 2048;
constexpr unsigned NGB_PART = 8;       // particles of a part of a heavy group
// A group whose list overflows stays with its wave all the same, which tests the
// list whenever it is full, where it is one of many alike: leaving it, the pass would
// walk the tree twice.  It is taken for such a group if it has no more than twice a
// wave's share of the particles, if NGB_LIKE of 64 radii taken evenly from its system
// reach NGB_ALIKE of its largest, and if its box is no denser than its system's.  Each
// depends on the input and the parameters alone.  Counts with these groups left to the
// later passes / staying, us (in brackets one wave for every group from the start), of
// uniform cubes: 60000 particles with 392 / 675 neighbours 119 / 80 (127), 197 / 124 (166),
// 100000 with 400 / 693 136 / 105 (156), 224 / 156 (195), 500000 with 421 / 737 612 / 474
// (513), 1010 / 683 (726), 2^20 with 427 1086 / 824 (870).  (Of 60000 particles whose
// radii are wide in a spot of the cube alone 98, staying there 405 (426).)
constexpr unsigned NGB_LIKE = 48;
constexpr float NGB_ALIKE = 0.7f;
constexpr unsigned NGB_ONE_PASS = 32768;  // particles up to which every group has NGB_WAVES waves
constexpr unsigned NGB_LIST_HEAVY = 4096;
constexpr float NGB_FAR = 1.0e18f;
// Candidates a group lists before its cells are tested against its particles
// one by one.  The test costs a group's wave 14 instructions per particle and
// step; a compact group (400-700 candidates on the spheres) loses by it, a
// group whose box spans more than its particles' radii wins: counts on the
// Plummer sphere (64 neighbours within 2h) with the test from the first cell /
// after 512 / 1024 / 2048 candidates / never: n = 2^17 390 / 394 / 397 / 417 /
// 7703 us, n = 2^20 674 / 659 / 684 / 742 / 4724, n = 2^22 2345 / 2169 / 2169 /
// 2209 / 2202.
constexpr unsigned NGB_REFINE = 512;

__device__ __forceinline__ unsigned lane64() { return __lane_id(); }
__device__ __forceinline__ unsigned uniform(unsigned v) { return __builtin_amdgcn_readfirstlane(v); }
__device__ __forceinline__ unsigned rank_below(unsigned long long mask) {
    return __builtin_amdgcn_mbcnt_hi((unsigned)(mask >> 32), __builtin_amdgcn_mbcnt_lo((unsigned)mask, 0u));
}

// exclusive prefix sum of small per-lane values (0 <= v < 16); *total = wave total
template <int BITS = 4>
__device__ __forceinline__ unsigned small_scan(unsigned v, unsigned *total) {
    unsigned r = 0, t = 0;
#pragma unroll
    for (int b = 0; b < BITS; b++) {
        const unsigned long long m = __ballot((v >> b) & 1u);
        r += rank_below(m) << b;
        t += (unsigned)__popcll(m) << b;
    }
    *total = t;
    return r;
}

__device__ __forceinline__ float readlane_f(float v, unsigned l) {
    return __int_as_float(__builtin_amdgcn_readlane(__float_as_int(v), l));
}

// Bits 0..K-1 of x in reverse order.
template <int K> __device__ __forceinline__ unsigned bitrev_k(unsigned x) {
    unsigned r = 0;
#pragma unroll
    for (int b = 0; b < K; b++) r |= ((x >> b) & 1u) << (K - 1 - b);
    return r;
}

// Sum over the wave of v[0..2^K): lane l ends with the total of
// v[bitrev_k<K>(l >> (6 - K))]; the particle of value p thus sits on the
// lanes bitrev_k<K>(p) << (6 - K) ... + 2^(6-K) - 1.
template <int K>
__device__ __forceinline__ float reduce_pow2(float (&v)[1 << K]) {
    const unsigned ln = lane64();
#pragma unroll
    for (int s = 0; s < K; s++) {
        const int o = 32 >> s;
        const int len = (1 << K) >> s;
        const bool hi = (ln & (unsigned)o) != 0;
#pragma unroll
        for (int p = 0; p < len / 2; p++) {
            const float keep = hi ? v[2 * p + 1] : v[2 * p];
            const float send = hi ? v[2 * p] : v[2 * p + 1];
            v[p] = keep + __shfl_xor(send, o, 64);
        }
    }
    float r = v[0];
#pragma unroll
    for (int o = 32 >> K; o > 0; o >>= 1) r += __shfl_xor(r, o, 64);
    return r;
}

// float32 squared distance, each operation rounded
__device__ __forceinline__ float dist2(float ax, float ay, float az, float bx, float by, float bz) {
#pragma clang fp contract(off)
    const float dx = bx - ax, dy = by - ay, dz = bz - az;
    return (dx * dx + dy * dy) + dz * dz;
}

// float32 squared distance from a particle to the nearest point of a box (min
// xyz, max xyz), each operation rounded, in dist2's order
__device__ __forceinline__ float box_gap2(const float (&b)[6], float4 q) {
#pragma clang fp contract(off)
    const float dx = fmaxf(fmaxf(b[0] - q.x, q.x - b[3]), 0.0f);
    const float dy = fmaxf(fmaxf(b[1] - q.y, q.y - b[4]), 0.0f);
    const float dz = fmaxf(fmaxf(b[2] - q.z, q.z - b[5]), 0.0f);
    return (dx * dx + dy * dy) + dz * dz;
}

// cubic spline W(r, h) with sig = 1/(pi h^3), ih = 1/h
__device__ __forceinline__ float spline(float r, float ih, float sig) {
    const float q = r * ih;
    const float t = 2.0f - q;
    const float inner = fmaf(0.75f * q, q * q, fmaf(-1.5f, q * q, 1.0f));
    const float outer = 0.25f * t * t * t;
    return sig * (q < 1.0f ? inner : (q < 2.0f ? outer : 0.0f));
}

struct NgbArgs {
    Header *hdr;
    unsigned *head;
    const uint4 *topo;
    const float *cbox;
    const float4 *spos;
    const uint32_t *perm;
    const uint2 *groups;
    const float *radius;     // per input particle: radius (count, list) or h (density)
    unsigned share;          // twice a wave's share of the particles
    uint32_t *wstack;
    const uint32_t *order;   // first pass: the groups in the queues' order (NULL: Morton)
    uint8_t *gflag;          // of each group: left by the first pass
    uint32_t *heavy;         // groups left to the second pass (NULL: no first pass, every group)
    uint32_t *count;         // per input particle
    const uint32_t *offset;  // list: first slot of each input particle
    uint32_t *index;         // list: neighbour input indices
    unsigned capacity;       // list: entries of index
    float *rho;              // density
};

enum { NGB_COUNT = 0, NGB_LISTS = 1, NGB_DENSITY = 2 };

// Candidate k of a list of n (a particle far away past the end), and its place.
__device__ __forceinline__ float4 candidate(const NgbArgs &a, const uint32_t *list, unsigned n, unsigned k,
                                            unsigned &e) {
    e = list[min(k, n - 1u)];
    const float4 s = a.spos[e];
    return k < n ? s : make_float4(NGB_FAR, NGB_FAR, NGB_FAR, 0.0f);
}

// Counts or lists the neighbours among the candidates of every NW-th tile of
// list[0..n), from tile w on; s_p: the group's gn particles and squared radii (-1
// past the last).  Bound by the latency of a tile's loads: a tile is loaded once
// for all of the group's particles, and while the one before it is tested.  With
// the positions broadcast into scalar registers, 8 particles per pass over the
// tiles, counts of 2^21 particles took 1080 us; they take 973.
template <bool LISTS, int NW>
__device__ void ngb_test(const NgbArgs &a, const uint32_t *list, unsigned n, unsigned w, unsigned gn,
                         const float4 *s_p, unsigned &cnt, unsigned obase, unsigned ocap) {
    constexpr unsigned STEP = 8;
    const unsigned ln = lane64();
    if (64 * w >= n) return;
    unsigned enext, onext = 0;
    float4 next = candidate(a, list, n, 64 * w + ln, enext);
    if (LISTS) onext = a.perm[enext];
#pragma unroll 1
    for (unsigned t0 = 64 * w; t0 < n; t0 += 64 * NW) {
        const float4 s = next;
        const unsigned oj = onext;
        if (t0 + 64 * NW < n) {
            next = candidate(a, list, n, t0 + 64 * NW + ln, enext);
            if (LISTS) onext = a.perm[enext];
        }
#pragma unroll 1
        for (unsigned j0 = 0; j0 < gn; j0 += STEP) {
#pragma unroll
            for (unsigned u = 0; u < STEP; u++) {
                const unsigned j = j0 + u;
                const float4 q = s_p[j];
                const bool in = dist2(q.x, q.y, q.z, s.x, s.y, s.z) <= q.w;
                const unsigned long long m = __ballot(in);
                if (LISTS) {
                    const unsigned base = __builtin_amdgcn_readlane(obase + cnt, j);
                    const unsigned cap = __builtin_amdgcn_readlane(ocap, j);
                    const unsigned slot = base + rank_below(m);
                    if (in && slot < cap) a.index[slot] = oj;
                }
                cnt += ln == j ? (unsigned)__popcll(m) : 0u;
            }
        }
    }
}

// Counts and density sums of the same candidates, 8 particles per pass over the
// tiles, their values in scalar registers (32 per pass, read from LDS, spilled 75
// scalar registers and took 887 us against 809 at 2^20 particles).
template <int NW>
__device__ void ngb_density(const NgbArgs &a, const uint32_t *list, unsigned n, unsigned w, unsigned gn, float px,
                            float py, float pz, float pr2, float ph, unsigned &cnt, double &rho) {
    constexpr int K = 3, CHUNK = 1 << K;
    const unsigned ln = lane64();
    if (64 * w >= n) return;
    for (unsigned c0 = 0; c0 < gn; c0 += CHUNK) {
        const unsigned cn = min((unsigned)CHUNK, gn - c0);
        float xi[CHUNK], yi[CHUNK], zi[CHUNK], r2i[CHUNK], ihi[CHUNK], sgi[CHUNK];
#pragma unroll
        for (int ii = 0; ii < CHUNK; ii++) {
            const unsigned src = c0 + min((unsigned)ii, cn - 1);
            xi[ii] = readlane_f(px, src);
            yi[ii] = readlane_f(py, src);
            zi[ii] = readlane_f(pz, src);
            // a padding particle (ii >= cn) admits nothing
            r2i[ii] = (unsigned)ii < cn ? readlane_f(pr2, src) : -1.0f;
            const float h = readlane_f(ph, src);
            ihi[ii] = 1.0f / h;
            sgi[ii] = ihi[ii] * ihi[ii] * ihi[ii] * 0.318309886183790672f;  // 1 / (pi h^3)
        }
        float acc[CHUNK];
#pragma unroll
        for (int ii = 0; ii < CHUNK; ii++) acc[ii] = 0.0f;
        unsigned e;
        float4 next = candidate(a, list, n, 64 * w + ln, e);
        for (unsigned t0 = 64 * w; t0 < n; t0 += 64 * NW) {
            const float4 s = next;
            if (t0 + 64 * NW < n) next = candidate(a, list, n, t0 + 64 * NW + ln, e);
#pragma unroll
            for (int ii = 0; ii < CHUNK; ii++) {
                const float d2 = dist2(xi[ii], yi[ii], zi[ii], s.x, s.y, s.z);
                const bool in = d2 <= r2i[ii];
                const unsigned nin = (unsigned)__popcll(__ballot(in));
                const float r = d2 > 0.0f ? d2 * __builtin_amdgcn_rsqf(d2) : 0.0f;
                acc[ii] += in ? s.w * spline(r, ihi[ii], sgi[ii]) : 0.0f;
                cnt += ln == c0 + (unsigned)ii ? nin : 0u;
            }
        }
        const float tot = reduce_pow2<K>(acc);
        const unsigned p = ln - c0;
        const float mine = __shfl(tot, (int)(bitrev_k<K>(p & (CHUNK - 1u)) << (6 - K)), 64);
        rho += ln >= c0 && ln < c0 + cn ? (double)mine : 0.0;
    }
}

// Three passes over the groups (one of NW = NGB_WAVES in small trees: see
// launch_passes).  The first (NW = 1) gives each group a wave and
// leaves those with more than NGB_LIST candidates, unless they are many alike (see
// NGB_LIKE), to the second, which gives each NGB_PART of their particles a
// workgroup of NGB_WAVES waves, as a group of their own (NGB_FEW heavy groups or
// fewer; else whole groups): a cell per thread and step of the traversal, and the
// tiles of candidates dealt to the waves.  Where most groups are heavy, more than
// NGB_MANY, the third pass (ALL, NW = 1) takes them instead, a wave each, and tests
// the list whenever it is full.  How many are heavy depends on the input alone.  The
// first pass takes large trees' groups in the walk's order, the end of each queue by
// size (density of 250007 particles 313 us in Morton order, 240 so).  In a sphere's
// outskirts a radius that reaches 64 neighbours may reach the whole core: with one
// wave for every group the pass lasted as long as that group, whatever n.
template <int MODE, int NW, bool ALL>
__global__ __launch_bounds__(64 * NW, 4) void k_neighbors(NgbArgs a) {
    constexpr bool HEAVY = NW > 1, REST = NW == 1 && ALL;  // REST: the third pass
    static_assert(ALL || NW == 1, "only a first pass leaves groups");
    constexpr float SCALE = MODE == NGB_DENSITY ? 2.0f : 1.0f;  // search radius to the caller's
    constexpr unsigned NT = 64 * NW, STEP = HEAVY ? 256u : 64u;  // cells taken per step at most
    constexpr unsigned RING = HEAVY ? 16u * STEP : NGB_LSTACK, MASK = RING - 1;
    constexpr unsigned LIST = HEAVY ? NGB_LIST_HEAVY : NGB_LIST;
    static_assert((RING & MASK) == 0 && RING >= 8 * STEP && STEP <= NT, "stack ring must hold one step's pushes");
    // Steps of 64 cells leave at most 512 pushes per level on the stack.  Wider
    // ones are taken from WIDE cells or fewer, so that they leave RING at most;
    // with 20 levels of 512 above those the spill, which moves in half rings,
    // stays within STACK_CAP.
    constexpr unsigned WIDE = RING / 2;
    static_assert(!HEAVY || (WIDE + 8 * STEP <= RING && KEY_LEVELS * 512u <= STACK_CAP / WIDE * WIDE), "stack bound");
    __shared__ uint32_t s_stk[RING];
    __shared__ uint32_t s_list[LIST];
    __shared__ float4 s_p[64];  // the group's particles and squared radii (-1 past the last)
    __shared__ unsigned s_cnt[2][NW][4];
    __shared__ unsigned s_pcnt[HEAVY ? NW : 1][64];  // each wave's counts
    __shared__ float s_rho[HEAVY ? NW : 1][64];
    const unsigned ln = lane64(), t = NW > 1 ? threadIdx.x : ln, w = NW > 1 ? uniform(threadIdx.x >> 6) : 0u;
    uint32_t *gstk = a.wstack + (size_t)blockIdx.x * STACK_CAP;
    if (a.hdr->flags & (FLAG_NONFINITE | FLAG_NEGMASS | FLAG_CELLCAP)) return;
    constexpr unsigned per_round = 8;  // particles per thread: a round always fits an empty list
    static_assert(per_round * STEP <= LIST, "a round fits");
    const unsigned nheavy = ALL && a.heavy ? uniform(a.hdr->ngb_heavy) : 0u;
    if (HEAVY && nheavy > NGB_MANY) return;
    if (REST && nheavy <= NGB_MANY) return;
    // slots: the groups, or the heavy ones' parts
    const unsigned part = HEAVY && a.heavy && nheavy <= NGB_FEW ? NGB_PART : 64u, nparts = 64u / part;
    const unsigned ngroups = (HEAVY && a.heavy ? nheavy : uniform(a.hdr->ngroups)) * nparts;
    QueueCursor qc = queue_start();
    unsigned par = 0;
    // sums over the workgroup of each wave's v (the same in all its lanes), before this wave and in all
    auto exchange = [&](const unsigned (&v)[4], unsigned (&before)[4], unsigned (&all)[4]) {
#pragma unroll
        for (int k = 0; k < 4; k++) {
            before[k] = 0;
            all[k] = v[k];
        }
        if (NW == 1) return;
        par ^= 1u;
#pragma unroll
        for (int k = 0; k < 4; k++) s_cnt[par][w][k] = v[k];
        __syncthreads();
#pragma unroll
        for (int k = 0; k < 4; k++) {
            all[k] = 0;
#pragma unroll
            for (unsigned u = 0; u < NW; u++) {
                const unsigned x = uniform(s_cnt[par][u][k]);
                before[k] += u < w ? x : 0u;
                all[k] += x;
            }
        }
    };
    for (unsigned slot = blockIdx.x;; slot += gridDim.x) {
        // every lane takes part in the queue atomic (see the walk's queue loop)
        if (!HEAVY) slot = queue_next(REST ? a.hdr->prefix_head : a.head, ngroups, qc);
        if (slot >= ngroups) break;
        const unsigned k = HEAVY ? slot / nparts : slot;
        const unsigned g = HEAVY ? (a.heavy ? uniform(a.heavy[k]) : k) : (a.order ? uniform(a.order[k]) : k);
        if (REST && uniform(a.gflag[g]) == 0u) continue;
        const uint2 gr = a.groups[g];
        const unsigned p0 = HEAVY ? slot % nparts * part : 0u, gall = uniform(gr.y & 255u);
        if (HEAVY && p0 >= gall) continue;  // the same for the whole workgroup
        const unsigned gf = uniform(gr.x) + p0, gn = min(gall - p0, part);
        const unsigned root = uniform(gr.y >> 16);
        const unsigned mine = gf + min(ln, gn - 1);
        const float4 p = a.spos[mine];
        const unsigned oi = a.perm[mine];
        const float hr = a.radius[oi];
        const float rr = SCALE * hr;
        const float pr2 = rr * rr;
        // (every wave writes the same values)
        s_p[ln] = make_float4(p.x, p.y, p.z, ln < gn ? pr2 : -1.0f);
        float bmin[3] = {p.x, p.y, p.z}, bmax[3] = {p.x, p.y, p.z};
        float rmax = rr;
#pragma unroll
        for (int o = 32; o > 0; o >>= 1) {
#pragma unroll
            for (int d = 0; d < 3; d++) {
                bmin[d] = fminf(bmin[d], __shfl_xor(bmin[d], o, 64));
                bmax[d] = fmaxf(bmax[d], __shfl_xor(bmax[d], o, 64));
            }
            rmax = fmaxf(rmax, __shfl_xor(rmax, o, 64));
        }
        const float open2 = rmax * rmax * (1.0f + 1.0e-5f);
        unsigned cnt = 0, cand = 0;  // cand: candidates listed so far
        double rho = 0.0;  // (in float32 the lists' sums of a group with several would each round)
        const unsigned obase = MODE == NGB_LISTS ? a.offset[oi] : 0u;
        const unsigned ocap = MODE == NGB_LISTS ? min(a.offset[oi] + a.count[oi], a.capacity) : 0u;

        // The root holds every particle, so every search opens it: its
        // children (the root itself when it is a leaf) start the stack.
        const uint4 tr = a.topo[root];
        const unsigned rn = uniform(tr.w & 255u);
        unsigned sb = 0, st = rn ? rn : 1u, gtop = 0, nl = 0;
        bool overflow = false, later = false, stay = false, full = false;
        unsigned m = 0, nl0 = 0;  // cells of a step, candidates listed before it
        auto test_list = [&]() {
            __syncthreads();
            if (MODE == NGB_DENSITY) {
                ngb_density<NW>(a, s_list, nl, w, gn, p.x, p.y, p.z, pr2, hr, cnt, rho);
            } else if (HEAVY && MODE == NGB_LISTS) {  // the waves' counts first: where each one's entries go
                unsigned own = 0;
                ngb_test<false, NW>(a, s_list, nl, w, gn, s_p, own, 0u, 0u);
                s_pcnt[w][ln] = own;
                __syncthreads();
                unsigned at = cnt;
#pragma unroll
                for (unsigned u = 0; u < NW; u++) {
                    const unsigned x = s_pcnt[u][ln];
                    at += u < w ? x : 0u;
                    cnt += x;
                }
                ngb_test<true, NW>(a, s_list, nl, w, gn, s_p, at, obase, ocap);
            } else {
                ngb_test<MODE == NGB_LISTS, NW>(a, s_list, nl, w, gn, s_p, cnt, obase, ocap);
            }
            nl = 0;
            __syncthreads();
        };
        const unsigned first = rn ? tr.z + min(ln, rn - 1) : root;
        if (ln < st) s_stk[ln] = first;
        __syncthreads();
        do {  // (once, but for a first pass whose list is full before the stack is empty)
        full = false;
        while (st != sb || gtop > 0) {
            if (st == sb) {  // refill the LDS part of the stack from the global spill
                const unsigned k = min(gtop, RING / 2);
                __threadfence_block();
                for (unsigned i = t; i < k; i += NT) s_stk[(sb - k + i) & MASK] = gstk[gtop - k + i];
                sb -= k;
                gtop -= k;
                __syncthreads();
            }
            nl0 = nl;
            m = min(st - sb, HEAVY && gtop + (st - sb) <= WIDE ? STEP : 64u);
            const bool valid = t < m;
            const unsigned c = valid ? s_stk[(st - m + t) & MASK] : 0u;
            st -= m;
            const uint4 tc = a.topo[c];
            const unsigned nch = tc.w & 255u;
            bool open = false;
            float bx[6] = {0.0f, 0.0f, 0.0f, 0.0f, 0.0f, 0.0f};  // the cell's particle box: min xyz, max xyz
            if (valid) {
#pragma clang fp contract(off)
                const float2 *cb = reinterpret_cast<const float2 *>(a.cbox + 6 * (size_t)c);
                const float2 b0 = cb[0], b1 = cb[1], b2 = cb[2];
                bx[0] = b0.x; bx[1] = b0.y; bx[2] = b1.x;
                bx[3] = b1.y; bx[4] = b2.x; bx[5] = b2.y;
                float gap2 = 0.0f;
#pragma unroll
                for (int d = 0; d < 3; d++) {
                    const float u = bx[d] - bmax[d];
                    const float v = bmin[d] - bx[3 + d];
                    const float gp = fmaxf(fmaxf(u, v), 0.0f);
                    gap2 = gap2 + gp * gp;
                }
                open = gap2 <= open2;
            }
            // The cells the group's box reaches, against its particles one by
            // one: a cell stays open when it is within some particle's radius.
            // Without it a group in a sphere's outskirts (a large box, large
            // radii) listed the whole core: one wave took 22 ms of a density
            // pass of 250007 particles that now takes 0.33 ms.
            // The gap to a particle is taken as the pair predicate takes the
            // distance (same operations, same order), and each rounded step of
            // it is at most the same step for any particle of the cell, so no
            // pair that the predicate admits is lost.
            if (cand >= NGB_REFINE && __ballot(open)) {
                bool hit = false;
                for (unsigned j0 = 0; j0 < gn; j0 += 4) {
#pragma unroll
                    for (unsigned u = 0; u < 4; u++) hit = hit | (box_gap2(bx, s_p[j0 + u]) <= s_p[j0 + u].w);
                    if (!__ballot(open & !hit)) break;
                }
                open = open & hit;
            }
            // opened leaves' particles go to the candidate list, opened internal
            // cells' children onto the stack: places by one scan of each.  Leaves
            // go whole where each holds fewer than 32 particles and they fit an
            // empty list, else in rounds; the list is tested when they do not fit.
            unsigned rem = open && nch == 0 ? tc.y : 0u, src = tc.x;
            const unsigned nc = open && nch != 0 ? nch : 0u;
            unsigned wsum[4], before[4], all[4];
            const bool big = __ballot(rem > 31u) != 0;
            unsigned loff = 0;
            wsum[0] = 0;
            if (!big && __ballot(rem > 0)) loff = small_scan<5>(rem, &wsum[0]);
            const unsigned coff = small_scan(nc, &wsum[1]);
            wsum[2] = big ? 1u : 0u;
            wsum[3] = 0;
            exchange(wsum, before, all);  // (the popped entries have been read by now)
            const unsigned nsum = all[1];
            if (all[2] == 0 && all[0] <= LIST) {
                if (all[0]) {
                    if (nl + all[0] > LIST) {
                        if (!ALL) {
                            full = true;
                            break;
                        }
                        test_list();
                    }
                    for (unsigned j = 0; j < rem; j++) s_list[nl + before[0] + loff + j] = src + j;
                    nl += all[0];
                    cand += all[0];
                }
            } else {
                for (;;) {
                    unsigned rsum[4] = {0u, 0u, 0u, 0u}, rb[4], ra[4];
                    const unsigned take = min(rem, per_round);
                    const unsigned off = small_scan(take, &rsum[0]);
                    exchange(rsum, rb, ra);
                    if (ra[0] == 0) break;
                    if (nl + ra[0] > LIST) {
                        if (!ALL) {
                            full = true;
                            break;
                        }
                        test_list();
                    }
                    for (unsigned j = 0; j < take; j++) s_list[nl + rb[0] + off + j] = src + j;
                    nl += ra[0];
                    cand += ra[0];
                    rem -= take;
                    src += take;
                }
                if (full) break;
            }
            const unsigned used = st - sb;
            if (used + nsum > RING) {  // spill the bottom of the LDS ring
                const unsigned need = used + nsum - RING;
                const unsigned sp = min(used, max(need, RING / 2));
                if (gtop + sp > STACK_CAP) {
                    overflow = true;
                    break;
                }
                for (unsigned i = t; i < sp; i += NT) gstk[gtop + i] = s_stk[(sb + i) & MASK];
                sb += sp;
                gtop += sp;
                __syncthreads();
            }
            for (unsigned j = 0; j < nc; j++) s_stk[(st + before[1] + coff + j) & MASK] = tc.z + j;
            st += nsum;
            __syncthreads();
        }
        if (!ALL && full) {  // the list does not take this step's candidates: the step is taken back
            cand -= nl - nl0;
            nl = nl0;
            st += m;
            if (!stay && nl > 0 && gn <= a.share) {
                const unsigned sample = tr.x + (unsigned)((2u * ln + 1u) * (unsigned long long)tr.y >> 7);
                const float other = SCALE * a.radius[a.perm[sample]];
                stay = (unsigned)__popcll(__ballot(other >= NGB_ALIKE * rmax)) >= NGB_LIKE;
                // the particles that the system's mean density would put into the group's
                // box, widened by their mean distance
                const float gap = cbrtf(1.0f / (float)tr.y);
                const float *rb = a.cbox + 6 * (size_t)root;
                float mean = (float)tr.y;
#pragma unroll
                for (int d = 0; d < 3; d++) {
                    const float ext = rb[3 + d] - rb[d];
                    mean *= ext > 0.0f ? fminf((bmax[d] - bmin[d]) / ext + gap, 1.0f) : 1.0f;
                }
                stay = stay && (float)gn <= readlane_f(mean, 0);
            }
            later = nl == 0 || !stay;
            if (later) break;
        }
        if (!overflow && nl > 0) test_list();
        } while (!ALL && full);
        if (!ALL) a.gflag[g] = later ? 1 : 0;
        if (later) {
            // (every lane stores the same word: no lane-dependent branch in this loop)
            a.heavy[uniform(atomicAdd(&a.hdr->ngb_heavy, ln == 0 ? 1u : 0u))] = g;
            continue;
        }
        if (overflow) {
            atomicOr(&a.hdr->flags, FLAG_STACK);
        } else if (HEAVY) {
            if (MODE != NGB_LISTS) {
                s_pcnt[w][ln] = cnt;
                s_rho[w][ln] = (float)rho;
                __syncthreads();
                if (w == 0 && ln < gn) {
                    // the waves' sums in float64, rounded once: added in float32 one
                    // after the other, the rms error of a density of 4096 particles
                    // was 8.0e-8 (7.7e-8 with one wave per group)
                    double sum = rho;
                    for (unsigned u = 1; u < NW; u++) {
                        cnt += s_pcnt[u][ln];
                        sum += (double)s_rho[u][ln];
                    }
                    a.count[oi] = cnt;
                    if (MODE == NGB_DENSITY) a.rho[oi] = (float)sum;
                }
            }
        } else if (ln < gn) {
            if (MODE != NGB_LISTS) a.count[oi] = cnt;
            if (MODE == NGB_DENSITY) a.rho[oi] = (float)rho;
        }
        if (HEAVY) __syncthreads();  // the LDS arrays are free again
    }
}

// Exclusive scan of n counts into off[0..n] (off[n] = total) in tiles of 1024:
// tile sums, one block scanning the tile sums, tiles scanned with their offset.
constexpr unsigned SCAN_TILE = 1024;

__global__ __launch_bounds__(256) void k_scan_tiles(const uint32_t *__restrict__ in, unsigned n,
                                                    uint32_t *__restrict__ tsum) {
    __shared__ unsigned s[4];
    const unsigned b = blockIdx.x * SCAN_TILE;
    unsigned v = 0;
    for (unsigned i = threadIdx.x; i < SCAN_TILE; i += 256) v += b + i < n ? in[b + i] : 0u;
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o, 64);
    if ((threadIdx.x & 63u) == 0u) s[threadIdx.x >> 6] = v;
    __syncthreads();
    if (threadIdx.x == 0) tsum[blockIdx.x] = s[0] + s[1] + s[2] + s[3];
}

__global__ __launch_bounds__(1024) void k_scan_sums(uint32_t *__restrict__ tsum, unsigned ntiles) {
    __shared__ unsigned s_w[16];
    const unsigned t = threadIdx.x, ln = lane64(), w = t >> 6;
    const unsigned per = (ntiles + 1023u) / 1024u;
    unsigned sum = 0;
    for (unsigned i = 0; i < per; i++) sum += t * per + i < ntiles ? tsum[t * per + i] : 0u;
    unsigned x = sum;
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) {
        const unsigned y = __shfl_up(x, o, 64);
        x += ln >= (unsigned)o ? y : 0u;
    }
    if (ln == 63) s_w[w] = x;
    __syncthreads();
    unsigned run = x - sum;
    for (unsigned i = 0; i < w; i++) run += s_w[i];
    for (unsigned i = 0; i < per; i++) {
        if (t * per + i < ntiles) {
            const unsigned v = tsum[t * per + i];
            tsum[t * per + i] = run;
            run += v;
        }
    }
}

__global__ __launch_bounds__(SCAN_TILE) void k_scan_apply(const uint32_t *__restrict__ in, unsigned n,
                                                           const uint32_t *__restrict__ tsum,
                                                           uint32_t *__restrict__ out) {
    __shared__ unsigned s_w[SCAN_TILE / 64];
    const unsigned t = threadIdx.x, ln = lane64(), w = t >> 6;
    const unsigned i = blockIdx.x * SCAN_TILE + t;
    const unsigned v = i < n ? in[i] : 0u;
    unsigned x = v;
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) {
        const unsigned y = __shfl_up(x, o, 64);
        x += ln >= (unsigned)o ? y : 0u;
    }
    if (ln == 63) s_w[w] = x;
    __syncthreads();
    unsigned run = tsum[blockIdx.x] + x - v;
    for (unsigned k = 0; k < w; k++) run += s_w[k];
    if (i < n) out[i] = run;
    if (i == n - 1) out[n] = run + v;
}

// With few groups each takes NGB_WAVES waves at once; with many their waves fill
// the chip and only the heavy ones do, in parts.  Density passes of a Plummer sphere
// (64 neighbours within 2h) one way / the other, us: 1000 46 / 103, 5000 74 / 175,
// 20000 202 / 273, 50000 480 / 407, 65536 823 / 500 (one wave for every group: 125,
// 315, 1096, -, 5196; heavy groups in one part: 65536 991, 70000 881 against 502,
// 131072 313 against 250; parts of 16 or 4: 70000 600, 517).
template <int MODE>
void launch_passes(NgbArgs a, unsigned n, unsigned waves, hipStream_t s) {
    const bool one = n <= NGB_ONE_PASS;
    if (one) a.heavy = nullptr;
    else hipLaunchKernelGGL((k_neighbors<MODE, 1, false>), dim3(waves), dim3(64), 0, s, a);
    hipLaunchKernelGGL((k_neighbors<MODE, NGB_WAVES, true>), dim3(one ? waves : min(waves, 512u)),
                       dim3(64 * NGB_WAVES), 0, s, a);
    if (!one) hipLaunchKernelGGL((k_neighbors<MODE, 1, true>), dim3(waves), dim3(64), 0, s, a);
}

}  // namespace

hipError_t launch_neighbors(const Buffers &b, int mode, const float *radius, uint32_t *count, const uint32_t *offset,
                            uint32_t *index, int64_t capacity, float *rho, unsigned n, unsigned nsys, hipStream_t s) {
    NgbArgs a;
    a.hdr = b.hdr;
    a.head = b.hdr->walk_head;
    a.topo = b.topo;
    a.cbox = b.cbox;
    a.spos = b.spos;
    a.perm = b.vals[0];
    a.groups = b.groups;
    a.radius = radius;
    a.share = (unsigned)std::min<uint64_t>(2ull * n / b.walk_waves, 64u);
    a.wstack = b.wstack;
    a.heavy = b.nheavy;
    a.gflag = b.gflag;
    a.order = nullptr;
    a.count = count;
    a.offset = offset;
    a.index = index;
    a.capacity = (unsigned)std::min<int64_t>(capacity, 0xffffffffll);
    a.rho = rho;
    // the heads of the first and third passes' queues and the number of heavy groups
    static_assert(offsetof(Header, prefix_head) == offsetof(Header, walk_head) + sizeof(Header::walk_head) + 256 &&
                      offsetof(Header, ngb_heavy) == offsetof(Header, walk_head) + sizeof(Header::walk_head),
                  "one fill");
    hipError_t e = launch_fill_u32(b.hdr->walk_head, 2 * WALK_QUEUES * QUEUE_STRIDE + 64, 0u, s);
    if (e != hipSuccess) return e;
    if (n > NGB_ONE_PASS && walk_sorts_groups(n)) {
        if ((e = launch_group_order(b, n, s)) != hipSuccess) return e;
        a.order = b.gorder;
    }
    if (mode == NGB_COUNT) launch_passes<NGB_COUNT>(a, n, b.walk_waves, s);
    else if (mode == NGB_LISTS) launch_passes<NGB_LISTS>(a, n, b.walk_waves, s);
    else launch_passes<NGB_DENSITY>(a, n, b.walk_waves, s);
    return hipGetLastError();
}

hipError_t launch_scan_u32(const uint32_t *in, unsigned n, uint32_t *out, uint32_t *tmp, hipStream_t s) {
    const unsigned ntiles = (n + SCAN_TILE - 1) / SCAN_TILE;
    hipLaunchKernelGGL(k_scan_tiles, dim3(ntiles), dim3(256), 0, s, in, n, tmp);
    hipLaunchKernelGGL(k_scan_sums, dim3(1), dim3(1024), 0, s, tmp, ntiles);
    hipLaunchKernelGGL(k_scan_apply, dim3(ntiles), dim3(SCAN_TILE), 0, s, in, n, tmp, out);
    return hipGetLastError();
}

}  // namespace mibh
