// Internal definitions shared by the HIP kernels and the host library.
#pragma once

#include <hip/hip_runtime.h>
#include <math.h>
#include <stdint.h>

namespace mibh {

constexpr int KEY_LEVELS = 20;          // 20 bits per axis, 60-bit keys, levels 0..20
constexpr int NCOUNTERS = 22;           // per-block counters of the build: levels 0..20, groups

constexpr int RADIX_BITS = 8;
constexpr int RADIX = 1 << RADIX_BITS;
constexpr int SORT_PASSES = 8;          // 64 bits in 8-bit digits (bits 60..63 are zero)
// Sort tiles of 512 threads x 8 keys: longer runs of each digit per tile, so
// the scatter's stores coalesce better (eight passes at N = 2^22: 256 x 8
// 475 us, 512 x 8 405 us, 512 x 6 or x 10 432 us, 768 x 8 468 us, 1024 x 8 421 us).
#ifndef MIBH_SORT_THREADS
#define MIBH_SORT_THREADS 512
#endif
constexpr int SORT_THREADS = MIBH_SORT_THREADS;  // a multiple of RADIX, <= 1024
#ifndef MIBH_SORT_ITEMS
#define MIBH_SORT_ITEMS 8
#endif
constexpr int SORT_ITEMS = MIBH_SORT_ITEMS;  // keys per thread per tile
constexpr int SORT_TILE = SORT_THREADS * SORT_ITEMS;

// particles per build block (tree construction at N = 2^22: 256 175 us, 512 150 us, 1024 162 us)
#ifndef MIBH_BUILD_THREADS
#define MIBH_BUILD_THREADS 512
#endif
constexpr int BUILD_THREADS = MIBH_BUILD_THREADS;
constexpr int MAX_WINDOW = 64;          // largest ncrit and group_cap (a build wave's window reach)
constexpr unsigned MP_FAN = 64;         // ranges per workgroup of the multipole pass' merge launches
// Particles per workgroup of the multipole pass.  Smaller chunks reach more compute
// units and have shorter chains of rounds, but more cells that leave them, whose
// merges take about 10 us for every MP_FAN chunks: so 1024 while one merge is enough
// (20000 particles, us: 2048 38, 1024 31, 512 31; 45000 with 1024 and two merges:
// a cube 28 against 26).  Leaves of few particles make many cells: with ncrit 1, us,
// 2048 / 1024 / 512: 3000 87 / 65 / 41, 20000 96 / 69 / 47, 100003 105 / 86 / 87,
// 300007 133 / 112 / -, 2^20 243 / 257 / 250; with ncrit 4 3000 45 / 40 / 32, 20000 52 /
// 42 / 34, 100003 57 / 55 / 66.
constexpr unsigned MP_SMALL_MAX = 512u * MP_FAN, MP_FINE_MAX = 1u << 19;
__host__ inline unsigned multipole_chunk(unsigned n, unsigned ncrit) {
    if (n <= 1024u) return 1024;
    if (n <= 2048u) return ncrit < 3u ? 512 : 2048;
    if (n <= MP_SMALL_MAX) return ncrit < 8u ? 512 : 1024;
    return n <= MP_FINE_MAX && ncrit < 3u ? 1024 : 2048;
}
constexpr int BBOX_BLOCKS = 1024;
constexpr int ENERGY_BLOCKS = 1024;
constexpr int ENERGY_THREADS = 256;

// Walk: one wave per workgroup; cell stack bound (see walk kernel): every
// traversal step pushes at most 64*8 children and at most one step's pushes
// per level are on the stack at any time, so 1 + 20*512 entries suffice.
constexpr unsigned STACK_CAP = 21u * 512u;

enum : unsigned {
    FLAG_NONFINITE = 1u,
    FLAG_NEGMASS = 2u,
    FLAG_STACK = 4u,
    FLAG_CELLCAP = 8u,
};

// Per-system root cube: corner lo (x, y, z) and side 2^k.
struct SysCube {
    float lo[3];
    int k;
};

constexpr int MAX_SYSTEMS = 256;        // systems per batch (one extra 8-bit sort pass)
constexpr int MLP_IN = 8, MLP_H = 64;   // work estimator 8 -> 64 -> 64 -> 1
constexpr int MLP_NPARAM = MLP_H * MLP_IN + MLP_H + MLP_H * MLP_H + MLP_H + MLP_H + 1;  // 4801
constexpr int BBOX_MIN_BLOCKS = 16;     // bounding-box blocks per system at least

// Device-resident per-context state, rewritten by every build (zeroed once
// when the context is created).
struct Header {
    unsigned nsys;          // systems in the current batch (1 for a single system)
    unsigned flags;         // conditions met since the current build started
    unsigned sticky;        // flags of the earlier builds since the drivers last cleared it
    unsigned n;
    unsigned ncells;
    unsigned ngroups;
    unsigned lvl_begin[24]; // cells of level l are [lvl_begin[l], lvl_begin[l+1]), l = 0..20
    // Heads of the walks' group queues (one per XCD, 256 bytes apart).  Every
    // wave of a walk increments them, so they sit on cache lines of their own:
    // sharing a line with the fields above, which every wave reads, made the
    // walk 1.8 times slower.
    alignas(256) unsigned walk_head[8 * 64];
    // Neighbour searches: number of groups left to the second pass (next to the
    // heads: cleared with them).
    alignas(256) unsigned ngb_heavy;
    // Shared-prefix walk: heads of the anchor pass's queues (as walk_head), then
    // the allocation head of the anchor-list pool and the number of anchors.
    alignas(256) unsigned prefix_head[8 * 64];
    alignas(256) unsigned long long pool_head;
    unsigned anchor_count;
    unsigned anchor_fail;  // anchors whose lists did not fit
    unsigned pool_pad[60];
};

// Group queues of the persistent walks.  gfx950 deals the workgroups of a
// launch to its 8 XCDs in turn (workgroup i to XCD i mod 8), and each XCD has
// its own L2.  Queue q holds the slots [q n / 8, (q + 1) n / 8) of the
// processing order (Morton order by default), so the waves of one XCD walk
// neighbouring groups, whose cells they then share in that XCD's L2.  A wave
// takes slots from its XCD's queue, then from the following queues in turn as
// each runs empty, and stops when all are empty.  Where the launch has a
// workgroup for every slot, each takes the slot of its number within its XCD's
// eighth and no queue is touched: the eight failing atomics in a row that end a
// wave took 20-30 us of such a walk.  ONCE = false leaves that case out, for the
// walk of large trees: the code cost its full register file 1.5% of a step.
// (Reading all eight heads at once when one runs empty cost it 2-3%.)
constexpr unsigned WALK_QUEUES = 8;
constexpr unsigned QUEUE_STRIDE = 64;  // words between queue heads

struct QueueCursor {
    unsigned q, tried;  // queue in use, queues found empty (one slot per workgroup: 0 until it was taken)
};

__device__ __forceinline__ QueueCursor queue_start() { return QueueCursor{blockIdx.x % WALK_QUEUES, 0u}; }

// Next slot for the calling wave, or n when there is none.  Every lane calls it
// (lane 0 adds 1, the others 0), so no lane-dependent branch is needed around
// it.
template <bool ONCE = true>
__device__ __forceinline__ unsigned queue_next(unsigned *heads, unsigned n, QueueCursor &qc) {
    const unsigned per = (n + WALK_QUEUES - 1u) / WALK_QUEUES;
    if (ONCE && per * WALK_QUEUES <= gridDim.x) {
        const unsigned k = blockIdx.x / WALK_QUEUES;
        const bool take = qc.tried == 0u && k < per;
        qc.tried = 1u;
        return take ? min(qc.q * per + k, n) : n;
    }
    while (qc.tried < WALK_QUEUES) {
        const unsigned lo = (unsigned)((unsigned long long)n * qc.q / WALK_QUEUES);
        const unsigned hi = (unsigned)((unsigned long long)n * (qc.q + 1u) / WALK_QUEUES);
        const unsigned s = __builtin_amdgcn_readfirstlane(
            atomicAdd(heads + QUEUE_STRIDE * qc.q, __lane_id() == 0 ? 1u : 0u));
        if (s < hi - lo) return lo + s;
        qc.tried++;
        qc.q = (qc.q + 1u) % WALK_QUEUES;
    }
    return n;
}

// Order of the walk's queue in large trees: the last GORD_WINDOW slots of each
// XCD's eighth by the groups' particle counts, largest first.  Blocks of
// GORD_BLOCK slots count their groups by (eighth, count); a block meets two
// eighths at most when there are GORD_MIN slots or more (shorter queues keep
// Morton order).  A walk ends when its last group does, and a group of 64
// particles takes about four times as long as one of 16: with the small groups
// last, the waves end together.  Only the end of a queue matters for that, and
// the order costs L2 hits (neighbouring groups read the same cells): walks with
// windows of 2048 / 4096 / 8192 / 16384 / all slots take, in us, 1430 / 1395 /
// 1418 / 1415 / 1440 at 2^20 Plummer particles, 2800 / 2680 / 2750 / 2780 / - at
// 2^21 and 5515 / 5470 / 5430 / 5565 / 5850 at 2^22 (Morton order: 1540 at 2^20,
// 5635 at 2^22).
constexpr unsigned GORD_BLOCK = 512;
constexpr unsigned GORD_CLASSES = 64;
constexpr unsigned GORD_MIN = WALK_QUEUES * GORD_BLOCK;
constexpr unsigned GORD_WINDOW = 4096;
__device__ __forceinline__ unsigned gord_begin(unsigned n, unsigned q) {  // first slot of queue q of n slots
    return (unsigned)((unsigned long long)n * q / WALK_QUEUES);
}
__device__ __forceinline__ unsigned gord_eighth(unsigned n, unsigned i) {  // the queue that holds slot i
    const unsigned q = (unsigned)((unsigned long long)WALK_QUEUES * i / n);
    return q + (gord_begin(n, q + 1u) <= i ? 1u : 0u);
}
__device__ __forceinline__ unsigned gord_window(unsigned n, unsigned q) {  // first slot of queue q's window
    const unsigned lo = gord_begin(n, q), hi = gord_begin(n, q + 1u);
    return hi - lo > GORD_WINDOW ? hi - GORD_WINDOW : lo;
}
__device__ __forceinline__ unsigned gord_class(uint2 group) { return (GORD_CLASSES - (group.y & 255u)) % GORD_CLASSES; }

// Counts of the groups in the queue's windows; `order` NULL: Morton order.  Called
// by whole workgroups of 256.
__device__ __forceinline__ void gord_count(const uint2 *groups, const uint32_t *order, unsigned n, uint32_t *ghist) {
    __shared__ unsigned s_h[2 * GORD_CLASSES];
    if (n < GORD_MIN) return;
    for (unsigned b = blockIdx.x; b * GORD_BLOCK < n; b += gridDim.x) {
        if (threadIdx.x < 2 * GORD_CLASSES) s_h[threadIdx.x] = 0;
        __syncthreads();
        const unsigned i0 = b * GORD_BLOCK, e0 = gord_eighth(n, i0);
        for (unsigned i = i0 + threadIdx.x; i < min(i0 + GORD_BLOCK, n); i += 256u) {
            const unsigned e = gord_eighth(n, i);
            if (i >= gord_window(n, e))
                atomicAdd(&s_h[(e - e0) * GORD_CLASSES + gord_class(groups[order ? order[i] : i])], 1u);
        }
        __syncthreads();
        if (threadIdx.x < 2 * GORD_CLASSES) ghist[(size_t)b * 2 * GORD_CLASSES + threadIdx.x] = s_h[threadIdx.x];
        __syncthreads();
    }
}

// Walk queue order by predicted or measured work: quarter-octave buckets of
// log2(work), heaviest first, Morton order within a bucket.
constexpr int ORDER_BUCKETS = 128;
constexpr int ORDER_BLOCKS = 256;

// Walk: LDS capacities per wave (one wave per workgroup).
constexpr unsigned WALK_LSTACK = 512;   // cell stack in LDS (spills to the global stack)
// Shared-prefix walk: per-wave scratch for an anchor cell's lists: the cells it
// accepts (F), then the cells left for each group, raw and sorted by level (S).
constexpr unsigned PREFIX_F_CAP = 3072;
constexpr unsigned PREFIX_S_CAP = 512;  // a seed of <= 512 cells fits the walk's LDS ring and keeps
                                        // the stack within STACK_CAP
constexpr unsigned PREFIX_SCRATCH = PREFIX_F_CAP + 2 * PREFIX_S_CAP;
// Pool words per particle for all anchors' lists: 16 >> (anchor_up - 1), as
// anchors get fewer and larger with their height (at N = 2^22 in a Plummer
// sphere the lists take about 0.8 words per particle at height 3); capped at
// 2^32 - 1 words, the reach of a 32-bit offset.  Anchors that find no room
// leave their groups to walk from the root.
constexpr unsigned PREFIX_POOL_WORDS_1 = 16;
constexpr unsigned PREFIX_WAVES = 4;    // waves that build an anchor's lists
constexpr unsigned PREFIX_THREADS = 64 * PREFIX_WAVES;
constexpr unsigned PREFIX_RING = 4096;  // LDS stack ring of the anchor-list pass
constexpr unsigned WALK_PC_LDS = 1024;  // particle-cell list
constexpr unsigned WALK_PP_LDS = 512;   // particle-particle list
static_assert(WALK_PC_LDS % 64 == 0 && WALK_PP_LDS % 64 == 0, "lists hold whole 64-entry tiles");
// A list's last tile is padded with a massless source this far away (its
// terms are exact zeros): the cell at index cap_cells (cmac, ceval) and the
// particle at index n_max (spos), one entry past the cells and particles.
constexpr float WALK_FAR = 1.0e18f;

// Device pointers carved from the caller's workspace.
struct BuildStart;

struct Buffers {
    Header *hdr;
    SysCube *cube;          // [max_systems]
    uint32_t *sys_off;      // [max_systems + 1] first particle of each system (input = sorted order)
    uint32_t *bkt_off;      // [max_systems + 1] first sort bucket of each system
    uint8_t *sys8;          // [n] system of each input particle (batches only)
    float *bbox_part;       // [max_systems][bbox blocks per system][8]
    uint64_t *keys[2];
    uint32_t *vals[2];
    uint32_t *hist;         // [RADIX][ntiles]
    uint32_t *btot;         // [RADIX]
    float4 *ppack;          // input x, y, z, m packed by the keys kernel (one line per gather)
    float4 *spos;           // sorted x, y, z, m
    int8_t *cl;             // common leading octal digits with the previous key (-1 at 0)
    uchar4 *lvinfo;         // per particle: first level started, leaf level, group level, group start
    uint32_t *blkcnt;       // [NCOUNTERS][nblk] counts of the build's blocks
    uint32_t *blkoff;       // their exclusive prefix sums over the blocks
    uint32_t *ctot;         // [NCOUNTERS]
    uint32_t *mlist;        // multipoles: cells that leave their range of particles, per range size and level
    uint4 *topo;            // cells: first, count, child_first, system<<16 | level<<8 | nchild
    double *mp;             // cells: [10] M, com xyz, S xx yy zz xy xz yz
    double *delta;          // cells: |com - centre|
    float *cbox;            // cells: [6] bounding box of the cell's particles (min xyz, max xyz)
    double *lside;          // cells: l' = max(side, 2 * largest per-axis distance of a particle from the centre)
    float4 *cmac;           // cells: com32 xyz, r_open^2
    float4 *ceval;          // cells: [2] (M, Qxx, Qyy, Qzz), (Qxy, Qxz, Qyz, 0)
    uint2 *groups;          // first, system<<16 | level<<8 | count
    uint2 *gcounts;         // n_pc, n_pp
    uint32_t *wstack;       // per walk wave: STACK_CAP (spill of the LDS stack)
    float *feat;            // work estimator: group features [n][8]
    float *pred;            // work estimator: predicted log2(1 + n_pc + n_pp) per group
    uint8_t *level;         // block time steps: level of every particle (input order)
    uint8_t *active;        // block time steps: particle due at the current tick
    uint32_t *gref;         // block time steps: work of a group at its first walk after a build (0: none)
    unsigned long long *bsum;  // block time steps: [0] work now, [1] reference work, [2] due particles
    uint32_t *qorder;       // walk queue: groups in processing order (work-ordered modes)
    uint32_t *ghist;        // [blocks of GORD_BLOCK groups][2][GORD_CLASSES] groups by eighth and count
    uint32_t *gahist;       // the same for an active walk's queue
    uint32_t *gorder;       // queue of large trees
    uint32_t *nheavy;       // neighbour searches: groups left to the second pass
    uint8_t *gflag;         // active walks: group holds an active particle
    uint32_t *acnt;         // active walks: such groups per 512
    uint32_t *anchor;       // shared-prefix walk: anchor cell of each group
    uint32_t *alist;        // shared-prefix walk: the anchor cells, each once
    uint4 *arec;            // shared-prefix walk, per cell: pool offset, |F|, |S|, 1 if the lists are valid
                            // (2 while claimed, before the lists are built)
    uint32_t *pool;         // shared-prefix walk: the anchors' F and S lists
    uint32_t *pscr;         // shared-prefix walk: PREFIX_SCRATCH words per walk wave
    unsigned long long pool_cap;  // words of the pool
    uint32_t *ohist;        // [ORDER_BUCKETS][ORDER_BLOCKS] bucket counts of the queue order
    double *epart;          // energy partials [ENERGY_BLOCKS][2]
    unsigned cap_cells, n_max, ntiles_max, nblk_max;
    unsigned walk_waves, pc_cap, pp_cap, max_systems, ncrit, group_cap;
};

// System of sorted or input position i: the s with sys_off[s] <= i < sys_off[s+1].
__device__ __forceinline__ unsigned system_of(const uint32_t *__restrict__ sys_off, unsigned nsys, unsigned i) {
    unsigned lo = 0, hi = nsys;  // sys_off[lo] <= i < sys_off[hi]
    while (hi - lo > 1) {
        const unsigned mid = (lo + hi) >> 1;
        if (sys_off[mid] <= i) lo = mid; else hi = mid;
    }
    return lo;
}

// Morton bit spreading: bit b of v (20 bits) moves to bit 3b.
__device__ __forceinline__ uint64_t spread3(uint64_t x) {
    x &= 0x1fffffull;
    x = (x | (x << 32)) & 0x1f00000000ffffull;
    x = (x | (x << 16)) & 0x1f0000ff0000ffull;
    x = (x | (x << 8)) & 0x100f00f00f00f00full;
    x = (x | (x << 4)) & 0x10c30c30c30c30c3ull;
    x = (x | (x << 2)) & 0x1249249249249249ull;
    return x;
}

// Morton key of a point in its system's cube: q_a = min(floor((x_a - lo_a)
// 2^(20-k)), 2^20 - 1), bits of q_x, q_y, q_z at 3b+2, 3b+1, 3b.
__device__ __forceinline__ uint64_t morton_key(const SysCube &c, float px, float py, float pz) {
    const double s = ldexp(1.0, KEY_LEVELS - c.k);
    const float x[3] = {px, py, pz};
    uint64_t q[3];
#pragma unroll
    for (int a = 0; a < 3; a++) {
        double f = floor(((double)x[a] - (double)c.lo[a]) * s);
        if (!(f >= 0.0)) f = 0.0;
        if (f > 1048575.0) f = 1048575.0;
        q[a] = (uint64_t)f;
    }
    return (spread3(q[0]) << 2) | (spread3(q[1]) << 1) | spread3(q[2]);
}

// Bounding box and input flags of a set of particles.
struct BoxFlags {
    float mn[3], mx[3];
    unsigned flags;
    __device__ BoxFlags() : mn{INFINITY, INFINITY, INFINITY}, mx{-INFINITY, -INFINITY, -INFINITY}, flags(0) {}
    __device__ void add(float x, float y, float z, float m) {
        if (!(isfinite(x) && isfinite(y) && isfinite(z) && isfinite(m))) flags |= FLAG_NONFINITE;
        if (m < 0.0f) flags |= FLAG_NEGMASS;
        const float p[3] = {x, y, z};
        for (int a = 0; a < 3; a++) {
            mn[a] = fminf(mn[a], p[a]);
            mx[a] = fmaxf(mx[a], p[a]);
        }
    }
    __device__ void add(const float *p) {  // a stored box: min xyz, max xyz, flags
        for (int a = 0; a < 3; a++) {
            mn[a] = fminf(mn[a], p[a]);
            mx[a] = fmaxf(mx[a], p[3 + a]);
        }
        flags |= __float_as_uint(p[6]);
    }
    __device__ void store(float *p) const {
        for (int a = 0; a < 3; a++) {
            p[a] = mn[a];
            p[3 + a] = mx[a];
        }
        p[6] = __uint_as_float(flags);
    }
};

// The box of all threads of a workgroup of NT, in every thread; s: one row per wave.
template <unsigned NT>
__device__ __forceinline__ void block_box(BoxFlags &b, float (*s)[8]) {
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) {
#pragma unroll
        for (int a = 0; a < 3; a++) {
            b.mn[a] = fminf(b.mn[a], __shfl_xor(b.mn[a], o, 64));
            b.mx[a] = fmaxf(b.mx[a], __shfl_xor(b.mx[a], o, 64));
        }
        b.flags |= __shfl_xor(b.flags, o, 64);
    }
    if ((threadIdx.x & 63u) == 0u) b.store(s[threadIdx.x >> 6]);
    __syncthreads();
    for (unsigned w = 0; w < NT / 64; w++) b.add(s[w]);
}

// Root cube of a box: corner = per-axis minimum, side 2^k with 2^k > largest
// extent (frexp of the float64 extent), k = 0 for a zero extent.
__device__ __forceinline__ SysCube root_cube(const BoxFlags &b) {
    double ext = 0.0;
    for (int a = 0; a < 3; a++) {
        const double e = (double)b.mx[a] - (double)b.mn[a];
        if (e > ext) ext = e;
    }
    int k = 0;
    if (ext > 0.0) frexp(ext, &k);
    // non-finite input: keep every later index computation tame
    const bool tame = (b.flags & FLAG_NONFINITE) != 0;
    SysCube c;
    for (int a = 0; a < 3; a++) c.lo[a] = tame ? 0.0f : b.mn[a];
    c.k = tame ? 0 : k;
    return c;
}

// Number of leading octal digits two 60-bit keys share (0..20).
__device__ __forceinline__ int shared_digits(uint64_t a, uint64_t b) {
    const uint64_t x = a ^ b;
    if (x == 0) return KEY_LEVELS;
    return (__clzll((long long)x) - 4) / 3;
}

// Host launchers (kernels live in the .hip files).
// boxes of *nparts stretches of each system into b.bbox_part
hipError_t launch_bbox_partial(const Buffers &b, const BuildStart &start, const float *pos, const float *mass,
                               unsigned nsys, unsigned *nparts, hipStream_t s);
// the same and the root cubes
hipError_t launch_bbox(const Buffers &b, const BuildStart &start, const float *pos, const float *mass, unsigned nsys,
                       hipStream_t s);
hipError_t launch_keys(const Buffers &b, const float *pos, const float *mass, unsigned n, unsigned nsys,
                       hipStream_t s);
hipError_t launch_sort(const Buffers &b, unsigned n, unsigned nsys, hipStream_t s);
// Both sorts leave the sorted keys and the permutation in keys[0] and vals[0].
// The radix sort's keys start in the buffer from which its passes end there.
inline int radix_first_buffer(unsigned nsys) { return nsys > 1 ? (SORT_PASSES + 1) & 1 : SORT_PASSES & 1; }
// Bucket sort (sort_kernels.hip): buckets of a system of n particles.
constexpr unsigned SORT_BUCKET = 4096;       // elements one workgroup sorts in LDS
// Elements of a bucket on average, for n in all systems.  Up to a chip's worth
// of workgroups the largest bucket sets the time, and one of more than 2048 elements
// takes two places per thread: sorting and moving with 512 / 768 / 1024 / 1365,
// in us: 70 / 72 / 72 / 87 at 32768, 88 / 87 / 85 / 98 at 100003, 106 / 105 / 104 /
// 107 at 300007, 155 / 149 / 131 / 141 at 2^20, 250 / 219 / 204 / 213 at 2^21.  At
// 2^22 the chip is full and the sample per bucket, 4096 of 8 lists at most, thin:
// 1024 330, 1365 312.
__host__ __device__ inline unsigned sort_bucket_mean(unsigned n) { return n <= 1u << 21 ? 1024u : 1365u; }
// The counting kernel keeps splitters and counts of all buckets in LDS, 16 bytes a
// bucket: 64 KB with this many, what a launch gets without asking for more, and two
// workgroups of 1024 threads, a full compute unit, fit.  Twice as many buckets would
// leave one of the two, and the dependent reads of each particle's search are what
// the kernel waits for; from memory they would take several times as long each.
// (Neither was built: larger inputs keep the radix sort, 1.55 ms at 2^24 particles.)
constexpr unsigned SORT_MAX_BUCKETS = 4096;
// shared digits of a particle that the tree build takes from its keys
constexpr int8_t CL_FROM_KEYS = 127;
__host__ __device__ inline unsigned sort_buckets(unsigned n, unsigned mean) {
    return n <= SORT_BUCKET ? 1u : (n + mean - 1u) / mean;
}
// System offsets travel to the device as a kernel argument, so a captured
// graph holds them by value and no host staging buffer is needed.
struct SysOffsets {
    unsigned nsys;
    unsigned off[MAX_SYSTEMS + 1];
};
// The start of a build: system offsets, the first sort bucket of each system,
// the header and the walk's padding entries.  The flags of the previous build
// move into the sticky word, so that a driver running many steps still sees a
// condition that one of its earlier builds met.  One workgroup of the build's
// first kernel does it, whose others need nothing of it (a launch of its own took
// 4.7 us).
struct BuildStart {
    SysOffsets o;
    uint32_t *sys_off, *bkt_off;
    Header *hdr;
    float4 *cmac, *ceval, *spos;
    unsigned cap_cells, n_max, bucket_mean;
};
__device__ inline void begin_build(const BuildStart &st) {
    const SysOffsets &o = st.o;
    Header *hdr = st.hdr;
    for (unsigned i = threadIdx.x; i <= o.nsys; i += blockDim.x) {
        st.sys_off[i] = o.off[i];
        unsigned nb = 0;
        for (unsigned s = 0; s < i; s++) nb += sort_buckets(o.off[s + 1] - o.off[s], st.bucket_mean);
        st.bkt_off[i] = nb;
    }
    if (threadIdx.x == 0) {
        // the walk's padding cell and particle: massless, far away
        st.cmac[st.cap_cells] = make_float4(WALK_FAR, WALK_FAR, WALK_FAR, 0.0f);
        st.ceval[2 * (size_t)st.cap_cells] = make_float4(0.0f, 0.0f, 0.0f, 0.0f);
        st.ceval[2 * (size_t)st.cap_cells + 1] = make_float4(0.0f, 0.0f, 0.0f, 0.0f);
        st.spos[st.n_max] = make_float4(WALK_FAR, WALK_FAR, WALK_FAR, 0.0f);
        hdr->nsys = o.nsys;
        hdr->sticky |= hdr->flags;
        hdr->flags = 0;
        hdr->n = o.off[o.nsys];
        hdr->ncells = 0;
        hdr->ngroups = 0;
        for (int l = 0; l < 24; l++) hdr->lvl_begin[l] = 0;
    }
    if (threadIdx.x < WALK_QUEUES) hdr->walk_head[QUEUE_STRIDE * threadIdx.x] = 0;
}
bool bucket_sort_fits(const Buffers &b, unsigned n, unsigned nb);
// The build's start is part of the partition, or, where every system is one
// bucket, of the sort if `start` is given (one system: no other workgroup).
hipError_t launch_bucket_partition(const Buffers &b, const BuildStart &start, const float *pos, const float *mass,
                                   unsigned n, unsigned nsys, unsigned nb, unsigned nb_max, hipStream_t s);
hipError_t launch_bucket_sort(const Buffers &b, const BuildStart *start, const float *pos, const float *mass,
                              unsigned n, unsigned nsys, unsigned nb, hipStream_t s);
hipError_t launch_reorder(const Buffers &b, unsigned n, unsigned nsys, hipStream_t s);
hipError_t launch_build(const Buffers &b, unsigned n, unsigned nsys, int ncrit, int gcap, hipStream_t s);
hipError_t launch_multipoles(const Buffers &b, unsigned n, unsigned nsys, hipStream_t s);
// theta: the float32 opening angle widened to float64
hipError_t launch_mac_prep(const Buffers &b, unsigned nsys, double theta, hipStream_t s);
// whether the walk of a tree of n particles takes the end of its queue by size
bool walk_sorts_groups(unsigned n);
// every group in that order into b.gorder
hipError_t launch_group_order(const Buffers &b, unsigned n, hipStream_t s);
// order: the queue (NULL: groups in Morton order); qlen: device count of queue
// entries to walk (NULL: every group)
// anchor_up > 0: groups share the traversal of their ancestor anchor_up levels up
hipError_t launch_walk(const Buffers &b, unsigned n, unsigned nsys, float eps2, float G, int precision,
                       const uint32_t *order, const uint32_t *qlen, const uint8_t *active, float *acc, float *pot,
                       int anchor_up, hipStream_t s);
hipError_t launch_features(const Buffers &b, float theta, float *feat, hipStream_t s);
hipError_t launch_mlp_forward(const void *w16, const float *x, unsigned rows, const Header *hdr, float *y,
                              hipStream_t s);
size_t mlp_scratch_bytes(unsigned batch);
hipError_t launch_mlp_grad(const void *w16, const float *x, const float *target, const int *idx, unsigned batch,
                           float *grad, float *loss, void *scratch, hipStream_t s);
hipError_t launch_adam(float *w32, void *w16, const float *grad, float *m, float *v, int step, float lr,
                       float beta1, float beta2, float eps, hipStream_t s);
// Writes b.qorder: the groups ordered by work, heaviest first; mode 1: work
// predicted by the estimator (b.pred), 2: exact counts of the last walk; mode
// ORDER_MODE_ACTIVE: groups holding a particle with active[input index] != 0
// first (their number, after the call, is b.ohist[ORDER_BLOCKS]), in Morton order.
constexpr int ORDER_MODE_ACTIVE = 3;
hipError_t launch_queue_order(const Buffers &b, int mode, const uint8_t *active, unsigned nsys, hipStream_t s);
// Packs input (x, y, z, m) into b.ppack and flags non-finite or negative values.
hipError_t launch_pack(const Buffers &b, const float *pos, const float *mass, unsigned n, hipStream_t s);
// v <- v + dt_kick a, then (dt_drift != 0) x <- x + dt_drift v, for n particles
hipError_t launch_kick_drift(float *pos, float *vel, const float *acc, unsigned n, float dt_kick, float dt_drift,
                             hipStream_t s);
// block time steps
enum : int { BLOCK_CLOSE = 1, BLOCK_LEVEL = 2, BLOCK_OPEN = 4 };
hipError_t launch_block_active(const uint8_t *level, unsigned n, unsigned tick, int R, uint8_t *active,
                               unsigned long long *nactive, hipStream_t s);
hipError_t launch_block_kick(float *vel, const float *acc, uint8_t *level, unsigned n, unsigned tick, int R,
                             float dt_max, int flags, double eta, double eps, hipStream_t s);
hipError_t launch_rebuild_check(const Buffers &b, const uint32_t *qlen, unsigned long long *sums, hipStream_t s);
hipError_t launch_fill_u32(uint32_t *p, unsigned n, uint32_t v, hipStream_t s);
// neighbour search (mode 0 counts, 1 lists, 2 SPH density); needs the cell boxes of compute_multipoles
hipError_t launch_neighbors(const Buffers &b, int mode, const float *radius, uint32_t *count, const uint32_t *offset,
                            uint32_t *index, int64_t capacity, float *rho, unsigned n, unsigned nsys, hipStream_t s);
// exclusive scan of n counts into out[0..n], out[n] = total; tmp holds (n + 1023) / 1024 words
hipError_t launch_scan_u32(const uint32_t *in, unsigned n, uint32_t *out, uint32_t *tmp, hipStream_t s);
hipError_t launch_energy(const Buffers &b, const float *mass, const float *pot, const float *vel,
                         unsigned n, double *d_out2, hipStream_t s);

}  // namespace mibh
