// Sorting by buckets: the particles' order along the Morton curve in one pass
// over memory and one sort in LDS, for up to SORT_MAX_BUCKETS buckets (about 5
// million particles); larger inputs take the eight-pass radix sort.
//
//   k_bucket_sample: per system, the root cube, and the keys of particles drawn
//     at hashed places (16 per bucket, up to 8 lists of 4096), sorted in LDS;
//   k_bucket_split: the lists' common quantiles (one list's own need no second
//     kernel): the buckets' splitters.
//   k_bucket_count: every particle's bucket (a binary search for its key over
//     the splitters in LDS) and the counts of each tile's buckets.
//   k_bucket_scan: the counts' prefix sums over the tiles, bucket by bucket (with
//     few tiles part of the next kernel).
//   k_bucket_scatter: particle records and indices to their buckets.
//   k_bucket_sort: one workgroup per bucket sorts it in LDS and writes keys,
//     permutation, records and shared digits in their final order: the moving
//     of the particles is part of it.
//
// Elements are ordered by (key, input index), so the order is the stable one
// whatever order the scatter left, equal keys are split between buckets like
// any others, and every run gives the same arrays.  A system of up to
// SORT_BUCKET particles is one bucket and needs only the last kernel.
//
// The radix sort reads and writes every key eight times in 24 launches, then
// gathers the records.  Sorting and moving, bounding cube to records in order:
// 27 / 64 / 77 / 125 / 297 us at n = 1000 / 20000 / 100003 / 2^20 / 2^22 against
// 124 / 161 / 169 / 216 / 488 us.  Small inputs are bound by the launches and
// the sort's chain of merges; at 2^22 the sort of the buckets takes 120 us (57
// bytes a particle, 0.4 of the copy rate; LDS latency of the merges), the
// scatter 48, the counting 37 (the search's dependent LDS reads), the sample 51.
#include "mibh_device.h"

namespace mibh {

namespace {

constexpr unsigned ITEMS = 8;            // elements per place of a workgroup's sort
constexpr unsigned SAMPLE_THREADS = 512;
constexpr unsigned SAMPLE_LIST = SAMPLE_THREADS * ITEMS;  // samples one workgroup sorts
constexpr unsigned SAMPLE_LISTS = 8;                      // workgroups per system at most
constexpr unsigned SAMPLE_PER_BUCKET = 16;
constexpr unsigned TILE_ITEMS = 8;       // particles per thread in the counting and scatter kernels
constexpr unsigned BS_THREADS = 256, BS_WAVES = 4;
constexpr unsigned BS_VT = SORT_BUCKET / (BS_THREADS * ITEMS);  // places per thread in a full bucket
static_assert(BS_VT == 2, "a bucket's sort takes one or two places per thread");
// Longest run of equal leading bits that one thread puts in order, its dependent
// loads one after the other.  Builds with 2 / 4 / 8 / 24, us: 2^22 particles at n / 24
// points 600 / 591 / 607 / 868 (radix sort 687), along a line (4 to a key, up to 14)
// 555 / 569 / 611 / 678 (609), 50 within a few grid cells of each of n / 50 points 595 /
// 588 / 532 / 533 (675); 3000 particles three to a point 88 / 70 / 70 / 70 (150).
constexpr unsigned BS_RUN = 8;

// Places in the LDS arrays, one in nine left free: neighbouring threads work 8
// or 16 elements apart, and such strides would meet in few banks.
__device__ __forceinline__ unsigned phys(unsigned i) { return i + (i >> 3); }
constexpr unsigned phys_size(unsigned n) { return n + n / 8; }

__device__ __forceinline__ bool before(uint64_t ka, uint32_t ia, uint64_t kb, uint32_t ib) {
    return ka < kb || (ka == kb && ia < ib);
}

__device__ __forceinline__ unsigned wave_incl(unsigned v) {
    const unsigned ln = __lane_id();
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) {
        const unsigned y = __shfl_up(v, o, 64);
        v += ln >= (unsigned)o ? y : 0u;
    }
    return v;
}

// Batcher's odd-even merge sort of N values of a thread; order(a, b) puts
// places a < b in order.
template <unsigned N, typename F>
__device__ __forceinline__ void sort_network(F order) {
#pragma unroll
    for (unsigned p = 1; p < N; p *= 2)
#pragma unroll
        for (unsigned k = p; k >= 1; k /= 2)
#pragma unroll
            for (unsigned j = k % p; j + k < N; j += 2 * k)
#pragma unroll
                for (unsigned i = 0; i < k; i++)
                    if (i + j + k < N && (i + j) / (2 * p) == (i + j + k) / (2 * p)) order(i + j, i + j + k);
}

// First output of one merge step, by the "merge path" method (Odeh, Green, Mwassi,
// Shmueli & Birk 2012; Green, McColl & Bader 2012): outputs d .. of the merge of
// A = [a0, a0 + la) and B = [a0 + la, a0 + la + lb) take lo elements of A and d - lo
// of B first; less(i, j): element i of A goes before element j of B.
template <typename F>
__device__ __forceinline__ unsigned merge_path(unsigned a0, unsigned la, unsigned lb, unsigned d, F less) {
    unsigned lo = d > lb ? d - lb : 0u, hi = min(d, la);
    while (lo < hi) {
        const unsigned mid = (lo + hi) >> 1;
        if (less(a0 + mid, a0 + la + d - 1u - mid)) lo = mid + 1u; else hi = mid;
    }
    return lo;
}

// Sorts the words v of the places t < active, ITEMS words each, together, into
// the LDS array sv; thread t of NT holds places t, t + NT, .. (VT of them, in
// v[0, ITEMS), v[ITEMS, 2 ITEMS), ..).  Every thread of the workgroup calls it.
// A network in registers, then merges of doubling length: each place finds where
// its outputs start by a binary search along the merge's diagonal and merges
// them.
template <unsigned NT, unsigned VT>
__device__ __forceinline__ void block_sort(uint64_t (&v)[VT * ITEMS], unsigned active, uint64_t *sv) {
    const unsigned total = active * ITEMS;
#pragma unroll
    for (unsigned x = 0; x < VT; x++)
        sort_network<ITEMS>([&](unsigned a, unsigned b) {
            const uint64_t va = v[x * ITEMS + a], vb = v[x * ITEMS + b];
            const bool sw = vb < va;
            v[x * ITEMS + a] = sw ? vb : va;
            v[x * ITEMS + b] = sw ? va : vb;
        });
    for (unsigned w = ITEMS;; w *= 2) {
#pragma unroll
        for (unsigned x = 0; x < VT; x++) {
            const unsigned t = threadIdx.x + x * NT;
            if (t < active) {
#pragma unroll
                for (unsigned u = 0; u < ITEMS; u++) sv[phys(t * ITEMS + u)] = v[x * ITEMS + u];
            }
        }
        __syncthreads();
        if (w >= total) return;
#pragma unroll
        for (unsigned x = 0; x < VT; x++) {
            const unsigned t = threadIdx.x + x * NT, o = t * ITEMS;
            if (t < active) {
                const unsigned a0 = o & ~(2u * w - 1u);
                const unsigned la = min(w, total - a0), lb = min(w, total - a0 - la), d = o - a0;
                const unsigned lo = merge_path(a0, la, lb, d,
                                               [&](unsigned i, unsigned j) { return sv[phys(i)] < sv[phys(j)]; });
                unsigned i = a0 + lo, j = a0 + la + (d - lo);
                const unsigned ea = a0 + la, eb = a0 + la + lb, last = total - 1u;
                uint64_t va = sv[phys(min(i, last))], vb = sv[phys(min(j, last))];
#pragma unroll
                for (unsigned u = 0; u < ITEMS; u++) {
                    const bool ta = i < ea && (j >= eb || va < vb);
                    v[x * ITEMS + u] = ta ? va : vb;
                    i += ta ? 1u : 0u;
                    j += ta ? 0u : 1u;
                    const uint64_t nx = sv[phys(min(ta ? i : j, last))];
                    va = ta ? nx : va;
                    vb = ta ? vb : nx;
                }
            }
        }
        __syncthreads();
    }
}

// Least and largest value over the workgroup of NT threads; s2 holds 2 * NT / 64 words.
template <unsigned NT>
__device__ __forceinline__ void block_minmax(uint64_t &lo, uint64_t &hi, uint64_t *s2) {
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) {
        lo = min(lo, (uint64_t)__shfl_xor((unsigned long long)lo, o, 64));
        hi = max(hi, (uint64_t)__shfl_xor((unsigned long long)hi, o, 64));
    }
    if ((threadIdx.x & 63u) == 0u) {
        s2[2 * (threadIdx.x >> 6)] = lo;
        s2[2 * (threadIdx.x >> 6) + 1] = hi;
    }
    __syncthreads();
    for (unsigned w = 0; w < NT / 64; w++) {
        lo = min(lo, s2[2 * w]);
        hi = max(hi, s2[2 * w + 1]);
    }
    __syncthreads();
}

// The sort word of an element: the leading bits of its key's distance from the
// smallest key, as many as leave room for the element's place, then the place.
struct Words {
    uint64_t kmin;
    int kbits;      // bits of the largest distance
    unsigned tb;    // bits of the place
    int sh;         // key bits that the words leave out
    __device__ Words(uint64_t lo, uint64_t hi, unsigned places) : kmin(lo) {
        kbits = hi > lo ? 64 - __clzll((long long)(hi - lo)) : 0;
        tb = 32u - (unsigned)__clz((int)(places - 1u));
        sh = max(0, kbits - (64 - (int)tb));
    }
    __device__ uint64_t word(uint64_t k, unsigned place) const { return ((k - kmin) >> sh) << tb | place; }
    __device__ unsigned place(uint64_t v) const { return (unsigned)v & ((1u << tb) - 1u); }
};

// Puts the runs of words in sv[0, m) whose key bits agree in order by (key,
// index), each by the thread that meets its first word; key(p), index(p): of
// the element at place p.  A run of more than BS_RUN words is left, and *s_long
// set.  The caller synchronises before and after.
template <unsigned NT, typename K, typename X>
__device__ __forceinline__ void order_runs(uint64_t *sv, unsigned m, const Words &wd, unsigned *s_long, K key, X index) {
    for (unsigned r = threadIdx.x; r + 1u < m; r += NT) {
        const uint64_t d = sv[phys(r)] >> wd.tb;
        // a run's first word is told by key bits alone, which no reordering changes
        if (d != sv[phys(r + 1u)] >> wd.tb || (r > 0 && d == sv[phys(r - 1u)] >> wd.tb)) continue;
        unsigned e = r + 2u;
        while (e < m && e - r <= BS_RUN && d == sv[phys(e)] >> wd.tb) e++;
        if (e - r > BS_RUN) {
            *s_long = 1;
            continue;
        }
        for (unsigned i = r + 1u; i < e; i++) {  // insertion sort
            const uint64_t v = sv[phys(i)];
            const unsigned p = wd.place(v);
            const uint64_t kp = key(p);
            const uint32_t xp = index(p);
            unsigned h = i;
            while (h > r) {
                const uint64_t u = sv[phys(h - 1u)];
                const unsigned pu = wd.place(u);
                if (!before(kp, xp, key(pu), index(pu))) break;
                sv[phys(h)] = u;
                h--;
            }
            sv[phys(h)] = v;
        }
    }
}

// Sorts the words in sv[0, m) again, those whose key bits agree by rest(p) (at most
// 64 - 2 tb bits: what the key bits leave out, then the index), then by place.  The
// words then hold the first place of their run, the rest, and the place.
template <unsigned NT, unsigned VT, typename R>
__device__ __forceinline__ void sort_runs(uint64_t *sv, unsigned m, const Words &wd, R rest) {
    const unsigned active = (m + ITEMS - 1) / ITEMS;
    uint64_t v[VT * ITEMS];
#pragma unroll
    for (unsigned x = 0; x < VT; x++) {
        const unsigned r0 = (threadIdx.x + x * NT) * ITEMS;
        uint64_t prev = 0;
        unsigned lo = 0;
#pragma unroll
        for (unsigned u = 0; u < ITEMS; u++) {
            const unsigned r = r0 + u;
            uint64_t w = ~0ull;
            if (r < m) {
                const uint64_t d = sv[phys(r)] >> wd.tb;
                if (u == 0) {  // the first word with these bits
                    lo = 0;
                    unsigned hi = r;
                    while (lo < hi) {
                        const unsigned mid = (lo + hi) >> 1;
                        if (sv[phys(mid)] >> wd.tb < d) lo = mid + 1u; else hi = mid;
                    }
                } else if (d != prev) {
                    lo = r;
                }
                prev = d;
                const unsigned p = wd.place(sv[phys(r)]);
                w = (uint64_t)lo << (64u - wd.tb) | rest(p) << wd.tb | p;
            }
            v[x * ITEMS + u] = w;
        }
    }
    __syncthreads();
    block_sort<NT, VT>(v, active, sv);
}

// A published 32-bit integer hash (two rounds of xor-shift and multiply, "lowbias32"
// of C. Wellons' hash prospector, 2018).
__device__ __forceinline__ unsigned mix32(unsigned v) {
    v ^= v >> 16;
    v *= 0x7feb352du;
    v ^= v >> 15;
    v *= 0x846ca68bu;
    v ^= v >> 16;
    return v;
}

// The sample of a system: m samples in `lists` sorted lists of m / lists each.
struct Sample {
    unsigned m, lists, len;
    uint64_t step;  // sample g: one particle of each of m stretches of the input, n / m long in 32-bit fixed point
    __device__ Sample(unsigned n, unsigned nb) {
        m = min(SAMPLE_PER_BUCKET * nb, SAMPLE_LISTS * SAMPLE_LIST);  // less than n: a bucket holds 1024 on average
        lists = (m + SAMPLE_LIST - 1u) / SAMPLE_LIST;
        len = (m / lists) & ~(ITEMS - 1u);
        m = len * lists;
        step = ((uint64_t)n << 32) / m;
    }
    __device__ unsigned particle(unsigned g, unsigned sys) const {  // at a hashed place of stretch g
        const unsigned lo = (unsigned)((step * g) >> 32), hi = (unsigned)((step * (g + 1u)) >> 32);
        return lo + __umulhi(mix32(g * 0x9e3779b9u + sys), hi - lo);
    }
};

// Root cubes, and the sorted samples: one workgroup per list (grid x) and system
// (grid y).  With one list its quantiles are the splitters: bucket r of system s
// starts at element (spl_key, spl_idx)[bkt_off[s] + r], r >= 1; several lists go
// to list_key and list_idx, system s' from SAMPLE_PER_BUCKET * bkt_off[s] on.
__global__ __launch_bounds__(SAMPLE_THREADS) void k_bucket_sample(
    const float *__restrict__ pos, const uint32_t *__restrict__ sys_off, const uint32_t *__restrict__ bkt_off,
    const float *__restrict__ part, unsigned nparts, Header *__restrict__ hdr, SysCube *__restrict__ cube,
    uint64_t *__restrict__ spl_key, uint32_t *__restrict__ spl_idx, uint64_t *__restrict__ list_key,
    uint32_t *__restrict__ list_idx) {
    __shared__ uint64_t sv[phys_size(SAMPLE_LIST)];
    __shared__ uint64_t s_mm[2 * SAMPLE_THREADS / 64];
    __shared__ float s_box[SAMPLE_THREADS / 64][8];
    __shared__ unsigned s_long;
    const unsigned s = blockIdx.y, t = threadIdx.x, w = blockIdx.x;
    const unsigned b0 = bkt_off[s], nb = bkt_off[s + 1] - b0;
    const unsigned o = sys_off[s], n = sys_off[s + 1] - o;
    const Sample sa(n, nb);
    if (w > 0 && (nb < 2u || w >= sa.lists)) return;
    BoxFlags bf;
    for (unsigned q = t; q < nparts; q += SAMPLE_THREADS) bf.add(part + ((size_t)s * nparts + q) * 8);
    block_box<SAMPLE_THREADS>(bf, s_box);
    const SysCube c = root_cube(bf);
    if (w == 0 && t == 0) {
        cube[s] = c;
        if (bf.flags) atomicOr(&hdr->flags, bf.flags);
    }
    if (nb < 2u) return;
    const unsigned m = sa.len, active = m / ITEMS;
    auto index = [&](unsigned j) { return o + sa.particle(j * sa.lists + w, s); };  // of the list's sample j
    auto key = [&](unsigned j) {
        const size_t i = 3 * (size_t)index(j);
        return morton_key(c, pos[i], pos[i + 1], pos[i + 2]);
    };
    uint64_t k[ITEMS], kmin = ~0ull, kmax = 0;
    if (t < active) {
#pragma unroll
        for (unsigned u = 0; u < ITEMS; u++) {
            k[u] = key(u * active + t);
            kmin = min(kmin, k[u]);
            kmax = max(kmax, k[u]);
        }
    }
    if (t == 0) s_long = 0;
    block_minmax<SAMPLE_THREADS>(kmin, kmax, s_mm);
    const Words wd(kmin, kmax, m);
#pragma unroll
    for (unsigned u = 0; u < ITEMS; u++) k[u] = t < active ? wd.word(k[u], u * active + t) : ~0ull;
    block_sort<SAMPLE_THREADS, 1>(k, active, sv);
    // Places rise with the indices, so only words that leave key bits out can be
    // out of order.
    if (wd.sh > 0) {
        order_runs<SAMPLE_THREADS>(sv, m, wd, &s_long, key, index);
        __syncthreads();
        if (s_long)
            sort_runs<SAMPLE_THREADS, 1>(sv, m, wd, [&](unsigned p) { return (key(p) - wd.kmin) & ((1ull << wd.sh) - 1ull); });
    }
    if (sa.lists == 1u) {
        for (unsigned r = 1 + t; r < nb; r += SAMPLE_THREADS) {
            const unsigned j = wd.place(sv[phys((unsigned)((uint64_t)m * r / nb))]);
            spl_key[b0 + r] = key(j);
            spl_idx[b0 + r] = index(j);
        }
    } else {
        const size_t l0 = SAMPLE_PER_BUCKET * (size_t)b0 + w * m;
        for (unsigned r = t; r < m; r += SAMPLE_THREADS) {
            const unsigned j = wd.place(sv[phys(r)]);
            list_key[l0 + r] = key(j);
            list_idx[l0 + r] = index(j);
        }
    }
}

// Splitters of the systems with several lists: a sample's rank in all of them is
// its place in its own plus the samples before it in every other.
__global__ __launch_bounds__(256) void k_bucket_split(const uint32_t *__restrict__ sys_off,
                                                      const uint32_t *__restrict__ bkt_off,
                                                      const uint64_t *__restrict__ list_key,
                                                      const uint32_t *__restrict__ list_idx,
                                                      uint64_t *__restrict__ spl_key, uint32_t *__restrict__ spl_idx) {
    const unsigned s = blockIdx.y;
    const unsigned b0 = bkt_off[s], nb = bkt_off[s + 1] - b0;
    if (nb < 2u) return;
    const Sample sa(sys_off[s + 1] - sys_off[s], nb);
    const unsigned g = blockIdx.x * 256u + threadIdx.x;
    if (sa.lists == 1u || g >= sa.m) return;
    const uint64_t *lk = list_key + SAMPLE_PER_BUCKET * (size_t)b0;
    const uint32_t *li = list_idx + SAMPLE_PER_BUCKET * (size_t)b0;
    const uint64_t k = lk[g];
    const uint32_t x = li[g];
    const unsigned own = g / sa.len;
    unsigned lo[SAMPLE_LISTS], hi[SAMPLE_LISTS];
#pragma unroll
    for (unsigned q = 0; q < SAMPLE_LISTS; q++) {
        lo[q] = 0;
        hi[q] = q < sa.lists && q != own ? sa.len : 0u;
    }
    for (unsigned span = sa.len; span > 0; span >>= 1) {  // the searches side by side
#pragma unroll
        for (unsigned q = 0; q < SAMPLE_LISTS; q++) {
            const unsigned mid = (lo[q] + hi[q]) >> 1;
            if (lo[q] < hi[q]) {
                const uint64_t km = lk[q * sa.len + mid];
                bool lt = km < k;
                if (km == k) lt = li[q * sa.len + mid] < x;
                lo[q] = lt ? mid + 1u : lo[q];
                hi[q] = lt ? hi[q] : mid;
            }
        }
    }
    unsigned r = g - own * sa.len;
#pragma unroll
    for (unsigned q = 0; q < SAMPLE_LISTS; q++) r += lo[q];
    // bucket c starts at the sample of rank m c / nb, rounded down
    const unsigned c = (unsigned)(((uint64_t)r * nb + sa.m - 1u) / sa.m);
    if (c >= 1u && c < nb && (unsigned)((uint64_t)sa.m * c / nb) == r) {
        spl_key[b0 + c] = k;
        spl_idx[b0 + c] = x;
    }
}

// Buckets of a tile of blockDim.x * TILE_ITEMS particles and the tile's row of
// counts[tile][nb].
__global__ __launch_bounds__(1024) void k_bucket_count(const float *__restrict__ pos, unsigned n, unsigned nsys,
                                                       const uint32_t *__restrict__ sys_off,
                                                       const uint32_t *__restrict__ bkt_off,
                                                       const SysCube *__restrict__ cube,
                                                       const uint64_t *__restrict__ spl_key,
                                                       const uint32_t *__restrict__ spl_idx, unsigned nb,
                                                       unsigned short *__restrict__ bkt,
                                                       uint32_t *__restrict__ counts) {
    extern __shared__ uint64_t s_dyn[];
    uint64_t *s_key = s_dyn;                                  // [nb]
    uint32_t *s_idx = reinterpret_cast<uint32_t *>(s_key + nb);  // [nb]
    uint32_t *s_cnt = s_idx + nb;                             // [nb]
    const unsigned t = threadIdx.x, nt = blockDim.x;
    for (unsigned b = t; b < nb; b += nt) {
        s_key[b] = spl_key[b];
        s_idx[b] = spl_idx[b];
        s_cnt[b] = 0;
    }
    const unsigned base = blockIdx.x * nt * TILE_ITEMS;
    float3 p[TILE_ITEMS];  // all of the thread's particles on their way at once
#pragma unroll
    for (unsigned u = 0; u < TILE_ITEMS; u++) {
        const size_t i = 3 * (size_t)min(base + u * nt + t, n - 1u);
        p[u] = make_float3(pos[i], pos[i + 1], pos[i + 2]);
    }
    __syncthreads();
#pragma unroll
    for (unsigned u = 0; u < TILE_ITEMS; u++) {
        const unsigned i = base + u * nt + t;
        if (i < n) {
            const unsigned s = nsys > 1 ? system_of(sys_off, nsys, i) : 0u;
            const uint64_t k = morton_key(cube[s], p[u].x, p[u].y, p[u].z);
            // the last bucket of the system whose splitter is not after (k, i)
            unsigned lo = bkt_off[s], hi = bkt_off[s + 1];
            while (hi - lo > 1) {
                const unsigned mid = (lo + hi) >> 1;
                const uint64_t km = s_key[mid];
                bool after = k < km;
                if (k == km) after = i < s_idx[mid];
                if (after) hi = mid; else lo = mid;
            }
            bkt[i] = (unsigned short)lo;
            atomicAdd(&s_cnt[lo], 1u);
        }
    }
    __syncthreads();
    for (unsigned b = t; b < nb; b += nt) counts[(size_t)blockIdx.x * nb + b] = s_cnt[b];
}

// Exclusive prefix sums of each column of counts[ntiles][nb], in place, and the
// columns' totals: 64 columns per workgroup, 8 stretches of tiles each.
constexpr unsigned SCAN_SEGS = 8;
__global__ __launch_bounds__(64 * SCAN_SEGS) void k_bucket_scan(uint32_t *__restrict__ counts, unsigned ntiles,
                                                                unsigned nb, uint32_t *__restrict__ total) {
    __shared__ unsigned s_sum[SCAN_SEGS][64];
    const unsigned col = blockIdx.x * 64u + (threadIdx.x & 63u), seg = threadIdx.x >> 6;
    const unsigned per = (ntiles + SCAN_SEGS - 1) / SCAN_SEGS;
    const unsigned t0 = min(seg * per, ntiles), t1 = min(t0 + per, ntiles);
    unsigned sum = 0;
    if (col < nb) {
#pragma unroll 8
        for (unsigned r = t0; r < t1; r++) sum += counts[(size_t)r * nb + col];
    }
    s_sum[seg][threadIdx.x & 63u] = sum;
    __syncthreads();
    unsigned run = 0, all = 0;
    for (unsigned v = 0; v < SCAN_SEGS; v++) {
        const unsigned c = s_sum[v][threadIdx.x & 63u];
        run += v < seg ? c : 0u;
        all += c;
    }
    if (col < nb) {
        if (seg == 0) total[col] = all;
#pragma unroll 8
        for (unsigned r = t0; r < t1; r++) {
            const unsigned c = counts[(size_t)r * nb + col];
            counts[(size_t)r * nb + col] = run;
            run += c;
        }
    }
}

// Elements to their buckets; the first workgroup also writes the buckets'
// starts.  A tile's elements are put in bucket order in LDS, one component at a
// time, so that neighbouring threads store neighbouring addresses: stored from
// where they were read, 2^22 records went to HBM in 287 MB of partial lines
// (84 MB of data) and 112 us.  Consecutive tiles go to one XCD (workgroup i runs
// on XCD i mod 8), so that the short runs they add to a bucket meet in its L2.
// SCAN: few tiles and no more buckets than threads; every workgroup adds up the
// columns of counts itself, a thread each (no launch between, 4.5 us).
constexpr unsigned SCATTER_SCAN_TILES = 64;
template <bool SCAN>
__global__ __launch_bounds__(1024) void k_bucket_scatter(const float *__restrict__ pos, const float *__restrict__ mass,
                                                         const unsigned short *__restrict__ bkt, unsigned n,
                                                         const uint32_t *__restrict__ counts, unsigned ntiles,
                                                         const uint32_t *__restrict__ total, unsigned nb,
                                                         uint32_t *__restrict__ start, uint32_t *__restrict__ vout,
                                                         float4 *__restrict__ rec) {
    extern __shared__ uint64_t s_dyn[];
    uint32_t *s_at = reinterpret_cast<uint32_t *>(s_dyn);  // [nb] next place in the tile
    uint32_t *s_out = s_at + nb;                           // [nb] output place of tile place i: s_out + i
    uint32_t *s_x = s_out + nb;                            // [tile] one component
    __shared__ unsigned s_w[2][17];
    const unsigned t = threadIdx.x, nt = blockDim.x;
    const unsigned per_xcd = gridDim.x / 8u;
    const unsigned tile = (blockIdx.x % 8u) * per_xcd + blockIdx.x / 8u;
    if (tile >= ntiles) return;  // workgroup 0 has tile 0
    // starts of the buckets in the output and of this tile's elements in the
    // tile: two block scans, `per` buckets per thread
    const unsigned per = (nb + nt - 1u) / nt;
    const unsigned c0 = min(t * per, nb), c1 = min(c0 + per, nb);
    const uint32_t *row = counts + (size_t)tile * nb;
    unsigned sum = 0, own = 0, earlier = 0;
    for (unsigned b = c0; b < c1; b++) {
        unsigned tot = 0, mine = 0;  // mine: this tile's elements of the bucket
        if (SCAN) {
#pragma unroll 8
            for (unsigned r = 0; r < ntiles; r++) {
                const unsigned c = counts[(size_t)r * nb + b];
                earlier += r < tile ? c : 0u;
                mine = r == tile ? c : mine;
                tot += c;
            }
        } else {
            tot = total[b];
            mine = (tile + 1u < ntiles ? row[nb + b] : tot) - row[b];
        }
        sum += tot;
        s_at[b] = mine;
        own += mine;
    }
    const unsigned inc = wave_incl(sum), inco = wave_incl(own);
    if ((t & 63u) == 63u) {
        s_w[0][t >> 6] = inc;
        s_w[1][t >> 6] = inco;
    }
    __syncthreads();
    unsigned run = inc - sum, runo = inco - own;
    for (unsigned v = 0; v < (t >> 6); v++) {
        run += s_w[0][v];
        runo += s_w[1][v];
    }
    for (unsigned b = c0; b < c1; b++) {
        const unsigned c = s_at[b];
        s_at[b] = runo;
        s_out[b] = run + (SCAN ? earlier : row[b]) - runo;  // modulo 2^32
        if (tile == 0) start[b] = run;
        run += SCAN ? sum : total[b];  // (one bucket per thread)
        runo += c;
    }
    if (tile == 0 && t == 0) start[nb] = n;
    __syncthreads();
    const unsigned base = tile * nt * TILE_ITEMS, cnt = min(nt * TILE_ITEMS, n - base);
    unsigned at[TILE_ITEMS], out[TILE_ITEMS], idx[TILE_ITEMS];
    float4 r[TILE_ITEMS];
#pragma unroll
    for (unsigned u = 0; u < TILE_ITEMS; u++) {
        const unsigned k = u * nt + t;
        const size_t i = base + min(k, cnt - 1u);
        const unsigned b = bkt[i];
        r[u] = make_float4(pos[3 * i], pos[3 * i + 1], pos[3 * i + 2], mass[i]);
        at[u] = k < cnt ? atomicAdd(&s_at[b], 1u) : 0u;
        out[u] = s_out[b] + at[u];
        idx[u] = (unsigned)i;
    }
    // x[u] of the element at tile place u * nt + t, for all of the tile
    auto exchange = [&](unsigned (&x)[TILE_ITEMS]) {
#pragma unroll
        for (unsigned u = 0; u < TILE_ITEMS; u++)
            if (u * nt + t < cnt) s_x[at[u]] = x[u];
        __syncthreads();
#pragma unroll
        for (unsigned u = 0; u < TILE_ITEMS; u++) x[u] = u * nt + t < cnt ? s_x[u * nt + t] : 0u;
        __syncthreads();
    };
    exchange(out);
    exchange(idx);
#pragma unroll
    for (unsigned u = 0; u < TILE_ITEMS; u++)
        if (u * nt + t < cnt) vout[out[u]] = idx[u];
    unsigned c[4][TILE_ITEMS];
#pragma unroll
    for (unsigned u = 0; u < TILE_ITEMS; u++) {
        c[0][u] = __float_as_uint(r[u].x);
        c[1][u] = __float_as_uint(r[u].y);
        c[2][u] = __float_as_uint(r[u].z);
        c[3][u] = __float_as_uint(r[u].w);
    }
#pragma unroll
    for (unsigned k = 0; k < 4; k++) exchange(c[k]);
#pragma unroll
    for (unsigned u = 0; u < TILE_ITEMS; u++)
        if (u * nt + t < cnt)
            rec[out[u]] = make_float4(__uint_as_float(c[0][u]), __uint_as_float(c[1][u]), __uint_as_float(c[2][u]),
                                      __uint_as_float(c[3][u]));
}

struct BucketArgs {
    const uint32_t *vin;
    const float4 *rec;
    const float *pos, *mass;
    const uint32_t *start;    // buckets' starts
    const uint32_t *sys_off;
    SysCube *cube;
    Header *hdr;
    unsigned nsys;
    uint64_t *kin;            // the elements' keys, written here first
    uint64_t *kout;
    uint32_t *vout;
    float4 *spos;
    int8_t *cl;
    uint64_t *tkey;           // pieces of a bucket larger than SORT_BUCKET
    uint32_t *tidx, *ttag;
};

// DIRECT: every system is one bucket, its elements in input order.
template <bool DIRECT>
__device__ __forceinline__ float4 bucket_record(const BucketArgs &a, unsigned e) {
    if (!DIRECT) return a.rec[e];
    return make_float4(a.pos[3 * (size_t)e], a.pos[3 * (size_t)e + 1], a.pos[3 * (size_t)e + 2], a.mass[e]);
}
template <bool DIRECT>
__device__ __forceinline__ uint32_t bucket_index(const BucketArgs &a, unsigned e) { return DIRECT ? e : a.vin[e]; }

// Sorts the m elements from q0 on into words in sv.  A direct bucket is a whole
// system, whose root cube is found here too.
template <bool DIRECT, unsigned VT>
__device__ __forceinline__ Words sort_piece(const BucketArgs &a, unsigned sys, unsigned q0, unsigned m, uint64_t *sv,
                                            uint64_t *s_mm, float (*s_box)[8]) {
    const unsigned active = (m + ITEMS - 1) / ITEMS;
    uint64_t v[VT * ITEMS], kmin = ~0ull, kmax = 0;
    SysCube cube;
    constexpr bool HOLD = DIRECT && VT == 1;  // positions kept in registers between the two passes
    float3 p[HOLD ? VT * ITEMS : 1];
    if (DIRECT) {
        BoxFlags bf;
#pragma unroll
        for (unsigned x = 0; x < VT; x++) {
            const unsigned t = threadIdx.x + x * BS_THREADS;
#pragma unroll
            for (unsigned u = 0; u < ITEMS; u++) {
                const unsigned j = u * active + t;
                if (t < active && j < m) {
                    const float4 r = bucket_record<DIRECT>(a, q0 + j);
                    if (HOLD) p[x * ITEMS + u] = make_float3(r.x, r.y, r.z);
                    bf.add(r.x, r.y, r.z, r.w);
                }
            }
        }
        block_box<BS_THREADS>(bf, s_box);
        cube = root_cube(bf);
        if (threadIdx.x == 0) {
            a.cube[sys] = cube;
            if (bf.flags) atomicOr(&a.hdr->flags, bf.flags);
        }
    } else {
        cube = a.cube[sys];
    }
#pragma unroll
    for (unsigned x = 0; x < VT; x++) {
        const unsigned t = threadIdx.x + x * BS_THREADS;
#pragma unroll
        for (unsigned u = 0; u < ITEMS; u++) {
            const unsigned j = u * active + t;
            uint64_t k = 0;
            if (t < active && j < m) {
                if (HOLD) {
                    k = morton_key(cube, p[x * ITEMS + u].x, p[x * ITEMS + u].y, p[x * ITEMS + u].z);
                } else {
                    const float4 r = bucket_record<DIRECT>(a, q0 + j);
                    k = morton_key(cube, r.x, r.y, r.z);
                }
                a.kin[q0 + j] = k;
                kmin = min(kmin, k);
                kmax = max(kmax, k);
            }
            v[x * ITEMS + u] = k;
        }
    }
    block_minmax<BS_THREADS>(kmin, kmax, s_mm);
    const Words wd(kmin, kmax, active * ITEMS);
#pragma unroll
    for (unsigned x = 0; x < VT; x++) {
        const unsigned t = threadIdx.x + x * BS_THREADS;
#pragma unroll
        for (unsigned u = 0; u < ITEMS; u++) {
            const unsigned j = u * active + t;
            v[x * ITEMS + u] = t < active && j < m ? wd.word(v[x * ITEMS + u], j) : ~0ull;  // padding comes last
        }
    }
    block_sort<BS_THREADS, VT>(v, active, sv);
    return wd;
}

// One workgroup per bucket.  What is sorted in LDS is one 64-bit word per
// element (struct Words): at least 52 bits of key distance and the place.
// Words that agree in those are then put in order by (key, index): a short run by
// one thread, and a bucket with a run longer than BS_RUN (particles that coincide
// or lie close) by a second sort of words that hold the run and the index
// in place of the key.  (Sorted by every digit of index and key instead, 2^22
// particles at n / 40 points took 812 us for the build; now 595, the radix sort 677.)
// BEGIN: the one workgroup of a one-bucket build also starts it.
template <bool DIRECT, bool BEGIN>
__global__ __launch_bounds__(BS_THREADS, BS_WAVES) void k_bucket_sort(BucketArgs a, BuildStart st) {
    __shared__ uint64_t sv[phys_size(SORT_BUCKET)];
    __shared__ uint64_t s_mm[2 * BS_THREADS / 64];
    __shared__ float s_box[BS_THREADS / 64][8];
    __shared__ unsigned s_long;
    const unsigned t = threadIdx.x, b = blockIdx.x;
    if (BEGIN) {
        begin_build(st);
        __syncthreads();
    }
    const unsigned b0 = BEGIN ? 0u : a.start[b], cnt = BEGIN ? st.o.off[1] : a.start[b + 1] - b0;
    if (cnt == 0) return;
    const unsigned sys = DIRECT ? b : a.nsys > 1 ? system_of(a.sys_off, a.nsys, b0) : 0u;
    const bool first = DIRECT || b0 == a.sys_off[sys];
    const unsigned pieces = (cnt + SORT_BUCKET - 1) / SORT_BUCKET;
    // key of a sorted word: from the word where it holds every key bit
    unsigned tb = 0, pmask = 0;
    uint64_t kmin = 0;
    bool whole = false;
    for (unsigned q = 0; q < pieces; q++) {
        const unsigned q0 = b0 + q * SORT_BUCKET, m = min((unsigned)SORT_BUCKET, cnt - q * SORT_BUCKET);
        if (t == 0) s_long = 0;
        const Words wd = m <= BS_THREADS * ITEMS ? sort_piece<DIRECT, 1>(a, sys, q0, m, sv, s_mm, s_box)
                                                 : sort_piece<DIRECT, BS_VT>(a, sys, q0, m, sv, s_mm, s_box);
        auto key = [&](unsigned p) { return a.kin[q0 + p]; };
        auto index = [&](unsigned p) { return bucket_index<DIRECT>(a, q0 + p); };
        // (places in input order need nothing where the words hold every key bit)
        if (!DIRECT || wd.sh > 0) order_runs<BS_THREADS>(sv, m, wd, &s_long, key, index);
        __syncthreads();
        const bool all = s_long != 0;  // the same for the whole workgroup
        if (all) {
            static_assert(SORT_BUCKET <= 4096, "words leave out 8 key bits at most: 8 + 32 + 2 * 12 bits");
            sort_runs<BS_THREADS, BS_VT>(sv, m, wd, [&](unsigned p) {
                const uint64_t low = wd.sh > 0 ? (key(p) - wd.kmin) & ((1ull << wd.sh) - 1ull) : 0ull;
                return low << 32 | index(p);
            });
        }
        tb = wd.tb;
        pmask = (1u << tb) - 1u;
        kmin = wd.kmin;
        whole = wd.sh == 0 && !all;
        if (pieces == 1) break;
        for (unsigned r = t; r < m; r += BS_THREADS) {
            const unsigned p = (unsigned)sv[phys(r)] & pmask;
            a.tkey[q0 + r] = a.kin[q0 + p];
            a.tidx[q0 + r] = bucket_index<DIRECT>(a, q0 + p);
            a.ttag[q0 + r] = q0 + p;
        }
        __syncthreads();
    }
    // A bucket's first element leaves its shared digits to the tree build
    // (CL_FROM_KEYS), which then sees the key before it.
    const int8_t lead = first ? (int8_t)-1 : CL_FROM_KEYS;
    if (pieces == 1) {
        auto word_key = [&](uint64_t v) { return whole ? kmin + (v >> tb) : a.kin[b0 + ((unsigned)v & pmask)]; };
        for (unsigned r = t; r < cnt; r += BS_THREADS) {
            const uint64_t v = sv[phys(r)];
            const unsigned e = b0 + ((unsigned)v & pmask);
            const uint64_t kr = word_key(v);
            a.kout[b0 + r] = kr;
            a.vout[b0 + r] = bucket_index<DIRECT>(a, e);
            a.spos[b0 + r] = bucket_record<DIRECT>(a, e);
            a.cl[b0 + r] = r == 0 ? lead : (int8_t)shared_digits(word_key(sv[phys(r - 1u)]), kr);
        }
        return;
    }
    // pieces ranked against each other: an element's place is its place in its
    // own piece plus the number of elements before it in every other
    for (unsigned j = t; j < cnt; j += BS_THREADS) {
        const uint64_t kj = a.tkey[b0 + j];
        const uint32_t xj = a.tidx[b0 + j];
        const unsigned own = j / SORT_BUCKET;
        unsigned r = j - own * SORT_BUCKET;
        for (unsigned q = 0; q < pieces; q++) {
            if (q == own) continue;
            const unsigned q0 = b0 + q * SORT_BUCKET;
            unsigned lo = 0, hi = min((unsigned)SORT_BUCKET, cnt - q * SORT_BUCKET);
            while (lo < hi) {
                const unsigned mid = (lo + hi) >> 1;
                if (before(a.tkey[q0 + mid], a.tidx[q0 + mid], kj, xj)) lo = mid + 1u; else hi = mid;
            }
            r += lo;
        }
        a.kout[b0 + r] = kj;
        a.vout[b0 + r] = xj;
        a.spos[b0 + r] = bucket_record<DIRECT>(a, a.ttag[b0 + j]);
    }
    __syncthreads();
    for (unsigned r = t; r < cnt; r += BS_THREADS)
        a.cl[b0 + r] = r == 0 ? lead : (int8_t)shared_digits(a.kout[b0 + r - 1u], a.kout[b0 + r]);
}

}  // namespace

// Scratch of the bucket sort in the cells' moment array, which the build leaves
// free until the multipole pass: 18 bytes per particle and the tiles' counts.
struct BucketScratch {
    uint64_t *tkey, *spl_key, *list_key;
    uint32_t *tidx, *ttag, *spl_idx, *list_idx, *counts, *total, *start;
    unsigned short *bkt;
};

// Particles per tile: small ones for small inputs, to reach more compute units.
static unsigned bucket_tile(unsigned n) {
    return (n <= (1u << 19) ? 256u : n <= (1u << 21) ? 512u : 1024u) * TILE_ITEMS;
}

static size_t bucket_scratch(unsigned n, unsigned nb, char *base, BucketScratch *sc) {
    size_t off = 0;
    auto take = [&](size_t bytes) -> char * {
        char *p = base + off;
        off = (off + bytes + 255) & ~(size_t)255;
        return p;
    };
    const unsigned ntiles = (n + bucket_tile(n) - 1) / bucket_tile(n);
    BucketScratch t;
    t.tkey = (uint64_t *)take(8 * (size_t)n);
    t.tidx = (uint32_t *)take(4 * (size_t)n);
    t.ttag = (uint32_t *)take(4 * (size_t)n);
    t.bkt = (unsigned short *)take(2 * (size_t)n);
    t.spl_key = (uint64_t *)take(8 * (size_t)nb);
    t.spl_idx = (uint32_t *)take(4 * (size_t)nb);
    t.list_key = (uint64_t *)take(8 * SAMPLE_PER_BUCKET * (size_t)nb);
    t.list_idx = (uint32_t *)take(4 * SAMPLE_PER_BUCKET * (size_t)nb);
    t.total = (uint32_t *)take(4 * (size_t)nb);
    t.start = (uint32_t *)take(4 * ((size_t)nb + 1));
    t.counts = (uint32_t *)take(4 * (size_t)nb * ntiles);
    if (sc) *sc = t;
    return off;
}

bool bucket_sort_fits(const Buffers &b, unsigned n, unsigned nb) {
    return nb <= SORT_MAX_BUCKETS && bucket_scratch(n, nb, nullptr, nullptr) <= 80 * (size_t)b.cap_cells;
}

// Root cubes and the partition into nb buckets (nothing to do where every system
// is one: its sort finds the cube).  nb_max: buckets of the largest system.
hipError_t launch_bucket_partition(const Buffers &b, const BuildStart &start, const float *pos, const float *mass,
                                   unsigned n, unsigned nsys, unsigned nb, unsigned nb_max, hipStream_t s) {
    if (nb == nsys) return hipSuccess;
    BucketScratch sc;
    bucket_scratch(n, nb, (char *)b.mp, &sc);
    const unsigned tile = bucket_tile(n), nt = tile / TILE_ITEMS, ntiles = (n + tile - 1) / tile;
    unsigned nparts;
    hipError_t e = launch_bbox_partial(b, start, pos, mass, nsys, &nparts, s);
    if (e != hipSuccess) return e;
    const unsigned lists = min((SAMPLE_PER_BUCKET * nb_max + SAMPLE_LIST - 1u) / SAMPLE_LIST, SAMPLE_LISTS);
    hipLaunchKernelGGL(k_bucket_sample, dim3(lists, nsys), dim3(SAMPLE_THREADS), 0, s, pos, b.sys_off, b.bkt_off,
                       b.bbox_part, nparts, b.hdr, b.cube, sc.spl_key, sc.spl_idx, sc.list_key, sc.list_idx);
    if (lists > 1)
        hipLaunchKernelGGL(k_bucket_split, dim3(lists * SAMPLE_LIST / 256u, nsys), dim3(256), 0, s, b.sys_off, b.bkt_off,
                           sc.list_key, sc.list_idx, sc.spl_key, sc.spl_idx);
    hipLaunchKernelGGL(k_bucket_count, dim3(ntiles), dim3(nt), 16 * (size_t)nb, s, pos, n, nsys, b.sys_off, b.bkt_off,
                       b.cube, sc.spl_key, sc.spl_idx, nb, sc.bkt, sc.counts);
    const unsigned grid = 8u * ((ntiles + 7u) / 8u);
    const size_t lds = 8 * (size_t)nb + 4 * (size_t)tile;
    if (ntiles <= SCATTER_SCAN_TILES && nb <= nt) {
        hipLaunchKernelGGL(k_bucket_scatter<true>, dim3(grid), dim3(nt), lds, s, pos, mass, sc.bkt, n, sc.counts, ntiles,
                           nullptr, nb, sc.start, b.vals[1], b.ppack);
    } else {
        hipLaunchKernelGGL(k_bucket_scan, dim3((nb + 63u) / 64u), dim3(64 * SCAN_SEGS), 0, s, sc.counts, ntiles, nb,
                           sc.total);
        hipLaunchKernelGGL(k_bucket_scatter<false>, dim3(grid), dim3(nt), lds, s, pos, mass, sc.bkt, n, sc.counts, ntiles,
                           sc.total, nb, sc.start, b.vals[1], b.ppack);
    }
    return hipGetLastError();
}

// Sorts the buckets into keys[0], vals[0], spos and cl.
hipError_t launch_bucket_sort(const Buffers &b, const BuildStart *start, const float *pos, const float *mass,
                              unsigned n, unsigned nsys, unsigned nb, hipStream_t s) {
    BucketScratch sc;
    bucket_scratch(n, nb, (char *)b.mp, &sc);
    BucketArgs a;
    const bool direct = nb == nsys;
    a.vin = b.vals[1];
    a.rec = b.ppack;
    a.pos = pos;
    a.mass = mass;
    a.start = direct ? b.sys_off : sc.start;
    a.sys_off = b.sys_off;
    a.cube = b.cube;
    a.hdr = b.hdr;
    a.nsys = nsys;
    a.kin = b.keys[1];
    a.kout = b.keys[0];
    a.vout = b.vals[0];
    a.spos = b.spos;
    a.cl = b.cl;
    a.tkey = sc.tkey;
    a.tidx = sc.tidx;
    a.ttag = sc.ttag;
    const bool begin = direct && start;
    BuildStart st = {};
    if (begin) st = *start;
    if (begin) hipLaunchKernelGGL((k_bucket_sort<true, true>), dim3(1), dim3(BS_THREADS), 0, s, a, st);
    else if (direct) hipLaunchKernelGGL((k_bucket_sort<true, false>), dim3(nb), dim3(BS_THREADS), 0, s, a, st);
    else hipLaunchKernelGGL((k_bucket_sort<false, false>), dim3(nb), dim3(BS_THREADS), 0, s, a, st);
    return hipGetLastError();
}

}  // namespace mibh
