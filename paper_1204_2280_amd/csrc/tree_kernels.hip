// Tree pipeline of the force step on gfx950: bounding cube, Morton keys,
// stable LSD radix sort, reorder ("moving"), breadth-first sparse octree and
// groups ("tree-construction"), float64 multipole moments and the per-theta
// opening radii.  The paper's parts are named in its Results section; the
// kernels here are this library's own design for CDNA4 (wave64 ballots,
// LDS-staged windows, no host synchronisation inside a step).
#include "mibh_device.h"

#include <math.h>

namespace mibh {

// --------------------------------------------------------------------------
// wave64 helpers
// --------------------------------------------------------------------------

__device__ __forceinline__ unsigned lane64() { return __lane_id(); }

// Number of set bits of mask in lanes below this one.
__device__ __forceinline__ unsigned rank_below(unsigned long long mask) {
    return __builtin_amdgcn_mbcnt_hi((unsigned)(mask >> 32),
                                     __builtin_amdgcn_mbcnt_lo((unsigned)mask, 0u));
}

// Lanes (among those in `active`) holding the same 8-bit digit as this lane.
__device__ __forceinline__ unsigned long long match_digit(unsigned d, unsigned long long active) {
    unsigned long long m = active;
#pragma unroll
    for (int b = 0; b < RADIX_BITS; b++) {
        const bool bit = (d >> b) & 1u;
        const unsigned long long v = __ballot(bit);
        m &= bit ? v : ~v;
    }
    return m;
}

// Inclusive scan over the 64 lanes of a wave.
__device__ __forceinline__ unsigned wave_incl_scan(unsigned v) {
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) {
        unsigned y = __shfl_up(v, o, 64);
        if (lane64() >= (unsigned)o) v += y;
    }
    return v;
}

// Exclusive scan of a block of NT threads (NT multiple of 64, <= 1024).
template <int NT>
__device__ __forceinline__ unsigned block_excl_scan(unsigned v, unsigned *s_wave, unsigned *total) {
    const unsigned w = threadIdx.x >> 6;
    const unsigned inc = wave_incl_scan(v);
    if (lane64() == 63) s_wave[w] = inc;
    __syncthreads();
    if (threadIdx.x == 0) {
        unsigned run = 0;
        for (int i = 0; i < NT / 64; i++) {
            unsigned t = s_wave[i];
            s_wave[i] = run;
            run += t;
        }
        s_wave[NT / 64] = run;
    }
    __syncthreads();
    const unsigned r = s_wave[w] + inc - v;
    *total = s_wave[NT / 64];
    __syncthreads();
    return r;
}

// Inverse of spread3: gathers bits 0, 3, 6, ... into a dense integer.
__device__ __forceinline__ uint32_t compact3(uint64_t x) {
    x &= 0x1249249249249249ull;
    x = (x ^ (x >> 2)) & 0x10c30c30c30c30c3ull;
    x = (x ^ (x >> 4)) & 0x100f00f00f00f00full;
    x = (x ^ (x >> 8)) & 0x1f0000ff0000ffull;
    x = (x ^ (x >> 16)) & 0x1f00000000ffffull;
    x = (x ^ (x >> 32)) & 0x1fffffull;
    return (uint32_t)x;
}

// First index j > i whose key differs from key i in the first `lev` octal
// digits (n if none) in the sorted keys.  A round reads WAYS - 1 keys side by side
// and cuts the range to a part in WAYS: first at distances 64 and up from i, then
// evenly in what is left.  A chain of dependent reads, 0.4 us each, is what the
// search costs where the chip is not full; in large trees it is the reads' bytes.
// The write kernel below by doubling and halving / with 4 / with 8 ways, us: n =
// 40000 13.6 / 9.3 / 8.6, 2^18 15.4 / 10.3 / 9.8, 2^19 17.3 / 12.8 / 12.6, 2^20 23.3 /
// 19.3 / 19.4, 2^21 34.8 / 30.8 / 34.0, 2^22 59.2 / 56.2 / 63.4, 12 million 164 / 153 /
// 177: 8 up to RUN_END_EIGHTHS particles, 4 beyond.
constexpr unsigned RUN_END_EIGHTHS = 1u << 19;
template <unsigned WAYS>
__device__ __forceinline__ unsigned run_end(const uint64_t *__restrict__ keys, unsigned n, unsigned i,
                                            int lev) {
    constexpr unsigned Q = WAYS - 1u, GROW = 21u / Q;  // the last of the first round's distances: 2^24 / 2^GROW
    // n is the end of i's system: keys of different systems are never compared
    if (lev == 0) return n;
    const int sh = 3 * (KEY_LEVELS - lev);
    const uint64_t p = keys[i] >> sh;
    unsigned lo = i, hi = n;  // lo is in the run, hi is not
    unsigned step = 0;
    do {
        unsigned pos[Q];
        uint64_t k[Q];
#pragma unroll
        for (unsigned q = 0; q < Q; q++) {
            pos[q] = min(step ? lo + step * (q + 1u) : lo + (64u << GROW * q), hi);
            k[q] = keys[min(pos[q], n - 1u)] >> sh;
        }
#pragma unroll
        for (unsigned q = 0; q < Q; q++) lo = pos[q] < hi && k[q] == p ? pos[q] : lo;
#pragma unroll
        for (int q = (int)Q - 1; q >= 0; q--) hi = pos[q] > lo ? pos[q] : hi;
        step = (hi - lo + Q) / WAYS;
    } while (hi - lo > 1);
    return hi;
}

// --------------------------------------------------------------------------
// Bounding cube, one per system (grid row y = system)
// --------------------------------------------------------------------------

__global__ __launch_bounds__(256) void k_bbox_partial(BuildStart start, const float *__restrict__ pos,
                                                      const float *__restrict__ mass, float *__restrict__ part) {
    __shared__ float s[4][8];
    const unsigned sys = blockIdx.y;
    const unsigned b0 = start.o.off[sys], b1 = start.o.off[sys + 1];
    if (blockIdx.x == 0 && sys == 0) begin_build(start);
    BoxFlags b;
    for (unsigned i = b0 + blockIdx.x * 256u + threadIdx.x; i < b1; i += gridDim.x * 256u) {
        const size_t p = (size_t)i * 3;
        b.add(pos[p], pos[p + 1], pos[p + 2], mass[i]);
    }
    block_box<256>(b, s);
    if (threadIdx.x == 0) b.store(part + ((size_t)sys * gridDim.x + blockIdx.x) * 8);
}

// Root cube of each system (one block per system).
__global__ __launch_bounds__(256) void k_bbox_final(const float *__restrict__ part, unsigned nblocks,
                                                    Header *__restrict__ hdr, SysCube *__restrict__ cube) {
    __shared__ float s[4][8];
    const unsigned sys = blockIdx.x;
    BoxFlags b;
    for (unsigned q = threadIdx.x; q < nblocks; q += 256) b.add(part + ((size_t)sys * nblocks + q) * 8);
    block_box<256>(b, s);
    if (threadIdx.x == 0) {
        cube[sys] = root_cube(b);
        if (b.flags) atomicOr(&hdr->flags, b.flags);
    }
}

hipError_t launch_bbox_partial(const Buffers &b, const BuildStart &start, const float *pos, const float *mass,
                               unsigned nsys, unsigned *nparts, hipStream_t s) {
    const unsigned per = max((unsigned)BBOX_MIN_BLOCKS, (unsigned)BBOX_BLOCKS / nsys);
    hipLaunchKernelGGL(k_bbox_partial, dim3(per, nsys), dim3(256), 0, s, start, pos, mass, b.bbox_part);
    *nparts = per;
    return hipGetLastError();
}

hipError_t launch_bbox(const Buffers &b, const BuildStart &start, const float *pos, const float *mass, unsigned nsys,
                       hipStream_t s) {
    unsigned per;
    hipError_t e = launch_bbox_partial(b, start, pos, mass, nsys, &per, s);
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(k_bbox_final, dim3(nsys), dim3(256), 0, s, b.bbox_part, per, b.hdr, b.cube);
    return hipGetLastError();
}

// --------------------------------------------------------------------------
// Morton keys: q_a = min(floor((x_a - lo_a) 2^(20-k)), 2^20 - 1), bits of
// q_x, q_y, q_z at 3b+2, 3b+1, 3b.
// --------------------------------------------------------------------------

// Also packs (x, y, z, m) of every particle into one float4, so that the
// reorder gathers one 16-byte record per particle instead of two.
__global__ __launch_bounds__(256) void k_keys(const float *__restrict__ pos, const float *__restrict__ mass,
                                              unsigned n, unsigned nsys, const uint32_t *__restrict__ sys_off,
                                              const SysCube *__restrict__ cube, uint64_t *__restrict__ keys,
                                              uint8_t *__restrict__ sys8, float4 *__restrict__ ppack) {
    const unsigned i = blockIdx.x * 256u + threadIdx.x;
    if (i >= n) return;
    const unsigned sys = nsys > 1 ? system_of(sys_off, nsys, i) : 0u;
    const float x = pos[(size_t)i * 3], y = pos[(size_t)i * 3 + 1], z = pos[(size_t)i * 3 + 2];
    ppack[i] = make_float4(x, y, z, mass[i]);
    keys[i] = morton_key(cube[sys], x, y, z);
    if (nsys > 1) sys8[i] = (uint8_t)sys;
}

// Refit input: packs (x, y, z, m) like the keys kernel and records non-finite
// values and negative masses in the header flags (the build does this in its
// bounding-box pass).
__global__ __launch_bounds__(256) void k_pack(const float *__restrict__ pos, const float *__restrict__ mass,
                                              unsigned n, Header *__restrict__ hdr, float4 *__restrict__ ppack) {
    for (unsigned i = blockIdx.x * 256u + threadIdx.x; i < n; i += gridDim.x * 256u) {
        const float4 p = make_float4(pos[(size_t)i * 3], pos[(size_t)i * 3 + 1], pos[(size_t)i * 3 + 2], mass[i]);
        ppack[i] = p;
        unsigned f = 0;
        if (!isfinite(p.x) || !isfinite(p.y) || !isfinite(p.z) || !isfinite(p.w)) f |= FLAG_NONFINITE;
        if (p.w < 0.0f) f |= FLAG_NEGMASS;
        if (f) atomicOr(&hdr->flags, f);
    }
}

hipError_t launch_pack(const Buffers &b, const float *pos, const float *mass, unsigned n, hipStream_t s) {
    const unsigned grid = min((n + 255u) / 256u, 8192u);
    hipLaunchKernelGGL(k_pack, dim3(grid), dim3(256), 0, s, pos, mass, n, b.hdr, b.ppack);
    return hipGetLastError();
}

hipError_t launch_keys(const Buffers &b, const float *pos, const float *mass, unsigned n, unsigned nsys,
                       hipStream_t s) {
    hipLaunchKernelGGL(k_keys, dim3((n + 255) / 256), dim3(256), 0, s, pos, mass, n, nsys, b.sys_off, b.cube,
                       b.keys[radix_first_buffer(nsys)], b.sys8, b.ppack);
    return hipGetLastError();
}

// --------------------------------------------------------------------------
// Stable LSD radix sort of (key, index), 8-bit digits, reduce-then-scan:
// per-tile digit histograms -> per-digit scan over tiles -> stable scatter.
// Ranks inside a tile come from wave64 digit matching (8 ballots) processed
// in key order, so equal digits keep their input order.
// --------------------------------------------------------------------------

// Digit of an element: 8 key bits at `shift`, or (shift < 0) the element's
// system, looked up by its original index (the last pass of a batch).
__device__ __forceinline__ unsigned radix_digit(uint64_t key, uint32_t val, int shift,
                                                const uint8_t *__restrict__ sys8) {
    return shift >= 0 ? (unsigned)(key >> shift) & (RADIX - 1) : (unsigned)sys8[val];
}

// AGG: equal digits of a wave are matched first (8 ballots) and their leader
// adds their number, one LDS atomic per distinct digit instead of per element:
// cheaper where digits are concentrated (the high digits of clustered keys,
// the system digit), where per-element atomics collide on one counter.
template <bool AGG>
__global__ __launch_bounds__(SORT_THREADS) void k_radix_hist(const uint64_t *__restrict__ keys,
                                                             const uint32_t *__restrict__ vals,
                                                             const uint8_t *__restrict__ sys8,
                                                             unsigned n, int shift,
                                                             uint32_t *__restrict__ hist,
                                                             unsigned ntiles) {
    __shared__ uint32_t h[SORT_THREADS / 64][RADIX];
    const unsigned w = threadIdx.x >> 6, ln = lane64();
    for (unsigned j = threadIdx.x; j < (SORT_THREADS / 64) * RADIX; j += SORT_THREADS) (&h[0][0])[j] = 0;
    __syncthreads();
    const unsigned base = blockIdx.x * SORT_TILE + w * (64 * SORT_ITEMS);
#pragma unroll
    for (int t = 0; t < SORT_ITEMS; t++) {
        const unsigned idx = base + t * 64 + ln;
        const bool valid = idx < n;
        const unsigned d = valid ? radix_digit(shift >= 0 ? keys[idx] : 0ull, shift >= 0 ? 0u : vals[idx], shift,
                                               sys8)
                                 : 0u;
        if (AGG) {
            const unsigned long long peers = match_digit(d, __ballot(valid));
            if (valid && ln == (unsigned)(__ffsll((long long)peers) - 1)) atomicAdd(&h[w][d], (unsigned)__popcll(peers));
        } else if (valid) {
            atomicAdd(&h[w][d], 1u);  // integer counts: the order of the adds does not matter
        }
    }
    __syncthreads();
    for (unsigned d = threadIdx.x; d < RADIX; d += SORT_THREADS) {
        unsigned s = 0;
        for (int v = 0; v < SORT_THREADS / 64; v++) s += h[v][d];
        hist[(size_t)d * ntiles + blockIdx.x] = s;
    }
}

// One block per digit: exclusive scan of its row over tiles; row total to btot.
__global__ __launch_bounds__(256) void k_radix_scan(uint32_t *__restrict__ hist, unsigned ntiles,
                                                    uint32_t *__restrict__ btot) {
    __shared__ unsigned s_wave[256 / 64 + 1];
    uint32_t *row = hist + (size_t)blockIdx.x * ntiles;
    const unsigned per = (ntiles + 255) / 256;
    const unsigned b = threadIdx.x * per, e = min(b + per, ntiles);
    unsigned sum = 0;
    for (unsigned j = b; j < e; j++) sum += row[j];
    unsigned total;
    unsigned run = block_excl_scan<256>(sum, s_wave, &total);
    for (unsigned j = b; j < e; j++) {
        const unsigned v = row[j];
        row[j] = run;
        run += v;
    }
    if (threadIdx.x == 0) btot[blockIdx.x] = total;
}

// Ranks every element of the tile (digit, then input order), stages the tile
// in LDS in that order and writes it out from there: consecutive threads then
// write consecutive addresses of each digit's run.
__global__ __launch_bounds__(SORT_THREADS) void k_radix_scatter(
    const uint64_t *__restrict__ kin, const uint32_t *__restrict__ vin, uint64_t *__restrict__ kout,
    uint32_t *__restrict__ vout, const uint8_t *__restrict__ sys8, unsigned n, int shift,
    const uint32_t *__restrict__ hist, const uint32_t *__restrict__ btot, unsigned ntiles) {
    constexpr int NW = SORT_THREADS / 64;
    static_assert(SORT_THREADS % RADIX == 0, "the first RADIX threads look after one digit each");
    __shared__ uint32_t wcnt[NW][RADIX];
    __shared__ uint32_t gshift[RADIX];  // output position of tile position i of digit d: gshift[d] + i
    __shared__ unsigned s_wave[NW + 1];
    __shared__ uint64_t s_key[SORT_TILE];  // the indices (as 32-bit words), then the keys
    const unsigned w = threadIdx.x >> 6, ln = lane64();
    const bool owner = threadIdx.x < (unsigned)RADIX;
    const unsigned dt = owner ? threadIdx.x : 0u;  // the digit this thread looks after
    unsigned total;
    // start of digit dt's run of this tile in the output
    const unsigned gstart = block_excl_scan<SORT_THREADS>(owner ? btot[dt] : 0u, s_wave, &total) +
                            (owner ? hist[(size_t)dt * ntiles + blockIdx.x] : 0u);
    if (owner)
        for (int v = 0; v < NW; v++) wcnt[v][dt] = 0;
    __syncthreads();
    const unsigned base = blockIdx.x * SORT_TILE + w * (64 * SORT_ITEMS);
    uint64_t key[SORT_ITEMS];
    uint32_t val[SORT_ITEMS], rank[SORT_ITEMS];
#pragma unroll
    for (int t = 0; t < SORT_ITEMS; t++) {
        const unsigned idx = base + t * 64 + ln;
        const bool valid = idx < n;
        key[t] = valid ? kin[idx] : 0ull;
        val[t] = valid ? (vin ? vin[idx] : idx) : 0u;
        const unsigned d = valid ? radix_digit(key[t], val[t], shift, sys8) : 0u;
        const unsigned long long peers = match_digit(d, __ballot(valid));
        const unsigned before = wcnt[w][d];
        rank[t] = before + rank_below(peers);
        if (valid && ln == (unsigned)(__ffsll((long long)peers) - 1)) wcnt[w][d] = before + __popcll(peers);
    }
    __syncthreads();
    {
        // tile position of the first element of digit dt from wave v: digits
        // before dt, then waves before v
        unsigned run = 0;
        if (owner)
            for (int v = 0; v < NW; v++) {
                const unsigned c = wcnt[v][dt];
                wcnt[v][dt] = run;
                run += c;
            }
        const unsigned lstart = block_excl_scan<SORT_THREADS>(run, s_wave, &total);
        if (owner) {
            for (int v = 0; v < NW; v++) wcnt[v][dt] += lstart;
            gshift[dt] = gstart - lstart;  // modulo 2^32; gshift + i >= 0 for the tile positions of dt
        }
    }
    __syncthreads();
    // the indices, then the keys, through the same LDS (a third less LDS, three
    // blocks per CU instead of two: sorting 402 -> 395 us at N = 2^22); each
    // thread keeps the indices of its tile positions between the two phases,
    // since the system pass needs an element's index for its digit
    unsigned lpos[SORT_ITEMS];
    uint32_t *s_val = reinterpret_cast<uint32_t *>(s_key);
#pragma unroll
    for (int t = 0; t < SORT_ITEMS; t++) {
        const unsigned idx = base + t * 64 + ln;
        const unsigned d = idx < n ? radix_digit(key[t], val[t], shift, sys8) : 0u;
        lpos[t] = wcnt[w][d] + rank[t];
    }
    const unsigned cnt = min((unsigned)SORT_TILE, n - blockIdx.x * SORT_TILE);
    uint32_t vpos[SORT_ITEMS];  // the index at tile position threadIdx.x + t * SORT_THREADS
    // phase 1: the indices
#pragma unroll
    for (int t = 0; t < SORT_ITEMS; t++)
        if (base + t * 64 + ln < n) s_val[lpos[t]] = val[t];
    __syncthreads();
#pragma unroll
    for (int t = 0; t < SORT_ITEMS; t++) {
        const unsigned i = threadIdx.x + t * SORT_THREADS;
        vpos[t] = i < cnt ? s_val[i] : 0u;
    }
    __syncthreads();
    // phase 2: the keys; position i's output slot from its digit
#pragma unroll
    for (int t = 0; t < SORT_ITEMS; t++)
        if (base + t * 64 + ln < n) s_key[lpos[t]] = key[t];
    __syncthreads();
#pragma unroll
    for (int t = 0; t < SORT_ITEMS; t++) {
        const unsigned i = threadIdx.x + t * SORT_THREADS;
        if (i < cnt) {
            const uint64_t k = s_key[i];
            const uint32_t v = vpos[t];
            const unsigned p = gshift[radix_digit(k, v, shift, sys8)] + i;
            kout[p] = k;
            vout[p] = v;
        }
    }
}

#ifndef MIBH_HIST_AGG_SHIFT
#define MIBH_HIST_AGG_SHIFT 48  // passes over key bits 48.. (and the system pass) match digits first
                                // (sorting at 2^22: 404 us without, 401 us with, 439 us for every pass)
#endif

// 8 passes over the 60-bit keys; a batch adds a last pass by system, which
// gathers each system's particles (in key order) into its input range.
hipError_t launch_sort(const Buffers &b, unsigned n, unsigned nsys, hipStream_t s) {
    const unsigned ntiles = (n + SORT_TILE - 1) / SORT_TILE;
    const int passes = SORT_PASSES + (nsys > 1 ? 1 : 0);
    for (int pass = 0; pass < passes; pass++) {
        const int src = (pass + radix_first_buffer(nsys)) & 1, dst = src ^ 1;
        const int shift = pass < SORT_PASSES ? pass * RADIX_BITS : -1;
        if (shift < 0 || shift >= MIBH_HIST_AGG_SHIFT)
            hipLaunchKernelGGL(k_radix_hist<true>, dim3(ntiles), dim3(SORT_THREADS), 0, s, b.keys[src], b.vals[src],
                               b.sys8, n, shift, b.hist, ntiles);
        else
            hipLaunchKernelGGL(k_radix_hist<false>, dim3(ntiles), dim3(SORT_THREADS), 0, s, b.keys[src], b.vals[src],
                               b.sys8, n, shift, b.hist, ntiles);
        hipLaunchKernelGGL(k_radix_scan, dim3(RADIX), dim3(256), 0, s, b.hist, ntiles, b.btot);
        hipLaunchKernelGGL(k_radix_scatter, dim3(ntiles), dim3(SORT_THREADS), 0, s, b.keys[src],
                           pass == 0 ? (const uint32_t *)nullptr : b.vals[src], b.keys[dst], b.vals[dst],
                           b.sys8, n, shift, b.hist, b.btot, ntiles);
    }
    return hipGetLastError();
}

// --------------------------------------------------------------------------
// Moving: gather (x, y, z, m) into key order; shared digits with the previous key.
// --------------------------------------------------------------------------

__global__ __launch_bounds__(256) void k_reorder(const float4 *__restrict__ ppack,
                                                 const uint64_t *__restrict__ keys,
                                                 const uint32_t *__restrict__ perm, unsigned n, unsigned nsys,
                                                 const uint32_t *__restrict__ sys_off,
                                                 float4 *__restrict__ spos, int8_t *__restrict__ cl) {
    const unsigned k = blockIdx.x * 256u + threadIdx.x;
    if (k >= n) return;
    spos[k] = ppack[perm[k]];
    // a system's first particle opens cells at every level, like particle 0
    const bool start = k == 0 || (nsys > 1 && sys_off[system_of(sys_off, nsys, k)] == k);
    cl[k] = start ? (int8_t)-1 : (int8_t)shared_digits(keys[k - 1], keys[k]);
}

hipError_t launch_reorder(const Buffers &b, unsigned n, unsigned nsys, hipStream_t s) {
    hipLaunchKernelGGL(k_reorder, dim3((n + 255) / 256), dim3(256), 0, s, b.ppack, b.keys[0], b.vals[0],
                       n, nsys, b.sys_off, b.spos, b.cl);
    return hipGetLastError();
}

// --------------------------------------------------------------------------
// Octree and groups, particle-parallel.
//
// With cl(i) the number of leading octal digits keys i-1 and i share, the
// level-l cell containing particle i starts at i iff cl(i) < l, and it holds
// more than w particles iff some window of w+1 consecutive particles around i
// has all its w inner cl values >= l.  So
//   lstar_w(i) = max over windows [a, a+w] containing i of min cl(a+1..a+w)
// is the deepest level whose cell around i holds more than w particles.  The
// leaf of i is at level min(lstar_ncrit + 1, 20) (0 if lstar < 0), its group at
// min(lstar_gcap + 1, 20); particle i starts the cells of levels
// cl(i)+1 .. leaf(i).  Cell numbers are per-level ranks, which gives the
// breadth-first order (level, then key).
// --------------------------------------------------------------------------

// Value at position `pos` (0..127, or 0..191 with three registers) of an array
// held as consecutive 64-lane registers r0, r1, r2: lane pos & 63 of register
// pos >> 6.  Every lane passes its own position; the lane index is shared by the
// shuffles, the register is picked afterwards.
__device__ __forceinline__ int wave_at3(int r0, int r1, int r2, unsigned pos) {
    const int lane = (int)(pos & 63u);
    const int v0 = __shfl(r0, lane, 64), v1 = __shfl(r1, lane, 64), v2 = __shfl(r2, lane, 64);
    return pos < 64u ? v0 : pos < 128u ? v1 : v2;
}
__device__ __forceinline__ int wave_at2(int r0, int r1, unsigned pos) {
    const int lane = (int)(pos & 63u);
    const int v0 = __shfl(r0, lane, 64), v1 = __shfl(r1, lane, 64);
    return pos < 64u ? v0 : v1;
}

__global__ __launch_bounds__(BUILD_THREADS) void k_build_count(
    const int8_t *__restrict__ cl, const uint64_t *__restrict__ keys, unsigned n, unsigned nsys,
    const uint32_t *__restrict__ sys_off, int ncrit, int gcap, uchar4 *__restrict__ lvinfo,
    uint32_t *__restrict__ blkcnt, unsigned nblk) {
    constexpr int NW = BUILD_THREADS / 64;
    __shared__ uint32_t s_cnt[NW][NCOUNTERS];
    const unsigned base = blockIdx.x * BUILD_THREADS;
    const unsigned i = base + threadIdx.x;
    const bool valid = i < n;
    // Each wave on its own, in registers: the cl values of positions wb - 64 ..
    // wb + 127 (wb = the wave's first particle; -1 outside the particles) cover
    // every window that contains one of the wave's particles (ncrit, gcap <= 64).
    // This replaced doubling tables in LDS with 13 block barriers (tree
    // construction at N = 2^22: 148 -> 139 us).
    static_assert(MAX_WINDOW <= 64, "windows reach at most one wave width either side");
    const unsigned ln_ = lane64();
    const long long wb = (long long)base + (long long)(threadIdx.x & ~63u);
    int t[3];
#pragma unroll
    for (int r = 0; r < 3; r++) {
        const long long j = wb - 64 + 64 * r + ln_;
        t[r] = (j >= 0 && j < (long long)n) ? (int)cl[j] : -1;
        if (t[r] == CL_FROM_KEYS) t[r] = shared_digits(keys[j - 1], keys[j]);  // a sort bucket's first particle
    }
    const int ci = t[1];
    // Minima by doubling: after step k, t[r] at lane l is the minimum of the 2^k
    // values from position 64 r + l on (positions past 191 are never asked for).
    const int kn = 31 - __clz(ncrit), kg = 31 - __clz(gcap), kmax = max(kn, kg);
    int tn[3] = {t[0], t[1], t[2]}, tg[3] = {t[0], t[1], t[2]};
    for (int k = 0; k < kmax; k++) {
        const unsigned sh = 1u << k;
        const int src = (int)((ln_ + sh) & 63u);
        const bool wrap = ln_ + sh >= 64u;
        const int a0 = __shfl(t[0], src, 64), a1 = __shfl(t[1], src, 64), a2 = __shfl(t[2], src, 64);
        t[0] = min(t[0], wrap ? a1 : a0);
        t[1] = min(t[1], wrap ? a2 : a1);
        t[2] = min(t[2], wrap ? t[2] : a2);
        if (k + 1 == kn) { tn[0] = t[0]; tn[1] = t[1]; tn[2] = t[2]; }
        if (k + 1 == kg) { tg[0] = t[0]; tg[1] = t[1]; tg[2] = t[2]; }
    }
    // Window minima for the window starts a = wb - 64 + 64 r + lane (r = 0, 1):
    // min cl[a+1 .. a+w] = min(T[a+1], T[a+1+w-2^k]); a start's position is its
    // array position, so a+1 sits at 64 r + lane + 1.
    int mn[2], mg[2];
#pragma unroll
    for (int r = 0; r < 2; r++) {
        const unsigned p = 64u * r + ln_ + 1u;
        mn[r] = min(wave_at3(tn[0], tn[1], tn[2], p), wave_at3(tn[0], tn[1], tn[2], p + (unsigned)(ncrit - (1 << kn))));
        mg[r] = min(wave_at3(tg[0], tg[1], tg[2], p), wave_at3(tg[0], tg[1], tg[2], p + (unsigned)(gcap - (1 << kg))));
    }
    // ln = max of the window minima over the starts tl - w .. tl (tl = the
    // particle's start position, 64 + lane), maxima by doubling over the 128 starts.
    int ln, lg;
    {
        const int kn2 = 31 - __clz(ncrit + 1), kg2 = 31 - __clz(gcap + 1), kmax2 = max(kn2, kg2);
        int un[2] = {mn[0], mn[1]}, ug[2] = {mg[0], mg[1]};
        int vn[2] = {mn[0], mn[1]}, vg[2] = {mg[0], mg[1]};  // the tables at kn2 and kg2
        for (int k = 0; k < kmax2; k++) {
            const unsigned sh = 1u << k;
            const int src = (int)((ln_ + sh) & 63u);
            const bool wrap = ln_ + sh >= 64u;
            const int b0 = __shfl(un[0], src, 64), b1 = __shfl(un[1], src, 64);
            const int c0 = __shfl(ug[0], src, 64), c1 = __shfl(ug[1], src, 64);
            un[0] = max(un[0], wrap ? b1 : b0);
            un[1] = max(un[1], wrap ? un[1] : b1);
            ug[0] = max(ug[0], wrap ? c1 : c0);
            ug[1] = max(ug[1], wrap ? ug[1] : c1);
            if (k + 1 == kn2) { vn[0] = un[0]; vn[1] = un[1]; }
            if (k + 1 == kg2) { vg[0] = ug[0]; vg[1] = ug[1]; }
        }
        const unsigned tl = 64u + ln_;
        ln = max(wave_at2(vn[0], vn[1], tl - (unsigned)ncrit), wave_at2(vn[0], vn[1], tl - (1u << kn2) + 1u));
        lg = max(wave_at2(vg[0], vg[1], tl - (unsigned)gcap), wave_at2(vg[0], vg[1], tl - (1u << kg2) + 1u));
    }
    const int leaf = ln < 0 ? 0 : min(ln + 1, KEY_LEVELS);
    const int glev = lg < 0 ? 0 : min(lg + 1, KEY_LEVELS);
    const int clo = ci + 1;
    bool gstart;
    unsigned oversized = 0;
    if (lg >= KEY_LEVELS && valid) {
        // a run of more than gcap identical keys: cut into chunks of gcap from its start
        oversized = 1;
        unsigned start = i;
        if (ci >= KEY_LEVELS) {
            const uint64_t key = keys[i];
            // first index of the run lies in [start of i's system, i]
            unsigned lo = nsys > 1 ? sys_off[system_of(sys_off, nsys, i)] : 0u, hi = i;
            while (lo < hi) {
                const unsigned mid = lo + (hi - lo) / 2;
                if (keys[mid] < key) lo = mid + 1; else hi = mid;
            }
            start = lo;
        }
        gstart = ((i - start) % (unsigned)gcap) == 0;
    } else {
        gstart = ci < glev;
    }
    if (valid) lvinfo[i] = make_uchar4((unsigned char)clo, (unsigned char)leaf, (unsigned char)glev,
                                       (unsigned char)((gstart ? 1 : 0) | (oversized << 1)));
    // Padding threads start no cell (first level 1 > leaf level 0) and no
    // group, so the ballot loops below need no per-lane validity branch; the
    // wave-uniform counts are stored by every lane.
    const int c_lo = valid ? clo : 1, c_hi = valid ? leaf : 0;
    const bool g_st = valid && gstart;
    const unsigned w = threadIdx.x >> 6;
    for (int l = 0; l <= KEY_LEVELS; l++) {
        const unsigned long long b = __ballot(c_lo <= l && l <= c_hi);
        s_cnt[w][l] = (uint32_t)__popcll(b);
    }
    {
        const unsigned long long b = __ballot(g_st);
        s_cnt[w][NCOUNTERS - 1] = (uint32_t)__popcll(b);
    }
    __syncthreads();
    if (threadIdx.x < NCOUNTERS) {
        uint32_t s = 0;
        for (int v = 0; v < NW; v++) s += s_cnt[v][threadIdx.x];
        blkcnt[(size_t)threadIdx.x * nblk + blockIdx.x] = s;
    }
}

// One block per counter: exclusive scan over blocks, totals to ctot.
__global__ __launch_bounds__(1024) void k_build_scan(const uint32_t *__restrict__ blkcnt, unsigned nblk,
                                                     uint32_t *__restrict__ blkoff, uint32_t *__restrict__ ctot) {
    __shared__ unsigned s_wave[1024 / 64 + 1];
    const uint32_t *row = blkcnt + (size_t)blockIdx.x * nblk;
    uint32_t *out = blkoff + (size_t)blockIdx.x * nblk;
    const unsigned per = (nblk + 1023) / 1024;
    const unsigned b = threadIdx.x * per, e = min(b + per, nblk);
    unsigned sum = 0;
    for (unsigned j = b; j < e; j++) sum += row[j];
    unsigned total;
    unsigned run = block_excl_scan<1024>(sum, s_wave, &total);
    for (unsigned j = b; j < e; j++) {
        out[j] = run;
        run += row[j];
    }
    if (threadIdx.x == 0) ctot[blockIdx.x] = total;
}

// Cell ends searched at the end of a block.  A cell whose end lies beyond its
// first particle's wave contains that wave's last particle, so a wave defers at
// most one cell per level: 16 waves x 21 levels fit (the inline search below
// is only a guard).
constexpr unsigned BUILD_PENDING = 512;
static_assert(BUILD_PENDING >= (BUILD_THREADS / 64) * (KEY_LEVELS + 1), "one deferred cell per wave and level");

// SCAN: up to 64 blocks, whose counts every block adds up itself (a wave per
// counter and a lane per block: no launch between, 4.6 us).
constexpr unsigned BUILD_SCAN_BLOCKS = 64;
template <bool SCAN, unsigned WAYS>
__global__ __launch_bounds__(BUILD_THREADS) void k_build_write(
    const uchar4 *__restrict__ lvinfo, const uint64_t *__restrict__ keys, unsigned n, unsigned nsys,
    const uint32_t *__restrict__ sys_off, int gcap, const uint32_t *__restrict__ blkcnt,
    uint32_t *__restrict__ blkoff, const uint32_t *__restrict__ ctot, unsigned nblk, Header *__restrict__ hdr, uint4 *__restrict__ topo,
    uint2 *__restrict__ groups, unsigned cap_cells) {
    constexpr int NW = BUILD_THREADS / 64;
    __shared__ uint32_t s_base[NCOUNTERS];   // first cell number of each level; 0 for groups
    __shared__ uint32_t s_blk[NCOUNTERS];    // this block's offset within each level
    __shared__ uint32_t s_wpre[NW][NCOUNTERS];
    // cells whose end lies beyond their wave: record (cell, first, child_first,
    // system | level word) and (system end, group + 1 or 0), searched at the end
    __shared__ uint4 s_prec[BUILD_PENDING];
    __shared__ uint2 s_pext[BUILD_PENDING];
    __shared__ unsigned s_np;
    __shared__ uint32_t s_tot[NCOUNTERS];    // totals of all blocks
    if (threadIdx.x == 0) s_np = 0;
    if (SCAN) {
        const unsigned ln = lane64();
        for (unsigned c = threadIdx.x >> 6; c < NCOUNTERS; c += NW) {
            const unsigned v = ln < nblk ? blkcnt[(size_t)c * nblk + ln] : 0u;
            const unsigned inc = wave_incl_scan(v);
            if (ln == blockIdx.x) {
                s_blk[c] = inc - v;
                blkoff[(size_t)c * nblk + ln] = inc - v;
            }
            if (ln == 63u) s_tot[c] = inc;
        }
    } else if (threadIdx.x < NCOUNTERS) {
        s_blk[threadIdx.x] = blkoff[(size_t)threadIdx.x * nblk + blockIdx.x];
        s_tot[threadIdx.x] = ctot[threadIdx.x];
    }
    __syncthreads();
    if (threadIdx.x == 0) {
        uint32_t run = 0;
        for (int l = 0; l <= KEY_LEVELS; l++) {
            s_base[l] = run;
            run += s_tot[l];
        }
        s_base[NCOUNTERS - 1] = 0;
        if (blockIdx.x == 0) {
            for (int l = 0; l <= KEY_LEVELS; l++) hdr->lvl_begin[l] = s_base[l];
            hdr->lvl_begin[KEY_LEVELS + 1] = run;
            hdr->ncells = run;
            hdr->ngroups = s_tot[NCOUNTERS - 1];
            if (run > cap_cells) atomicOr(&hdr->flags, FLAG_CELLCAP);
        }
    }
    const unsigned i = blockIdx.x * BUILD_THREADS + threadIdx.x;
    const bool valid = i < n;
    // padding threads: first level 1 > leaf level 0 and no group start
    const uchar4 info = valid ? lvinfo[i] : make_uchar4(1, 0, 0, 0);
    const int clo = info.x, leaf = info.y, glev = info.z;
    const bool gstart = (info.w & 1) != 0;
    const unsigned w = threadIdx.x >> 6;
    for (int c = 0; c < NCOUNTERS; c++) {
        const bool pred = c < NCOUNTERS - 1 ? (clo <= c && c <= leaf) : gstart;
        const unsigned long long b = __ballot(pred);
        s_wpre[w][c] = (uint32_t)__popcll(b);
    }
    __syncthreads();
    if (threadIdx.x < NCOUNTERS) {
        uint32_t run = 0;
        for (int v = 0; v < NW; v++) {
            const uint32_t t = s_wpre[v][threadIdx.x];
            s_wpre[v][threadIdx.x] = run;
            run += t;
        }
    }
    __syncthreads();
    // the system of this particle and its end: runs never cross systems
    const unsigned sys = (nsys > 1 && valid) ? system_of(sys_off, nsys, i) : 0u;
    const unsigned send = nsys > 1 ? (valid ? sys_off[sys + 1] : n) : n;
    // cells, deepest level first so that each cell knows its first child's number.
    // A level-l cell starting at i ends at the first j > i with cl(j) < l (or
    // where the particles end): the wave finds it from a ballot of those
    // boundaries when it lies inside the wave, else by searching the keys.
    // Ends found by searching the keys are deferred to the end of the kernel,
    // where the block's threads take one search each: a particle that starts
    // large cells at many levels (the first particles of the big cells) would
    // otherwise run its searches one after the other, the kernel's longest path.
    const int ci = clo - 1;
    const unsigned ln = lane64();
    unsigned next = 0, gend = 0, gpend = 0;
    for (int l = KEY_LEVELS; l >= 0; l--) {
        const bool pred = clo <= l && l <= leaf;
        const unsigned long long b = __ballot(pred);
        if (b == 0) continue;
        const unsigned long long bnd = __ballot(!valid || ci < l);
        if (pred) {
            const unsigned idx = s_base[l] + s_blk[l] + s_wpre[w][l] + rank_below(b);
            const unsigned long long after = ln < 63 ? bnd >> (ln + 1) : 0ull;
            const unsigned cf = l < leaf ? next : 0u;
            const unsigned word = (sys << 16) | ((unsigned)l << 8);
            const unsigned k = after ? BUILD_PENDING : atomicAdd(&s_np, 1u);
            if (k < BUILD_PENDING) {
                s_prec[k] = make_uint4(idx, i, cf, word);
                s_pext[k] = make_uint2(send, 0u);
                if (l == glev) gpend = k + 1;
            } else {  // end inside the wave, or no room left to defer
                const unsigned end = after ? i + (unsigned)__ffsll((long long)after) : run_end<WAYS>(keys, send, i, l);
                if (idx < cap_cells) topo[idx] = make_uint4(i, end - i, cf, word);
                if (l == glev) gend = end;
            }
            next = idx;
        }
    }
    {
        const unsigned long long b = __ballot(gstart);
        if (gstart) {
            const unsigned g = s_blk[NCOUNTERS - 1] + s_wpre[w][NCOUNTERS - 1] + rank_below(b);
            const unsigned gword = (sys << 16) | ((unsigned)glev << 8);
            if (info.w & 2) {
                groups[g] = make_uint2(i, gword | min((unsigned)gcap, run_end<WAYS>(keys, send, i, KEY_LEVELS) - i));
            } else if (gend == 0 && gpend) {
                s_pext[gpend - 1].y = g + 1;  // written with its cell's end below
            } else {
                groups[g] = make_uint2(i, gword | ((gend ? gend : run_end<WAYS>(keys, send, i, glev)) - i));
            }
        }
    }
    __syncthreads();
    const unsigned np = min(s_np, BUILD_PENDING);
    for (unsigned k = threadIdx.x; k < np; k += BUILD_THREADS) {
        const uint4 r = s_prec[k];
        const uint2 e = s_pext[k];
        const unsigned end = run_end<WAYS>(keys, e.x, r.y, (int)((r.w >> 8) & 255u));
        if (r.x < cap_cells) topo[r.x] = make_uint4(r.y, end - r.y, r.z, r.w);
        if (e.y) groups[e.y - 1] = make_uint2(r.y, r.w | (end - r.y));
    }
}

// Children of an internal cell are the consecutive next-level cells that start
// inside it.  The kernel also counts the groups for the order of the walk.
__global__ __launch_bounds__(256) void k_build_nchild(const Header *__restrict__ hdr, const uint2 *__restrict__ groups,
                                                      uint4 *__restrict__ topo, unsigned cap_cells,
                                                      uint32_t *__restrict__ ghist) {
    if (hdr->flags & FLAG_CELLCAP) return;  // cell numbers beyond the capacity were never written
    if (ghist) gord_count(groups, nullptr, hdr->ngroups, ghist);
    const unsigned nc = min(hdr->ncells, cap_cells);
    for (unsigned c = blockIdx.x * 256u + threadIdx.x; c < nc; c += gridDim.x * 256u) {
        const uint4 t = topo[c];
        if (t.z == 0) continue;
        const unsigned l = (t.w >> 8) & 255u;
        const unsigned lend = min(hdr->lvl_begin[l + 2], nc);
        const unsigned end = t.x + t.y;
        unsigned nch = 0;
        for (unsigned k = t.z; k < lend && nch < 8; k++) {
            if (topo[k].x < end) nch++;
            else break;
        }
        reinterpret_cast<unsigned *>(topo)[4 * (size_t)c + 3] = (t.w & 0xffff0000u) | (l << 8) | nch;
    }
}

hipError_t launch_build(const Buffers &b, unsigned n, unsigned nsys, int ncrit, int gcap, hipStream_t s) {
    const unsigned nblk = (n + BUILD_THREADS - 1) / BUILD_THREADS;
    const uint64_t *keys = b.keys[0];
    hipLaunchKernelGGL(k_build_count, dim3(nblk), dim3(BUILD_THREADS), 0, s, b.cl, keys, n, nsys, b.sys_off,
                       ncrit, gcap, b.lvinfo, b.blkcnt, nblk);
    auto write = nblk <= BUILD_SCAN_BLOCKS ? k_build_write<true, 8>
                 : n <= RUN_END_EIGHTHS    ? k_build_write<false, 8>
                                           : k_build_write<false, 4>;
    if (nblk > BUILD_SCAN_BLOCKS)
        hipLaunchKernelGGL(k_build_scan, dim3(NCOUNTERS), dim3(1024), 0, s, b.blkcnt, nblk, b.blkoff, b.ctot);
    hipLaunchKernelGGL(write, dim3(nblk), dim3(BUILD_THREADS), 0, s, b.lvinfo, keys, n, nsys, b.sys_off, gcap, b.blkcnt,
                       b.blkoff, b.ctot, nblk, b.hdr, b.topo, b.groups, b.cap_cells);
    const unsigned grid = min((b.cap_cells + 255u) / 256u, 4096u);
    hipLaunchKernelGGL(k_build_nchild, dim3(grid), dim3(256), 0, s, b.hdr, b.groups, b.topo, b.cap_cells,
                       walk_sorts_groups(n) ? b.ghist : nullptr);
    return hipGetLastError();
}

// --------------------------------------------------------------------------
// Multipole moments, float64, bottom-up:
//   leaf:     M = sum m, com = (sum fma(m, x, .)) / M, S_ab = sum fma(m d_a, d_b, .)
//   internal: M = sum M_c, com = (sum fma(M_c, com_c, .)) / M,
//             S_ab = sum (S_c,ab + (M_c e_a) e_b), e = com_c - com
//   Q = 3 S - tr(S) I, delta = |com - geometric centre|
//   box = float32 min/max of the cell's particles (children's boxes for an
//   internal cell); l' = max(l, 2 max_a max(centre_a - min_a, max_a - centre_a)):
//   the side of the smallest cube about the geometric centre that holds the
//   particles, never below the cell side.  A freshly built cell holds its
//   particles, so l' = l; after a refit (particles moved, tree kept) l' grows
//   with the particles that left their cells.
// The operation order is fixed and nothing is contracted except the explicit
// fma calls, so every run gives the same bits.
// --------------------------------------------------------------------------

// Eight lanes take an internal cell together.  Lane q of the octet sums second
// moment min(q, 5) of (xx, yy, zz, xy, xz, yz), centre-of-mass axis q mod 3 and
// box component min(q, 5); every lane sums the mass.  Each sum keeps its own
// order, so the bits are those of one thread per cell; that form held the 8
// children in 234 registers (two waves per SIMD) and ran the sums one after the
// other.  Stores are the same for every lane but for their address and value:
// no branch on the lane alone sits beside the shuffles (see the walk's queue
// loop).
constexpr unsigned OCT = 8;

struct CellBuffers {
    const SysCube *cube;
    const uint4 *topo;
    const uint64_t *keys;
    const float4 *spos;
    double *mp, *delta;
    float *cbox;
    double *lside;
    float4 *cmac, *ceval;
};

struct Octet {
    unsigned q;        // lane of the octet
    unsigned ax;       // centre-of-mass axis
    unsigned ma, mb;   // second moment's axes
    unsigned qb;       // second moment and box component
};

__device__ __forceinline__ Octet octet() {
    Octet o;
    o.q = threadIdx.x & (OCT - 1u);
    o.ax = o.q % 3u;
    o.qb = min(o.q, 5u);
    o.ma = o.qb < 3u ? o.qb : (o.qb == 5u ? 1u : 0u);
    o.mb = o.qb < 3u ? o.qb : (o.qb == 3u ? 1u : 2u);
    return o;
}

__device__ __forceinline__ double oct_shfl(double v, unsigned lane) { return __shfl(v, (int)lane, OCT); }
__device__ __forceinline__ float oct_shfl(float v, unsigned lane) { return __shfl(v, (int)lane, OCT); }

// Side of the cell of level lev that starts at particle `first` (system sys)
// and its geometric centre along axis ax (corner from the key prefix).
__device__ __forceinline__ double cell_geometry(const CellBuffers &a, unsigned first, unsigned lev, unsigned sys,
                                                unsigned ax, double *centre) {
#pragma clang fp contract(off)
    const SysCube *cb = a.cube + sys;
    const double l = ldexp(1.0, cb->k - (int)lev);
    const uint64_t pre = a.keys[first] >> (3 * (KEY_LEVELS - (int)lev));
    const double corner = (double)cb->lo[ax] + (double)compact3(pre >> (2u - ax)) * l;
    *centre = corner + 0.5 * l;
    return l;
}

// Quantities derived from the moments of cell c, one thread: |com - centre|,
// the opening size and the walk's float32 data.
__device__ __forceinline__ void store_derived(const CellBuffers &a, unsigned c, double l, const double centre[3],
                                              double M, const double com[3], const double S[6], const float bn[3],
                                              const float bx[3]) {
#pragma clang fp contract(off)
    const double tr = (S[0] + S[1]) + S[2];
    const double Q0 = 3.0 * S[0] - tr, Q1 = 3.0 * S[1] - tr, Q2 = 3.0 * S[2] - tr;
    const double dx = com[0] - centre[0], dy = com[1] - centre[1], dz = com[2] - centre[2];
    a.delta[c] = sqrt((dx * dx + dy * dy) + dz * dz);
    double reach = 0.0;
    for (int k = 0; k < 3; k++) {
        reach = fmax(reach, centre[k] - (double)bn[k]);
        reach = fmax(reach, (double)bx[k] - centre[k]);
    }
    a.lside[c] = fmax(l, 2.0 * reach);
    a.cmac[c] = make_float4((float)com[0], (float)com[1], (float)com[2], 0.0f);
    a.ceval[2 * (size_t)c] = make_float4((float)M, (float)Q0, (float)Q1, (float)Q2);
    a.ceval[2 * (size_t)c + 1] = make_float4((float)(3.0 * S[3]), (float)(3.0 * S[4]), (float)(3.0 * S[5]), 0.0f);
}

// Leaf c of `cnt` particles from sorted position `first`, one thread: the first
// `nl` of them are in LDS at sp, the others are read from the sorted array.
__device__ __forceinline__ void leaf_cell(const CellBuffers &a, unsigned c, unsigned first, unsigned cnt,
                                          unsigned lev, unsigned sys, const float4 *sp, unsigned nl) {
#pragma clang fp contract(off)
    double centre[3], l = 0.0;
    for (unsigned ax = 0; ax < 3; ax++) l = cell_geometry(a, first, lev, sys, ax, centre + ax);
    const float4 *gp = a.spos + first;
    double M = 0.0, cm[3] = {0.0, 0.0, 0.0}, com[3], S[6] = {0.0, 0.0, 0.0, 0.0, 0.0, 0.0};
    float bn[3] = {sp[0].x, sp[0].y, sp[0].z}, bx[3] = {bn[0], bn[1], bn[2]};
    auto first_pass = [&](const float4 p) {
        bn[0] = fminf(bn[0], p.x);
        bx[0] = fmaxf(bx[0], p.x);
        bn[1] = fminf(bn[1], p.y);
        bx[1] = fmaxf(bx[1], p.y);
        bn[2] = fminf(bn[2], p.z);
        bx[2] = fmaxf(bx[2], p.z);
        const double m = (double)p.w;
        M = M + m;
        cm[0] = fma(m, (double)p.x, cm[0]);
        cm[1] = fma(m, (double)p.y, cm[1]);
        cm[2] = fma(m, (double)p.z, cm[2]);
    };
    auto second_pass = [&](const float4 p) {
#pragma clang fp contract(off)
        const double m = (double)p.w;
        const double dx = (double)p.x - com[0], dy = (double)p.y - com[1], dz = (double)p.z - com[2];
        S[0] = fma(m * dx, dx, S[0]);
        S[1] = fma(m * dy, dy, S[1]);
        S[2] = fma(m * dz, dz, S[2]);
        S[3] = fma(m * dx, dy, S[3]);
        S[4] = fma(m * dx, dz, S[4]);
        S[5] = fma(m * dy, dz, S[5]);
    };
#pragma unroll 4
    for (unsigned j = 0; j < nl; j++) first_pass(sp[j]);
#pragma unroll 4
    for (unsigned j = nl; j < cnt; j++) first_pass(gp[j]);
    for (int k = 0; k < 3; k++) com[k] = M > 0.0 ? cm[k] / M : centre[k];
#pragma unroll 4
    for (unsigned j = 0; j < nl; j++) second_pass(sp[j]);
#pragma unroll 4
    for (unsigned j = nl; j < cnt; j++) second_pass(gp[j]);
    double *o = a.mp + 10 * (size_t)c;
    o[0] = M;
    o[1] = com[0];
    o[2] = com[1];
    o[3] = com[2];
    for (int k = 0; k < 6; k++) o[4 + k] = S[k];
    for (int k = 0; k < 3; k++) {
        a.cbox[6 * (size_t)c + k] = bn[k];
        a.cbox[6 * (size_t)c + 3 + k] = bx[k];
    }
    store_derived(a, c, l, centre, M, com, S, bn, bx);
}

// An internal cell: (c, first child, system << 16 | level << 8 | children, first particle).
__device__ __forceinline__ uint4 cell_entry(unsigned c, const uint4 &t) { return make_uint4(c, t.z, t.w, t.x); }

// Internal cell of entry e, its children (NJ at most) done: the children's values
// are loaded together, then combined in child order.
template <unsigned NJ>
__device__ __forceinline__ void internal_cell(const CellBuffers &a, const Octet &o, const uint4 &e) {
#pragma clang fp contract(off)
    const unsigned nch = e.z & 255u;
    double Mc[NJ], xa[NJ], xb[NJ], Sc[NJ];
    float bc[NJ];
#pragma unroll
    for (unsigned j = 0; j < NJ; j++) {
        const unsigned k = e.y + min(j, nch - 1u);  // the last child again: its values are not used
        const double *m = a.mp + 10 * (size_t)k;
        Mc[j] = m[0];
        xa[j] = m[1 + o.ma];
        xb[j] = m[1 + o.mb];
        Sc[j] = m[4 + o.qb];
        bc[j] = a.cbox[6 * (size_t)k + o.qb];
    }
    // Lanes 0..2 hold their centre-of-mass axis in xa (ma = ax there); the other
    // lanes' own axes differ, so their sums are not used.
    double M = 0.0, cm = 0.0, S = 0.0;
    float box = bc[0];
#pragma unroll
    for (unsigned j = 0; j < NJ; j++) {
        const bool in = j < nch;
        const double M1 = M + Mc[j], c1 = fma(Mc[j], xa[j], cm);
        M = in ? M1 : M;
        cm = in ? c1 : cm;
        box = o.q < 3u ? fminf(box, bc[j]) : fmaxf(box, bc[j]);
    }
    double own = cm / M;
    if (__ballot(!(M > 0.0))) {  // massless cells take their centre
        double centre;
        cell_geometry(a, e.w, (e.z >> 8) & 255u, e.z >> 16, o.ax, &centre);
        own = M > 0.0 ? own : centre;
    }
    const double com = oct_shfl(own, o.ax);
    const double ca = oct_shfl(own, o.ma), cb = oct_shfl(own, o.mb);
#pragma unroll
    for (unsigned j = 0; j < NJ; j++) {
        const double ea = xa[j] - ca, eb = xb[j] - cb;
        const double S1 = S + (Sc[j] + (Mc[j] * ea) * eb);
        S = j < nch ? S1 : S;
    }
    double *m = a.mp + 10 * (size_t)e.x;
    m[o.q < 6u ? 4u + o.q : 0u] = o.q < 6u ? S : M;
    m[1 + o.ax] = com;
    a.cbox[6 * (size_t)e.x + o.qb] = box;
}

// A cell with one child, one thread: the same sums.  Above points that coincide
// there are chains of up to 19 of these.
__device__ __forceinline__ void chain_cell(const CellBuffers &a, const uint4 &e) {
#pragma clang fp contract(off)
    const double *c = a.mp + 10 * (size_t)e.y;
    const float *cb = a.cbox + 6 * (size_t)e.y;
    double v[10], com[3];
    float box[6];
    for (int k = 0; k < 10; k++) v[k] = c[k];
    for (int k = 0; k < 6; k++) box[k] = cb[k];
    const double M = 0.0 + v[0];
    for (int k = 0; k < 3; k++) com[k] = fma(v[0], v[1 + k], 0.0) / M;
    if (!(M > 0.0))
        for (unsigned ax = 0; ax < 3; ax++) cell_geometry(a, e.w, (e.z >> 8) & 255u, e.z >> 16, ax, com + ax);
    const double d[3] = {v[1] - com[0], v[2] - com[1], v[3] - com[2]};
    double *o = a.mp + 10 * (size_t)e.x;
    o[0] = M;
    for (int k = 0; k < 3; k++) o[1 + k] = com[k];
    o[4] = 0.0 + (v[4] + (v[0] * d[0]) * d[0]);
    o[5] = 0.0 + (v[5] + (v[0] * d[1]) * d[1]);
    o[6] = 0.0 + (v[6] + (v[0] * d[2]) * d[2]);
    o[7] = 0.0 + (v[7] + (v[0] * d[0]) * d[1]);
    o[8] = 0.0 + (v[8] + (v[0] * d[0]) * d[2]);
    o[9] = 0.0 + (v[9] + (v[0] * d[1]) * d[2]);
    for (int k = 0; k < 6; k++) a.cbox[6 * (size_t)e.x + k] = box[k];
}

// The derived quantities of the internal cell of entry e, its moments done: one thread.
__device__ __forceinline__ void derive_cell(const CellBuffers &a, const uint4 &e) {
    double centre[3], l = 0.0, com[3], S[6];
    float bn[3], bx[3];
    const double *m = a.mp + 10 * (size_t)e.x;
    const float *cb = a.cbox + 6 * (size_t)e.x;
    const double M = m[0];
    for (int k = 0; k < 3; k++) com[k] = m[1 + k];
    for (int k = 0; k < 6; k++) S[k] = m[4 + k];
    for (int k = 0; k < 3; k++) {
        bn[k] = cb[k];
        bx[k] = cb[3 + k];
    }
    for (unsigned ax = 0; ax < 3; ax++) l = cell_geometry(a, e.w, (e.z >> 8) & 255u, e.z >> 16, ax, centre + ax);
    store_derived(a, e.x, l, centre, M, com, S, bn, bx);
}

// All cells in a few launches.  The particles are cut into chunks (multipole_chunk),
// whole build blocks; the cells of one level that start in a chunk are
// consecutive (the build's block counts give their range), and all but the last
// of them end in it.
//   k_multipole_chunk: one workgroup per chunk, the chunk's particles in LDS:
//     every leaf that starts in the chunk, then the internal cells that end in
//     it, level by level from the deepest with workgroup barriers between
//     (their children lie in the chunk too).  An internal cell that does not
//     end in its chunk, at most one per level, goes on the list of the chunk.
//   k_multipole_merge: one workgroup per MP_FAN chunks takes the listed cells
//     that end within its range in the same way and lists the others; it is
//     launched until one range covers everything.
// What bounds it: the chain of levels, more than 1 us each (float64 sums and a
// division, the barrier), so the quantities that no parent needs are derived
// after the last level, and a cell's centre, which the moments need only of
// massless cells, too.  A leaf pass and one launch per level (21 launches) took,
// with the launching call, 60-80 / 67-84 / 70-85 / 111 / 189 us at n = 1000 / 20000 /
// 100003 / 2^20 / 2^22 (Plummer sphere, ncrit 16); this takes 16 / 31 / 39 / 66 / 139
// (one workgroup for all listed cells instead of MP_FAN-way merges: 567 us at 2^22).
// A chunk's moments kept in LDS for the parents change nothing up to 2^19 particles
// and take 85 / 217 us at 2^20 / 2^22: one workgroup per compute unit.
// Deep trees are bound by the number of cells: 24 particles at each of n / 24 points
// are a chain of 16 cells with one child each per point.  With eight lanes for each
// of those, and 8 rounds of loads, 152 / 231 / 664 us at 100003 / 2^20 / 2^22; with one
// thread for each (chain_cell) 69 / 120 / 321 (one launch per level: 80 / 134 / 343).
constexpr unsigned MP_THREADS = 256;
constexpr unsigned MP_OCTS = MP_THREADS / OCT;
constexpr unsigned MP_MERGE_THREADS = 512;
// internal cells of a chunk listed in LDS as they are met (more: some levels at a
// time): with chunks of 2048, room for four workgroups per compute unit
constexpr unsigned MP_CELLS = 512;
constexpr unsigned MP_NONE = 0xffffffffu;

template <unsigned CHUNK>
__global__ __launch_bounds__(MP_THREADS, 4) void k_multipole_chunk(const Header *__restrict__ hdr, CellBuffers a,
                                                                   const uint32_t *__restrict__ blkoff, unsigned nblk,
                                                                   unsigned n, unsigned nchunks,
                                                                   uint32_t *__restrict__ out) {
    static_assert(CHUNK % BUILD_THREADS == 0, "chunks are whole build blocks");
    static_assert(MP_CELLS <= CHUNK, "the list by level takes the particles' place");
    static_assert(CHUNK <= 2048 && KEY_LEVELS < 32 && MAX_SYSTEMS <= 256, "11 + 8 + 5 + 4 bits of a packed cell");
    __shared__ float4 s_p[CHUNK];                       // the particles, then the internal cells by level
    // internal cells as met: number, first child, and first particle << 17 | system << 9 | level << 4 | children
    __shared__ uint32_t s_raw[3][MP_CELLS];
    __shared__ unsigned short s_rank[MP_CELLS];         // their ranks in their levels
    __shared__ unsigned s_lo[KEY_LEVELS + 1];           // first cell of a level that starts here
    __shared__ unsigned s_pre[KEY_LEVELS + 2];          // prefix sums of the numbers of these
    __shared__ unsigned s_cnt[KEY_LEVELS + 1];          // internal cells of a level
    __shared__ unsigned s_at[KEY_LEVELS + 1], s_end[KEY_LEVELS + 1];  // their places in the list by level
    __shared__ unsigned s_nint;
    uint4 *s_int = reinterpret_cast<uint4 *>(s_p);  // once the leaves are done
    constexpr unsigned PB = CHUNK / BUILD_THREADS;
    if (hdr->flags & FLAG_CELLCAP) return;
    const unsigned t = threadIdx.x;
    const unsigned b = blockIdx.x * CHUNK, e = min(b + CHUNK, n);
    if (t < 64u) {  // the first wave: ranges of the levels and their prefix sums
        const bool lev = t <= (unsigned)KEY_LEVELS;
        const unsigned l = lev ? t : 0u;
        const unsigned b0 = blockIdx.x * PB, b1 = b0 + PB;
        const unsigned lb = hdr->lvl_begin[l], le = hdr->lvl_begin[l + 1];
        const unsigned lo = lb + blkoff[(size_t)l * nblk + b0];
        const unsigned hi = b1 < nblk ? lb + blkoff[(size_t)l * nblk + b1] : le;
        const unsigned cnt = lev ? hi - lo : 0u;
        const unsigned inc = wave_incl_scan(cnt);
        if (lev) {
            s_lo[l] = lo;
            s_pre[l] = inc - cnt;
            s_cnt[l] = 0;
            if (out && l < (unsigned)KEY_LEVELS) out[l * nchunks + blockIdx.x] = MP_NONE;
        }
        if (t == 63u) s_pre[KEY_LEVELS + 1] = inc;
        if (t == 63u) s_nint = 0;
    }
    for (unsigned i = b + t; i < e; i += MP_THREADS) s_p[i - b] = a.spos[i];
    __syncthreads();
    // the chunk's cells: leaves are done at once, internal cells that end here listed
    const unsigned total = s_pre[KEY_LEVELS + 1];
    for (unsigned i = t; i < total; i += MP_THREADS) {
        unsigned l = 0, h = KEY_LEVELS + 1;  // s_pre[l] <= i < s_pre[h]
        while (h - l > 1) {
            const unsigned mid = (l + h) >> 1;
            if (s_pre[mid] <= i) l = mid; else h = mid;
        }
        const unsigned c = s_lo[l] + (i - s_pre[l]);
        const uint4 tc = a.topo[c];
        if ((tc.w & 255u) == 0) {
            leaf_cell(a, c, tc.x, tc.y, l, tc.w >> 16, s_p + (tc.x - b), min(tc.y, e - tc.x));
        } else if (tc.x + tc.y > b + CHUNK) {
            out[l * nchunks + blockIdx.x] = c;  // leaves the chunk: there is more than one, so a list
        } else {
            const unsigned r = atomicAdd(&s_cnt[l], 1u), k = atomicAdd(&s_nint, 1u);
            if (k < MP_CELLS) {
                s_raw[0][k] = c;
                s_raw[1][k] = tc.z;
                s_raw[2][k] = (tc.x - b) << 17 | (tc.w >> 16) << 9 | l << 4 | (tc.w & 15u);
                s_rank[k] = (unsigned short)r;
            }
        }
    }
    __syncthreads();
    const unsigned nint = s_nint;
    const bool listed = nint <= MP_CELLS;
    const Octet o = octet();
    const unsigned oct = t / OCT;
    if (listed) {
        if (t < 64u) {
            const unsigned cnt = t <= (unsigned)KEY_LEVELS ? s_cnt[t] : 0u;
            const unsigned inc = wave_incl_scan(cnt);
            if (t <= (unsigned)KEY_LEVELS) s_at[t] = inc - cnt;
        }
        __syncthreads();
        for (unsigned k = t; k < nint; k += MP_THREADS) {
            const unsigned v = s_raw[2][k], l = (v >> 4) & 31u;
            s_int[s_at[l] + s_rank[k]] =
                make_uint4(s_raw[0][k], s_raw[1][k], ((v >> 9) & 255u) << 16 | l << 8 | (v & 15u), b + (v >> 17));
        }
        __syncthreads();
        for (int l = KEY_LEVELS - 1; l >= 0; l--) {
            const unsigned cnt = s_cnt[l];
            if (cnt == 0) continue;  // the same for the whole workgroup
            const unsigned at = s_at[l];
            for (unsigned i = oct; i < cnt; i += MP_OCTS) internal_cell<8>(a, o, s_int[at + i]);
            __syncthreads();
        }
        // the derived quantities at the end, off the chain of the levels
        for (unsigned k = t; k < nint; k += MP_THREADS) derive_cell(a, s_int[k]);
        return;
    }
    // More cells than that list holds: gathered again from their ranges, as many
    // levels at a time as fit the particles' place (one at least: an internal cell has
    // two particles or more), those with one child first in each level.  Where points
    // coincide most cells are such, and along a line most have two children at most:
    // the octets of a wave take the short form where all of theirs have.
    for (int l1 = KEY_LEVELS; l1 > 0;) {
        int l0 = l1;
        unsigned sum = 0;
        while (l0 > 0 && sum + s_cnt[l0 - 1] <= CHUNK) sum += s_cnt[--l0];  // the same for the whole workgroup
        if (t == 0) {
            unsigned at = 0;
            for (int l = l1 - 1; l >= l0; l--) {
                s_at[l] = at;
                at += s_cnt[l];
                s_end[l] = at;
            }
        }
        __syncthreads();
        for (unsigned i = s_pre[l0] + t; i < s_pre[l1]; i += MP_THREADS) {
            unsigned l = l0, h = l1;  // s_pre[l] <= i < s_pre[h]
            while (h - l > 1) {
                const unsigned mid = (l + h) >> 1;
                if (s_pre[mid] <= i) l = mid; else h = mid;
            }
            const unsigned c = s_lo[l] + (i - s_pre[l]);
            const uint4 tc = a.topo[c];
            const unsigned nch = tc.w & 255u;
            if (nch != 0 && tc.x + tc.y <= b + CHUNK)
                s_int[nch == 1 ? atomicAdd(&s_at[l], 1u) : atomicSub(&s_end[l], 1u) - 1u] = cell_entry(c, tc);
        }
        __syncthreads();
        unsigned at = 0;
        for (int l = l1 - 1; l >= l0; l--) {
            const unsigned one = s_at[l], end = at + s_cnt[l];  // cells with one child end at `one` now
            if (at == end) continue;
            for (unsigned i = at + t; i < one; i += MP_THREADS) chain_cell(a, s_int[i]);
            for (unsigned i = one + oct; i < end; i += MP_OCTS) {
                const uint4 e = s_int[i];
                if (__ballot((e.z & 255u) > 2u)) internal_cell<8>(a, o, e);
                else internal_cell<2>(a, o, e);
            }
            __syncthreads();
            at = end;
        }
        for (unsigned k = t; k < sum; k += MP_THREADS) derive_cell(a, s_int[k]);
        __syncthreads();  // the list is free again
        l1 = l0;
    }
}

// in[level][nin]: listed cells of the ranges below, MP_FAN of them per
// workgroup; `span`: particles of this workgroup's range; out as above
__global__ __launch_bounds__(MP_MERGE_THREADS) void k_multipole_merge(const Header *__restrict__ hdr, CellBuffers a,
                                                                const uint32_t *__restrict__ in, unsigned nin,
                                                                unsigned long long span, unsigned nout,
                                                                uint32_t *__restrict__ out) {
    __shared__ uint4 s_int[KEY_LEVELS][MP_FAN];
    __shared__ unsigned s_cnt[KEY_LEVELS];  // cells of the level; in the high half those with more than one child
    if (hdr->flags & FLAG_CELLCAP) return;
    const unsigned t = threadIdx.x;
    const unsigned r0 = blockIdx.x * MP_FAN;
    const unsigned long long end = (blockIdx.x + 1ull) * span;
    if (t < (unsigned)KEY_LEVELS) {
        s_cnt[t] = 0;
        if (out) out[t * nout + blockIdx.x] = MP_NONE;
    }
    __syncthreads();
    for (unsigned i = t; i < (unsigned)KEY_LEVELS * MP_FAN; i += MP_MERGE_THREADS) {
        const unsigned l = i / MP_FAN, k = r0 + i % MP_FAN;
        const unsigned c = k < nin ? in[l * nin + k] : MP_NONE;
        if (c != MP_NONE) {
            const uint4 tc = a.topo[c];
            if (tc.x + (unsigned long long)tc.y > end) out[l * nout + blockIdx.x] = c;
            else s_int[l][atomicAdd(&s_cnt[l], (tc.w & 255u) > 1u ? 0x10001u : 1u) & 0xffffu] = cell_entry(c, tc);
        }
    }
    __syncthreads();
    const Octet o = octet();
    const unsigned oct = t / OCT;
    for (int l = KEY_LEVELS - 1; l >= 0; l--) {
        const unsigned cnt = s_cnt[l] & 0xffffu, wide = s_cnt[l] >> 16;
        if (cnt == 0) continue;  // the same for the whole workgroup
        if (wide) {
            for (unsigned i = oct; i < cnt; i += MP_MERGE_THREADS / OCT) internal_cell<8>(a, o, s_int[l][i]);
        } else {
            for (unsigned i = t; i < cnt; i += MP_MERGE_THREADS) chain_cell(a, s_int[l][i]);
        }
        __syncthreads();
    }
    for (unsigned i = t; i < (unsigned)KEY_LEVELS * MP_FAN; i += MP_MERGE_THREADS)
        if (i % MP_FAN < (s_cnt[i / MP_FAN] & 0xffffu)) derive_cell(a, s_int[i / MP_FAN][i % MP_FAN]);
}

hipError_t launch_multipoles(const Buffers &b, unsigned n, unsigned nsys, hipStream_t s) {
    const CellBuffers a = {b.cube, b.topo, b.keys[0], b.spos, b.mp, b.delta, b.cbox, b.lside,
                           b.cmac, b.ceval};
    const unsigned nblk = (n + BUILD_THREADS - 1) / BUILD_THREADS;
    const unsigned chunk = multipole_chunk(n, b.ncrit);
    unsigned nr = (n + chunk - 1) / chunk;
    uint32_t *list = b.mlist;
    unsigned long long span = chunk;
    auto k = chunk == 512 ? k_multipole_chunk<512> : chunk == 1024 ? k_multipole_chunk<1024> : k_multipole_chunk<2048>;
    hipLaunchKernelGGL(k, dim3(nr), dim3(MP_THREADS), 0, s, b.hdr, a, b.blkoff, nblk, n, nr, nr > 1 ? list : nullptr);
    while (nr > 1) {
        const unsigned nout = (nr + MP_FAN - 1) / MP_FAN;
        uint32_t *next = list + (size_t)KEY_LEVELS * nr;
        span *= MP_FAN;
        hipLaunchKernelGGL(k_multipole_merge, dim3(nout), dim3(MP_MERGE_THREADS), 0, s, b.hdr, a, list, nr, span, nout,
                           nout > 1 ? next : nullptr);
        list = next;
        nr = nout;
    }
    return hipGetLastError();
}

// r_open = l'/theta + delta in float64 (a correctly rounded division; for a
// fresh cell l' = 2^(k - level) and the quotient is the exact scaling of
// fl(1/theta)), squared in float64, rounded once to float32.
__global__ __launch_bounds__(256) void k_mac_prep(Header *__restrict__ hdr, const double *__restrict__ lside,
                                                  const double *__restrict__ delta, double theta,
                                                  float4 *__restrict__ cmac, uint4 *__restrict__ arec,
                                                  unsigned cap_cells) {
#pragma clang fp contract(off)
    if (hdr->flags & FLAG_CELLCAP) return;
    const unsigned nc = min(hdr->ncells, cap_cells);
    if (blockIdx.x == 0 && threadIdx.x < WALK_QUEUES) {  // queues of the walk that follows
        hdr->walk_head[QUEUE_STRIDE * threadIdx.x] = 0;
        hdr->prefix_head[QUEUE_STRIDE * threadIdx.x] = 0;
    }
    if (blockIdx.x == 0 && threadIdx.x == 0) {
        hdr->pool_head = 0;
        hdr->anchor_count = 0;
        hdr->anchor_fail = 0;
    }
    for (unsigned c = blockIdx.x * 256u + threadIdx.x; c < nc; c += gridDim.x * 256u) {
        const double ro = lside[c] / theta + delta[c];
        cmac[c].w = (float)(ro * ro);
        if (arec) arec[c] = make_uint4(0u, 0u, 0u, 0u);  // no anchor yet
    }
}

hipError_t launch_mac_prep(const Buffers &b, unsigned nsys, double theta, hipStream_t s) {
    (void)nsys;
    const unsigned grid = min((b.cap_cells + 255u) / 256u, 4096u);
    hipLaunchKernelGGL(k_mac_prep, dim3(grid), dim3(256), 0, s, b.hdr, b.lside, b.delta, theta, b.cmac,
                       b.arec, b.cap_cells);
    return hipGetLastError();
}

// --------------------------------------------------------------------------
// Energies: W = 1/2 sum m phi, T = 1/2 sum m v^2 in float64; every block sums
// a fixed strided set, then one block sums the partials in a fixed order.
// --------------------------------------------------------------------------

__global__ __launch_bounds__(ENERGY_THREADS) void k_energy_partial(const float *__restrict__ mass,
                                                                   const float *__restrict__ pot,
                                                                   const float *__restrict__ vel,
                                                                   unsigned n, double *__restrict__ part) {
    double w = 0.0, t = 0.0;
    for (unsigned i = blockIdx.x * ENERGY_THREADS + threadIdx.x; i < n; i += ENERGY_BLOCKS * ENERGY_THREADS) {
        const double m = (double)mass[i];
        w += m * (double)pot[i];
        if (vel) {
            const double vx = vel[3 * (size_t)i], vy = vel[3 * (size_t)i + 1], vz = vel[3 * (size_t)i + 2];
            t += m * (vx * vx + vy * vy + vz * vz);
        }
    }
    __shared__ double sw[ENERGY_THREADS], st[ENERGY_THREADS];
    sw[threadIdx.x] = w;
    st[threadIdx.x] = t;
    __syncthreads();
    for (int o = ENERGY_THREADS / 2; o > 0; o >>= 1) {
        if (threadIdx.x < (unsigned)o) {
            sw[threadIdx.x] += sw[threadIdx.x + o];
            st[threadIdx.x] += st[threadIdx.x + o];
        }
        __syncthreads();
    }
    if (threadIdx.x == 0) {
        part[2 * blockIdx.x] = sw[0];
        part[2 * blockIdx.x + 1] = st[0];
    }
}

__global__ __launch_bounds__(ENERGY_THREADS) void k_energy_final(const double *__restrict__ part,
                                                                 double *__restrict__ out) {
    __shared__ double sw[ENERGY_THREADS], st[ENERGY_THREADS];
    double w = 0.0, t = 0.0;
    for (int b = threadIdx.x; b < ENERGY_BLOCKS; b += ENERGY_THREADS) {
        w += part[2 * b];
        t += part[2 * b + 1];
    }
    sw[threadIdx.x] = w;
    st[threadIdx.x] = t;
    __syncthreads();
    for (int o = ENERGY_THREADS / 2; o > 0; o >>= 1) {
        if (threadIdx.x < (unsigned)o) {
            sw[threadIdx.x] += sw[threadIdx.x + o];
            st[threadIdx.x] += st[threadIdx.x + o];
        }
        __syncthreads();
    }
    if (threadIdx.x == 0) {
        out[0] = 0.5 * st[0];
        out[1] = 0.5 * sw[0];
    }
}

hipError_t launch_energy(const Buffers &b, const float *mass, const float *pot, const float *vel,
                         unsigned n, double *d_out2, hipStream_t s) {
    hipLaunchKernelGGL(k_energy_partial, dim3(ENERGY_BLOCKS), dim3(ENERGY_THREADS), 0, s, mass, pot, vel, n,
                       b.epart);
    hipLaunchKernelGGL(k_energy_final, dim3(1), dim3(ENERGY_THREADS), 0, s, b.epart, d_out2);
    return hipGetLastError();
}

}  // namespace mibh
