// Group tree walk ("tree-traverse", the >90% part of a step in the paper's
// Results section) on gfx950.
//
// One wave64 per group (the vector-machine idea of Barnes 1990: one
// interaction list shared by a group of nearby particles; two to eight waves where
// groups are few, see walk_group_waves), persistent waves pulling groups from
// eight queues, one per XCD, each an atomic head on a cache line of its own over
// one eighth of the processing order: the groups in Morton order (the waves of an
// XCD then walk spatial neighbours, whose cells they share in that XCD's L2), in
// large trees with the end of each queue by group size, or a
// work-ordered permutation, heaviest groups first.  A wave whose queue is empty
// takes groups from the others.
//
// Traversal: lanes hold up to 64 candidate cells popped from a per-wave stack
// kept in LDS (circular, spilling its bottom to a per-wave global stack when
// full); each lane applies the opening test of Barnes (1994) for the group's
// bounding box (float32, fixed operation order); ballots + mbcnt compact
// accepted cells into the particle-cell list, opened leaves into the
// particle-particle list (expanded to particle indices) and opened internal
// cells' children onto the stack.  Lanes pop in stack order and push in lane
// order, so stack levels never decrease towards the top; then at most one
// step's pushes (<= 64*8) per level are on the stack at any time, which bounds
// it by 1 + 20*512 entries.  Both lists live in LDS and are evaluated in whole
// 64-entry tiles when they fill (the remainder stays), the last partial tile at
// the end of the group.
//
// Evaluation: groups average ~20 particles, so lanes run over the list
// entries (64 sources per tile) and a wave-uniform loop runs over the group's
// particles, 16 at a time; each lane keeps 16 x 4 partial sums, folded across
// lanes by a 63-shuffle transposed reduction (lane l receives the total of
// accumulator bitrev6(l)) when a full list is flushed, and once for both lists
// at the end of the group.  An active walk (block time
// steps) evaluates only the group's active particles, packed into the first
// lanes; its lists are still built from the whole group's box.  No
// floating-point atomics: results are bitwise reproducible run to run.
#include "mibh_device.h"

namespace mibh {

namespace {

__device__ __forceinline__ unsigned lane64() { return __lane_id(); }

__device__ __forceinline__ unsigned rank_below(unsigned long long mask) {
    return __builtin_amdgcn_mbcnt_hi((unsigned)(mask >> 32),
                                     __builtin_amdgcn_mbcnt_lo((unsigned)mask, 0u));
}

__device__ __forceinline__ unsigned uniform(unsigned v) { return __builtin_amdgcn_readfirstlane(v); }

// Orders this wave's own LDS and global accesses: its lanes then read what its
// other lanes wrote.  The hardware runs one wave's accesses in order, so this
// costs nothing beyond keeping the compiler from moving them, where a workgroup
// barrier waits for every outstanding access.
__device__ __forceinline__ void wave_sync() {
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    __builtin_amdgcn_wave_barrier();
}

__device__ __forceinline__ unsigned bitrev6(unsigned l) {
    return ((l & 1u) << 5) | ((l & 2u) << 3) | ((l & 4u) << 1) | ((l & 8u) >> 1) | ((l & 16u) >> 3) |
           ((l & 32u) >> 5);
}

// Exclusive prefix sum over the wave of small per-lane values (0 <= v < 2^BITS),
// from BITS ballots; *total gets the wave total.
template <int BITS = 4>
__device__ __forceinline__ unsigned small_excl_scan(unsigned v, unsigned *total) {
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

// Inclusive prefix sum over the wave, in lane order, of unsigned per-lane
// values whose sums do not overflow: Hillis-Steele steps inside each row of 16
// lanes (DPP row shifts 1, 2, 4, 8; a lane with no source lane adds 0), then the
// row totals carried across rows by the GFX9 row broadcasts (lane 15 into rows 1
// and 3, lane 31 into rows 2 and 3).  Six DPP steps (a move and an add each,
// where the compiler does not fuse them) against two ballots and a shift-add
// per bit for a ballot scan; the whole wave must be active.
__device__ __forceinline__ unsigned wave_incl_scan(unsigned v) {
    v += (unsigned)__builtin_amdgcn_update_dpp(0, (int)v, 0x111, 0xf, 0xf, false);  // row_shr:1
    v += (unsigned)__builtin_amdgcn_update_dpp(0, (int)v, 0x112, 0xf, 0xf, false);  // row_shr:2
    v += (unsigned)__builtin_amdgcn_update_dpp(0, (int)v, 0x114, 0xf, 0xf, false);  // row_shr:4
    v += (unsigned)__builtin_amdgcn_update_dpp(0, (int)v, 0x118, 0xf, 0xf, false);  // row_shr:8
    v += (unsigned)__builtin_amdgcn_update_dpp(0, (int)v, 0x142, 0xa, 0xf, false);  // row_bcast:15
    v += (unsigned)__builtin_amdgcn_update_dpp(0, (int)v, 0x143, 0xc, 0xf, false);  // row_bcast:31
    return v;
}

// Sums each of the NV per-lane values v[0..NV) (NV = 64 or 32) over the wave.
// With NV = 64 lane l gets the total of v[bitrev6(l)]; with NV = 32 lanes l and
// l ^ 1 both get the total of v[bitrev6(l) & 31].  Stage with offset o pairs
// v[2p], v[2p+1]: lanes whose bit o is clear keep the pair sum of v[2p], the
// others of v[2p+1].  The offsets 32 and 16 are the gfx950 half/row swaps
// (v_permlane32_swap exchanges the upper half of its first operand with the
// lower half of its second, so one swap and one add finish a pair); the others
// use shuffles, and for NV = 32 a last shuffle adds the two lanes of a pair.
template <int NV>
__device__ __forceinline__ float transpose_reduce(float (&v)[NV]) {
    static_assert(NV == 64 || NV == 32, "64 or 32 values");
    const unsigned ln = lane64();
#pragma unroll
    for (int p = 0; p < NV / 2; p++) {
        const auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(v[2 * p]), __float_as_uint(v[2 * p + 1]),
                                                        false, false);
        v[p] = __uint_as_float(r[0]) + __uint_as_float(r[1]);
    }
#pragma unroll
    for (int p = 0; p < NV / 4; p++) {
        const auto r = __builtin_amdgcn_permlane16_swap(__float_as_uint(v[2 * p]), __float_as_uint(v[2 * p + 1]),
                                                        false, false);
        v[p] = __uint_as_float(r[0]) + __uint_as_float(r[1]);
    }
#pragma unroll
    for (int s = 2; (NV >> s) >= 2; s++) {
        const int o = 32 >> s;
        const int len = NV >> s;
        const bool hi = (ln & (unsigned)o) != 0;
#pragma unroll
        for (int p = 0; p < len / 2; p++) {
            const float keep = hi ? v[2 * p + 1] : v[2 * p];
            const float send = hi ? v[2 * p] : v[2 * p + 1];
            v[p] = keep + __shfl_xor(send, o, 64);
        }
    }
    return NV == 64 ? v[0] : v[0] + __shfl_xor(v[0], 1, 64);
}

// The opening test, float32 with every operation rounded (no contraction):
// d_a = max(max(bmin_a - c_a, c_a - bmax_a), 0), d2 = (dx dx + dy dy) + dz dz,
// accept iff d2 > r_open^2.  The inputs are finite (the walk refuses others),
// so fmaxf (one v_max_f32) gives the maxima; where it may pick -0 instead of
// +0 the square is +0 all the same.
__device__ __forceinline__ bool mac_accept(float3 bmin, float3 bmax, float4 m) {
#pragma clang fp contract(off)
    const float dx = fmaxf(fmaxf(bmin.x - m.x, m.x - bmax.x), 0.0f);
    const float dy = fmaxf(fmaxf(bmin.y - m.y, m.y - bmax.y), 0.0f);
    const float dz = fmaxf(fmaxf(bmin.z - m.z, m.z - bmax.z), 0.0f);
    const float d2 = (dx * dx + dy * dy) + dz * dz;
    return d2 > m.w;
}

// The opening test's distance taken to the box's farthest point instead of its
// nearest: d_a = max(max(bmax_a - c_a, c_a - bmin_a), 0), same operation order.
// For any box B' inside [bmin, bmax] each rounded step of the nearest-point
// distance of B' is at most the same step here, so d2(B') <= far_d2: a cell with
// far_d2 <= r_open^2 is opened for every group inside the box.
__device__ __forceinline__ float far_d2(float3 bmin, float3 bmax, float4 m) {
#pragma clang fp contract(off)
    const float dx = fmaxf(fmaxf(bmax.x - m.x, m.x - bmin.x), 0.0f);
    const float dy = fmaxf(fmaxf(bmax.y - m.y, m.y - bmin.y), 0.0f);
    const float dz = fmaxf(fmaxf(bmax.z - m.z, m.z - bmin.z), 0.0f);
    return (dx * dx + dy * dy) + dz * dz;
}

template <bool KAHAN>
__device__ __forceinline__ void add(float &s, float &c, float x) {
    if (KAHAN) {
        const float y = x - c;
        const float t = s + y;
        c = (t - s) - y;
        s = t;
    } else {
        s += x;
    }
}

struct WalkArgs {
    Header *hdr;
    const uint4 *topo;
    const float4 *cmac;
    const float4 *ceval;
    const float4 *spos;
    const uint32_t *perm;
    const uint2 *groups;
    uint2 *gcounts;
    uint32_t *wstack;
    const uint32_t *order;   // queue order (NULL: Morton order)
    const uint32_t *qlen;    // number of queue entries to walk (NULL: all groups)
    const uint8_t *active;   // per input particle, nonzero = evaluate it (NULL: every particle)
    unsigned *head;          // heads of the group queues (one per XCD)
    float *acc, *pot;
    float eps2, G;
    unsigned pc_cap, pp_cap;
    unsigned dcell, dpart;   // padding cell and particle (massless, far)
    // shared-prefix walk
    const float *cbox;       // cells' particle boxes
    const uint32_t *anchor;  // anchor cell of each group
    const uint4 *arec;       // per anchor cell: pool offset, |F|, |S|, valid
    const uint32_t *pool;    // the anchors' lists
};

// Accumulation modes (the library's precision parameter):
//   0 plain float32;
//   1 compensated across flushes: within one evaluation of the lists each lane
//     sums its <= 16 tiles in plain float32 and the lanes are folded by a
//     six-level tree, and the per-particle totals of successive evaluations
//     (one per flush of a full list, one at the end of the group) are added
//     with Kahan compensation: the long sums of a particle are the ones across
//     evaluations, while those inside one are short and pairwise;
//   2 compensated per term: every term is added to its lane's sum with Kahan
//     compensation, and the evaluations' totals as in mode 1.
// Group particles per evaluation pass: 16 (64 sums per lane), or 8 per term
// compensated (32 sums and 32 compensations), so that every mode keeps 64
// accumulator registers per lane.
template <int PREC> constexpr int chunk_of() { return PREC == 2 ? 8 : 16; }
// Slot of a lane's reduced value for chunk c in the per-group result array
// (256 floats: 4 chunks x 64 values, or 8 chunks x 32 values).
template <int PREC> __device__ __forceinline__ unsigned res_slot(unsigned c, unsigned ln) {
    return chunk_of<PREC>() == 8 ? c * 32u + (ln >> 1) : c * 64u + ln;
}
// Evaluates the particle-cell entries `fl` (`nfl`, an anchor's shared cells in
// the pool, or none) and `pcl` (`npcl`, in LDS) and the particle-particle
// entries `ppl` (`nppl`), all whole 64-entry tiles (a list's last tile is padded
// with the massless far cell or particle), for the group particles [g0, g1) and
// adds the results into s_res (one value per lane per chunk): one reduction per
// chunk covers all the lists.  Whole tiles need no per-lane test or substitute
// in the tile loops.  A particle's sums depend on the lists alone, not on the
// chunk or the wave that holds it.
template <int PREC>
__device__ void evaluate(const WalkArgs &a, const uint32_t *fl, unsigned nfl, const uint32_t *pcl, unsigned npcl,
                         const uint32_t *ppl, unsigned nppl, unsigned g0, unsigned g1, float px, float py, float pz,
                         float *s_res, float *s_cmp) {
    constexpr int CHUNK = chunk_of<PREC>();
    constexpr int NV = 4 * CHUNK;
    constexpr bool TERM = PREC == 2;
    const unsigned ln = lane64();
    const float eps2 = a.eps2;
    for (unsigned c0 = g0; c0 < g1; c0 += CHUNK) {
        const unsigned cn = min((unsigned)CHUNK, g1 - c0);
        float xi[CHUNK], yi[CHUNK], zi[CHUNK];
#pragma unroll
        for (int ii = 0; ii < CHUNK; ii++) {
            const unsigned src = c0 + min((unsigned)ii, cn - 1);
            xi[ii] = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(px), src));
            yi[ii] = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(py), src));
            zi[ii] = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(pz), src));
        }
        float v[NV], cv[NV];
#pragma unroll
        for (int j = 0; j < NV; j++) { v[j] = 0.0f; cv[j] = 0.0f; }
        // particle-cell tiles: the shared list in the pool (fl), then the
        // group's own list in LDS (pcl), one loop over both
        const uint32_t *lst = fl;
        unsigned nl = nfl;
#pragma unroll 1
        for (int seg = 0; seg < 2; seg++, lst = pcl, nl = npcl)
        for (unsigned t0 = 0; t0 < nl; t0 += 64) {
            // The particle count of the chunk is taken as new in every tile, so
            // that its 16 comparisons are made in place (scalar compares) instead
            // of being kept as 16 lane masks across the loop: 32 scalar registers
            // more than the wave can hold, spilled to vector-register lanes and
            // read back in every tile.
            unsigned cn_t = cn;
            asm volatile("" : "+s"(cn_t));
            const unsigned e = lst[t0 + ln];
            const float4 m = a.cmac[e], q0 = a.ceval[2 * (size_t)e], q1 = a.ceval[2 * (size_t)e + 1];
#pragma unroll
            for (int ii = 0; ii < CHUNK; ii++) {
                if ((unsigned)ii < cn_t) {
                    // R = x - com; r2 = R.R + eps2
                    const float Rx = xi[ii] - m.x, Ry = yi[ii] - m.y, Rz = zi[ii] - m.z;
                    const float r2 = fmaf(Rz, Rz, fmaf(Ry, Ry, fmaf(Rx, Rx, eps2)));
                    const float rinv = __builtin_amdgcn_rsqf(r2);
                    const float rinv2 = rinv * rinv;
                    const float r3 = rinv * rinv2;
                    const float r5 = r3 * rinv2;
                    // Q R with Q = (xx, yy, zz | xy, xz, yz)
                    const float QRx = fmaf(q0.y, Rx, fmaf(q1.x, Ry, q1.y * Rz));
                    const float QRy = fmaf(q1.x, Rx, fmaf(q0.z, Ry, q1.z * Rz));
                    const float QRz = fmaf(q1.y, Rx, fmaf(q1.z, Ry, q0.w * Rz));
                    const float RQR = fmaf(Rx, QRx, fmaf(Ry, QRy, Rz * QRz));
                    const float Mr3 = q0.x * r3;
                    const float u = RQR * r5;
                    // a = -M R/r^3 + Q R/r^5 - (5/2)(RQR) R/r^7 ; phi = -(M/r + RQR/(2 r^5))
                    const float coef = fmaf(2.5f * u, rinv2, Mr3);
                    if (TERM) {
                        add<true>(v[4 * ii + 0], cv[4 * ii + 0], fmaf(QRx, r5, -coef * Rx));
                        add<true>(v[4 * ii + 1], cv[4 * ii + 1], fmaf(QRy, r5, -coef * Ry));
                        add<true>(v[4 * ii + 2], cv[4 * ii + 2], fmaf(QRz, r5, -coef * Rz));
                        add<true>(v[4 * ii + 3], cv[4 * ii + 3], -fmaf(0.5f, u, q0.x * rinv));
                    } else {  // the term goes into the sum as two fused multiply-adds
                        v[4 * ii + 0] = fmaf(-coef, Rx, fmaf(QRx, r5, v[4 * ii + 0]));
                        v[4 * ii + 1] = fmaf(-coef, Ry, fmaf(QRy, r5, v[4 * ii + 1]));
                        v[4 * ii + 2] = fmaf(-coef, Rz, fmaf(QRz, r5, v[4 * ii + 2]));
                        v[4 * ii + 3] = fmaf(-q0.x, rinv, fmaf(-0.5f, u, v[4 * ii + 3]));
                    }
                }
            }
        }
        for (unsigned t0 = 0; t0 < nppl; t0 += 64) {
            unsigned cn_t = cn;  // in place in every tile, as above
            asm volatile("" : "+s"(cn_t));
            const float4 s = a.spos[ppl[t0 + ln]];
#pragma unroll
            for (int ii = 0; ii < CHUNK; ii++) {
                if ((unsigned)ii < cn_t) {
                    const float dx = s.x - xi[ii], dy = s.y - yi[ii], dz = s.z - zi[ii];
                    const float r2 = fmaf(dz, dz, fmaf(dy, dy, dx * dx));
                    float rinv = __builtin_amdgcn_rsqf(r2 + eps2);
                    rinv = r2 > 0.0f ? rinv : 0.0f;  // self and coincident pairs contribute nothing
                    const float mr = s.w * rinv;
                    const float mr3 = mr * rinv * rinv;
                    add<TERM>(v[4 * ii + 0], cv[4 * ii + 0], mr3 * dx);
                    add<TERM>(v[4 * ii + 1], cv[4 * ii + 1], mr3 * dy);
                    add<TERM>(v[4 * ii + 2], cv[4 * ii + 2], mr3 * dz);
                    add<TERM>(v[4 * ii + 3], cv[4 * ii + 3], -mr);
                }
            }
        }
        if (TERM) {
#pragma unroll
            for (int j = 0; j < NV; j++) v[j] = v[j] - cv[j];
        }
        const float r = transpose_reduce<NV>(v);
        const unsigned slot = res_slot<PREC>((c0 - g0) / CHUNK, ln);
        if (PREC) add<true>(s_res[slot], s_cmp[slot], r);
        else s_res[slot] += r;
    }
}

// What the first wave of a workgroup asks the others to evaluate.
enum : unsigned { EVAL_PC = 0, EVAL_PP = 1, EVAL_LAST = 2, EVAL_NONE = 3 };
struct EvalCmd {
    unsigned what, npc, npp;
};

// Evaluates the list's whole 64-entry tiles (the first wave's call; with NW > 1
// the other waves take their particles meanwhile), moves the remaining entries
// to the front and returns their number.
template <int PREC, bool PC, int NW>
__device__ unsigned flush_list(const WalkArgs &a, uint32_t *list, unsigned n, unsigned g1, float px, float py,
                               float pz, float *s_res, float *s_cmp, EvalCmd *s_cmd) {
    const unsigned ne = n & ~63u;
    wave_sync();  // list entries written by other lanes are visible
    if (ne) {
        if (NW > 1) {
            *s_cmd = EvalCmd{PC ? EVAL_PC : EVAL_PP, ne, ne};
            __syncthreads();
        }
        if (PC) evaluate<PREC>(a, nullptr, 0u, list, ne, list, 0u, 0u, g1, px, py, pz, s_res, s_cmp);
        else evaluate<PREC>(a, nullptr, 0u, list, 0u, list, ne, 0u, g1, px, py, pz, s_res, s_cmp);
        if (NW > 1) __syncthreads();  // the others are done with the list
    }
    const unsigned r = n - ne;
    if (r) {
        const unsigned ln = lane64();
        const unsigned v = ln < r ? list[ne + ln] : 0u;
        wave_sync();
        if (ln < r) list[ln] = v;
        wave_sync();
    }
    return r;
}

// One group per workgroup of NW waves.  The first wave builds the group's lists;
// all of them evaluate the lists, each for its share of the particles.  NW = 1
// is the walk of a full chip.  Where there are fewer groups than the chip holds
// waves, the walk lasts as long as its heaviest group, and NW waves shorten
// that: see walk_group_waves.
template <int PREC, bool SHARED, int NW>
__global__ __launch_bounds__(64 * NW, 4) void k_walk(WalkArgs a) {
    constexpr unsigned MASK = WALK_LSTACK - 1;
    static_assert((WALK_LSTACK & MASK) == 0 && WALK_LSTACK >= 512, "stack ring must hold one step's pushes");
    static_assert(PREFIX_S_CAP <= WALK_LSTACK, "an anchor's cells left fit the empty ring");
    __shared__ uint32_t s_stk[WALK_LSTACK];
    // the compensated walks' compensations take 768 more bytes of LDS: their
    // particle-cell list is shorter by as much, so 16 waves still fit a CU
    constexpr unsigned PC_LDS = PREC ? WALK_PC_LDS - 192 : WALK_PC_LDS;
    __shared__ uint32_t s_pc[PC_LDS];
    __shared__ uint32_t s_pp[WALK_PP_LDS];
    // results of 64 particles, at least one chunk's per wave
    constexpr unsigned RES = NW <= 4 ? 256u / NW : 64u;
    __shared__ float s_res_all[NW * RES];
    __shared__ float s_cmp_all[PREC ? NW * RES : 64];
    __shared__ uint32_t s_idx[64];  // group particle evaluated in each lane
    __shared__ uint32_t s_perm[64];  // caller's index of each group particle
    __shared__ EvalCmd s_cmd;
    __shared__ unsigned s_slot;
    const unsigned ln = lane64();
    const unsigned wid = NW > 1 ? uniform(threadIdx.x >> 6) : 0u;
    float *const s_res = s_res_all + wid * RES;
    float *const s_cmp = s_cmp_all + (PREC ? wid * RES : 0u);
    uint32_t *gstk = a.wstack + (size_t)blockIdx.x * STACK_CAP;
    if (a.hdr->flags & (FLAG_NONFINITE | FLAG_NEGMASS | FLAG_CELLCAP)) return;
    // particles a lane may add to the particle-particle list per round, so that
    // a round (<= 64 * per_round) fits after a flush leaves < 64 entries
    const unsigned per_round = max(1u, (a.pp_cap - 64u) >> 6);  // < 16 since pp_cap <= 1024
    static_assert(WALK_PP_LDS <= 1024, "per-round counts must fit the 4-bit prefix sums");
    const unsigned ngroups = a.qlen ? uniform(*a.qlen) : uniform(a.hdr->ngroups);
    const unsigned pc_cap = min(a.pc_cap, PC_LDS);
    QueueCursor qc = queue_start();
    for (;;) {
        // Every lane executes the queue atomic (only lane 0 adds 1) so that no
        // lane-dependent branch sits inside this loop: the compiler may split a
        // loop on a loop-invariant divergent condition, which would separate
        // lane 0 from the cross-lane operations of the other lanes.
        unsigned slot;
        if (NW > 1) {
            if (wid == 0) s_slot = queue_next(a.head, ngroups, qc);
            __syncthreads();
            slot = uniform(s_slot);
        } else {
            slot = queue_next<false>(a.head, ngroups, qc);  // many groups: more than workgroups by default
        }
        if (slot >= ngroups) break;
        const unsigned g = a.order ? uniform(a.order[slot]) : slot;
        const uint2 gr = a.groups[g];
        // the anchor's record (its lists' place in the pool) is read now, so that
        // it arrives while the group's box is formed
        const uint4 rec = SHARED ? a.arec[uniform(a.anchor[g])] : make_uint4(0u, 0u, 0u, 0u);
        const unsigned gf = uniform(gr.x), gn = uniform(gr.y & 255u), glev = uniform((gr.y >> 8) & 255u);
        const unsigned root = uniform(gr.y >> 16);  // level-0 cells are the systems' roots, in system order
        const unsigned gl = min(ln, gn - 1);
        const float4 p0 = a.spos[gf + gl];
        // each lane's particle in the caller's order, kept in LDS for the results
        const unsigned pm = a.perm[gf + gl];
        float3 bmin = make_float3(p0.x, p0.y, p0.z), bmax = bmin;
#pragma unroll
        for (int o = 32; o > 0; o >>= 1) {
            bmin.x = fminf(bmin.x, __shfl_xor(bmin.x, o, 64));
            bmin.y = fminf(bmin.y, __shfl_xor(bmin.y, o, 64));
            bmin.z = fminf(bmin.z, __shfl_xor(bmin.z, o, 64));
            bmax.x = fmaxf(bmax.x, __shfl_xor(bmax.x, o, 64));
            bmax.y = fmaxf(bmax.y, __shfl_xor(bmax.y, o, 64));
            bmax.z = fmaxf(bmax.z, __shfl_xor(bmax.z, o, 64));
        }
        // The particles evaluated: all of the group's, or only its active ones
        // (an active walk), packed into the first `ge` lanes.  The interaction
        // lists are the whole group's either way (its box above).
        const bool due = ln < gn && (!a.active || a.active[pm] != 0);
        const unsigned long long dm = __ballot(due);
        const unsigned ge = (unsigned)__popcll(dm);
        // (every wave of the workgroup writes the same values)
        if (due) s_idx[rank_below(dm)] = ln;
        s_perm[ln] = pm;
        wave_sync();
        const unsigned pv = s_idx[ln];
        const unsigned pj = ln < ge ? pv : 0u;
        float4 p;
        p.x = __shfl(p0.x, pj, 64);
        p.y = __shfl(p0.y, pj, 64);
        p.z = __shfl(p0.z, pj, 64);
        p.w = 0.0f;
#pragma unroll
        for (int c = 0; c < (int)(RES / 64u); c++) {
            s_res[c * 64 + ln] = 0.0f;
            if (PREC) s_cmp[c * 64 + ln] = 0.0f;
        }
        // this wave's particles
        const unsigned share = (ge + NW - 1u) / NW;
        const unsigned g0 = min(wid * share, ge), g1 = min(g0 + share, ge);

        unsigned f_off = 0, f_n = 0;  // the shared accepted cells, whole tiles in the pool
        bool seeded = false;
        if (SHARED) {
            seeded = uniform(rec.w) == 1u;
            if (seeded) {
                f_off = uniform(rec.x);
                f_n = (uniform(rec.y) + 63u) & ~63u;
            }
        }
        unsigned npc = 0, npp = 0;
        bool overflow = false;
        if (wid == 0) {
        // logical stack = global spill [0, gtop) followed by the LDS ring [sb, st)
        unsigned sb = 0, st = 0, gtop = 0;
        unsigned tot_pc = 0, tot_pp = 0;
        if (SHARED) {
            // the lists shared by the groups below this group's anchor cell: its
            // accepted cells are evaluated in place, from the pool, with the
            // group's own lists at its end, and the stack starts with the cells
            // left (sorted by level, shallowest at the bottom, so that stack levels
            // never decrease towards the top), in the LDS ring, which is empty here
            // and holds all of them (<= PREFIX_S_CAP)
            if (seeded) {
                const unsigned ns = uniform(rec.z);
                for (unsigned i = ln; i < ns; i += 64) s_stk[i] = a.pool[f_off + f_n + i];
                st = ns;
                tot_pc += uniform(rec.y);
            }
        }
        if (!seeded) {
            // The root is an ancestor of every group, so the walk always opens it:
            // its children (the root itself when it is a leaf) start the stack, in
            // the order its opening would push them.
            const uint4 tr = a.topo[root];
            const unsigned rn = uniform(tr.w & 255u);
            st = rn ? rn : 1u;
            const unsigned first = rn ? tr.z + min(ln, rn - 1) : root;
            if (ln < st) s_stk[ln] = first;
        }
        wave_sync();
        while (st != sb || gtop > 0) {
            if (st == sb) {  // LDS part empty: refill from the top of the global spill
                const unsigned k = min(gtop, WALK_LSTACK / 2);
                wave_sync();
                for (unsigned i = ln; i < k; i += 64) s_stk[(sb - k + i) & MASK] = gstk[gtop - k + i];
                sb -= k;
                gtop -= k;
                wave_sync();
            }
            const unsigned m = min(st - sb, 64u);
            const bool valid = ln < m;
            const unsigned c = valid ? s_stk[(st - m + ln) & MASK] : 0u;
            st -= m;
            const uint4 t = a.topo[c];
            const float4 mc = a.cmac[c];
            const unsigned lvl = (t.w >> 8) & 255u, nch = t.w & 255u;
            const bool anc = t.x <= gf && gf < t.x + t.y && lvl <= glev;
            // The opening test is taken in every lane and combined without
            // short-circuit: were it skipped for ancestors, the compiler would
            // issue the cell's MAC load only after its topology had arrived,
            // two dependent round trips per step instead of one.
            const bool far = mac_accept(bmin, bmax, mc);
            const bool accept = valid & !anc & far;
            const bool opened = valid && !accept;
            const bool leaf = opened && nch == 0;
            const bool push = opened && nch != 0;

            // accepted cells -> particle-cell list
            const unsigned long long am = __ballot(accept);
            const unsigned na = (unsigned)__popcll(am);
            if (npc + na > pc_cap)
                npc = flush_list<PREC, true, NW>(a, s_pc, npc, g1, p.x, p.y, p.z, s_res, s_cmp, &s_cmd);
            if (accept) s_pc[npc + rank_below(am)] = c;
            npc += na;
            tot_pc += na;

            // One prefix sum gives the list offsets of both the opened leaves'
            // particles (low half; leaves of 32 or more particles count 0 here
            // and go by rounds below) and the opened internal cells' children
            // (high half): sums stay below 64 * 32 and 64 * 8.
            unsigned rem = leaf ? t.y : 0u, src = t.x;
            const unsigned nc = push ? nch : 0u;
            const bool big = __ballot(rem > 31u) != 0;
            const unsigned packed = (big ? 0u : rem) | (nc << 16);
            const unsigned incl = wave_incl_scan(packed);
            const unsigned excl = incl - packed;
            const unsigned both = uniform(__builtin_amdgcn_readlane(incl, 63));

            // opened leaves -> particle-particle list: whole leaves in one round
            // when every leaf holds fewer than 32 particles and they fit after a
            // flush, else in rounds of at most per_round particles per lane
            if (!big && (both & 0xffffu)) {
                const unsigned sum = both & 0xffffu;
                const unsigned off = excl & 0xffffu;
                if (sum + 63u <= a.pp_cap) {
                    if (npp + sum > a.pp_cap)
                        npp = flush_list<PREC, false, NW>(a, s_pp, npp, g1, p.x, p.y, p.z, s_res, s_cmp, &s_cmd);
                    for (unsigned j = 0; j < rem; j++) s_pp[npp + off + j] = src + j;
                    npp += sum;
                    tot_pp += sum;
                    rem = 0;
                }
            }
            while (__ballot(rem > 0)) {
                const unsigned take = min(rem, per_round);
                unsigned sum;
                const unsigned off = small_excl_scan(take, &sum);
                if (npp + sum > a.pp_cap)
                    npp = flush_list<PREC, false, NW>(a, s_pp, npp, g1, p.x, p.y, p.z, s_res, s_cmp, &s_cmd);
                for (unsigned j = 0; j < take; j++) s_pp[npp + off + j] = src + j;
                npp += sum;
                tot_pp += sum;
                rem -= take;
                src += take;
            }

            // opened internal cells -> children onto the stack
            const unsigned nsum = both >> 16;
            const unsigned off = excl >> 16;
            const unsigned used = st - sb;
            if (used + nsum > WALK_LSTACK) {  // spill the bottom of the LDS ring
                const unsigned need = used + nsum - WALK_LSTACK;
                const unsigned sp = min(used, max(need, WALK_LSTACK / 2));
                if (gtop + sp > STACK_CAP) {
                    overflow = true;
                    break;
                }
                for (unsigned i = ln; i < sp; i += 64) gstk[gtop + i] = s_stk[(sb + i) & MASK];
                sb += sp;
                gtop += sp;
                wave_sync();
            }
            for (unsigned j = 0; j < nc; j++) s_stk[(st + off + j) & MASK] = t.z + j;
            st += nsum;
            wave_sync();
        }
        if (overflow) {
            atomicOr(&a.hdr->flags, FLAG_STACK);
        } else {
            // both lists' last tiles padded with the massless far cell and
            // particle (npc <= pc_cap and npp <= pp_cap, so the padded lists
            // stay within their LDS arrays, whole tiles long)
            const unsigned npc_t = (npc + 63u) & ~63u, npp_t = (npp + 63u) & ~63u;
            if (npc + ln < npc_t) s_pc[npc + ln] = a.dcell;
            if (npp + ln < npp_t) s_pp[npp + ln] = a.dpart;
            npc = npc_t;
            npp = npp_t;
            a.gcounts[g] = make_uint2(tot_pc, tot_pp);  // same value from every lane
        }
        wave_sync();  // list entries written by other lanes are visible
        if (NW > 1) {
            s_cmd = EvalCmd{overflow ? EVAL_NONE : EVAL_LAST, npc, npp};
            __syncthreads();
        }
        } else {  // the other waves: their particles of each evaluation the first one asks for
            for (;;) {
                __syncthreads();
                const unsigned what = uniform(s_cmd.what);
                npc = uniform(s_cmd.npc);
                npp = uniform(s_cmd.npp);
                overflow = what == EVAL_NONE;
                if (what >= EVAL_LAST) break;
                evaluate<PREC>(a, nullptr, 0u, s_pc, what == EVAL_PC ? npc : 0u, s_pp, what == EVAL_PP ? npp : 0u, g0, g1,
                               p.x, p.y, p.z, s_res, s_cmp);
                __syncthreads();
            }
        }
        if (overflow) continue;
        if (f_n + npc + npp)
            evaluate<PREC>(a, f_n ? a.pool + f_off : nullptr, f_n, s_pc, npc, s_pp, npp, g0, g1, p.x, p.y, p.z, s_res,
                           s_cmp);

        // results back to the caller's order
        constexpr int CHUNK = chunk_of<PREC>();
        constexpr bool HALF = CHUNK == 8;
        // value held by this lane: bitrev6(ln) (64 per chunk) or its low five
        // bits (32 per chunk, lanes ln and ln ^ 1 alike: the even one stores)
        const unsigned idx = HALF ? (bitrev6(ln) & 31u) : bitrev6(ln);
        const unsigned comp = idx & 3u;
        for (unsigned c = 0; c * CHUNK < g1 - g0; c++) {
            const unsigned pi = g0 + c * CHUNK + (idx >> 2) + ((HALF && (ln & 1u)) ? 64u : 0u);
            if (pi < g1) {
                const unsigned slot = res_slot<PREC>(c, ln);
                float val = s_res[slot];
                if (PREC) val = val - s_cmp[slot];
                val *= a.G;
                const size_t orig = s_perm[s_idx[pi]];
                if (comp < 3) a.acc[3 * orig + comp] = val;
                else a.pot[orig] = val;
            }
        }
    }
}

// --------------------------------------------------------------------------
// Shared-prefix walk: the groups below one anchor cell A (the ancestor `up`
// levels above each group) share the part of their traversals that A's
// particle box decides for all of them.  From the root, with A's box:
//   * a cell that is an ancestor-or-self of A, or whose opening radius reaches
//     the farthest point of A's box, is opened by every group inside A: its
//     children are visited, and a leaf among them is left to each group (it
//     lands in the group's particle-particle list);
//   * a cell A's box accepts (the group MAC with A's box) is accepted by every
//     group inside A: the group's box lies inside A's, so its rounded distance
//     is no smaller; such a cell is never an ancestor of a group (it would
//     either contain A, and ancestors of A are opened, or lie inside A, with
//     its centre of mass inside A's box at distance 0);
//   * any other cell is left to each group.
// Each group then starts with the cells left (S) on its stack and walks on as
// usual, and evaluates the accepted cells (F, whole tiles in the pool) in place
// with its own lists at its end: the same cells are accepted and opened as in
// a walk from the root, and summed in another order.
// --------------------------------------------------------------------------

// Anchor of every group the walk visits (every group, or the queue's first *qlen
// entries): the cell at level max(level - up, 0) that holds the group's first
// particle (cells of one level are numbered in particle order).  Each anchor is
// listed once, by the group that claims it: a compare-and-swap of its record's
// valid word from 0, where the MAC kernel left it, to 2.  Only entries whose anchor
// differs from the previous entry's try: in Morton order an anchor's groups are
// contiguous unless groups of deeper levels sit between them, so few entries
// compete (a wave's first entry tries without a look at the entry before: a
// claiming kernel of its own, which had that, took 4.5 us more).
// With `gorder` the kernel also (without ANCHORS: only) places the queue's groups:
// each eighth's window by particle count, largest first, in the old order within a
// count.  Every workgroup adds up the counts of its
// eighths' window blocks; the ranks inside a block come from ballots, so the order
// is the same on every run.
template <bool ANCHORS>
__global__ __launch_bounds__(GORD_BLOCK) void k_walk_anchor(const Header *__restrict__ hdr,
                                                            const uint2 *__restrict__ groups,
                                                            const uint4 *__restrict__ topo, int up,
                                                            uint32_t *__restrict__ anchor, uint4 *__restrict__ arec,
                                                            const uint32_t *__restrict__ order,
                                                            const uint32_t *__restrict__ qlen,
                                                            const uint32_t *__restrict__ ghist,
                                                            uint32_t *__restrict__ gorder,
                                                            uint32_t *__restrict__ alist,
                                                            unsigned *__restrict__ acount) {
    constexpr unsigned NW = GORD_BLOCK / 64, STRIPS = GORD_BLOCK / GORD_CLASSES;
    static_assert(NW == STRIPS && GORD_CLASSES == 64, "one wave per strip of blocks");
    __shared__ unsigned s_sum[2][2][STRIPS][GORD_CLASSES];  // [half][before this block, all]
    __shared__ unsigned s_at[2][GORD_CLASSES];              // first slot of this block's groups
    __shared__ unsigned s_cnt[NW][2 * GORD_CLASSES];
    if (hdr->flags & (FLAG_NONFINITE | FLAG_NEGMASS | FLAG_CELLCAP)) return;
    const unsigned ng = hdr->ngroups;
    const unsigned nq = qlen ? min(*qlen, ng) : ng;
    const unsigned t = threadIdx.x, w = t >> 6, c = lane64();
    for (unsigned blk = blockIdx.x; blk * GORD_BLOCK < nq; blk += gridDim.x) {
        const unsigned i = blk * GORD_BLOCK + t;
        const unsigned g = i < nq ? (order ? order[i] : i) : 0u;
        const uint2 gr = i < nq ? groups[g] : make_uint2(0u, 0u);
        if (ANCHORS) {
            const int glev = (int)((gr.y >> 8) & 255u);
            const int lev = glev > up ? glev - up : 0;
            unsigned lo = hdr->lvl_begin[lev], hi = hdr->lvl_begin[lev + 1];  // topo[lo].x <= gr.x
            while (hi - lo > 1) {
                const unsigned mid = lo + (hi - lo) / 2;
                if (topo[mid].x <= gr.x) lo = mid; else hi = mid;
            }
            const unsigned prev = __shfl_up(lo, 1, 64);
            if (i < nq) {
                anchor[g] = lo;
                if ((c == 0 || prev != lo) && atomicCAS(&arec[lo].w, 0u, 2u) == 0u) alist[atomicAdd(acount, 1u)] = lo;
            }
        }
        if (!gorder) continue;  // the same for the whole launch
        if (nq < GORD_MIN) {
            if (i < nq) gorder[i] = g;
            continue;
        }
        const unsigned e0 = gord_eighth(nq, blk * GORD_BLOCK);
        const unsigned elast = gord_eighth(nq, min(blk * GORD_BLOCK + GORD_BLOCK, nq) - 1u);
#pragma unroll
        for (unsigned h = 0; h < 2; h++) {  // sums of class c over strip w of the blocks
            unsigned before = 0, all = 0;
            if (e0 + h <= elast) {
                const unsigned lo = gord_begin(nq, e0 + h), hi = gord_begin(nq, e0 + h + 1u);
                for (unsigned b = gord_window(nq, e0 + h) / GORD_BLOCK + w; b * GORD_BLOCK < hi; b += STRIPS) {
                    // an eighth is a block's second one only in the block it starts in
                    const unsigned half = b * GORD_BLOCK < lo ? 1u : 0u;
                    const unsigned v = ghist[((size_t)b * 2 + half) * GORD_CLASSES + c];
                    all += v;
                    before += b < blk ? v : 0u;
                }
            }
            s_sum[h][0][w][c] = before;
            s_sum[h][1][w][c] = all;
        }
        (&s_cnt[0][0])[t] = 0;
        (&s_cnt[0][0])[t + GORD_BLOCK] = 0;
        __syncthreads();
        if (w < 2u) {  // wave h: slots of eighth e0 + h by class
            unsigned before = 0, all = 0;
#pragma unroll
            for (unsigned v = 0; v < STRIPS; v++) {
                before += s_sum[w][0][v][c];
                all += s_sum[w][1][v][c];
            }
            s_at[w][c] = gord_window(nq, min(e0 + w, WALK_QUEUES - 1u)) + (wave_incl_scan(all) - all) + before;
        }
        // rank among the wave's groups of the same eighth and class
        const unsigned e = i < nq ? gord_eighth(nq, i) : 0u;
        const bool ranked = i < nq && i >= gord_window(nq, e);
        const unsigned d = ranked ? (e - e0) * GORD_CLASSES + gord_class(gr) : 0u;
        unsigned long long peers = __ballot(ranked);
#pragma unroll
        for (int bit = 0; bit < 7; bit++) {
            const bool v = (d >> bit) & 1u;
            const unsigned long long m = __ballot(v);
            peers &= v ? m : ~m;
        }
        const unsigned rank = rank_below(peers);
        if (ranked && rank == 0) s_cnt[w][d] = (unsigned)__popcll(peers);
        __syncthreads();
        if (i < nq) {
            unsigned pos = i;
            if (ranked) {
                pos = s_at[d / GORD_CLASSES][d % GORD_CLASSES] + rank;
                for (unsigned v = 0; v < w; v++) pos += s_cnt[v][d];
            }
            gorder[pos] = g;
        }
        __syncthreads();
    }
}

// Counts of an active walk's queue (a full walk's come with the tree).
__global__ __launch_bounds__(256) void k_walk_count(const Header *__restrict__ hdr, const uint2 *__restrict__ groups,
                                                    const uint32_t *__restrict__ order,
                                                    const uint32_t *__restrict__ qlen, uint32_t *__restrict__ ghist) {
    if (hdr->flags & (FLAG_NONFINITE | FLAG_NEGMASS | FLAG_CELLCAP)) return;
    gord_count(groups, order, min(*qlen, hdr->ngroups), ghist);
}

// F and S of anchor cell A into this workgroup's scratch (F at pf, S sorted by
// level at pf + PREFIX_F_CAP + PREFIX_S_CAP).  False when a list outgrows its
// room or the stack its bound (the groups then walk from the root).  A step takes
// up to 256 cells off the stack, one per thread: the pass is bound by the
// dependent round trips of its traversals, about 10 steps each.  One wave taking
// 4 cells per lane had a step's four batches one after the other: the pass took
// 65 / 71 / 80 us at n = 32768 / 2^20 / 2^22, with four waves 42 / 45 / 55, and
// without eight empty queues tried at its end 19 / 23 / 33.
struct PrefixShared {
    uint32_t stk[PREFIX_RING];
    unsigned cnt[2][PREFIX_WAVES][3];               // accepted, left, children of each wave, by parity of the step
    unsigned lev[KEY_LEVELS + 1][PREFIX_S_CAP / 64];  // cells of a level in each batch of 64
    unsigned off[2];
};

__device__ bool anchor_lists(const WalkArgs &a, unsigned A, PrefixShared &sh, uint32_t *gstk, uint32_t *pf,
                             unsigned *nf_out, unsigned *ns_out) {
    constexpr unsigned NT = PREFIX_THREADS, RING = PREFIX_RING, MASK = RING - 1;
    static_assert((RING & MASK) == 0 && RING >= 2 * NT * 8, "ring must hold one step's pushes");
    const unsigned t = threadIdx.x, ln = lane64(), w = uniform(t >> 6);
    uint32_t *praw = pf + PREFIX_F_CAP, *pseed = praw + PREFIX_S_CAP;
    const uint4 ta = a.topo[A];
    const unsigned af = uniform(ta.x), alev = uniform((ta.w >> 8) & 255u), root = uniform(ta.w >> 16);
    const float *cb = a.cbox + 6 * (size_t)A;
    const float3 bmin = make_float3(cb[0], cb[1], cb[2]), bmax = make_float3(cb[3], cb[4], cb[5]);
    const uint4 tr = a.topo[root];
    const unsigned rn = uniform(tr.w & 255u);
    unsigned sb = 0, st = rn ? rn : 1u, gtop = 0, nf = 0, ns = 0;
    bool ok = true;
    if (t < st) sh.stk[t] = rn ? tr.z + t : root;
    __syncthreads();
    for (unsigned par = 0; st != sb || gtop > 0; par ^= 1u) {
        if (st == sb) {  // LDS part empty: refill from the top of the global spill
            const unsigned k = min(gtop, RING / 2);
            for (unsigned i = t; i < k; i += NT) sh.stk[(sb - k + i) & MASK] = gstk[gtop - k + i];
            sb -= k;
            gtop -= k;
            __syncthreads();
        }
        const unsigned m = min(st - sb, NT);
        const bool valid = t < m;
        const unsigned c = valid ? sh.stk[(st - m + t) & MASK] : 0u;
        st -= m;
        const uint4 tc = a.topo[c];
        const float4 mc = a.cmac[c];
        const unsigned lvl = (tc.w >> 8) & 255u, nch = tc.w & 255u;
        const bool anc = tc.x <= af && af < tc.x + tc.y && lvl <= alev;
        // both tests in every lane, no short-circuit: the MAC load then goes
        // out with the topology load (see the group walk)
        const bool reach = !(far_d2(bmin, bmax, mc) > mc.w);
        const bool far = mac_accept(bmin, bmax, mc);
        const bool open = valid & (anc | reach);
        const bool accept = valid & !open & far;
        const bool left = valid && !accept && (!open || nch == 0);
        const unsigned long long am = __ballot(accept), lm = __ballot(left);
        const unsigned nc = open ? nch : 0u;
        unsigned tk;
        const unsigned o = small_excl_scan(nc, &tk);
        // this wave's counts to the others, theirs back: the popped entries have
        // been read when the barrier is passed
        sh.cnt[par][w][0] = (unsigned)__popcll(am);
        sh.cnt[par][w][1] = (unsigned)__popcll(lm);
        sh.cnt[par][w][2] = tk;
        __syncthreads();
        unsigned before[3] = {0u, 0u, 0u}, all[3] = {0u, 0u, 0u};
#pragma unroll
        for (unsigned v = 0; v < PREFIX_WAVES; v++) {
#pragma unroll
            for (unsigned k = 0; k < 3; k++) {
                const unsigned x = uniform(sh.cnt[par][v][k]);
                before[k] += v < w ? x : 0u;
                all[k] += x;
            }
        }
        if (nf + all[0] > PREFIX_F_CAP || ns + all[1] > PREFIX_S_CAP) {  // the same for the whole workgroup
            ok = false;
            break;
        }
        if (accept) pf[nf + before[0] + rank_below(am)] = c;
        if (left) praw[ns + before[1] + rank_below(lm)] = c;
        nf += all[0];
        ns += all[1];
        const unsigned nsum = all[2], used = st - sb;
        if (used + nsum > RING) {  // spill the bottom of the LDS ring
            const unsigned need = used + nsum - RING;
            const unsigned sp = min(used, max(need, RING / 2));
            if (gtop + sp > STACK_CAP) {
                ok = false;
                break;
            }
            for (unsigned i = t; i < sp; i += NT) gstk[gtop + i] = sh.stk[(sb + i) & MASK];
            sb += sp;
            gtop += sp;
            __syncthreads();
        }
        for (unsigned j = 0; j < nc; j++) sh.stk[(st + before[2] + o + j) & MASK] = tc.z + j;
        st += nsum;
        __syncthreads();
    }
    __syncthreads();
    if (ok) {  // S by level, shallowest first, in order within a level: ranks in batches of 64
        constexpr unsigned NB = PREFIX_S_CAP / 64, PER = NB / PREFIX_WAVES;
        for (unsigned k = t; k < (KEY_LEVELS + 1u) * NB; k += NT) (&sh.lev[0][0])[k] = 0;
        __syncthreads();
        unsigned cell[PER], lv[PER], rank[PER];
#pragma unroll
        for (unsigned x = 0; x < PER; x++) {
            const unsigned b = w * PER + x, i = b * 64 + ln;
            const bool in = i < ns;
            cell[x] = in ? praw[i] : 0u;
            lv[x] = in ? (a.topo[cell[x]].w >> 8) & 255u : 0u;
            unsigned long long peers = __ballot(in);
#pragma unroll
            for (int bit = 0; bit < 5; bit++) {
                static_assert(KEY_LEVELS < 32, "5-bit levels");
                const bool v = (lv[x] >> bit) & 1u;
                const unsigned long long bm = __ballot(v);
                peers &= v ? bm : ~bm;
            }
            rank[x] = rank_below(peers);
            if (in && rank[x] == 0) sh.lev[lv[x]][b] = (unsigned)__popcll(peers);
        }
        __syncthreads();
        if (t < 64u) {  // places of the level's batches: a scan of the table, level by level
            constexpr unsigned N = (KEY_LEVELS + 1) * NB, P = (N + 63u) / 64u;
            unsigned *tab = &sh.lev[0][0];
            unsigned v[P], sum = 0;
#pragma unroll
            for (unsigned k = 0; k < P; k++) {
                v[k] = t * P + k < N ? tab[t * P + k] : 0u;
                sum += v[k];
            }
            unsigned run = wave_incl_scan(sum) - sum;
#pragma unroll
            for (unsigned k = 0; k < P; k++) {
                if (t * P + k < N) tab[t * P + k] = run;
                run += v[k];
            }
        }
        __syncthreads();
#pragma unroll
        for (unsigned x = 0; x < PER; x++) {
            const unsigned b = w * PER + x;
            if (b * 64 + ln < ns) pseed[sh.lev[lv[x]][b] + rank[x]] = cell[x];
        }
        __syncthreads();
    }
    *nf_out = nf;
    *ns_out = ns;
    return ok;
}

// One pass over the anchor list (persistent workgroups, per-XCD queues as in the
// walk; one anchor per queue slot): a workgroup builds its anchor's lists, stores
// them in the pool and their place in arec[anchor] (valid word 1; all zero when
// they did not fit, and the anchor's groups walk from the root).
__global__ __launch_bounds__(PREFIX_THREADS) void k_walk_prefix(WalkArgs a, unsigned *__restrict__ prefix_head,
                                                                const unsigned *__restrict__ acount,
                                                                const uint32_t *__restrict__ alist,
                                                                unsigned long long *__restrict__ pool_head,
                                                                uint4 *__restrict__ arec, uint32_t *__restrict__ pool,
                                                                unsigned long long pool_cap,
                                                                uint32_t *__restrict__ pscr,
                                                                unsigned *__restrict__ nfail) {
    __shared__ PrefixShared sh;
    const unsigned t = threadIdx.x, ln = lane64(), w = uniform(t >> 6);
    uint32_t *gstk = a.wstack + (size_t)blockIdx.x * STACK_CAP;
    uint32_t *pf = pscr + (size_t)blockIdx.x * PREFIX_SCRATCH;
    if (a.hdr->flags & (FLAG_NONFINITE | FLAG_NEGMASS | FLAG_CELLCAP)) return;
    const unsigned nanchor = uniform(*acount);
    QueueCursor qc = queue_start();
    for (;;) {
        if (w == 0) sh.off[0] = queue_next(prefix_head, nanchor, qc);
        __syncthreads();
        const unsigned slot = uniform(sh.off[0]);
        if (slot >= nanchor) break;
        const unsigned A = uniform(alist[slot]);
        unsigned nf, ns;
        bool ok = anchor_lists(a, A, sh, gstk, pf, &nf, &ns);
        // F takes whole 64-entry tiles in the pool (padded with the massless far
        // cell): the groups evaluate it in place
        const unsigned nfp = (nf + 63u) & ~63u;
        if (w == 0) {
            unsigned long long off64 = ~0ull;
            if (ok) off64 = atomicAdd(pool_head, ln == 0 ? (unsigned long long)(nfp + ns) : 0ull);
            off64 = ((unsigned long long)uniform((unsigned)(off64 >> 32)) << 32) | uniform((unsigned)off64);
            const bool fits = ok && off64 + nfp + ns <= pool_cap;
            if (!fits) atomicAdd(nfail, ln == 0 ? 1u : 0u);  // the same for the whole wave
            sh.off[0] = (unsigned)off64;  // < 2^32 when it fits
            sh.off[1] = fits ? 1u : 0u;
        }
        __syncthreads();
        const unsigned off = uniform(sh.off[0]);
        ok = uniform(sh.off[1]) != 0u;
        if (ok) {
            for (unsigned i = t; i < nfp; i += PREFIX_THREADS) pool[off + i] = i < nf ? pf[i] : a.dcell;
            const uint32_t *pseed = pf + PREFIX_F_CAP + PREFIX_S_CAP;
            for (unsigned i = t; i < ns; i += PREFIX_THREADS) pool[off + nfp + i] = pseed[i];
        }
        // every thread stores the same record: no lane-dependent branch in this loop
        arec[A] = ok ? make_uint4(off, nf, ns, 1u) : make_uint4(0u, 0u, 0u, 0u);
        __syncthreads();  // sh.off and the scratch are free again
    }
}

// Waves per group for a tree of n particles in groups of up to `cap`.  A chip full of
// groups wants one: the waves that wait while the first builds the lists hold
// registers that another group's wave could use.  With few groups the heaviest one
// sets the time.  Groups of up to 64, walk stage with 1 / 2 / 4 waves per group
// (Plummer sphere, theta 0.75, us): n = 1000 96 / 66 / 52, 20000 195 / 131 / 121,
// 32768 209 / 148 / 146, 65536 260 / 217 / 229, 131072 390 / 370 / 415, 200000 480 /
// 481 / 555, 300007 617 / 636 / 746, 2^20 1513 / 1731 / 2334.  The results are the
// same bits.  With the queue's end by size one wave gains more than two, so the
// second line lies between where these meet at theta 0.75 (115000) and 0.5 (128000):
// with one wave and with two, us, 100003 278 / 483 and 265 / 446, 125000 278 / 548
// and 298 / 522, 140000 288 / 562 and 318 / 568, 160000 303 / 577 and 354 / 638.
// Eight waves against four, theta 0.75, us with the anchor pass: 1000 47.8 / 50.1,
// 3000 63.2 / 67.8, 6000 77.3 / 83.9, 10000 106 / 88.
// Smaller groups are more (they hold about 0.27 cap + 0.7 particles), so the lines
// are taken at m, the particles that make as many groups of up to 64; and a group of
// few particles leaves the further waves little, so the lines come sooner.  Forces,
// theta 0.5, us, with 1 / 2 / 4 / 8 waves: cap 32, n = 5000 178 / 92 / 84 / 110, 20000
// 262 / 180 / 223 / 346, 50000 342 / 331 / 476, 100003 395 / 506; cap 16, 5000 138 /
// 87 / 81 / 130, 10000 163 / 135 / 165, 20000 191 / 213 / 338 (a cube 113 / 79 / 117);
// cap 8, 2000 106 / 54 / 55 / 76, 10000 149 / 136 / 210, 20000 206 / 251 / 430; cap 1,
// 1000 105 / 58 / 59 / 83, 2000 111 / 68 / 100, 5000 162 / 185 / 303.
// An active walk takes the waves of its whole tree: how many groups it visits is
// known on the device alone (*qlen), and the launch's form is fixed before.  With few
// groups due in a large tree the heaviest of them, on one wave, then sets the time;
// the results do not depend on it.
int walk_group_waves(unsigned n, unsigned cap) {
    const unsigned long long m = 67ull * n / (cap + 3u);
    return m <= 8192u ? 8 : m <= 15360u + 272u * cap ? 4 : m <= 73728u + 768u * cap ? 2 : 1;
}

// As many workgroups as the launch parameter's waves have spill stacks.  Of 4096
// workgroups of 2, 4 or 8 waves the chip holds a part at once; the
// others follow as those end, so up to 4096 groups need no queue.
template <int PREC, int NW>
void launch_walk_groups(const WalkArgs &a, bool shared, unsigned grid, hipStream_t s) {
    if (shared) hipLaunchKernelGGL((k_walk<PREC, true, NW>), dim3(grid), dim3(64 * NW), 0, s, a);
    else hipLaunchKernelGGL((k_walk<PREC, false, NW>), dim3(grid), dim3(64 * NW), 0, s, a);
}
template <int PREC>
void launch_walk_waves(const WalkArgs &a, bool shared, int nw, unsigned waves, hipStream_t s) {
    if (nw == 8) launch_walk_groups<PREC, 8>(a, shared, waves, s);
    else if (nw == 4) launch_walk_groups<PREC, 4>(a, shared, waves, s);
    else if (nw == 2) launch_walk_groups<PREC, 2>(a, shared, waves, s);
    else launch_walk_groups<PREC, 1>(a, shared, waves, s);
}

}  // namespace

// Small trees give every group a workgroup at once: the order is the hardware's,
// and one by size spreads each XCD's heavy groups over fewer CUs (the walk of a
// 65536-particle Plummer sphere by work: 282 us against 217 in Morton order).  With
// more groups than workgroups the walk gains from 80000 particles (230 us against
// 270) over 300007 (485 against 630) to 2^20 (1395 against 1540); an active walk
// of 15% of 2^20 particles takes 364 us against 450.
bool walk_sorts_groups(unsigned n) { return n > 65536u; }

hipError_t launch_group_order(const Buffers &b, unsigned n, hipStream_t s) {
    const unsigned blocks = min((n + GORD_BLOCK - 1u) / GORD_BLOCK, 1024u);
    hipLaunchKernelGGL(k_walk_anchor<false>, dim3(blocks), dim3(GORD_BLOCK), 0, s, b.hdr, b.groups, b.topo, 0, nullptr,
                       nullptr, nullptr, nullptr, b.ghist, b.gorder, nullptr, nullptr);
    return hipGetLastError();
}

hipError_t launch_walk(const Buffers &b, unsigned n, unsigned nsys, float eps2, float G, int precision,
                       const uint32_t *order, const uint32_t *qlen, const uint8_t *active, float *acc, float *pot,
                       int anchor_up, hipStream_t s) {
    WalkArgs a;
    a.hdr = b.hdr;
    a.topo = b.topo;
    a.cmac = b.cmac;
    a.ceval = b.ceval;
    a.spos = b.spos;
    a.perm = b.vals[0];
    a.groups = b.groups;
    a.gcounts = b.gcounts;
    a.wstack = b.wstack;
    a.order = order;
    a.qlen = qlen;
    a.active = active;
    a.head = b.hdr->walk_head;
    a.acc = acc;
    a.pot = pot;
    a.eps2 = eps2;
    a.G = G;
    a.pc_cap = b.pc_cap;
    a.pp_cap = b.pp_cap;
    a.dcell = b.cap_cells;
    a.dpart = b.n_max;
    a.cbox = b.cbox;
    a.anchor = b.anchor;
    a.arec = b.arec;
    a.pool = b.pool;
    const bool shared = anchor_up > 0 && b.anchor;
    if (shared) {
        // a queue in Morton order is put in order of size; the work-ordered ones are taken as they are
        const unsigned ablk = min((n + GORD_BLOCK - 1u) / GORD_BLOCK, 1024u);
        uint32_t *gorder = (!order || qlen) && walk_sorts_groups(n) ? b.gorder : nullptr;
        uint32_t *ghist = qlen ? b.gahist : b.ghist;
        if (gorder && qlen)
            hipLaunchKernelGGL(k_walk_count, dim3(ablk), dim3(256), 0, s, b.hdr, b.groups, order, qlen, ghist);
        hipLaunchKernelGGL(k_walk_anchor<true>, dim3(ablk), dim3(GORD_BLOCK), 0, s, b.hdr, b.groups, b.topo, anchor_up, b.anchor,
                           b.arec, order, qlen, ghist, gorder, b.alist, &b.hdr->anchor_count);
        if (gorder) a.order = gorder;
        hipLaunchKernelGGL(k_walk_prefix, dim3(min(b.walk_waves, 1024u)), dim3(PREFIX_THREADS), 0, s, a, b.hdr->prefix_head,
                           &b.hdr->anchor_count, b.alist, &b.hdr->pool_head, b.arec, b.pool, b.pool_cap, b.pscr,
                           &b.hdr->anchor_fail);
    }
    const int nw = walk_group_waves(n, b.group_cap);
    if (precision == 2) launch_walk_waves<2>(a, shared, nw, b.walk_waves, s);
    else if (precision == 1) launch_walk_waves<1>(a, shared, nw, b.walk_waves, s);
    else launch_walk_waves<0>(a, shared, nw, b.walk_waves, s);
    return hipGetLastError();
}

// --------------------------------------------------------------------------
// Queue of an active walk: the groups that hold an active particle, then the
// others, both in Morton order.  Bound by the latency of perm and the mask behind
// it: a wave reads a group's particles at once, eight groups in flight.  20 us at
// 2^20 particles (15 + 5); by the counting sort below, with one thread per group
// that read its particles one after the other in two of the three kernels, 52 us.
// A block's first slot is the sum of the counts of the blocks before it.
// --------------------------------------------------------------------------
namespace {

constexpr unsigned ACT_BLOCK = 512;  // groups per workgroup and threads

__global__ __launch_bounds__(ACT_BLOCK) void k_active_flag(const Header *__restrict__ hdr,
                                                           const uint2 *__restrict__ groups,
                                                           const uint32_t *__restrict__ perm,
                                                           const uint8_t *__restrict__ active,
                                                           uint8_t *__restrict__ gflag, uint32_t *__restrict__ bcnt) {
    constexpr unsigned IN_FLIGHT = 8;
    __shared__ unsigned s_cnt[ACT_BLOCK / 64];
    if (hdr->flags & (FLAG_NONFINITE | FLAG_NEGMASS | FLAG_CELLCAP)) return;
    const unsigned ng = hdr->ngroups, ln = lane64(), w = uniform(threadIdx.x >> 6);
    for (unsigned blk = blockIdx.x; blk * ACT_BLOCK < ng; blk += gridDim.x) {
        const unsigned g0 = blk * ACT_BLOCK + w * 64;  // this wave's groups, one per lane
        const uint2 gr = groups[min(g0 + ln, ng - 1u)];
        unsigned long long any = 0;  // bit k: group g0 + k holds an active particle
        for (unsigned k0 = 0; k0 < 64; k0 += IN_FLIGHT) {
            uint8_t v[IN_FLIGHT];
#pragma unroll
            for (unsigned u = 0; u < IN_FLIGHT; u++) {
                const unsigned first = __builtin_amdgcn_readlane(gr.x, k0 + u);
                const unsigned cnt = __builtin_amdgcn_readlane(gr.y, k0 + u) & 255u;
                v[u] = active[perm[first + min(ln, cnt - 1u)]];
            }
#pragma unroll
            for (unsigned u = 0; u < IN_FLIGHT; u++) any |= __ballot(v[u] != 0) ? 1ull << (k0 + u) : 0ull;
        }
        const bool mine = g0 + ln < ng && ((any >> ln) & 1ull);
        if (g0 + ln < ng) gflag[g0 + ln] = mine ? 1 : 0;
        const unsigned cnt = (unsigned)__popcll(__ballot(mine));
        if (ln == 0) s_cnt[w] = cnt;
        __syncthreads();
        if (threadIdx.x == 0) {
            unsigned sum = 0;
            for (unsigned v = 0; v < ACT_BLOCK / 64; v++) sum += s_cnt[v];
            bcnt[blk] = sum;
        }
        __syncthreads();
    }
}

__global__ __launch_bounds__(ACT_BLOCK) void k_active_queue(const Header *__restrict__ hdr,
                                                            const uint8_t *__restrict__ gflag,
                                                            const uint32_t *__restrict__ bcnt,
                                                            uint32_t *__restrict__ order, uint32_t *__restrict__ qlen) {
    __shared__ unsigned s_sum[2][ACT_BLOCK / 64];
    if (hdr->flags & (FLAG_NONFINITE | FLAG_NEGMASS | FLAG_CELLCAP)) return;
    const unsigned ng = hdr->ngroups, ln = lane64(), w = threadIdx.x >> 6;
    const unsigned nblk = (ng + ACT_BLOCK - 1u) / ACT_BLOCK;
    for (unsigned blk = blockIdx.x; blk < nblk; blk += gridDim.x) {
        unsigned before = 0, all = 0;  // visited groups of the blocks before, of all blocks
        for (unsigned b = threadIdx.x; b < nblk; b += ACT_BLOCK) {
            const unsigned v = bcnt[b];
            all += v;
            before += b < blk ? v : 0u;
        }
#pragma unroll
        for (int o = 32; o > 0; o >>= 1) {
            before += __shfl_xor(before, o, 64);
            all += __shfl_xor(all, o, 64);
        }
        if (ln == 0) {
            s_sum[0][w] = before;
            s_sum[1][w] = all;
        }
        __syncthreads();
        before = all = 0;
        for (unsigned v = 0; v < ACT_BLOCK / 64; v++) {
            before += s_sum[0][v];
            all += s_sum[1][v];
        }
        __syncthreads();
        const unsigned g = blk * ACT_BLOCK + threadIdx.x;
        const bool mine = g < ng && gflag[g] != 0;
        const unsigned long long m = __ballot(mine);
        if (ln == 0) s_sum[0][w] = (unsigned)__popcll(m);
        __syncthreads();
        unsigned vis = before + rank_below(m);  // visited groups before g
        for (unsigned v = 0; v < w; v++) vis += s_sum[0][v];
        if (g < ng) order[mine ? vis : all + (g - vis)] = g;
        if (blk == 0 && threadIdx.x == 0) *qlen = all;
        __syncthreads();
    }
}

}  // namespace

// --------------------------------------------------------------------------
// Queue order: a stable counting sort of the groups by work bucket, heaviest
// bucket first.  work = count * 2^prediction (estimator) or
// count * (1 + n_pc + n_pp) (exact counts of the last walk); bucket =
// floor(4 log2 work), clamped to ORDER_BUCKETS values.  Block b owns a
// contiguous slice of the groups; the blocks' bucket counts, scanned
// bucket-major (heaviest first) then block-minor, place every group, and ranks
// inside a block are taken tile by tile in group order, so groups of equal
// bucket keep their Morton order.  Integer counts only: the order is the same
// on every run.
// --------------------------------------------------------------------------
namespace {

constexpr int ORDER_THREADS = 256;
constexpr int ORDER_SCAN_THREADS = 1024;
constexpr unsigned ORDER_SKIP = FLAG_NONFINITE | FLAG_NEGMASS | FLAG_CELLCAP;  // the walk does nothing then

struct OrderArgs {
    const Header *hdr;
    unsigned n_max;
    const uint2 *groups;
    const float *pred;       // mode 1
    const uint2 *counts;     // mode 2
    int mode;
};

// Queue bucket of group g: 0 for the heaviest work.
__device__ __forceinline__ unsigned work_bucket(const OrderArgs &o, unsigned g) {
    const uint2 gr = o.groups[g];
    const float gn = (float)(gr.y & 255u);
    const float *pred = o.pred;
    const uint2 *counts = o.counts;
    const int mode = o.mode;
    float l2;
    if (mode == 1) {
        const float p = pred[g];
        l2 = log2f(gn) + (isfinite(p) ? fminf(fmaxf(p, 0.0f), 40.0f) : 0.0f);
    } else {
        const uint2 c = counts[g];
        l2 = log2f(gn * (float)(1u + c.x + c.y));
    }
    const int b = min(max((int)floorf(4.0f * l2), 0), ORDER_BUCKETS - 1);
    return (unsigned)(ORDER_BUCKETS - 1 - b);
}

__device__ __forceinline__ void order_slice(const Header *hdr, unsigned n_max, unsigned *beg, unsigned *end) {
    const unsigned ng = min(hdr->ngroups, n_max);
    const unsigned chunk = (ng + ORDER_BLOCKS - 1) / ORDER_BLOCKS;
    *beg = min(ng, blockIdx.x * chunk);
    *end = min(ng, *beg + chunk);
}

__global__ __launch_bounds__(ORDER_THREADS) void k_order_hist(OrderArgs o, uint32_t *__restrict__ ohist) {
    __shared__ unsigned s_h[ORDER_BUCKETS];
    if (o.hdr->flags & ORDER_SKIP) return;
    const unsigned t = threadIdx.x;
    if (t < ORDER_BUCKETS) s_h[t] = 0;
    __syncthreads();
    unsigned beg, end;
    order_slice(o.hdr, o.n_max, &beg, &end);
    for (unsigned g = beg + t; g < end; g += ORDER_THREADS) atomicAdd(&s_h[work_bucket(o, g)], 1u);
    __syncthreads();
    if (t < ORDER_BUCKETS) ohist[t * ORDER_BLOCKS + blockIdx.x] = s_h[t];
}

// Exclusive prefix sum, in place, of ohist[ORDER_BUCKETS][ORDER_BLOCKS] read
// as one row-major sequence.  It skips with the histogram and scatter kernels.
__global__ __launch_bounds__(ORDER_SCAN_THREADS) void k_order_scan(const Header *__restrict__ hdr,
                                                                   uint32_t *__restrict__ ohist) {
    constexpr int PER = ORDER_BUCKETS * ORDER_BLOCKS / ORDER_SCAN_THREADS;
    static_assert(PER * ORDER_SCAN_THREADS == ORDER_BUCKETS * ORDER_BLOCKS, "scan covers the table");
    __shared__ unsigned s_w[ORDER_SCAN_THREADS / 64];
    if (hdr->flags & ORDER_SKIP) return;
    const unsigned t = threadIdx.x, ln = lane64(), w = t >> 6;
    unsigned v[PER], sum = 0;
#pragma unroll
    for (int i = 0; i < PER; i++) {
        v[i] = ohist[t * PER + i];
        sum += v[i];
    }
    unsigned x = sum;  // inclusive scan over the wave
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) {
        const unsigned y = __shfl_up(x, o, 64);
        x += ln >= (unsigned)o ? y : 0u;
    }
    if (ln == 63) s_w[w] = x;
    __syncthreads();
    unsigned run = x - sum;
    for (unsigned i = 0; i < w; i++) run += s_w[i];
#pragma unroll
    for (int i = 0; i < PER; i++) {
        ohist[t * PER + i] = run;
        run += v[i];
    }
}

__global__ __launch_bounds__(ORDER_THREADS) void k_order_scatter(OrderArgs o, const uint32_t *__restrict__ ohist,
                                                                 uint32_t *__restrict__ order) {
    constexpr int NW = ORDER_THREADS / 64;
    static_assert(NW * ORDER_BUCKETS == 2 * ORDER_THREADS, "two counters per thread to clear");
    __shared__ unsigned s_base[ORDER_BUCKETS];
    __shared__ unsigned s_wcnt[NW][ORDER_BUCKETS];
    if (o.hdr->flags & ORDER_SKIP) return;
    const unsigned t = threadIdx.x, w = t >> 6;
    if (t < ORDER_BUCKETS) s_base[t] = ohist[t * ORDER_BLOCKS + blockIdx.x];
    unsigned beg, end;
    order_slice(o.hdr, o.n_max, &beg, &end);
    // No branch below depends on the thread alone (see the walk's queue loop).
    for (unsigned t0 = beg; t0 < end; t0 += ORDER_THREADS) {
        (&s_wcnt[0][0])[t] = 0;
        (&s_wcnt[0][0])[t + ORDER_THREADS] = 0;
        __syncthreads();
        const unsigned g = t0 + t;
        const bool valid = g < end;
        const unsigned d = valid ? work_bucket(o, g) : 0u;
        // lanes of this wave with the same bucket
        unsigned long long peers = __ballot(valid);
#pragma unroll
        for (int bit = 0; bit < 7; bit++) {
            static_assert(ORDER_BUCKETS <= 128, "7-bit buckets");
            const unsigned long long m = __ballot((d >> bit) & 1u);
            peers &= ((d >> bit) & 1u) ? m : ~m;
        }
        const unsigned rank = rank_below(peers), cnt = (unsigned)__popcll(peers);
        const bool leader = valid && rank == 0;
        if (leader) s_wcnt[w][d] = cnt;
        __syncthreads();
        if (valid) {
            unsigned pos = s_base[d] + rank;
            for (unsigned w2 = 0; w2 < w; w2++) pos += s_wcnt[w2][d];
            order[pos] = g;
        }
        __syncthreads();
        if (leader) atomicAdd(&s_base[d], cnt);
        __syncthreads();
    }
}

}  // namespace

hipError_t launch_queue_order(const Buffers &b, int mode, const uint8_t *active, unsigned nsys, hipStream_t s) {
    if (mode == ORDER_MODE_ACTIVE) {
        // the number of visited groups goes where the counting sort would leave it
        const unsigned grid = min((b.n_max + ACT_BLOCK - 1u) / ACT_BLOCK, 1024u);
        hipLaunchKernelGGL(k_active_flag, dim3(grid), dim3(ACT_BLOCK), 0, s, b.hdr, b.groups, b.vals[0], active, b.gflag,
                           b.acnt);
        hipLaunchKernelGGL(k_active_queue, dim3(grid), dim3(ACT_BLOCK), 0, s, b.hdr, b.gflag, b.acnt, b.qorder,
                           b.ohist + ORDER_BLOCKS);
        return hipGetLastError();
    }
    OrderArgs o;
    o.hdr = b.hdr;
    o.n_max = b.n_max;
    o.groups = b.groups;
    o.pred = b.pred;
    o.counts = b.gcounts;
    o.mode = mode;
    hipLaunchKernelGGL(k_order_hist, dim3(ORDER_BLOCKS), dim3(ORDER_THREADS), 0, s, o, b.ohist);
    hipLaunchKernelGGL(k_order_scan, dim3(1), dim3(ORDER_SCAN_THREADS), 0, s, b.hdr, b.ohist);
    hipLaunchKernelGGL(k_order_scatter, dim3(ORDER_BLOCKS), dim3(ORDER_THREADS), 0, s, o, b.ohist, b.qorder);
    return hipGetLastError();
}

}  // namespace mibh
