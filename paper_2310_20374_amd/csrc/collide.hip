// Collision search on the candidate cell pairs of the collision walk (Alg. 2 with
// "do nothing" for well-separated cells) and the pair test of Sect. 3.1:
//   Delta = (dr.dv)^2 + dv^2 [(R1 + R2)^2 - dr^2]                      (Eq. 1)
//   dt_c  = -(dr.dv + sqrt(Delta)) / dv^2, collision iff 0 <= dt_c <= dt (Eq. 2)
// The arithmetic is FP64 with a fixed operation order and no contraction, and it is
// symmetric under swapping the two moonlets bit for bit (dr and dv only change
// sign), so the pair set is reproducible exactly.
#include "contact.h"

namespace ncorp {

// Value of lane `src` (the same for every lane of the wave) on all lanes: scalar
// reads, where a general shuffle would go through LDS permutes.
__device__ __forceinline__ int bcast_i(int v, int src) {
    return __builtin_amdgcn_readlane(v, src);
}
__device__ __forceinline__ double bcast_d(double v, int src) {
    const long long b = __double_as_longlong(v);
    const int lo = __builtin_amdgcn_readlane((int)(b & 0xffffffffll), src);
    const int hi = __builtin_amdgcn_readlane((int)(b >> 32), src);
    return __longlong_as_double(((long long)hi << 32) | (long long)(unsigned)lo);
}
__device__ __forceinline__ double4 bcast4(double4 v, int src) {
    return make_double4(bcast_d(v.x, src), bcast_d(v.y, src), bcast_d(v.z, src),
                        bcast_d(v.w, src));
}

__device__ __forceinline__ int wave_excl_sum_c(int v, int lane, int &total) {
    int x = v;
#pragma unroll
    for (int o = 1; o < kWave; o <<= 1) {
        const int t = __shfl_up(x, o);
        if (lane >= o) x += t;
    }
    total = __shfl(x, kWave - 1);
    return x - v;
}

// One wave per candidate cell pair.  B's moonlets are staged in LDS 64 at a time;
// A's moonlets sit on the lanes, and when A has fewer than 64 the lanes split
// B's moonlets into groups.  In a self pair only j > i is tested.
struct PState {
    double x, y, z, vx, vy, vz, R, reach;    // reach = R + dt |v|
    uint32_t id;
};

// A pair that touches at a time t in [0, dt] starts at most R_a + R_b + dt |v_a - v_b|
// <= reach_a + reach_b apart: the cheap distance check rejects nearly every pair before
// Eqs. (1)-(2) are evaluated (relative margin 1e-9, far above rounding).
__device__ __forceinline__ bool within_reach(const PState &a, const PState &b) {
    const double dx = a.x - b.x, dy = a.y - b.y, dz = a.z - b.z;
    const double rs = a.reach + b.reach;
    return dx * dx + dy * dy + dz * dz <= rs * rs * (1.0 + 1e-9);
}

// Colliding pairs a wave has found, listed together at its end (beyond kPairBuf one by
// one): an atomic on the pair count takes some 15 ns and holds up the wave's next loads, so
// one a pair bounded a search that finds many (66000 pairs at 4e6 clumped moonlets: 1256 ->
// 890 us).
constexpr int kPairBuf = 96;         // as much LDS as its allocation step leaves unused
struct PairOut {
    int64_t *out;
    int64_t cap;
    DevState *st;
    int64_t *buf;                        // LDS, kPairBuf keys
    int *n;                              // LDS, keys pushed
};

__device__ __forceinline__ void flush_pairs(const PairOut &P, int lane) {
    __syncthreads();
    const int n = *P.n < kPairBuf ? *P.n : kPairBuf;
    if (n == 0) return;
    unsigned long long base = 0;
    if (lane == 0) base = atomicAdd((unsigned long long *)&P.st->npairs, (unsigned long long)n);
    base = ((unsigned long long)__shfl((unsigned)(base >> 32), 0) << 32) |
           (unsigned)__shfl((unsigned)base, 0);
    for (int k = lane; k < n; k += kWave)
        if ((int64_t)base + k < P.cap) P.out[base + k] = P.buf[k];
}

__device__ __forceinline__ void test_pair(const PState &p, const PState &o, double dt,
                                          const PairOut &P) {
    if (within_reach(p, o) &&
        pair_test(p.x, p.y, p.z, p.vx, p.vy, p.vz, p.R, o.x, o.y, o.z, o.vx, o.vy, o.vz, o.R,
                  dt)) {
        const int k = atomicAdd(P.n, 1);
        if (k < kPairBuf) P.buf[k] = pair_key(p.id, o.id);
        else record(P.out, P.cap, (unsigned long long *)&P.st->npairs, p.id, o.id);
    }
}

// Can moonlet p = (x, y, z, R + dt |v|) meet a moonlet of the other cell within the
// step?  A pair that touches at a time t in [0, dt] starts at most R_a + R_b +
// dt (|v_a| + |v_b|) apart.  Spheres (BOXES = false, from the collision climb): the
// other cell's moonlets lie within r_crit - (R + dt |v|) of its centre, so
// |r_a - s| <= R_a + dt |v_a| + r_crit (a = centre, radius).  Boxes (BOXES = true):
// the other leaf's moonlets lie in the box [a.xyz, b.xyz], each with a reach of at
// most a.w, so the distance from r_a to the box is at most R_a + dt |v_a| + a.w.
// The relative margin 1e-9 dwarfs the rounding of either side, so no pair the exact
// test accepts is dropped.
template <bool BOXES>
__device__ __forceinline__ bool can_reach(const double4 &p, const double4 &a, const double4 &b) {
    if (BOXES) {
        const double gx = fmax(0.0, fmax(a.x - p.x, p.x - b.x));
        const double gy = fmax(0.0, fmax(a.y - p.y, p.y - b.y));
        const double gz = fmax(0.0, fmax(a.z - p.z, p.z - b.z));
        const double rs = p.w + a.w;
        return gx * gx + gy * gy + gz * gz <= rs * rs * (1.0 + 1e-9);
    }
    const double reach = p.w + a.w;
    const double dx = p.x - a.x, dy = p.y - a.y, dz = p.z - a.z;
    return dx * dx + dy * dy + dz * dz <= reach * reach * (1.0 + 1e-9);
}

// Moonlets of cell C (first f, count n) that can reach the other cell within the
// step (can_reach).  The survivors are compacted into out[] in moonlet order;
// returns their number, or -1 if more than `limit` survive.
template <bool BOXES>
__device__ __forceinline__ int cull_cell(int f, int n, double4 oa, double4 ob,
                                         const double4 *__restrict__ pcol,
                                         const double4 *__restrict__ vcol,
                                         const uint32_t *__restrict__ perm, PState *out,
                                         int limit) {
    const int lane = threadIdx.x;
    int kept = 0;
    for (int c0 = 0; c0 < n; c0 += kWave) {
        bool keep = false;
        PState ps;
        int k = 0;
        if (c0 + lane < n) {
            k = f + c0 + lane;
            // position and R + dt |v|, as the climb or the box pass stored them
            const double4 p = pcol[k];
            ps.x = p.x; ps.y = p.y; ps.z = p.z; ps.reach = p.w;
            keep = can_reach<BOXES>(p, oa, ob);
        }
        if (keep) {
            const double4 v = vcol[k];
            ps.vx = v.x; ps.vy = v.y; ps.vz = v.z; ps.R = v.w;
            ps.id = perm[k];
        }
        const uint64_t m = __ballot(keep);
        const int nk = __popcll(m);
        if (kept + nk > limit) return -1;
        const uint64_t lt = lane == 0 ? 0ull : (~0ull >> (64 - lane));
        if (keep) out[kept + __popcll(m & lt)] = ps;
        kept += nk;
    }
    return kept;
}

// All pairs of one cell of n <= 64 moonlets staged in sb: (i, i + d mod n) for
// d = 1 .. n/2 (for even n, d = n/2 only from i < n/2) is every unordered pair once.
// Lane groups of S >= n lanes take different d, so the rounds stay full instead of
// shrinking as i grows.
__device__ __forceinline__ void self_pairs_staged(int n, const PState *sb,
                                                  const double4 *spos, double dt,
                                                  const PairOut &P,
                                                  unsigned long long &tests) {
    const int lane = threadIdx.x;
    int S = 1;
    while (S < n) S <<= 1;
    const int G = kWave / S, i = lane % S, grp = lane / S, dmax = n / 2;
    if (i >= n) return;
    const PState me = sb[i];
    for (int d0 = 1; d0 <= dmax; d0 += G) {
        const int d = d0 + grp;
        if (d > dmax || (2 * d == n && i >= d)) continue;
        int j = i + d;
        if (j >= n) j -= n;
        tests++;
        const double4 o = spos[j];
        const double dx = me.x - o.x, dy = me.y - o.y, dz = me.z - o.z;
        const double rs = me.reach + o.w;
        if (dx * dx + dy * dy + dz * dz <= rs * rs * (1.0 + 1e-9)) test_pair(me, sb[j], dt, P);
    }
}

// Every moonlet pair of the candidate cell pair (A, B) (i < j when A == B): lanes
// take moonlets of A, B's moonlets are staged in LDS 64 at a time and split over
// lane groups when A holds fewer than 64.
__device__ __forceinline__ void test_cell_pair(
    int2 pr, PState *sb, double4 *spos, const int32_t *__restrict__ c_first,
    const int32_t *__restrict__ c_count, const uint32_t *__restrict__ perm,
    const double4 *__restrict__ pcol, const double4 *__restrict__ vcol, double dt,
    const PairOut &P, unsigned long long &tests) {
    const int lane = threadIdx.x;
    const int fa = c_first[pr.x], na = c_count[pr.x];
    const int fb = c_first[pr.y], nb = c_count[pr.y];
    const bool self = pr.x == pr.y;
    if (self && na <= kWave) {
        __syncthreads();
        if (lane < na) {
            const int b = fa + lane;
            PState ps;
            const double4 p = pcol[b], v = vcol[b];
            ps.x = p.x; ps.y = p.y; ps.z = p.z; ps.reach = p.w;
            ps.vx = v.x; ps.vy = v.y; ps.vz = v.z; ps.R = v.w;
            ps.id = perm[b];
            sb[lane] = ps;
            spos[lane] = p;
        }
        __syncthreads();
        self_pairs_staged(na, sb, spos, dt, P, tests);
        return;
    }
    for (int a0 = 0; a0 < na; a0 += 64) {
        const int nac = na - a0 < 64 ? na - a0 : 64;
        int S = 1;
        while (S < nac) S <<= 1;
        const int G = 64 / S, tl = lane % S, grp = lane / S;
        const bool act = tl < nac;
        const int ia = a0 + (act ? tl : 0);
        const int a = fa + ia;
        PState me;
        {
            const double4 p = pcol[a], v = vcol[a];
            me.x = p.x; me.y = p.y; me.z = p.z; me.reach = p.w;
            me.vx = v.x; me.vy = v.y; me.vz = v.z; me.R = v.w;
        }
        me.id = perm[a];
        for (int b0 = self ? a0 : 0; b0 < nb; b0 += 64) {
            const int nbc = nb - b0 < 64 ? nb - b0 : 64;
            __syncthreads();
            if (lane < nbc) {
                const int b = fb + b0 + lane;
                PState ps;
                const double4 p = pcol[b], v = vcol[b];
                ps.x = p.x; ps.y = p.y; ps.z = p.z; ps.reach = p.w;
                ps.vx = v.x; ps.vy = v.y; ps.vz = v.z; ps.R = v.w;
                ps.id = perm[b];
                sb[lane] = ps;
            }
            __syncthreads();
            if (!act) continue;
            const int jlo = self ? (ia + 1 - b0 > 0 ? ia + 1 - b0 : 0) : 0;
            // first j >= jlo with j = grp (mod G)
            int j = jlo + ((grp - jlo % G) % G + G) % G;
            for (; j < nbc; j += G) {
                tests++;
                test_pair(me, sb[j], dt, P);
            }
        }
    }
}

// candidate slots a wave reads at a time; the cell ranges and spheres of both
// sides of all of them are loaded in one go
constexpr int kCandRound = 8;
static_assert(kCandRegions == kWave && kWalkClasses == kWave, "a lane per counter line");

// BOXES: the candidates are leaf pairs with bounding boxes (cbox: low corner and
// largest reach, high corner, per cell); otherwise cell pairs with the collision
// climb's spheres (ccell).
template <bool BOXES>
__global__ void __launch_bounds__(64)
k_collide(DevState *st, const CandOut C, const int32_t *__restrict__ walk_ctr,
          int64_t visit_cap,
          const int32_t *__restrict__ c_first, const int32_t *__restrict__ c_count,
          const double4 *__restrict__ ccell, const double4 *__restrict__ cbox,
          const uint32_t *__restrict__ perm, const double4 *__restrict__ pcol,
          const double4 *__restrict__ vcol, const int32_t *__restrict__ ent_cell, double dt,
          int64_t *out, int64_t cap, unsigned long long *tests_part) {
    __shared__ PState sp[kWave];    // survivors of both sides (or a staged tile of B)
    __shared__ double4 spos[kWave];
    __shared__ int64_t pair_buf[kPairBuf];
    __shared__ int pair_n;
    const PairOut P = {out, cap, st, pair_buf, &pair_n};
    if (threadIdx.x == 0) pair_n = 0;
    if (st->status & kSkipMask) {
        if (threadIdx.x == 0) tests_part[blockIdx.x] = 0;
        return;
    }
    const int lane = threadIdx.x;
    if (!BOXES && blockIdx.x == 0) {
        // the collision walk's visits, summed over its classes
        unsigned long long v = *(const unsigned long long *)(walk_ctr + lane * kCtrStride +
                                                             kCtrVisited);
        for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o);
        if (lane == 0 && (int64_t)v > visit_cap) {
            atomicOr(&st->status, (int32_t)ST_CAP_QUEUE);
            atomicMax((unsigned long long *)&st->required, v);
        }
    }
    // lane k: the candidates of region k, in rounds of kCandRound slots
    const int my_len = C.ctr[lane * kCtrStride];
    int nround;
    const int my_rounds = (my_len + kCandRound - 1) / kCandRound;
    const int my_first = wave_excl_sum_c(my_rounds, lane, nround);
    const uint64_t lt = lane == 0 ? 0ull : (~0ull >> (64 - lane));
    unsigned long long tests = 0;
    for (int q = blockIdx.x; q < nround; q += gridDim.x) {
        // the region of round q: the last that starts at or before it and is not empty
        const int reg = __popcll(__ballot(my_first + my_rounds <= q));
        const int q0 = (q - __builtin_amdgcn_readlane(my_first, reg)) * kCandRound;
        const int len = __builtin_amdgcn_readlane(my_len, reg);
        int2 cq = make_int2(-1, -1);
        if (lane < kCandRound && q0 + lane < len) cq = C.list[(int64_t)reg * C.per + q0 + lane];
        // lane l < R: side A of candidate l (with B's sphere, for its cull); lane R + l:
        // side B (with A's sphere)
        const int src = lane < kCandRound ? lane : lane - kCandRound;
        const int qa = __shfl(cq.x, src & (kWave - 1)), qb = __shfl(cq.y, src & (kWave - 1));
        const bool side = lane < 2 * kCandRound && qa >= 0;
        const int mine = lane < kCandRound ? qa : qb, other = lane < kCandRound ? qb : qa;
        int cf = 0, cn = 0;
        double4 sph = make_double4(0.0, 0.0, 0.0, 0.0), shi = sph;
        if (side) {
            cf = c_first[mine];
            cn = c_count[mine];
            if (BOXES) {
                sph = cbox[2 * (int64_t)other];
                shi = cbox[2 * (int64_t)other + 1];
            } else {
                sph = ccell[other];
            }
        }
        uint64_t live = __ballot(lane < kCandRound && cq.x >= 0);   // gaps are skipped
        while (live) {
            const int l = __ffsll((unsigned long long)live) - 1;
            live &= live - 1;
            const int2 pr = make_int2(bcast_i(cq.x, l), bcast_i(cq.y, l));
            if (pr.x != pr.y) {
                // distinct cells: keep only moonlets that can reach the other cell
                const int lb = kCandRound + l;
                const int fa = bcast_i(cf, l), na = bcast_i(cn, l);
                const int fb = bcast_i(cf, lb), nb = bcast_i(cn, lb);
                int ka = -1, kb = -1;
                __syncthreads();
                if (BOXES && na + nb <= 2 * kWave) {
                    // both sides at once, two moonlets per lane (item t = lane, lane + 64
                    // is A[t] for t < na, else B[t - na]), whole records loaded together:
                    // one dependent round trip per candidate
                    const double4 oA = bcast4(sph, l), hA = bcast4(shi, l);
                    const double4 oB = bcast4(sph, lb), hB = bcast4(shi, lb);
                    PState ps[2];
                    bool keep[2], isA[2];
#pragma unroll
                    for (int u = 0; u < 2; u++) {
                        const int t = lane + u * kWave;
                        isA[u] = t < na;
                        keep[u] = false;
                        if (t < na + nb) {
                            const int k = isA[u] ? fa + t : fb + (t - na);
                            const double4 p = pcol[k], v = vcol[k];
                            ps[u].x = p.x; ps[u].y = p.y; ps[u].z = p.z; ps[u].reach = p.w;
                            ps[u].vx = v.x; ps[u].vy = v.y; ps[u].vz = v.z; ps[u].R = v.w;
                            ps[u].id = perm[k];
                            // an A moonlet is culled against B's box and the other way round
                            keep[u] = isA[u] ? can_reach<true>(p, oA, hA)
                                             : can_reach<true>(p, oB, hB);
                        }
                    }
                    const uint64_t mA0 = __ballot(keep[0] && isA[0]);
                    const uint64_t mA1 = __ballot(keep[1] && isA[1]);
                    const uint64_t mB0 = __ballot(keep[0] && !isA[0]);
                    const uint64_t mB1 = __ballot(keep[1] && !isA[1]);
                    const int a0 = __popcll(mA0), b0 = __popcll(mB0);
                    ka = a0 + __popcll(mA1);
                    kb = b0 + __popcll(mB1);
                    if (ka + kb <= kWave) {
                        if (keep[0])
                            sp[isA[0] ? __popcll(mA0 & lt) : ka + __popcll(mB0 & lt)] = ps[0];
                        if (keep[1])
                            sp[isA[1] ? a0 + __popcll(mA1 & lt) : ka + b0 + __popcll(mB1 & lt)] =
                                ps[1];
                    } else {
                        ka = kb = -1;
                    }
                } else if (na + nb <= kWave) {
                    // both sides in one round: lanes [0, na) hold A, [na, na + nb) hold B
                    const bool inA = lane < na, inB = !inA && lane < na + nb;
                    const int sl = inA ? l : lb;
                    const double4 s4 = make_double4(__shfl(sph.x, sl), __shfl(sph.y, sl),
                                                    __shfl(sph.z, sl), __shfl(sph.w, sl));
                    double4 h4 = s4;
                    if (BOXES)
                        h4 = make_double4(__shfl(shi.x, sl), __shfl(shi.y, sl),
                                          __shfl(shi.z, sl), 0.0);
                    bool keep = false;
                    int k = 0;
                    double4 p = make_double4(0.0, 0.0, 0.0, 0.0);
                    if (inA || inB) {
                        k = inA ? fa + lane : fb + (lane - na);
                        p = pcol[k];
                        keep = can_reach<BOXES>(p, s4, h4);
                    }
                    const uint64_t mA = __ballot(keep && inA), mB = __ballot(keep && inB);
                    ka = __popcll(mA);
                    kb = __popcll(mB);
                    if (keep) {
                        PState ps;
                        ps.x = p.x; ps.y = p.y; ps.z = p.z; ps.reach = p.w;
                        const double4 v = vcol[k];
                        ps.vx = v.x; ps.vy = v.y; ps.vz = v.z; ps.R = v.w;
                        ps.id = perm[k];
                        sp[inA ? __popcll(mA & lt) : ka + __popcll(mB & lt)] = ps;
                    }
                } else {
                    const double4 sA = bcast4(sph, l), sB = bcast4(sph, lb);
                    const double4 hA = bcast4(shi, l), hB = bcast4(shi, lb);
                    ka = cull_cell<BOXES>(fa, na, sA, hA, pcol, vcol, perm, sp, kWave);
                    kb = ka < 0 ? -1
                                : cull_cell<BOXES>(fb, nb, sB, hB, pcol, vcol, perm, sp + ka,
                                                   kWave - ka);
                }
                __syncthreads();
                if (ka >= 0 && kb >= 0) {
                    const int tot = ka * kb;
                    for (int t = lane; t < tot; t += kWave) {
                        tests++;
                        test_pair(sp[t / kb], sp[ka + t % kb], dt, P);
                    }
                    continue;
                }
            }
            test_cell_pair(pr, sp, spos, c_first, c_count, perm, pcol, vcol, dt, P, tests);
        }
    }
    if (BOXES) {
        // then every leaf with itself (the candidates hold distinct leaves only); blocks
        // that finish their candidates early start here, so both kinds of work overlap
        const int K = st->nleaves;
        for (int e = blockIdx.x; e < K; e += gridDim.x) {
            const int c = ent_cell[e];
            const int n = c_count[c];
            if (n < 2) continue;
            if (n > kWave) {
                test_cell_pair(make_int2(c, c), sp, spos, c_first, c_count, perm, pcol, vcol, dt,
                               P, tests);
                continue;
            }
            __syncthreads();
            if (lane < n) {
                const int k = c_first[c] + lane;
                const double4 p = pcol[k], v = vcol[k];
                PState ps;
                ps.x = p.x; ps.y = p.y; ps.z = p.z; ps.reach = p.w;
                ps.vx = v.x; ps.vy = v.y; ps.vz = v.z; ps.R = v.w;
                ps.id = perm[k];
                sp[lane] = ps;
                spos[lane] = p;
            }
            __syncthreads();
            self_pairs_staged(n, sp, spos, dt, P, tests);
        }
    }
    flush_pairs(P, lane);
    // per-block partials, summed by the pair ranking that follows: one atomic per wave
    // on a single counter would serialise all blocks of the grid
    for (int o = 32; o > 0; o >>= 1) tests += __shfl_xor(tests, o);
    if (lane == 0) tests_part[blockIdx.x] = tests;
}

// dst (+)= the sum of n partials, in a fixed order
__global__ void __launch_bounds__(1024)
k_sum_u64(const unsigned long long *__restrict__ part, int64_t n, unsigned long long *dst,
          int add) {
    __shared__ unsigned long long red[1024 / kWave];
    unsigned long long v = 0;
    for (int64_t i = threadIdx.x; i < n; i += 1024) v += part[i];
    for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o);
    if ((threadIdx.x & (kWave - 1)) == 0) red[threadIdx.x / kWave] = v;
    __syncthreads();
    if (threadIdx.x == 0) {
        unsigned long long t = 0;
        for (int k = 0; k < 1024 / kWave; k++) t += red[k];
        *dst = add ? *dst + t : t;
    }
}

hipError_t launch_sum_u64(const unsigned long long *part, int64_t n, unsigned long long *dst,
                          bool add, hipStream_t s) {
    k_sum_u64<<<1, 1024, 0, s>>>(part, n, dst, add ? 1 : 0);
    return hipGetLastError();
}

__global__ void k_collide_init(DevState *st) {
    if (threadIdx.x == 0 && blockIdx.x == 0) { st->npairs = 0; st->col_tests = 0; }
}

hipError_t launch_collide_reset(const Workspace &ws, hipStream_t s) {
    k_collide_init<<<1, 64, 0, s>>>(ws.st);
    return hipGetLastError();
}

// Rank sort of the (distinct) pair keys: rank = number of smaller keys.  Up to
// kRankDirect pairs by counting all of them: a block of
// kRankSplit waves takes 64 keys (a lane each); wave w counts the smaller keys in the
// w-th of kRankSplit equal segments of the list, walking it in chunks of 256 keys
// loaded coalesced (the next chunk while the current one is compared) and read back
// from LDS as wave-wide broadcasts; the block then adds the counts of its waves.
constexpr int kRankSplit = 8;
constexpr int kRankGrid = 512;     // 64 keys each up to kRankDirect, a range each beyond
constexpr int kRankSumBlocks = 16;   // blocks that also add up the pair-test counts
constexpr int kRankChunk = 4 * kWave;
// The resolution's per-pair start (when dtc is non-null): contact time (Eq. 2) of
// every ranked pair at its rank, its live flag, and its moonlets' matched flags cleared
struct RankResolve {
    const double *x, *y, *z, *vx, *vy, *vz, *R;
    double dt;
    double *dtc;
    int32_t *flag, *mmatch, *mbest;      // mbest: no earliest pair yet (-1)
};

// The report's output: pairs as (i, j), or (step, i, j) after the earlier steps' (triple)
struct RankReport {
    int64_t *pairs;                      // nullptr: none
    int64_t cap;
    const int64_t *cursor;
    int triple, step;
};

// What is done with the pair of key v and rank r.
__device__ __forceinline__ void ranked(int64_t v, int64_t r, int64_t *out,
                                       const RankResolve &RR, bool resolve,
                                       const RankReport &RP) {
    if (RP.pairs) {
        const int64_t o = (RP.triple ? *RP.cursor : 0) + r;
        if (o < RP.cap) {
            int64_t *q = RP.pairs + (RP.triple ? 3 : 2) * o;
            if (RP.triple) *q++ = RP.step;
            q[0] = v >> 32;
            q[1] = v & 0xffffffffll;
        }
        return;
    }
    out[r] = v;
    if (!resolve) return;
    const int a = (int)(v >> 32), b = (int)(v & 0xffffffffll);
    const double t = contact_time(RR.x[a], RR.y[a], RR.z[a], RR.vx[a], RR.vy[a], RR.vz[a], RR.R[a],
                                  RR.x[b], RR.y[b], RR.z[b], RR.vx[b], RR.vy[b], RR.vz[b],
                                  RR.R[b], RR.dt);
    RR.dtc[r] = t;
    RR.flag[r] = t >= 0.0 ? 1 : 0;
    RR.mmatch[a] = 0;
    RR.mmatch[b] = 0;
    RR.mbest[a] = -1;
    RR.mbest[b] = -1;
}

// Beyond kRankDirect pairs: block g of G ranks the keys between splitters g and g + 1 of a
// sorted sample of the list (four samples a block, the same sample and sort in every
// block).  It reads the whole list once, counts the keys below its range, gathers its own
// in LDS (about kRankOwn of them) and counts those against each other.  A range of more
// than kRankRoom keys (a list of millions, or an uneven sample) is gathered in memory, in
// the block's part of a buffer of the list's size, counted against itself by way of LDS
// and ranked in place.  Counting all against all took 946 us for the 66000 pairs of 4e6
// clumped moonlets, this 95.
constexpr int64_t kRankDirect = 4096;
constexpr int kRankOwn = 512, kRankSamples = 2048, kRankRoom = 4096;
constexpr int kRankHeld = 8;         // keys a thread counts at a time, of a large range
union RankLds {
    struct {
        int64_t tile[kRankSplit][kRankChunk];
        int64_t part[kRankSplit][kWave];
    } d;
    struct {
        int64_t sample[kRankSamples];
        int64_t own[kRankRoom];
        int nown;
        unsigned long long below;
    } l;
};

__device__ __forceinline__ void rank_long(int64_t n, const int64_t *__restrict__ in,
                                          int64_t *out, int64_t *tmp, RankLds &lds,
                                          const RankResolve &RR, bool resolve,
                                          const RankReport &RP) {
    constexpr int T = kWave * kRankSplit;
    int G = 1;                                    // ranges: a power of two
    while (G < (int)gridDim.x && G < kRankSamples / 4 && (int64_t)G * kRankOwn < n) G <<= 1;
    if (G > (int)gridDim.x) G >>= 1;
    const int g = blockIdx.x, t = threadIdx.x;
    if (g >= G) return;
    const int S = 4 * G;                          // <= kRankSamples
    for (int k = t; k < S; k += T) lds.l.sample[k] = in[(int64_t)k * n / S];
    if (t == 0) { lds.l.nown = 0; lds.l.below = 0; }
    __syncthreads();
    for (int k = 2; k <= S; k <<= 1)              // bitonic, ascending
        for (int j = k >> 1; j > 0; j >>= 1) {
            for (int q = t; q < S / 2; q += T) {
                const int a = 2 * q - (q & (j - 1)), b = a + j;
                const int64_t va = lds.l.sample[a], vb = lds.l.sample[b];
                if ((vb < va) == ((a & k) == 0)) { lds.l.sample[a] = vb; lds.l.sample[b] = va; }
            }
            __syncthreads();
        }
    // keys in [lo, hi): distinct keys, so distinct splitters
    const int64_t lo = g == 0 ? INT64_MIN : lds.l.sample[4 * g];
    const int64_t hi = g == G - 1 ? INT64_MAX : lds.l.sample[4 * (g + 1)];
    unsigned long long below = 0;
    constexpr int U = 4;
    for (int64_t q0 = t; q0 < n; q0 += U * T) {
        int64_t v[U];
#pragma unroll
        for (int u = 0; u < U; u++) v[u] = q0 + u * T < n ? in[q0 + u * T] : INT64_MAX;
#pragma unroll
        for (int u = 0; u < U; u++) {
            below += v[u] < lo ? 1 : 0;
            if (v[u] >= lo && v[u] < hi) {
                const int at = atomicAdd(&lds.l.nown, 1);
                if (at < kRankRoom) lds.l.own[at] = v[u];
            }
        }
    }
    for (int o = kWave / 2; o > 0; o >>= 1) below += __shfl_xor(below, o);
    if (t % kWave == 0) atomicAdd(&lds.l.below, below);
    __syncthreads();
    const int m = lds.l.nown;
    const int64_t base = (int64_t)lds.l.below;
    if (m <= kRankRoom) {
        for (int a = t; a < m; a += T) {
            const int64_t v = lds.l.own[a];
            int rk = 0;
            for (int k = 0; k < m; k++) rk += lds.l.own[k] < v;
            ranked(v, base + rk, out, RR, resolve, RP);
        }
        return;
    }
    // ranks base .. base + m - 1 are this block's: so are those places of tmp and out
    int64_t *keys = tmp + base, *sorted = out + base;
    __syncthreads();
    if (t == 0) lds.l.nown = 0;
    __syncthreads();
    for (int64_t q = t; q < n; q += T) {
        const int64_t v = in[q];
        if (v >= lo && v < hi) keys[atomicAdd(&lds.l.nown, 1)] = v;
    }
    __syncthreads();
    for (int64_t a0 = 0; a0 < m; a0 += kRankHeld * T) {
        int64_t v[kRankHeld];
        int rk[kRankHeld];
#pragma unroll
        for (int u = 0; u < kRankHeld; u++) {
            const int64_t a = a0 + u * T + t;
            v[u] = a < m ? keys[a] : INT64_MIN;          // (none below it)
            rk[u] = 0;
        }
        for (int k0 = 0; k0 < m; k0 += kRankRoom) {
            const int len = m - k0 < kRankRoom ? m - k0 : kRankRoom;
            __syncthreads();
            for (int k = t; k < len; k += T) lds.l.own[k] = keys[k0 + k];
            __syncthreads();
            for (int k = 0; k < len; k++) {
                const int64_t w = lds.l.own[k];
#pragma unroll
                for (int u = 0; u < kRankHeld; u++) rk[u] += w < v[u];
            }
        }
#pragma unroll
        for (int u = 0; u < kRankHeld; u++)
            if (a0 + u * T + t < m) sorted[rk[u]] = v[u];
    }
    __syncthreads();
    for (int64_t a = t; a < m; a += T) ranked(sorted[a], base + a, out, RR, resolve, RP);
}

__global__ void __launch_bounds__(kWave * kRankSplit)
k_rank_pairs(DevState *__restrict__ st, const int64_t *__restrict__ in, int64_t cap,
             int64_t *out, int64_t *tmp, const unsigned long long *__restrict__ tests_part,
             int n_part, const RankResolve RR, const RankReport RP,
             int32_t *__restrict__ walk_ctr) {
    __shared__ RankLds lds;
    auto &tile_all = lds.d.tile;
    auto &part = lds.d.part;
    // the next search's reaches start at zero
    if (blockIdx.x == 0 && threadIdx.x < kWalkClasses)
        *(double *)(walk_ctr + threadIdx.x * kCtrStride + kCtrReach) = 0.0;
    const int sum_b = (int)blockIdx.x - ((int)gridDim.x - kRankSumBlocks);
    if (tests_part && sum_b >= 0) {
        // the pair tests' per-block counts, summed by the last kRankSumBlocks blocks
        // (which have no keys to rank unless the list is long), one integer atomic each
        const int per = (n_part + kRankSumBlocks - 1) / kRankSumBlocks;
        const int i0 = sum_b * per, i1 = i0 + per < n_part ? i0 + per : n_part;
        unsigned long long v = 0;
        for (int i = i0 + threadIdx.x; i < i1; i += blockDim.x) v += tests_part[i];
        for (int o = kWave / 2; o > 0; o >>= 1) v += __shfl_xor(v, o);
        unsigned long long *red = (unsigned long long *)&part[0][0];
        __syncthreads();
        if ((threadIdx.x & (kWave - 1)) == 0) red[threadIdx.x / kWave] = v;
        __syncthreads();
        if (threadIdx.x == 0) {
            unsigned long long t = 0;
            for (int k = 0; k < (int)blockDim.x / kWave; k++) t += red[k];
            atomicAdd((unsigned long long *)&st->col_tests, t);
        }
        __syncthreads();
    }
    int64_t n = st->npairs;
    // the resolution takes no pair of an overflowed list or after a failed pass
    const bool resolve = RR.dtc && n <= cap && !(st->status & kSkipMask);
    if (n > cap) n = cap;
    if (n > kRankDirect) {
        // (tmp is the contact times' buffer: a block's places there are its own, and it
        // writes its contact times after its last use of them)
        rank_long(n, in, out, tmp, lds, RR, resolve, RP);
        return;
    }
    const int lane = threadIdx.x % kWave, w = threadIdx.x / kWave;
    int64_t *tile = tile_all[w];
    // this wave's segment of the list
    const int64_t seg = (n + kRankSplit - 1) / kRankSplit;
    const int64_t s0 = seg * w < n ? seg * w : n;
    const int64_t s1 = s0 + seg < n ? s0 + seg : n;
    for (int64_t base = (int64_t)blockIdx.x * kWave; base < n; base += (int64_t)gridDim.x * kWave) {
        const int64_t i = base + lane;
        const int64_t v = i < n ? in[i] : INT64_MAX;
        int64_t r0 = 0, r1 = 0;
        int64_t nxt[4];
#pragma unroll
        for (int u = 0; u < 4; u++) {
            const int64_t q = s0 + u * kWave + lane;
            nxt[u] = q < s1 ? in[q] : INT64_MAX;
        }
        for (int64_t t0 = s0; t0 < s1; t0 += kRankChunk) {
            wave_sync();
#pragma unroll
            for (int u = 0; u < 4; u++) tile[u * kWave + lane] = nxt[u];
            wave_sync();
            const int64_t t1 = t0 + kRankChunk;
#pragma unroll
            for (int u = 0; u < 4; u++) {
                const int64_t q = t1 + u * kWave + lane;
                nxt[u] = q < s1 ? in[q] : INT64_MAX;
            }
            // padding keys (INT64_MAX) are never below a real key
#pragma unroll 8
            for (int k = 0; k < kRankChunk; k += 2) {
                r0 += tile[k] < v;
                r1 += tile[k + 1] < v;
            }
        }
        part[w][lane] = r0 + r1;
        __syncthreads();
        if (w == 0 && i < n) {
            int64_t r = 0;
#pragma unroll
            for (int k = 0; k < kRankSplit; k++) r += part[k][lane];
            ranked(v, r, out, RR, resolve, RP);
        }
        __syncthreads();
    }
}

__global__ void k_pairs_done(DevState *st, int64_t *n_pairs_dev, int64_t cap, int64_t tmp_cap,
                             int triple, int64_t *cursor) {
    if (threadIdx.x != 0 || blockIdx.x != 0) return;
    int64_t n = st->npairs;
    *n_pairs_dev = n;
    int64_t base = triple ? *cursor : 0;
    if (n > tmp_cap || base + n > cap) {
        atomicOr(&st->status, (int32_t)ST_CAP_PAIRS);
        atomicMax((unsigned long long *)&st->required, (unsigned long long)(base + n));
    }
    if (triple) *cursor = base + n;
}
// ---------------------------------------------------------------- candidates from lists
// Collision candidates from the gravity walk's lists of the same tree (each leaf's
// direct-sum sources, and the M2L partners of the leaf and its ancestors).  Those lists
// cover every moonlet pair exactly once from either side, so the leaf pairs below their
// entries, minus those that provably cannot collide, are candidates covering every
// colliding pair once: the pair set is the collision walk's.  A pair that touches
// within the step starts at most R_a + R_b + dt (|v_a| + |v_b|) apart, so two leaves can
// hold a colliding pair only if their bounding boxes (the tight boxes of their moonlets,
// k_leaf_boxes), each grown by its largest R + dt |v|, overlap.  The pairs inside each
// leaf are searched apart from the candidates (by k_collide, after them).
struct CBox {
    double lx, ly, lz, hx, hy, hz, r;
};

__device__ __forceinline__ bool boxes_meet(const CBox &a, const CBox &b) {
    const double gx = fmax(0.0, fmax(b.lx - a.hx, a.lx - b.hx));
    const double gy = fmax(0.0, fmax(b.ly - a.hy, a.ly - b.hy));
    const double gz = fmax(0.0, fmax(b.lz - a.hz, a.lz - b.hz));
    const double rs = (a.r + b.r) * (1.0 + 1e-9);
    return gx * gx + gy * gy + gz * gz <= rs * rs;
}

__device__ __forceinline__ CBox leaf_box(const double4 *__restrict__ cbox, int c) {
    const double4 lo = cbox[2 * (int64_t)c], hi = cbox[2 * (int64_t)c + 1];
    return CBox{lo.x, lo.y, lo.z, hi.x, hi.y, hi.z, lo.w};
}

// One wave per leaf: every moonlet's (x, y, z, R + dt |v|) record for the culling, the
// tight box of the leaf's moonlets with their largest R + dt |v|, and the largest of
// all moonlets (for the M2L lists), as maxima on the 64 counter lines, which the walk's init
// or the last search's ranking left at zero: a line takes a few hundred atomics at most
// (16384 waves), some 4 us among the other work, where a block adding up partial maxima took
// 5 to 7 us in a launch of its own.  The pair, test and candidate counts of the search
// start here.
__global__ void __launch_bounds__(kWave)
k_leaf_boxes(DevState *st, const double *__restrict__ xs, const double *__restrict__ ys,
             const double *__restrict__ zs, const double4 *__restrict__ pack4,
             const uint32_t *__restrict__ perm, double dt, const int32_t *__restrict__ ent_cell,
             const int32_t *__restrict__ c_first, const int32_t *__restrict__ c_count,
             double4 *__restrict__ cbox, double4 *__restrict__ pcol,
             double4 *__restrict__ vcol, int32_t *__restrict__ walk_ctr,
             int32_t *__restrict__ cand_ctr) {
    if (blockIdx.x == 0) {
        if (threadIdx.x == 0) { st->npairs = 0; st->col_tests = 0; }
        cand_ctr[threadIdx.x * kCtrStride] = 0;
        if (threadIdx.x == 0) cand_ctr[kCandRefused] = 0;
    }
    if (st->status & kSkipMask) return;
    const int K = st->nleaves;
    const int lane = threadIdx.x;
    double wmax = 0.0;
    for (int e = blockIdx.x; e < K; e += gridDim.x) {
        const int c = ent_cell[e];
        const int f = c_first[c], cnt = c_count[c];
        double lx = INFINITY, ly = INFINITY, lz = INFINITY;
        double hx = -INFINITY, hy = -INFINITY, hz = -INFINITY, ex = 0.0;
        for (int c0 = lane; c0 < cnt; c0 += kWave) {
            const int k = f + c0;
            const double x = xs[k], y = ys[k], z = zs[k];
            const double4 w = pack4[perm[k]];          // (vx, vy, vz, R), input order
            const double v = sqrt(w.x * w.x + w.y * w.y + w.z * w.z);
            const double ee = (w.w + dt * v) - 0.0;
            pcol[k] = make_double4(x, y, z, ee);
            vcol[k] = w;
            lx = fmin(lx, x); ly = fmin(ly, y); lz = fmin(lz, z);
            hx = fmax(hx, x); hy = fmax(hy, y); hz = fmax(hz, z);
            ex = fmax(ex, ee);
        }
        for (int o = kWave / 2; o > 0; o >>= 1) {
            lx = fmin(lx, __shfl_xor(lx, o)); ly = fmin(ly, __shfl_xor(ly, o));
            lz = fmin(lz, __shfl_xor(lz, o));
            hx = fmax(hx, __shfl_xor(hx, o)); hy = fmax(hy, __shfl_xor(hy, o));
            hz = fmax(hz, __shfl_xor(hz, o));
            ex = fmax(ex, __shfl_xor(ex, o));
        }
        if (lane == 0) {
            cbox[2 * (int64_t)c] = make_double4(lx, ly, lz, ex);
            cbox[2 * (int64_t)c + 1] = make_double4(hx, hy, hz, 0.0);
        }
        wmax = fmax(wmax, ex);
    }
    // reaches are >= 0, so their bit patterns order like the values
    if (lane == 0 && wmax > 0.0)
        atomicMax((unsigned long long *)(walk_ctr + blockIdx.x % kWalkClasses * kCtrStride +
                                         kCtrReach),
                  (unsigned long long)__double_as_longlong(wmax));
}

// waves of the box pass: 16384, or one per leaf slot of a small tree
constexpr int kBoxGrid = 16384;

hipError_t launch_leaf_boxes(const Workspace &ws, int64_t n, double dt, hipStream_t s) {
    (void)n;
    const int64_t g = ws.leaf_cap < kBoxGrid ? ws.leaf_cap : kBoxGrid;
    k_leaf_boxes<<<(int)g, kWave, 0, s>>>(ws.st, ws.xs, ws.ys, ws.zs, ws.pack4, ws.idx, dt,
                                          ws.ent_cell, ws.c_first, ws.c_count,
                                          ws.cbox, ws.pcol, ws.vcol, ws.walk_ctr, cand_out(ws).ctr);
    return hipGetLastError();
}

struct CandArgs {
    const DevState *st;
    const double4 *cbox;
    const double4 *gcell;                // gravity climb: centre of mass
    const double *c_rmax;                // bounds every moonlet's distance from it
    const WCell *wg;
    const int32_t *ent_cell, *c_nent, *c_entry;
    const int32_t *p2p_cnt, *p2p_seg, *m2l_cnt, *m2l_seg;
    int p2p_stride, m2l_stride;
    const float *leaf_slack;
    const uint16_t *seg;                 // batched: disk of every tree position, else nullptr
    const double *disk_L;
    const int32_t *walk_ctr;
};

// The candidate leaf pairs (c, l), l later than c in leaf order, below the lanes' list
// entries B (-1: none): the leaves of B whose box meets that of the wave's leaf c.
__device__ __forceinline__ void emit_leaves(const CandArgs &A, int c, int e, const CBox &box,
                                            int B, int lane, int2 *buf, int &nb, int cls,
                                            const CandOut &C, DevState *st) {
    const uint64_t lt = lane == 0 ? 0ull : (~0ull >> (64 - lane));
    int eb = 0, left = 0;
    if (B >= 0) {
        eb = A.c_entry[B];
        left = A.c_nent[B];
        if (eb <= e) {                   // only leaves after e: each pair once
            left -= e + 1 - eb;
            eb = e + 1;
        }
    }
    while (__any(left > 0)) {
        bool take = false;
        int l = 0;
        if (left > 0) {
            l = A.ent_cell[eb];
            take = boxes_meet(box, leaf_box(A.cbox, l));
            eb++;
            left--;
        }
        const uint64_t m = __ballot(take);
        if (!m) continue;
        if (take) buf[nb + __popcll(m & lt)] = make_int2(c, l);
        nb += __popcll(m);
        if (nb > kCandBuf - kWave) flush_cand(buf, nb, lane, cls, C, st);
    }
}

constexpr int kCandWaves = 4;            // independent waves per block
constexpr int kCandGrid = 2048;

// One wave per leaf.  Its direct-sum sources give nearly all candidates.  A
// well-separated pair lies at least slack_A + slack_B apart (slack = r_crit - r_max), so
// the M2L lists of a leaf's chain matter only where the chain's smallest slack (formed
// by the walk) is within twice the largest reach of any moonlet; 23 + 9 + 31 us of
// count, scan and write passes over the cell-pair lists took 63 us before at N = 1e6.
__global__ void __launch_bounds__(kWave * kCandWaves)
k_cand_leaves(DevState *st, const CandArgs A, const CandOut C) {
    __shared__ int2 bufs[kCandWaves][kCandBuf];
    if (st->status & kSkipMask) return;
    const int lane = threadIdx.x % kWave, wid = threadIdx.x / kWave;
    int2 *const buf = bufs[wid];
    const int cls = (int)blockIdx.x % kCandRegions;
    const int K = st->nleaves;
    // the largest reach of all moonlets: a line a lane
    double r = *(const double *)(A.walk_ctr + lane * kCtrStride + kCtrReach);
    for (int o = kWave / 2; o > 0; o >>= 1) r = fmax(r, __shfl_xor(r, o));
    int nb = 0;
    for (int e = blockIdx.x * kCandWaves + wid; e < K; e += gridDim.x * kCandWaves) {
        const int c = A.ent_cell[e];
        const CBox box = leaf_box(A.cbox, c);
        const int np = A.p2p_cnt[e];
        const float slack = A.leaf_slack[e];
        const int32_t *row = A.p2p_seg + (int64_t)e * A.p2p_stride;
        for (int q = lane; q - lane < np; q += kWave)
            emit_leaves(A, c, e, box, q < np ? row[q] : -1, lane, buf, nb, cls, C, st);
        const double L = A.seg ? A.disk_L[A.seg[A.wg[c].first]] : st->L;
        const double far = 2.0 * r * (1.0 + 1e-6) + 1e-12 * L;
        if ((double)slack > far) continue;
        for (int a = c; a >= 0;) {
            const WCell wa = A.wg[a];
            const int up = wa.parent;
            if (wa.rcrit - A.c_rmax[a] <= far) {
                const int nm = A.m2l_cnt[a];
                const int32_t *mrow = A.m2l_seg + (int64_t)a * A.m2l_stride;
                for (int q = lane; q - lane < nm; q += kWave) {
                    int B = q < nm ? mrow[q] : -1;
                    if (B >= 0) {
                        // B's moonlets lie within r_max of its centre of mass
                        const double4 g = A.gcell[B];
                        const double gx = fmax(0.0, fmax(box.lx - g.x, g.x - box.hx));
                        const double gy = fmax(0.0, fmax(box.ly - g.y, g.y - box.hy));
                        const double gz = fmax(0.0, fmax(box.lz - g.z, g.z - box.hz));
                        const double rs = (A.c_rmax[B] + box.r + r) * (1.0 + 1e-9);
                        if (gx * gx + gy * gy + gz * gz > rs * rs) B = -1;
                    }
                    if (__any(B >= 0)) emit_leaves(A, c, e, box, B, lane, buf, nb, cls, C, st);
                }
            }
            a = up;
        }
    }
    flush_cand(buf, nb, lane, cls, C, st);
}

hipError_t launch_candidates_from_lists(const Workspace &ws, hipStream_t s) {
    int64_t g = (ws.leaf_cap + kCandWaves - 1) / kCandWaves;
    if (g > kCandGrid) g = kCandGrid;
    CandArgs A;
    A.st = ws.st; A.cbox = ws.cbox; A.gcell = ws.gcell; A.c_rmax = ws.c_rmax; A.wg = ws.wg;
    A.ent_cell = ws.ent_cell; A.c_nent = ws.c_nent; A.c_entry = ws.c_entry;
    A.p2p_cnt = ws.p2p_cnt; A.p2p_seg = ws.p2p_seg; A.m2l_cnt = ws.m2l_cnt; A.m2l_seg = ws.m2l_seg;
    A.p2p_stride = ws.p2p_stride; A.m2l_stride = ws.m2l_stride;
    A.leaf_slack = ws.leaf_slack;
    A.seg = ws.ndisks > 1 ? ws.seg : nullptr;
    A.disk_L = ws.disk_L;
    A.walk_ctr = ws.walk_ctr;
    k_cand_leaves<<<(int)g, kWave * kCandWaves, 0, s>>>(ws.st, A, cand_out(ws));
    return hipGetLastError();
}

// ---------------------------------------------------------------- resolution
// Hard-sphere resolution of the pairs found (Sect. 5.1-5.2), one block.  Pairs are
// taken in increasing (dt_c, i, j) and a moonlet collides at most once per step:
// this greedy matching is reached in rounds, each accepting every live pair that
// is the earliest live pair of both its moonlets (the earliest live pair of all is
// always one, so every round makes progress) and dropping the live pairs that
// touch a moonlet just matched -- the same set as taking the pairs one by one.
// Each round visits only the pairs still live.
// The pair list is sorted by (i, j), so its index breaks ties of dt_c.
__device__ __forceinline__ bool earlier(const double *dtc, int p, int q) {
    return dtc[p] < dtc[q] || (dtc[p] == dtc[q] && p < q);
}

__device__ __forceinline__ void keep_earliest(int32_t *slot, int p, const double *dtc) {
    int cur = *slot;
    while (cur < 0 || earlier(dtc, p, cur)) {
        const int old = atomicCAS(slot, cur, p);
        if (old == cur) break;
        cur = old;
    }
}

constexpr int kResolveThreads = 1024;
constexpr int kResolveBlocks = 32;     // most blocks of the matching's first half round
constexpr int kResolveGrid = 512;      // blocks of the per-pair passes

// exclusive prefix of v >= 0 over the block (wsum: one word per wave), and the
// block's total
__device__ __forceinline__ int block_int_prefix(int v, int *wsum, int *total) {
    const int lane = threadIdx.x % kWave, w = threadIdx.x / kWave;
    int x = v;
#pragma unroll
    for (int o = 1; o < kWave; o <<= 1) {
        const int y = __shfl_up(x, o);
        if (lane >= o) x += y;
    }
    if (lane == kWave - 1) wsum[w] = x;
    __syncthreads();
    int before = 0, tot = 0;
    for (int k = 0; k < (int)blockDim.x / kWave; k++) {
        if (k < w) before += wsum[k];
        tot += wsum[k];
    }
    __syncthreads();
    *total = tot;
    return before + x - v;
}

__device__ __forceinline__ int pair_i(int64_t key) { return (int)(key >> 32); }
__device__ __forceinline__ int pair_j(int64_t key) { return (int)(key & 0xffffffffll); }

// pairs per thread and pass of the one-block rounds
constexpr int kResolveUnroll = 4;

// number of pairs the resolution takes: 0 when the list overflowed (the status then
// says so) or an earlier pass failed
__device__ __forceinline__ int resolve_count(const DevState *st, int64_t pair_cap) {
    const int64_t np = st->npairs;
    if (np > pair_cap || (st->status & kSkipMask)) return 0;
    return (int)np;                       // pair indices are 32-bit (the capacity is)
}

// The rounds of the matching and the list of resolved pairs.  Every live pair's bid for
// its two moonlets in the first round, which has by far the most pairs, is spread over as
// many blocks as there are 4096 pairs; the last of them to finish goes on alone (nobody
// waits).  The ranking left the moonlets' slots empty.  66000 pairs: 1404 us in one block
// from the start, 655 now.
__global__ void __launch_bounds__(kResolveThreads)
k_resolve(DevState *st, const int64_t *__restrict__ keys, int64_t pair_cap,
          const double *__restrict__ dtc, int32_t *flag, int32_t *mbest, int32_t *mmatch,
          int32_t *live, int64_t *pairs, int64_t cap, int64_t *n_pairs_dev, int step,
          int64_t *cursor) {
    constexpr int U = kResolveUnroll;
    __shared__ int wsum[kResolveThreads / kWave];
    __shared__ int last;
    const int tid = threadIdx.x;
    const int T = blockDim.x;
    const int np = resolve_count(st, pair_cap);
    int blocks = (np + U * T - 1) / (U * T);
    blocks = blocks < 1 ? 1 : (blocks > (int)gridDim.x ? (int)gridDim.x : blocks);
    if ((int)blockIdx.x >= blocks) return;
    // flag: 0 dropped, 1 live, 2 resolved
    for (int c0 = blockIdx.x * U * T; c0 < np; c0 += blocks * U * T)
#pragma unroll
        for (int u = 0; u < U; u++) {
            const int p = c0 + u * T + tid;
            if (p < np && flag[p] == 1) {
                const int64_t k = keys[p];
                keep_earliest(&mbest[pair_i(k)], p, dtc);
                keep_earliest(&mbest[pair_j(k)], p, dtc);
            }
        }
    if (blocks > 1) {
        __threadfence();
        __syncthreads();
        if (tid == 0) last = atomicAdd(&st->resolve_done, 1) == blocks - 1 ? 1 : 0;
        __syncthreads();
        if (!last) return;
        __threadfence();
        if (tid == 0) st->resolve_done = 0;
    }
    if (st->npairs > pair_cap && !(st->status & kSkipMask) && tid == 0) {
        // the list is incomplete: nothing is resolved
        atomicOr(&st->status, (int32_t)ST_CAP_PAIRS);
        atomicMax((unsigned long long *)&st->required, (unsigned long long)st->npairs);
    }
    __syncthreads();
    // the first round's matches; the pairs still live after it are then kept compacted in
    // `live`, so later rounds visit only what is left
    for (int c0 = 0; c0 < np; c0 += U * T)
#pragma unroll
        for (int u = 0; u < U; u++) {
            const int p = c0 + u * T + tid;
            if (p < np && flag[p] == 1) {
                const int64_t k = keys[p];
                const int i = pair_i(k), j = pair_j(k);
                // (other blocks wrote the slots)
                if (__hip_atomic_load(&mbest[i], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) == p &&
                    __hip_atomic_load(&mbest[j], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) == p) {
                    flag[p] = 2;
                    mmatch[i] = 1;
                    mmatch[j] = 1;
                }
            }
        }
    __syncthreads();
    int nlive = 0;
    for (int c0 = 0; c0 < np; c0 += U * T) {
        int cnt = 0;
        bool ok[U];
#pragma unroll
        for (int u = 0; u < U; u++) {
            const int p = c0 + U * tid + u;
            ok[u] = false;
            if (p < np && flag[p] == 1) {
                const int64_t k = keys[p];
                if (mmatch[pair_i(k)] || mmatch[pair_j(k)]) flag[p] = 0;
                else ok[u] = true;
            }
            cnt += ok[u] ? 1 : 0;
        }
        int tot;
        int o = nlive + block_int_prefix(cnt, wsum, &tot);
#pragma unroll
        for (int u = 0; u < U; u++)
            if (ok[u]) live[o++] = c0 + U * tid + u;
        nlive += tot;
    }
    __syncthreads();
    while (nlive > 0) {
        for (int c0 = 0; c0 < nlive; c0 += U * T)
#pragma unroll
            for (int u = 0; u < U; u++) {
                const int q = c0 + u * T + tid;
                if (q < nlive) {
                    const int64_t k = keys[live[q]];
                    mbest[pair_i(k)] = -1;
                    mbest[pair_j(k)] = -1;
                }
            }
        __syncthreads();
        for (int c0 = 0; c0 < nlive; c0 += U * T)
#pragma unroll
            for (int u = 0; u < U; u++) {
                const int q = c0 + u * T + tid;
                if (q < nlive) {
                    const int p = live[q];
                    const int64_t k = keys[p];
                    keep_earliest(&mbest[pair_i(k)], p, dtc);
                    keep_earliest(&mbest[pair_j(k)], p, dtc);
                }
            }
        __syncthreads();
        for (int c0 = 0; c0 < nlive; c0 += U * T)
#pragma unroll
            for (int u = 0; u < U; u++) {
                const int q = c0 + u * T + tid;
                if (q < nlive) {
                    const int p = live[q];
                    const int64_t k = keys[p];
                    const int i = pair_i(k), j = pair_j(k);
                    if (mbest[i] == p && mbest[j] == p) {
                        flag[p] = 2;
                        mmatch[i] = 1;
                        mmatch[j] = 1;
                    }
                }
            }
        __syncthreads();
        // drop what touches a moonlet just matched; compact the rest in place (a pass
        // reads all its entries before any is written, and writes only below them)
        int kept = 0;
        for (int c0 = 0; c0 < nlive; c0 += U * T) {
            bool keep[U];
            int pv[U];
#pragma unroll
            for (int u = 0; u < U; u++) {
                const int q = c0 + u * T + tid;
                keep[u] = false;
                pv[u] = 0;
                if (q < nlive) {
                    pv[u] = live[q];
                    if (flag[pv[u]] == 1) {
                        const int64_t k = keys[pv[u]];
                        if (mmatch[pair_i(k)] || mmatch[pair_j(k)]) flag[pv[u]] = 0;
                        else keep[u] = true;
                    }
                }
            }
            int cnt = 0;
#pragma unroll
            for (int u = 0; u < U; u++) cnt += keep[u] ? 1 : 0;
            int tot;
            int o = kept + block_int_prefix(cnt, wsum, &tot);
#pragma unroll
            for (int u = 0; u < U; u++)
                if (keep[u]) live[o++] = pv[u];
            kept += tot;
        }
        nlive = kept;
        __syncthreads();
    }
    // the resolved pairs, in (i, j) order, as (step, i, j) after the earlier steps';
    // a thread takes U consecutive pairs per pass
    const int64_t base = *cursor;
    int64_t run = 0;
    for (int c0 = 0; c0 < np; c0 += U * T) {
        bool acc[U];
        int cnt = 0;
#pragma unroll
        for (int u = 0; u < U; u++) {
            const int p = c0 + U * tid + u;
            acc[u] = p < np && flag[p] == 2;
            cnt += acc[u] ? 1 : 0;
        }
        int tot;
        int64_t o = base + run + block_int_prefix(cnt, wsum, &tot);
#pragma unroll
        for (int u = 0; u < U; u++)
            if (acc[u]) {
                const int p = c0 + U * tid + u;
                if (o < cap) {
                    pairs[3 * o] = step;
                    pairs[3 * o + 1] = keys[p] >> 32;
                    pairs[3 * o + 2] = keys[p] & 0xffffffffll;
                }
                o++;
            }
        run += tot;
    }
    if (tid == 0) {
        *n_pairs_dev = run;
        if (base + run > cap) {
            atomicOr(&st->status, (int32_t)ST_CAP_PAIRS);
            atomicMax((unsigned long long *)&st->required, (unsigned long long)(base + run));
        }
        *cursor = base + run;
    }
}

// Impulses of the resolved pairs (disjoint moonlets: 1 = i, 2 = j), over the whole GPU.
__global__ void __launch_bounds__(256)
k_resolve_apply(const DevState *__restrict__ st, const int64_t *__restrict__ keys,
                int64_t pair_cap, const int32_t *__restrict__ flag,
                const double *__restrict__ dtc, double *__restrict__ x,
                double *__restrict__ y, double *__restrict__ z, double *__restrict__ vx,
                double *__restrict__ vy, double *__restrict__ vz, const double *__restrict__ m,
                const double *__restrict__ R, double f) {
    const int np = resolve_count(st, pair_cap);
    for (int p = blockIdx.x * blockDim.x + threadIdx.x; p < np; p += gridDim.x * blockDim.x) {
        if (flag[p] != 2) continue;
        const int64_t k = keys[p];
        const int i = pair_i(k), j = pair_j(k);
        const double t = dtc[p];
        const double x1 = x[i] + t * vx[i], y1 = y[i] + t * vy[i], z1 = z[i] + t * vz[i];
        const double x2 = x[j] + t * vx[j], y2 = y[j] + t * vy[j], z2 = z[j] + t * vz[j];
        const double drx = x1 - x2, dry = y1 - y2, drz = z1 - z2;
        const double dvx = vx[i] - vx[j], dvy = vy[i] - vy[j], dvz = vz[i] - vz[j];
        const double sdot = drx * dvx + dry * dvy + drz * dvz;
        const double Rs = R[i] + R[j];
        const double alpha = f * m[i] * m[j] / ((m[i] + m[j]) * (Rs * Rs));
        const double Jx = alpha * sdot * drx, Jy = alpha * sdot * dry, Jz = alpha * sdot * drz;
        const double u1x = vx[i] - Jx / m[i], u1y = vy[i] - Jy / m[i], u1z = vz[i] - Jz / m[i];
        const double u2x = vx[j] + Jx / m[j], u2y = vy[j] + Jy / m[j], u2z = vz[j] + Jz / m[j];
        // old velocity up to contact, new one after: the drift adds dt u
        x[i] = x[i] + t * (vx[i] - u1x); y[i] = y[i] + t * (vy[i] - u1y);
        z[i] = z[i] + t * (vz[i] - u1z);
        x[j] = x[j] + t * (vx[j] - u2x); y[j] = y[j] + t * (vy[j] - u2y);
        z[j] = z[j] + t * (vz[j] - u2z);
        vx[i] = u1x; vy[i] = u1y; vz[i] = u1z;
        vx[j] = u2x; vy[j] = u2y; vz[j] = u2z;
    }
}

hipError_t launch_resolve(const Workspace &ws, double *x, double *y, double *z, double *vx,
                          double *vy, double *vz, const double *m, const double *R, double dt,
                          double f, int64_t *pairs, int64_t cap, int64_t *n_pairs_dev, int step,
                          int64_t *cursor, const unsigned long long *tests_part, int n_part,
                          hipStream_t s) {
    const RankResolve RR = {x, y, z, vx, vy, vz, R, dt, ws.pair_dt, ws.pair_flag, ws.mmatch,
                            ws.mbest};
    k_rank_pairs<<<kRankGrid, kWave * kRankSplit, 0, s>>>(ws.st, ws.pairs_tmp, ws.pair_cap,
                                                          ws.pairs_alt, (int64_t *)ws.pair_dt,
                                                          tests_part, n_part, RR,
                                                          RankReport{}, ws.walk_ctr);
    // the unsorted list is no longer needed: its buffer holds the live pair indices
    k_resolve<<<kResolveBlocks, kResolveThreads, 0, s>>>(ws.st, ws.pairs_alt, ws.pair_cap, ws.pair_dt,
                                            ws.pair_flag, ws.mbest, ws.mmatch,
                                            (int32_t *)ws.pairs_tmp, pairs, cap, n_pairs_dev,
                                            step, cursor);
    k_resolve_apply<<<kResolveGrid, 256, 0, s>>>(ws.st, ws.pairs_alt, ws.pair_cap, ws.pair_flag,
                                                 ws.pair_dt, x, y, z, vx, vy, vz, m, R, f);
    return hipGetLastError();
}

hipError_t launch_collide_pairs(const Workspace &ws, int64_t n, double dt, bool boxes,
                                hipStream_t s) {
    (void)n;
    // the pair and test counts start at zero: cleared by the box pass or the walk's init
    const auto kernel = boxes ? k_collide<true> : k_collide<false>;
    kernel<<<collide_grid(ws), 64, 0, s>>>(ws.st, cand_out(ws), ws.walk_ctr, ws.queue_cap,
                                           ws.c_first, ws.c_count, ws.ccell, ws.cbox, ws.idx,
                                           ws.pcol, ws.vcol, ws.ent_cell, dt, ws.pairs_tmp,
                                           ws.pair_cap, ws.count_part);
    return hipGetLastError();
}

hipError_t launch_emit_pairs(const Workspace &ws, int64_t *pairs, int64_t cap,
                             int64_t *n_pairs_dev, int triple, int step, int64_t *cursor,
                             const unsigned long long *tests_part, int n_part, hipStream_t s) {
    const RankReport RP = {pairs, cap, cursor, triple, step};
    k_rank_pairs<<<kRankGrid, kWave * kRankSplit, 0, s>>>(ws.st, ws.pairs_tmp, ws.pair_cap,
                                                          ws.pairs_alt, (int64_t *)ws.pair_dt,
                                                          tests_part, n_part, RankResolve{}, RP,
                                                          ws.walk_ctr);
    k_pairs_done<<<1, 64, 0, s>>>(ws.st, n_pairs_dev, cap, ws.pair_cap, triple, cursor);
    return hipGetLastError();
}

}  // namespace ncorp
