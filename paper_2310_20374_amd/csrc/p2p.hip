// Downward pass (Eq. 26) and evaluation at the moonlets: direct sums of the
// walk's brute-force pairs plus the leaf expansion.
//
// Descent: C^(m)(s_1) = sum_{|b| <= p-m} C_{a+b}(s_0) (s_1 - s_0)^b / b!.  Applied
// from the root down the paper's way, every leaf ends up with the sum of its own
// and its ancestors' walk tensors, each shifted to the leaf's centre; that sum is
// formed directly per leaf (shifts compose exactly), so no pass waits on another.
//
// Evaluation: one wave per leaf, or several where a leaf's sums would outlast the others'.
// Its sources (every cell the walk paired with the leaf or one of its ancestors for a
// direct sum) are prefix-summed 64 cells at a time into one flat range and streamed
// through LDS 256 moonlets at a time; leaves with fewer than 64 moonlets split each tile
// over lane groups.  In the FP32-bulk form offsets from the leaf centre are formed in FP64
// and rounded, each source tile is summed in FP32, and the tile sums are added with Kahan
// compensation.  The leaf's C tensors then give
// a_i += sum_{|b| <= p-1} C_{e+b}(s_leaf) (x_i - s_leaf)^b / b!.
#include "ncorp_internal.h"
#include "expansion.h"

namespace ncorp {

template <int P>
__device__ __forceinline__ void scaled_pow(double ux, double uy, double uz, double *px,
                                           double *py, double *pz) {
    px[0] = py[0] = pz[0] = 1.0;
#pragma unroll
    for (int a = 1; a <= P; a++) {
        const double inv = 1.0 / (double)a;
        px[a] = px[a - 1] * ux * inv;
        py[a] = py[a - 1] * uy * inv;
        pz[a] = pz[a - 1] * uz * inv;
    }
}

// Descent without inter-cell waiting.  Shifting a degree-p local expansion is an
// exact re-expansion, so shifts compose: C(leaf) = sum over the leaf and its
// ancestors a of shift(C_walk(a), s_leaf - s_a).  One thread per (leaf, output
// order m) sums that chain; threads are ordered by m so a wave runs one order.
template <int P, int M>
__device__ __forceinline__ void leaf_local_order(int cl, const int32_t *__restrict__ c_parent,
                                                 const double4 *__restrict__ gcell,
                                                 const double *__restrict__ local,
                                                 const int32_t *__restrict__ m2l_cnt,
                                                 double *__restrict__ out) {
    constexpr int NL = n_local(P), NR = P - M, NC = ncomp(M);
    double acc[NC];
#pragma unroll
    for (int k = 0; k < NC; k++) acc[k] = 0.0;
    const double4 gl = gcell[cl];
    int a = cl;
    for (int up = 0; up <= kMaxDepth && a >= 0; up++) {
        if (m2l_cnt[a] != 0) {                       // cells without M2L hold zeros
            const double4 ga = gcell[a];
            double px[NR + 1], py[NR + 1], pz[NR + 1];
            scaled_pow<NR>(gl.x - ga.x, gl.y - ga.y, gl.z - ga.z, px, py, pz);
            const double *ca = local + (int64_t)a * NL;
#pragma unroll
            for (int b = 0; b <= M; b++)
#pragma unroll
                for (int c = 0; c <= M - b; c++) {
                    const int aa = M - b - c;
                    double sum = acc[tri(b + c) + c];
#pragma unroll
                    for (int n = 0; n <= NR; n++)
#pragma unroll
                        for (int b2 = 0; b2 <= n; b2++)
#pragma unroll
                            for (int c2 = 0; c2 <= n - b2; c2++) {
                                const int a2 = n - b2 - c2;
                                sum += ca[cidx(aa + a2, b + b2, c + c2)] *
                                       (px[a2] * py[b2] * pz[c2]);
                            }
                    acc[tri(b + c) + c] = sum;
                }
        }
        a = c_parent[a];
    }
#pragma unroll
    for (int k = 0; k < NC; k++) out[cidx(M, 0, 0) + k] = acc[k];
}

// The gravity walk's totals (its classes' counter lines, one per lane) against the
// capacities the caller gave; later passes stop on a list that is too long.
struct WalkCaps {
    int64_t visited, m2l, p2p;
};
__device__ __forceinline__ void walk_totals(DevState *st, const int32_t *ctr,
                                            const WalkCaps &caps) {
    static_assert(kWalkClasses == kWave, "a lane per class");
    const int lane = threadIdx.x & (kWave - 1);
    unsigned long long v = *(const unsigned long long *)(ctr + lane * kCtrStride + kCtrVisited);
    long long m = ctr[lane * kCtrStride + kCtrM2L], p = ctr[lane * kCtrStride + kCtrP2P];
    for (int o = kWave / 2; o > 0; o >>= 1) {
        v += __shfl_xor(v, o);
        m += __shfl_xor(m, o);
        p += __shfl_xor(p, o);
    }
    if (lane != 0) return;
    int32_t bits = 0;
    unsigned long long need = 0;
    if ((int64_t)v > caps.visited) { bits |= ST_CAP_QUEUE; need = v; }
    if (m > caps.m2l) { bits |= ST_CAP_M2L; need = (unsigned long long)m > need ? m : need; }
    if (p > caps.p2p) { bits |= ST_CAP_P2P; need = (unsigned long long)p > need ? p : need; }
    if (bits) {
        atomicOr(&st->status, bits);
        atomicMax((unsigned long long *)&st->required, need);
    }
}

constexpr int kP2PSrc = kWave;      // source cells per batch, one per lane (prefix sums in LDS)

// FP32 sums of a list are added up in strands, each by itself: a list of one batch is one
// strand, a longer one has kLongSlots of them (or as many as it has batches), strand v
// taking the batches v, v + kLongSlots, ...  A leaf's waves share its strands, so what is
// added up in FP32 is the same however many waves it has; the strands' sums are then added
// in FP64, in an order that depends on them.
__device__ __forceinline__ int list_strands(int len) {
    const int nb = (len + kP2PSrc - 1) / kP2PSrc;
    return nb < kLongSlots ? nb : kLongSlots;
}

// How many waves share a leaf's direct sums (up to kLongSlots): as many as it has shares
// of about `quantum` moonlet interactions.  The chip holds some 5000 waves and an average
// leaf has 15000 to 60000 interactions (s = 48 and 96), so a small tree's leaves are
// all split, and in a large one only those that would outlast the others.  A share costs
// about 10 us of dependent loads before its first tile, hence the lower limit; in between
// four interactions a leaf, and never so many that the heaviest leaves are left whole.
// The rule knows its own tree only, so a disk's sums are the same in a batch and alone.
// Unsplit -> split, direct sums alone (FP32 at four waves a SIMD): 9973 moonlets in 519
// leaves (FP64) 129 -> 46 us, 1e6 in 2.7e4 FP32 582 -> 433 us; a quantum of 2048 instead
// for 1e5 in 2700: 88 -> 103 us.
constexpr int64_t kQuantumMin = 2048, kQuantumMax = 49152;
constexpr uint32_t kListed = 0x100;     // a leaf's slots: it is in the list
struct SplitArgs {
    const int32_t *p2p_cnt, *c_count, *c_first, *c_nent;
    const uint16_t *seg;                 // batched: disk of every tree position, else nullptr
    const int32_t *disk_root;
    uint32_t *src;                       // per leaf: source moonlets in, slots out
    int32_t *longs;                      // leaves whose list is beyond one LDS batch
    int32_t *split;                      // slots (leaf | slot << 24) of the leaves with more
                                         // than one or a long list: kLongSlots a leaf fit
    bool fp32;
};
__device__ __forceinline__ void split_leaf(DevState *st, const SplitArgs &S, int e, int c) {
    const int64_t src = S.src[e];
    const int K = S.seg ? S.c_nent[S.disk_root[S.seg[S.c_first[c]]]] : st->nleaves;
    int64_t quantum = 4 * (int64_t)K;
    quantum = quantum < kQuantumMin ? kQuantumMin : (quantum > kQuantumMax ? kQuantumMax : quantum);
    const int64_t work = src * S.c_count[c];
    int64_t slots = (work + quantum / 2) / quantum;
    // what there is to hand out: in FP32 the strands of every chunk of 64 targets, in FP64 64
    // source moonlets at a time
    const int64_t units = S.fp32 ? list_strands(S.p2p_cnt[e]) *
                                       (int64_t)((S.c_count[c] + kWave - 1) / kWave)
                                 : (src + kWave - 1) / kWave;
    slots = slots < units ? slots : units;
    slots = slots > kLongSlots ? kLongSlots : (slots < 1 ? 1 : slots);
    // one atomic per wave for the list's length
    const bool lng = S.p2p_cnt[e] > kP2PListLDS;
    if (const uint64_t ml = __ballot(lng)) {
        const int ln = threadIdx.x & (kWave - 1), first = __ffsll((unsigned long long)ml) - 1;
        int at = 0;
        if (ln == first) at = atomicAdd(&st->nlong, __popcll(ml));
        at = __shfl(at, first);
        if (lng) S.longs[at + __popcll(ml & (ln == 0 ? 0ull : (~0ull >> (64 - ln))))] = e;
    }
    // listed, to start first: what is split, long or heavy.  Heavy in FP32 from a quantum on, in FP64 from half of one: at
    // N = 1e6 without the heavy ones 515 us (FP32, four waves a SIMD) and 603 us, from a
    // quantum on 433 and 581 us, from half of one 502 and 542 us.
    const bool heavy = (S.fp32 ? work : 2 * work) > quantum;
    const int add = slots > 1 || lng || heavy ? (int)slots : 0;
    S.src[e] = (uint32_t)slots | (add > 0 ? kListed : 0u);
    if (!__any(add)) return;
    const int lane = threadIdx.x & (kWave - 1);
    const int lead = __ffsll((unsigned long long)__ballot(1)) - 1;
    int off = 0, tot = 0;                // the slots of the lanes below and of all
    for (uint64_t act = __ballot(add > 0); act; act &= act - 1) {
        const int l = __ffsll((unsigned long long)act) - 1;
        if (lane == l) off = tot;
        tot += __shfl(add, l);
    }
    int base = 0;
    if (lane == lead) base = atomicAdd(&st->nsplit, tot);
    base = __shfl(base, lead) + off;
    for (int k = 0; k < add; k++) S.split[base + k] = e | (k << 24);
}

template <int P>
__global__ void __launch_bounds__(128)
k_leaf_local(DevState *st, const int32_t *__restrict__ ent_cell,
             const int32_t *__restrict__ c_parent, const double4 *__restrict__ gcell,
             const double *__restrict__ local, const int32_t *__restrict__ m2l_cnt,
             double *__restrict__ cleaf, const SplitArgs S,
             const int32_t *__restrict__ walk_ctr, const WalkCaps caps) {
    constexpr int NL = n_local(P);
    if (blockIdx.x == 0 && threadIdx.x < kWave) walk_totals(st, walk_ctr, caps);
    if (st->status & kSkipMask) return;
    const int K = st->nleaves;
    const int64_t total = (int64_t)K * P;
    for (int64_t t = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; t < total;
         t += (int64_t)gridDim.x * blockDim.x) {
        const int m = (int)(t / K) + 1, e = (int)(t % K);
        if (m == 1) split_leaf(st, S, e, ent_cell[e]);
        const int cl = ent_cell[e];
        double *out = cleaf + (int64_t)e * NL;
        switch (m) {
            case 1: leaf_local_order<P, 1>(cl, c_parent, gcell, local, m2l_cnt, out); break;
            case 2: if constexpr (P >= 2) leaf_local_order<P, (P >= 2 ? 2 : 1)>(cl, c_parent, gcell, local, m2l_cnt, out); break;
            case 3: if constexpr (P >= 3) leaf_local_order<P, (P >= 3 ? 3 : 1)>(cl, c_parent, gcell, local, m2l_cnt, out); break;
            case 4: if constexpr (P >= 4) leaf_local_order<P, (P >= 4 ? 4 : 1)>(cl, c_parent, gcell, local, m2l_cnt, out); break;
            case 5: if constexpr (P >= 5) leaf_local_order<P, (P >= 5 ? 5 : 1)>(cl, c_parent, gcell, local, m2l_cnt, out); break;
            case 6: if constexpr (P >= 6) leaf_local_order<P, (P >= 6 ? 6 : 1)>(cl, c_parent, gcell, local, m2l_cnt, out); break;
            default: break;
        }
    }
}

// ------------------------------------------------------------------ evaluation
template <typename T> struct Acc3;
template <> struct Acc3<double> {
    double x = 0, y = 0, z = 0;
    __device__ void open_tile(double &px, double &py, double &pz) const { px = x; py = y; pz = z; }
    __device__ void close_tile(double px, double py, double pz) { x = px; y = py; z = pz; }
    __device__ void fold(double &ox, double &oy, double &oz) const { ox = x; oy = y; oz = z; }
};
// Kahan-compensated FP32 sums of FP32 tile partials
template <> struct Acc3<float> {
    float x = 0, y = 0, z = 0, cx = 0, cy = 0, cz = 0;
    __device__ static void kahan(float &s, float &c, float v) {
        float yv = v - c;
        float t = s + yv;
        c = (t - s) - yv;
        s = t;
    }
    __device__ void open_tile(float &px, float &py, float &pz) const { px = py = pz = 0.0f; }
    __device__ void close_tile(float px, float py, float pz) {
        kahan(x, cx, px); kahan(y, cy, py); kahan(z, cz, pz);
    }
    __device__ void fold(double &ox, double &oy, double &oz) const {
        ox = (double)x - (double)cx; oy = (double)y - (double)cy; oz = (double)z - (double)cz;
    }
};

__device__ __forceinline__ int wave_excl_sum_p(int v, int lane, int &total) {
    int x = v;
#pragma unroll
    for (int o = 1; o < kWave; o <<= 1) {
        int t = __shfl_up(x, o);
        if (lane >= o) x += t;
    }
    total = __shfl(x, kWave - 1);
    return x - v;
}

template <typename T> __device__ __forceinline__ T fmat(T a, T b, T c);
template <> __device__ __forceinline__ double fmat<double>(double a, double b, double c) { return fma(a, b, c); }
template <> __device__ __forceinline__ float fmat<float>(float a, float b, float c) { return fmaf(a, b, c); }

template <typename T> struct Vec4;
template <> struct Vec4<float> { using type = float4; };
template <> struct Vec4<double> { using type = double4; };
// r^2 floor: a moonlet meets itself (dx = 0) in its own leaf; the floor keeps
// 1/r^3 finite there so the term is exactly 0; it is added to r^2 and far below any pair
// distance.  m / floor^(3/2) stays finite for G m up to ~3e11 (FP32) and ~1e158 (FP64).
template <typename T> __device__ __forceinline__ T r2_floor();
template <> __device__ __forceinline__ float r2_floor<float>() { return 1e-18f; }
template <> __device__ __forceinline__ double r2_floor<double>() { return 1e-100; }

constexpr int kP2PTile = 256;       // source moonlets staged per LDS tile (default)

// Exclusive prefix sums of the moonlet counts of a batch's source cells (one per
// lane) into s_pref[0..kP2PSrc]; returns the total.
__device__ __forceinline__ int batch_prefix(int cnt, int32_t *s_pref, int lane) {
    int tot;
    const int ex = wave_excl_sum_p(cnt, lane, tot);
    s_pref[lane] = ex;
    if (lane == 0) s_pref[kP2PSrc] = tot;
    return tot;
}

// An offset from the leaf centre: in FP64 held to +-1e150, so that r2 stays finite (at
// such distances the term is 0 either way).
template <typename T> __device__ __forceinline__ T offset_of(double d) {
    if constexpr (sizeof(T) == 8) {
        const double lim = 1e150;
        return d > lim ? lim : (d < -lim ? -lim : d);
    }
    return (T)d;
}

// One source against the NT targets a lane holds.
template <typename T, int NT>
__device__ __forceinline__ void interact(const typename Vec4<T>::type &v, const T (&xi)[NT],
                                         const T (&yi)[NT], const T (&zi)[NT], T (&px)[NT],
                                         T (&py)[NT], T (&pz)[NT]) {
    const T floor2 = r2_floor<T>();
#pragma unroll
    for (int k = 0; k < NT; k++) {
        const T dx = v.x - xi[k], dy = v.y - yi[k], dz = v.z - zi[k];
        // the floor enters as an addend, so r2 is a normal number and the hardware
        // reciprocal square root needs no handling of small ones
        const T r2 = fmat<T>(dz, dz, fmat<T>(dy, dy, fmat<T>(dx, dx, floor2)));
        T w;
        if constexpr (sizeof(T) == 4) {
            const T rinv = __builtin_amdgcn_rsqf(r2);
            w = v.w * (rinv * rinv) * rinv;
        } else {
            w = over_r3(v.w, r2);
        }
        px[k] = fmat<T>(dx, w, px[k]);
        py[k] = fmat<T>(dy, w, py[k]);
        pz[k] = fmat<T>(dz, w, pz[k]);
    }
}

// Slot `slot` of nslots of a batch of tot moonlets (FP64): an equal share of them, [q0, q1).
struct TileRange {
    int q0, q1;
};
__device__ __forceinline__ TileRange slot_range(int tot, int slot, int nslots) {
    const int per = ((tot + nslots - 1) / nslots + kWave - 1) / kWave * kWave;
    const int q0 = slot * per;
    return TileRange{q0, q0 + per < tot ? q0 + per : tot};
}

// Direct sums of the NT targets a lane holds over a range of a batch of source cells
// whose moonlet ranges are s_first[k] .. + (s_pref[k+1] - s_pref[k]), k < nsb; the
// range is streamed through LDS TILE moonlets at a time and the lane's group takes
// sources j0, j0 + G, ... of every tile.
template <typename T, int NT, int TILE>
__device__ __forceinline__ void p2p_batch(const TileRange tr, int nsb, const int32_t *s_first,
                                          const int32_t *s_pref,
                                          typename Vec4<T>::type *tile,
                                          const double4 *__restrict__ pos4, const double4 g,
                                          const T (&xi)[NT], const T (&yi)[NT], const T (&zi)[NT],
                                          int j0, int G, Acc3<T> (&acc)[NT]) {
    using V = typename Vec4<T>::type;
    const int lane = threadIdx.x & (kWave - 1);
    for (int p0 = tr.q0; p0 < tr.q1; p0 += TILE) {
        const int nj = tr.q1 - p0 < TILE ? tr.q1 - p0 : TILE;
        // stage the tile: source moonlet q of the batch -> its cell by binary
        // search over the prefix sums
#pragma unroll
        for (int k = 0; k < TILE / 64; k++) {
            const int q = p0 + lane + 64 * k;
            if (q < tr.q1) {
                int lo = 0, hi = nsb;          // s_pref[lo] <= q < s_pref[hi]
                while (hi - lo > 1) {
                    const int mid = (lo + hi) >> 1;
                    if (s_pref[mid] <= q) lo = mid; else hi = mid;
                }
                const int j = s_first[lo] + (q - s_pref[lo]);
                const double4 s = pos4[j];
                V v;
                v.x = offset_of<T>(s.x - g.x);
                v.y = offset_of<T>(s.y - g.y);
                v.z = offset_of<T>(s.z - g.z);
                v.w = (T)s.w;
                tile[lane + 64 * k] = v;
            }
        }
        wave_sync();
        // FP64 adds to the running sums; FP32 sums each tile by itself
        T px[NT], py[NT], pz[NT];
#pragma unroll
        for (int k = 0; k < NT; k++) acc[k].open_tile(px[k], py[k], pz[k]);
        if constexpr (NT == 1) {
#pragma unroll 4
            for (int j = j0; j < nj; j += G) interact<T, NT>(tile[j], xi, yi, zi, px, py, pz);
        } else if constexpr (NT == 2) {
#pragma unroll 2
            for (int j = j0; j < nj; j += G) interact<T, NT>(tile[j], xi, yi, zi, px, py, pz);
        } else {
            for (int j = j0; j < nj; j += G) interact<T, NT>(tile[j], xi, yi, zi, px, py, pz);
        }
#pragma unroll
        for (int k = 0; k < NT; k++) acc[k].close_tile(px[k], py[k], pz[k]);
        wave_sync();
    }
}

// Stages batch b of a leaf's source list: the moonlet ranges of its up to kP2PSrc cells
// in s_first and s_pref; returns the batch's moonlets.  FP64 takes the cells in the
// walk's order.  FP32 takes them in cell order, which its tile sums are rounded in: a
// list of one batch is ranked here (`rank`: scratch of kP2PSrc ints, free until the
// first tile), a longer one was sorted by the pre-pass.
template <typename T>
__device__ __forceinline__ int stage_batch(const int32_t *__restrict__ list, int len, int b,
                                           const int32_t *__restrict__ c_first,
                                           const int32_t *__restrict__ c_count,
                                           int32_t *s_first, int32_t *s_pref, int32_t *rank) {
    const int lane = threadIdx.x & (kWave - 1);
    const bool in = b * kP2PSrc + lane < len;
    const int v = in ? list[b * kP2PSrc + lane] : 0x7fffffff;
    int cf = 0, cn = 0;
    if (in) {
        cf = c_first[v];
        cn = c_count[v];
    }
    wave_sync();                                  // the last batch is done with
    if (sizeof(T) == 4 && len <= kP2PSrc) {
        rank[lane] = v;
        wave_sync();
        if (in) {
            const int4 *s4 = reinterpret_cast<const int4 *>(rank);
            int rk = 0;
#pragma unroll
            for (int j = 0; j < kP2PSrc / 4; j++) {
                const int4 t = s4[j];
                rk += (t.x < v) + (t.y < v) + (t.z < v) + (t.w < v);
            }
            s_first[rk] = cf;
            s_pref[rk] = cn;
        }
        wave_sync();
        cn = in ? s_pref[lane] : 0;
        wave_sync();
    } else {
        s_first[lane] = cf;
    }
    const int tot = batch_prefix(cn, s_pref, lane);
    wave_sync();
    return tot;
}

// Direct sums for ntc <= 64 targets (moonlets tb .. tb+ntc-1) of one leaf, over slot
// `slot` of nslots of its list.  FP32: the strands slot, slot + nslots, ...  FP64: the
// batches of kP2PSrc source cells are dealt to the slots, and where there are fewer batches
// than slots, each batch's moonlets to its share of them.  The lanes form G = 64 / lpg
// groups of lpg = ceil(ntc / NT) lanes; lane li of a group holds targets li, li + lpg, ...,
// and the groups split every tile's sources.  The group partials are added in a fixed tree
// and written to out[d * n + i], d = x, y, z.
template <typename T, int NT, int TILE>
__device__ __forceinline__ void p2p_targets(int ntc, int tb, int len, int slot, int nslots,
                                            const int32_t *__restrict__ list, int32_t *s_first,
                                            int32_t *s_pref, typename Vec4<T>::type *tile,
                                            const double4 *__restrict__ pos4,
                                            const int32_t *__restrict__ c_first,
                                            const int32_t *__restrict__ c_count, const double4 g,
                                            double *__restrict__ out, int64_t n) {
    const int lane = threadIdx.x & (kWave - 1);
    const int lpg = (ntc + NT - 1) / NT;
    const int G = kWave / lpg;
    const int grp = lane / lpg, li = lane % lpg;
    T xi[NT], yi[NT], zi[NT];
#pragma unroll
    for (int k = 0; k < NT; k++) {
        const int t = li + k * lpg;
        const int i = tb + (t < ntc ? t : 0);
        const double4 p = pos4[i];
        xi[k] = offset_of<T>(p.x - g.x);
        yi[k] = offset_of<T>(p.y - g.y);
        zi[k] = offset_of<T>(p.z - g.z);
    }
    const int j0 = grp < G ? grp : TILE;           // lanes beyond the groups idle
    const int nb = (len + kP2PSrc - 1) / kP2PSrc;
    double px[NT], py[NT], pz[NT];
    if constexpr (sizeof(T) == 4) {
#pragma unroll
        for (int k = 0; k < NT; k++) px[k] = py[k] = pz[k] = 0.0;
        for (int v = slot; v < list_strands(len); v += nslots) {
            Acc3<T> acc[NT];
            for (int b = v; b < nb; b += kLongSlots) {
                const int tot = stage_batch<T>(list, len, b, c_first, c_count, s_first, s_pref,
                                               reinterpret_cast<int32_t *>(tile));
                const int nsb = len - b * kP2PSrc < kP2PSrc ? len - b * kP2PSrc : kP2PSrc;
                p2p_batch<T, NT, TILE>(TileRange{0, __builtin_amdgcn_readfirstlane(tot)}, nsb,
                                       s_first, s_pref, tile, pos4, g, xi, yi, zi, j0, G, acc);
            }
#pragma unroll
            for (int k = 0; k < NT; k++) {
                double ox, oy, oz;
                acc[k].fold(ox, oy, oz);
                px[k] += ox; py[k] += oy; pz[k] += oz;
            }
        }
    } else {
        Acc3<T> acc[NT];
        const int b0 = nb < nslots ? slot * nb / nslots : slot;
        // the slots that share batch b0: those with slot * nb / nslots = b0
        const int s0 = nb < nslots ? (b0 * nslots + nb - 1) / nb : slot;
        const int s1 = nb < nslots ? ((b0 + 1) * nslots + nb - 1) / nb : slot + 1;
        for (int b = b0; b < nb; b += nb < nslots ? nb : nslots) {
            const int tot = stage_batch<T>(list, len, b, c_first, c_count, s_first, s_pref,
                                           reinterpret_cast<int32_t *>(tile));
            const int nsb = len - b * kP2PSrc < kP2PSrc ? len - b * kP2PSrc : kP2PSrc;
            p2p_batch<T, NT, TILE>(slot_range(__builtin_amdgcn_readfirstlane(tot), slot - s0,
                                              s1 - s0),
                                   nsb, s_first, s_pref, tile, pos4, g, xi, yi, zi, j0, G, acc);
        }
#pragma unroll
        for (int k = 0; k < NT; k++) acc[k].fold(px[k], py[k], pz[k]);
    }
    // the groups' partials, added pairwise in a fixed tree (a leaf of 5 targets has 32
    // groups: one after the other they took as long as its sums)
    for (int o = 1; o < G; o <<= 1) {
        const bool add = (grp & (2 * o - 1)) == 0 && grp + o < G;
#pragma unroll
        for (int k = 0; k < NT; k++) {
            const double ox = __shfl_down(px[k], o * lpg);
            const double oy = __shfl_down(py[k], o * lpg);
            const double oz = __shfl_down(pz[k], o * lpg);
            if (add) { px[k] += ox; py[k] += oy; pz[k] += oz; }
        }
    }
#pragma unroll
    for (int k = 0; k < NT; k++) {
        const int t = li + k * lpg;
        if (grp == 0 && t < ntc) {
            out[tb + t] = px[k];
            out[n + tb + t] = py[k];
            out[2 * n + tb + t] = pz[k];
        }
    }
}

// Targets per lane for a chunk of ntc <= 64 targets: lpg = ceil(ntc / NT) lanes hold
// them, G = 64 / lpg lane groups split every tile, so a round keeps ntc * G of the
// 64 * NT lane slots busy.  The NT in 1..4 with the largest share wins (the smaller
// on ties): 43 targets use 3 per lane (4 groups of 15 lanes, 90 % busy) where one or
// two per lane leave a third of the lanes idle.
__device__ __forceinline__ int targets_per_lane(int ntc, int tmax) {
    int best = 1, best_score = -1;
#pragma unroll
    for (int nt = 1; nt <= 4; nt++) {
        if (nt > tmax) break;
        const int lpg = (ntc + nt - 1) / nt;
        const int score = ntc * (kWave / lpg) * (12 / nt);
        if (score > best_score) { best = nt; best_score = score; }
    }
    return best;
}

template <typename T, int TILE>
__device__ __forceinline__ void p2p_targets_any(int ntc, int tmax, int tb, int len, int slot,
                                                int nslots, const int32_t *__restrict__ list,
                                                int32_t *s_first, int32_t *s_pref,
                                                typename Vec4<T>::type *tile,
                                                const double4 *__restrict__ pos4,
                                                const int32_t *__restrict__ c_first,
                                                const int32_t *__restrict__ c_count,
                                                const double4 g, double *__restrict__ out,
                                                int64_t n) {
    switch (targets_per_lane(ntc, tmax)) {
        case 1:
            p2p_targets<T, 1, TILE>(ntc, tb, len, slot, nslots, list, s_first, s_pref, tile, pos4,
                                    c_first, c_count, g, out, n);
            break;
        case 2:
            p2p_targets<T, 2, TILE>(ntc, tb, len, slot, nslots, list, s_first, s_pref, tile, pos4,
                                    c_first, c_count, g, out, n);
            break;
        case 3:
            p2p_targets<T, 3, TILE>(ntc, tb, len, slot, nslots, list, s_first, s_pref, tile, pos4,
                                    c_first, c_count, g, out, n);
            break;
        default:
            p2p_targets<T, 4, TILE>(ntc, tb, len, slot, nslots, list, s_first, s_pref, tile, pos4,
                                    c_first, c_count, g, out, n);
            break;
    }
}

// FP32: the first strand that slot `slot` takes of the chunk of targets at t0 (strand v of
// chunk k is unit k * strands + v, the units are dealt in turn; none: beyond the strands)
template <typename T>
__device__ __forceinline__ int first_strand(int slot, int nslots, int t0, int len) {
    if (sizeof(T) == 8) return slot;
    return (slot + nslots - t0 / kWave * list_strands(len) % nslots) % nslots;
}

constexpr int kP2PRun = 8;
constexpr int64_t kP2PGrid = 65536;  // most blocks, of one wave each
static_assert(kP2PListLDS == kP2PSrc, "one LDS batch holds a list that is not long");

// Direct sums of every leaf, one wave per work item: a leaf, or one of the slots of a
// leaf that is split (split_leaf), whose partial sums the evaluation kernel adds in slot
// order.  The split and the long leaves come first, so they start first and the others
// fill in around them within the same launch, which the hardware deals out as waves end:
// blocks of one wave, an item each.  Four waves a block and items by position took 582 us
// at N = 1e6, s = 96 in FP32, where this takes 423; persistent waves with counters 490.
//
// Five waves a SIMD, 96 registers: vector instructions of different waves overlap in part,
// and a fifth wave is worth more than the registers it spills between the tiles.  FP32 with
// four waves (125 registers, none spilled) 434 us at 1e6, 342 for 64 batched disks, 3100
// for 4e6 in clumps; with five 423, 331, 2920; with six (91 spilled) 429, 334, 2920 and
// 1e5 moonlets 86.7 instead of 83.
template <typename T, int TILE>
__global__ void __launch_bounds__(kWave, 5)
k_p2p(const DevState *__restrict__ st, const double4 *__restrict__ pos4,
      const int32_t *__restrict__ ent_cell,
      const int32_t *__restrict__ c_first, const int32_t *__restrict__ c_count,
      const double4 *__restrict__ gcell, const int32_t *__restrict__ p2p_cnt,
      const int32_t *__restrict__ p2p_seg, int stride, const int32_t *__restrict__ split,
      const uint32_t *__restrict__ slots, double *__restrict__ part,
      double *__restrict__ acc_s, int64_t n, int tmax) {
    using V = typename Vec4<T>::type;
    static_assert(TILE % 64 == 0, "a tile is staged one moonlet per lane");
    __shared__ __align__(16) V tile[TILE];
    __shared__ int32_t firsts[kP2PSrc], prefs[kP2PSrc + 1];
    if (st->status & kSkipMask) return;
    const int K = st->nleaves;
    const int nsplit = st->nsplit;
    const int items = nsplit + K;
    // runs of kP2PRun items (the slots of a leaf, neighbouring leaves) stay on an XCD
    constexpr int kRound = kXcds * kP2PRun;
    for (int b = blockIdx.x; b < (items + kRound - 1) / kRound * kRound; b += gridDim.x) {
        const int w = (b / kRound * kXcds + b % kXcds) * kP2PRun + b / kXcds % kP2PRun;
        if (w >= items) continue;
        const bool lng = w < nsplit;
        const int ent = lng ? split[w] : w - nsplit;
        const int e = ent & 0xffffff, slot = ent >> 24;
        const uint32_t sl = slots[e];
        const int nslots = (int)(sl & 0xffu), len = p2p_cnt[e];
        if (!lng && (sl & kListed)) continue;
        const int c = ent_cell[e];
        const int f = c_first[c], nt = c_count[c];
        double *out = nslots > 1 ? part + (int64_t)slot * 3 * n : acc_s;
        for (int t0 = 0; t0 < nt; t0 += kWave)
            p2p_targets_any<T, TILE>(nt - t0 < kWave ? nt - t0 : kWave, tmax, f + t0, len,
                                     first_strand<T>(slot, nslots, t0, len), nslots, p2p_seg + (int64_t)e * stride, firsts, prefs,
                                     tile, pos4, c_first, c_count, gcell[c], out, n);
    }
}

// evaluation of the leaf's expansion at its moonlets (Eq. 26 down to C^(1)),
// added to the direct sums and written in input order
constexpr int kL2PWaves = 4;        // independent waves per block

template <int P>
__global__ void __launch_bounds__(kWave * kL2PWaves)
k_l2p(const DevState *__restrict__ st, const double *__restrict__ xs,
      const double *__restrict__ ys, const double *__restrict__ zs,
      const uint32_t *__restrict__ perm, const int32_t *__restrict__ ent_cell,
      const int32_t *__restrict__ c_first, const int32_t *__restrict__ c_count,
      const double4 *__restrict__ gcell, const double *__restrict__ cleaf,
      const double *__restrict__ acc_s, const uint32_t *__restrict__ slots,
      const double *__restrict__ part, int64_t n, double *__restrict__ ax,
      double *__restrict__ ay, double *__restrict__ az, double4 *__restrict__ acc4) {
    constexpr int NL = n_local(P);
    if (st->status & kSkipMask) return;
    const int K = st->nleaves;
    const int lane = threadIdx.x & (kWave - 1), wid = threadIdx.x / kWave;
    for (int e = blockIdx.x * kL2PWaves + wid; e < K; e += gridDim.x * kL2PWaves) {
        const int c = ent_cell[e];
        const int f = c_first[c], nt = c_count[c];
        const double4 g = gcell[c];
        const int nsl = (int)(slots[e] & 0xffu);      // direct sums in nsl parts
        // the leaf's C is wave-uniform: scalar loads, no copy in LDS
        const double *__restrict__ cle = cleaf + (int64_t)__builtin_amdgcn_readfirstlane(e) * NL;
        for (int t0 = 0; t0 < nt; t0 += 64) {
            const int t = t0 + lane;
            if (t >= nt) continue;
            const int i = f + t;
            double px[P], py[P], pz[P];
            const double ux = xs[i] - g.x, uy = ys[i] - g.y, uz = zs[i] - g.z;
            px[0] = py[0] = pz[0] = 1.0;
#pragma unroll
            for (int a = 1; a < P; a++) {
                const double inv = 1.0 / (double)a;
                px[a] = px[a - 1] * ux * inv;
                py[a] = py[a - 1] * uy * inv;
                pz[a] = pz[a - 1] * uz * inv;
            }
            double lx = 0.0, ly = 0.0, lz = 0.0;
#pragma unroll
            for (int nn = 0; nn < P; nn++)
#pragma unroll
                for (int b2 = 0; b2 <= nn; b2++)
#pragma unroll
                    for (int c2 = 0; c2 <= nn - b2; c2++) {
                        const int a2 = nn - b2 - c2;
                        const double w = px[a2] * py[b2] * pz[c2];
                        lx += cle[cidx(1 + a2, b2, c2)] * w;
                        ly += cle[cidx(a2, 1 + b2, c2)] * w;
                        lz += cle[cidx(a2, b2, 1 + c2)] * w;
                    }
            double dx = 0.0, dy = 0.0, dz = 0.0;       // direct sums
            if (nsl > 1) {
                for (int sl = 0; sl < nsl; sl++) {
                    const double *ps = part + (int64_t)sl * 3 * n;
                    dx += ps[i];
                    dy += ps[n + i];
                    dz += ps[2 * n + i];
                }
            } else {
                dx = acc_s[i];
                dy = acc_s[n + i];
                dz = acc_s[2 * n + i];
            }
            const uint32_t o = perm[i];
            if (acc4) {
                acc4[o] = make_double4(dx + lx, dy + ly, dz + lz, 0.0);
            } else {
                ax[o] = dx + lx;
                ay[o] = dy + ly;
                az[o] = dz + lz;
            }
        }
    }
}

template <int P>
static void launch_leaf_local(const Workspace &ws, bool fp32, hipStream_t s) {
    const SplitArgs S = {ws.p2p_cnt, ws.c_count, ws.c_first, ws.c_nent,
                         ws.ndisks > 1 ? ws.seg : nullptr, ws.disk_root, ws.ent_work,
                         ws.long_p2p, ws.split_p2p, fp32};
    int64_t g = ((int64_t)ws.n_max * P + 127) / 128;
    if (g > 8192) g = 8192;
    if (g < 1) g = 1;
    k_leaf_local<P><<<(int)g, 128, 0, s>>>(ws.st, ws.ent_cell, ws.c_parent, ws.gcell, ws.local,
                                           ws.m2l_cnt, ws.cleaf, S, ws.walk_ctr,
                                           WalkCaps{ws.queue_cap, ws.m2l_cap, ws.p2p_cap});
}

// Direct-sum lists beyond one LDS batch, sorted in place, one block per list (rank sort
// in LDS, the keys split over four waves).  Only the FP32 form needs it: its tile sums
// are rounded in cell order.
constexpr int kSortThreads = 256;
constexpr int kSortLongBlocks = 2048;

__global__ void __launch_bounds__(kSortThreads)
k_sort_long_lists(const DevState *__restrict__ st, const int32_t *__restrict__ cnt,
                  int32_t *seg, int stride, const int32_t *__restrict__ longs) {
    extern __shared__ __align__(16) int32_t scr[];   // round_up(stride, 4) ints
    if (st->status & kSkipMask) return;
    const int nl = st->nlong;
    for (int q = blockIdx.x; q < nl; q += gridDim.x) {
        const int t = longs[q];
        const int len = cnt[t];
        int32_t *list = seg + (int64_t)t * stride;
        const int len4 = (len + 3) & ~3;
        __syncthreads();
        for (int i = threadIdx.x; i < len4; i += kSortThreads)
            scr[i] = i < len ? list[i] : 0x7fffffff;
        __syncthreads();
        const int4 *s4 = reinterpret_cast<const int4 *>(scr);
        for (int i = threadIdx.x; i < len; i += kSortThreads) {
            const int v = scr[i];
            int r = 0;
            #pragma unroll 8
            for (int j = 0; j < len4 / 4; j++) {
                const int4 w = s4[j];
                r += (w.x < v) + (w.y < v) + (w.z < v) + (w.w < v);
            }
            list[r] = v;
        }
    }
}

hipError_t launch_l2l(const Workspace &ws, int p, int precision, hipStream_t s) {
    const bool fp32 = precision == NCORP_FP32_BULK;
    switch (p) {
        case 1: launch_leaf_local<1>(ws, fp32, s); break;
        case 2: launch_leaf_local<2>(ws, fp32, s); break;
        case 3: launch_leaf_local<3>(ws, fp32, s); break;
        case 4: launch_leaf_local<4>(ws, fp32, s); break;
        case 5: launch_leaf_local<5>(ws, fp32, s); break;
        case 6: launch_leaf_local<6>(ws, fp32, s); break;
        default: break;
    }
    if (fp32) {
        const size_t lds = (size_t)((ws.p2p_stride + 3) & ~3) * sizeof(int32_t);
        k_sort_long_lists<<<kSortLongBlocks, kSortThreads, lds, s>>>(ws.st, ws.p2p_cnt, ws.p2p_seg,
                                                                     ws.p2p_stride, ws.long_p2p);
    }
    return hipGetLastError();
}

template <typename T, int TILE>
static void launch_p2p_t(const Workspace &ws, int64_t n, int tmax, hipStream_t s) {
    // about 1 ns a block to deal out, empty or not: no more than a small tree can use
    const int64_t most = ws.leaf_cap + 2048;
    const int64_t g = most < kP2PGrid ? most : kP2PGrid;
    k_p2p<T, TILE><<<(int)g, kWave, 0, s>>>(
        ws.st, ws.vcol, ws.ent_cell, ws.c_first, ws.c_count, ws.gcell, ws.p2p_cnt, ws.p2p_seg,
        ws.p2p_stride, ws.split_p2p, ws.ent_work, ws.p2p_part, ws.acc_s, n, tmax);
}

template <typename T>
static void launch_p2p_tile(const Workspace &ws, int64_t n, int tile, int tmax, hipStream_t s) {
    switch (tile) {
        case 128: launch_p2p_t<T, 128>(ws, n, tmax, s); break;
        case 512: launch_p2p_t<T, 512>(ws, n, tmax, s); break;
        default: launch_p2p_t<T, kP2PTile>(ws, n, tmax, s); break;
    }
}

// tile: source moonlets per LDS tile (128, 256, 512; 0 = 256); tmax: most targets per
// lane (1..4; 0 = 4)
hipError_t launch_p2p(const Workspace &ws, int64_t n, int precision, int tile, int tmax,
                      hipStream_t s) {
    const int tm = tmax > 0 ? tmax : 4;
    if (precision == NCORP_FP32_BULK) launch_p2p_tile<float>(ws, n, tile, tm, s);
    else launch_p2p_tile<double>(ws, n, tile, tm, s);
    return hipGetLastError();
}

template <int P>
static void launch_l2p_p(const Workspace &ws, int64_t n, double *ax, double *ay, double *az,
                         hipStream_t s, double4 *acc4) {
    int64_t g = (ws.leaf_cap + kL2PWaves - 1) / kL2PWaves;
    g = g < 1 ? 1 : (g > 16384 ? 16384 : g);
    k_l2p<P><<<(int)g, kWave * kL2PWaves, 0, s>>>(ws.st, ws.xs, ws.ys, ws.zs, ws.idx, ws.ent_cell, ws.c_first,
                              ws.c_count, ws.gcell, ws.cleaf, ws.acc_s, ws.ent_work, ws.p2p_part, n,
                              ax, ay, az, acc4);
}

hipError_t launch_l2p(const Workspace &ws, int64_t n, int p, double *ax, double *ay, double *az,
                      hipStream_t s, double4 *acc4) {
    switch (p) {
        case 1: launch_l2p_p<1>(ws, n, ax, ay, az, s, acc4); break;
        case 2: launch_l2p_p<2>(ws, n, ax, ay, az, s, acc4); break;
        case 3: launch_l2p_p<3>(ws, n, ax, ay, az, s, acc4); break;
        case 4: launch_l2p_p<4>(ws, n, ax, ay, az, s, acc4); break;
        case 5: launch_l2p_p<5>(ws, n, ax, ay, az, s, acc4); break;
        case 6: launch_l2p_p<6>(ws, n, ax, ay, az, s, acc4); break;
        default: break;
    }
    return hipGetLastError();
}

}  // namespace ncorp
