// The falcON dual tree walk (Alg. 2) on the GPU, one wave per target cell.
//
// The paper's recursion visits unordered pairs of cells from (root, root) down.  Here
// every cell A works through the pairs that hold it, by itself: its wave takes the
// pairs its parent left to be opened on the parent's side, classifies each (A, B)
// exactly as Alg. 2 does (self pair / brute force before the opening test / well
// separated / brute force after it / split the cell with the larger critical radius)
// and
//   - where B is split, goes on with (A, B's children) at once, from a stack in LDS;
//   - where A is split, leaves B in A's hand-down list, which A's children start from;
//   - where the pair is well separated or summed directly, appends B to A's own lists (if
//     A is not a leaf, a direct-sum pair goes into the hand-down list: the leaves below A
//     inherit it).
// Classification is symmetric in A and B bit for bit (sums, squares and comparisons
// that commute, and ties broken by which cell holds the earlier moonlets), so the wave
// of B takes the same decision on the same pair: the pairs are those of the recursion,
// each seen once from either side.  That doubles the classifications, which are
// cheap, and makes every list the property of one wave: no queue, no atomic and no
// sort of a list whose order would depend on timing.  A cell's lists come out in an
// order fixed by the tree alone.
//
// The cells are dealt in runs of 8 (siblings mostly) to kWalkClasses classes and taken
// in breadth-first order within each, by the waves of that class, from a ticket counter
// (atomics on one address take about 15 ns each, so counters are many and nothing else
// is counted per cell).  A wave waits until its cell's parent has published its list;
// a class hands out its cells in ascending order and a parent precedes its children.
// Where another stream's kernel leaves room for a few workgroups only, the waves that run
// take the cells they wait for from classes that have none (walk_plan.h), so the launch
// ends whatever runs beside it.  A wave that polls for too long without progress latches
// ST_WALK_STALL and leaves.
//
// What bounds it: the chain of levels, about 6 us each (the parent's list, one or two
// rounds of cell loads, publication), and for large or deep trees the rounds' loads.
// A queue of cell pairs with atomics on its head and tail and on every list took 283 us
// at N = 1e6 (s = 96, p = 6), 244 us at 1e5 (s = 52) and 1030 us for 2.6e5 moonlets in
// leaves of 17; this takes 94, 60 and 176 us, and no list needs a sort afterwards.
#include <atomic>

#include "ncorp_internal.h"
#include "rcrit.h"

namespace ncorp {

constexpr uint32_t kSpinLimit = 1u << 20;    // empty polls in a row before giving up

__device__ __forceinline__ uint64_t ld_relaxed(const uint64_t *p) {
    return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ int32_t ld_relaxed(const int32_t *p) {
    return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ void st_relaxed(int32_t *p, int32_t v) {
    __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// Sets up a walk: hand-down headers empty, counters at zero; with do_rcrit also the
// cells' opening angles, critical radii and walk records (the gravity climb then leaves
// them out).
__global__ void k_walk_init(DevState *st, WalkQueue *wq, uint64_t *hdr, int32_t *ctr, int nctr,
                            int mode, const RcritArgs R, int do_rcrit) {
    const int nc = st->ncells;
    const bool go = nc > 0 && !(st->status & kSkipMask);
    const int64_t gid = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    const int64_t gstride = (int64_t)gridDim.x * blockDim.x;
    if (go)
        for (int64_t c = gid; c < nc; c += gstride) {
            hdr[c] = 0ull;
            if (do_rcrit) rcrit_cell(R, (int)c);
        }
    for (int64_t t = gid; t < nctr; t += gstride) ctr[t] = 0;
    if (gid != 0) return;
    wq->ncells = go ? nc : 0;
    if (mode == 0) {
        st->nsplit = 0; st->nlong = 0;
    } else {
        st->npairs = 0; st->col_tests = 0;      // of the search on this walk's candidates
    }
}

// Per-wave LDS.  kStack bounds the open pairs of a cell: a round is cut down until
// what it pushes leaves kStackFree entries, and below that the walk is depth first on
// one pair (at most 7 more entries a level, 21 levels).
constexpr int kStack = 640;
constexpr int kStackFree = 160;
static_assert(7 * kMaxDepth < kStackFree, "a depth-first descent must fit");
// hand-down entries staged: the cell's own, and what it inherits (as much as a slot holds)
constexpr int kDownOwn = 192, kDownInherit = 64, kDown = kDownOwn + kDownInherit;
static_assert(kDownInherit == kWalkInline && kDownOwn >= kWave, "a slot, and a round");
struct WalkLds {
    int32_t stack[kStack];
    int32_t down[kDown];
    int held[kWalkHeld];                     // cells put aside
};
static_assert(kMaxDepth + 2 < kWalkHeld, "a cell a level, and the next one");
template <int MODE> struct WalkPairs { int2 p[kCandBuf]; };      // collisions: candidates staged
template <> struct WalkPairs<0> { int2 p[1]; };

// A hand-down list is published as one 64-bit header per cell: valid | inline | linked |
// above | slack (16 bits, see below) | direct | entry count (9 bits) | offset (32 bits) of
// its last segment in the list space.  A list of up to WalkArgs.inl entries sits in the
// cell's own slot of inl entries; a longer one in segments of the shared space, of which
// all but the first start with the offset and the size (and link) of the one before.  An
// entry is a cell B, with kDownDirect set where (A, B) is a direct-sum pair ("direct": the
// list has some).
//
// A leaf below A inherits A's direct-sum pairs.  A cell that comes in between copies what
// its parent's list has of them into its own slot, after its own entries, if all that fits;
// if not it copies none and is marked "above": the leaf then goes up its ancestors' lists,
// from the parent to the first that is not marked, and takes their direct-sum pairs.  The
// leaf meets them in the same order either way.  So the shared space holds nobody's
// inheritance, and what it needs is bounded by the visits (list_space).
constexpr int32_t kDownDirect = (int32_t)0x80000000;
constexpr int kDownCount = 0x1ff, kDownLinked = 0x200;       // a segment's size and link
constexpr uint32_t kHdrInline = 1u << 30, kHdrLinked = 1u << 29, kHdrAbove = 1u << 28,
                   kHdrDirect = 1u << 11;                    // in the header's upper half
static_assert(kDownOwn <= kDownCount && kWalkInline <= kDownCount, "counts of 9 bits");
__device__ __forceinline__ uint64_t down_header(uint32_t flags, uint32_t slack16, int n,
                                                uint32_t off) {
    return ((uint64_t)(0x80000000u | flags | (slack16 << 12) | (uint32_t)n) << 32) | off;
}
// The smallest r_crit - r_max of a cell and its ancestors, as the upper half of a float,
// rounded towards zero: the moonlets of a cell and of any well-separated partner are at
// least that far apart, which spares the collision search most M2L lists.
__device__ __forceinline__ uint32_t slack_bits(double v) {
    return v > 0.0 ? (uint32_t)__float_as_int(__double2float_rz(v)) >> 16 : 0u;
}

struct WalkArgs {
    DevState *st;
    WalkQueue *wq;
    const WCell *__restrict__ cell;
    int ncs, ncc_pre, ncc_post;
    uint64_t *hdr;                       // hand-down header of every cell
    int32_t *space;                      // hand-down lists: inl entries a cell, then shared
    int32_t *ctr;                        // counters of the classes (walk_ctr)
    int inl;
    int64_t shared0, shared_n;           // shared part: kXcds regions of shared_n entries
    int64_t visit_cap;                   // most pairs a walk may visit
    CandOut cand;                        // collisions: candidate cell pairs
    // gravity: per-target lists; per leaf, the slack of its chain
    int32_t *m2l_cnt, *m2l_seg, *p2p_cnt, *p2p_seg;
    int m2l_stride, p2p_stride;
    const double *c_rmax;
    float *leaf_slack;
    uint32_t *leaf_src;                  // per leaf: source moonlets of its direct sums
    int timing;                          // record the waves' busy cycles
};

__device__ __forceinline__ void latch_cap(DevState *st, int32_t bit, int64_t need) {
    atomicOr(&st->status, bit);
    atomicMax((unsigned long long *)&st->required, (unsigned long long)need);
}

// n words of the shared list space, from this XCD's region or the next with room; returns
// their offset, or -1 when no region has any: the walk then visits more than queue_cap
// pairs, by how many is not known, and twice the capacity is asked for.
__device__ __forceinline__ int64_t take_space(const WalkArgs &A, int xcd, int n, int lane) {
    for (int t = 0; t < kXcds; t++) {
        const int x = (xcd + t) % kXcds;
        int old = 0;
        if (lane == 0) old = atomicAdd(walk_ctr(A.ctr, x, kCtrSpace), n);
        old = __builtin_amdgcn_readfirstlane(old);
        if (old >= 0 && (int64_t)old + n <= A.shared_n)
            return A.shared0 + (int64_t)x * A.shared_n + old;
        if (lane == 0) atomicSub(walk_ctr(A.ctr, x, kCtrSpace), n);   // no room: taken back
    }
    const int64_t twice = 2 * A.visit_cap;
    if (lane == 0)
        latch_cap(A.st, ST_CAP_QUEUE,
                  twice > kMaxQueue && A.visit_cap < kMaxQueue ? kMaxQueue : twice);
    return -1;
}

// Writes the staged hand-down entries as a segment after (poff, pn), which it replaces.
__device__ __forceinline__ void flush_down(const WalkArgs &A, int xcd, const int32_t *down, int &n,
                                           int lane, int &poff, int &pn) {
    const int head = poff >= 0 ? 2 : 0;
    const int64_t off = take_space(A, xcd, n + head, lane);
    if (off >= 0) {
        wave_sync();
        if (lane < head) st_relaxed(&A.space[off + lane], lane == 0 ? poff : pn);
        for (int i = lane; i < n; i += kWave) st_relaxed(&A.space[off + head + i], down[i]);
        wave_sync();
        poff = (int)off;
        pn = n | (head ? kDownLinked : 0);
    }
    n = 0;
}

// a cell's header, wave-uniform (upper 0: not published)
struct Header {
    uint32_t lower, upper;
};
__device__ __forceinline__ Header read_header(const WalkArgs &A, int cell) {
    const uint64_t h = ld_relaxed(&A.hdr[cell]);
    return {(uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)h),
            (uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)(h >> 32))};
}

// What is left to take of a hand-down list: one segment, and the one before it.
struct DownReader {
    int64_t off = 0;
    int n = 0, prev = -1, prev_n = 0;

    // the segment of size and link `pn` at o
    __device__ __forceinline__ void segment(const int32_t *space, int64_t o, int pn) {
        n = pn & kDownCount;
        prev = -1;
        if (pn & kDownLinked) {
            prev = __builtin_amdgcn_readfirstlane(ld_relaxed(&space[o]));
            prev_n = __builtin_amdgcn_readfirstlane(ld_relaxed(&space[o + 1]));
            o += 2;
        }
        off = o;
    }
    // the list of a cell with header h
    __device__ __forceinline__ void list(const WalkArgs &A, int cell, const Header &h) {
        const int count = (int)(h.upper & kDownCount);
        if (h.upper & kHdrInline) segment(A.space, (int64_t)cell * A.inl, count);
        else segment(A.space, h.lower, count | (h.upper & kHdrLinked ? kDownLinked : 0));
    }
};

// the classes' ticket counters (WaveTurns)
struct Tickets {
    int32_t *ctr;
    int lane;
    __device__ int take(int cls) const {
        return lane == 0 ? atomicAdd(walk_ctr(ctr, cls, kCtrTicket), 1) : 0;
    }
    __device__ int value(int v) const { return __builtin_amdgcn_readlane(v, 0); }
    __device__ int taken(int cls) const {
        return __builtin_amdgcn_readfirstlane(ld_relaxed(walk_ctr(ctr, cls, kCtrTicket)));
    }
    __device__ bool claim(int cls, int t) const {
        int old = 0;
        if (lane == 0) old = atomicCAS(walk_ctr(ctr, cls, kCtrTicket), t, t + 1);
        return __builtin_amdgcn_readlane(old, 0) == t;
    }
};

template <int MODE>
__global__ void __launch_bounds__(kWalkBlock, 6) k_walk(const WalkArgs A) {
    constexpr int WPB = kWalkBlock / kWave;
    __shared__ WalkLds lds_all[WPB];
    __shared__ WalkPairs<MODE> pairs_all[WPB];
    __shared__ unsigned long long s_visited, s_busy, s_busymax;
    __shared__ int s_m2l, s_p2p, s_longm, s_longp, s_left;
    const int lane = threadIdx.x % kWave;
    WalkLds &W = lds_all[threadIdx.x / kWave];
    int2 *const pbuf = pairs_all[threadIdx.x / kWave].p;
    if (threadIdx.x == 0) { s_visited = s_busy = s_busymax = 0; s_m2l = s_p2p = s_longm = s_longp = 0; s_left = WPB; }
    __syncthreads();
    const int nc = A.wq->ncells;
    const int cls = (int)blockIdx.x % kWalkClasses, xcd = cls % kXcds;
    const uint64_t lt = lane == 0 ? 0ull : (~0ull >> (64 - lane));
    const long long t_start = (MODE == 0 && A.timing) ? clock64() : 0;
    unsigned long long visited = 0;
    int nm2l = 0, np2p = 0, nlongm = 0, nlongp = 0;           // pairs of the cells taken; long lists
    int npb = 0;                                  // candidates staged
    const Tickets tickets = {A.ctr, lane};
    WaveTurns turns;
    turns.start(tickets, cls);
    int c = 0;
    while (turns.get(tickets, W.held, nc, c)) {
        const WCell wa = A.cell[c];
        const int par = wa.parent;
        const bool leaf = wa.nchild == 0;
        int top = 0;                              // open pairs on the stack
        uint32_t slack = 0;
        if (MODE == 0) slack = slack_bits(wa.rcrit - A.c_rmax[c]);
        DownReader in;                            // the parent's list (then its ancestors')
        int anc = par;                            // whose it is
        bool above = false;                       // direct-sum pairs to inherit from beyond it
        if (par < 0) {
            if (lane == 0) W.stack[0] = c;
            top = 1;
        } else {
            Header h;
            uint32_t spins = 0;
            bool aside = false;
            for (;;) {
                h = read_header(A, par);
                if (h.upper != 0 || ++spins > kSpinLimit) break;
                if ((spins & (turns.patience - 1)) == 0 && (aside = turns.help(tickets, W.held, c, par)))
                    break;
                if (spins < 16) __builtin_amdgcn_s_sleep(4);
                else __builtin_amdgcn_s_sleep(16);
            }
            if (aside) continue;
            if (h.upper == 0) {                   // waited too long
                if (lane == 0) atomicOr(&A.st->status, (int32_t)ST_WALK_STALL);
                break;
            }
            const uint32_t ps = (h.upper >> 12) & 0xffffu;
            slack = ps < slack ? ps : slack;
            above = MODE == 0 && (h.upper & kHdrAbove);
            in.list(A, par, h);
        }
        unsigned src = 0;                         // this lane's direct-sum sources
        int nm = 0, np = 0, nd = 0, ni = 0;       // own lists, staged own and inherited entries
        bool direct_down = false;                 // own direct-sum pairs among those
        int seg_off = -1, seg_n = 0;              // last hand-down segment written
        int32_t *const mrow = MODE == 0 ? A.m2l_seg + (int64_t)c * A.m2l_stride : nullptr;
        int32_t *const prow = MODE == 0 ? A.p2p_seg + (int64_t)wa.entry * A.p2p_stride : nullptr;
        for (;;) {
            // ---- take entries of the parent's list while the stack is short
            while (top < kWave) {
                if (in.n == 0) {
                    if (in.prev >= 0) {           // the segment before this one
                        in.segment(A.space, in.prev, in.prev_n);
                    } else if (leaf && above) {   // what the ancestor above has to inherit
                        anc = A.cell[anc].parent;
                        const Header h = read_header(A, anc);   // its child has waited for it
                        above = h.upper & kHdrAbove;
                        if (h.upper & kHdrDirect) in.list(A, anc, h);
                        if (h.upper == 0 && lane == 0)
                            atomicOr(&A.st->status, (int32_t)ST_BAD_ITEM);
                    } else {
                        break;
                    }
                    continue;
                }
                const int m = in.n;               // a whole segment
                constexpr int kRounds = kDownOwn / kWave;
                static_assert(kRounds * kWave == kDownOwn && kWalkInline <= kDownOwn, "whole rounds");
                int32_t e[kRounds];
#pragma unroll
                for (int u = 0; u < kRounds; u++)
                    e[u] = u * kWave + lane < m ? ld_relaxed(&A.space[in.off + u * kWave + lane]) : 0;
                in.n = 0;
#pragma unroll
                for (int u = 0; u < kRounds; u++) {
                    if (u * kWave >= m) break;
                    const bool have = u * kWave + lane < m;
                    const uint64_t md = MODE == 0 ? __ballot(have && e[u] < 0) : 0ull;
                    if (md == 0 && anc == par) {
                        if (have) W.stack[top + lane] = e[u];
                        top += m - u * kWave < kWave ? m - u * kWave : kWave;
                        continue;
                    }
                    // direct-sum pairs, and of an ancestor's list nothing else
                    if (leaf) {
                        const int B = e[u] & 0x7fffffff, pos = np + __popcll(md & lt);
                        if (have && e[u] < 0) {
                            if ((uint32_t)B >= (uint32_t)nc) {       // cannot happen either
                                atomicOr(&A.st->status, (int32_t)ST_BAD_ITEM);
                            } else {
                                if (pos < A.p2p_stride) prow[pos] = B;
                                src += (unsigned)A.cell[B].count;
                            }
                        }
                        np += __popcll(md);
                        if (anc != par) continue;
                    } else {
                        const int pos = ni + __popcll(md & lt);
                        if (have && e[u] < 0 && pos < kDownInherit) W.down[kDownOwn + pos] = e[u];
                        ni += __popcll(md);
                    }
                    const uint64_t mo = __ballot(have && e[u] >= 0);
                    if ((mo >> lane) & 1) W.stack[top + __popcll(mo & lt)] = e[u];
                    top += __popcll(mo);
                }
            }
            if (top == 0) break;
            wave_sync();
            // ---- classify up to 64 open pairs (A, B)
            int k = top < kWave ? top : kWave;
            int kind = 0, B = 0, child = 0, npush = 0, tot = 0, off = 0, cnt = 0;
            int32_t down = 0;
            for (;;) {
                kind = 0; npush = 0; down = 0; B = -1; child = 0; cnt = 0;
                if (lane < k) {
                    B = W.stack[top - 1 - lane];
                    if ((uint32_t)B >= (uint32_t)nc) {    // cannot happen; never follow it
                        atomicOr(&A.st->status, (int32_t)ST_BAD_ITEM);
                        B = -1;
                    } else if (B == c) {
                        if (wa.count <= A.ncs || leaf) { kind = 2; down = B | kDownDirect; cnt = wa.count; }
                        else { kind = 4; down = B; }
                    } else {
                        const WCell wb = A.cell[B];
                        child = wb.child;
                        if (B == par) {
                            kind = 5;                     // the parent's self pair: all siblings
                            npush = wb.nchild;
                        } else {
                            const int64_t prod = (int64_t)wa.count * (int64_t)wb.count;
                            if (prod < (int64_t)A.ncc_pre) {
                                kind = 2;
                            } else {
                                const double dx = wa.x - wb.x, dy = wa.y - wb.y, dz = wa.z - wb.z;
                                const double d = sqrt(dx * dx + dy * dy + dz * dz);
                                if (wa.rcrit + wb.rcrit <= d) {
                                    kind = 1;
                                } else if (prod < (int64_t)A.ncc_post ||
                                           (leaf && wb.nchild == 0)) {
                                    kind = 2;
                                } else {
                                    // Alg. 2 opens the first of the pair (the one with
                                    // the earlier moonlets) if the second is a leaf or
                                    // has the smaller critical radius, else the second
                                    const bool early = wa.first < wb.first;
                                    const int n1 = early ? wa.nchild : wb.nchild;
                                    const int n2 = early ? wb.nchild : wa.nchild;
                                    const double r1 = early ? wa.rcrit : wb.rcrit;
                                    const double r2 = early ? wb.rcrit : wa.rcrit;
                                    const bool open1 = n2 == 0 || (n1 != 0 && r1 > r2);
                                    if (open1 == early) { kind = 4; down = B; }
                                    else { kind = 6; npush = wb.nchild; }
                                }
                            }
                            if (kind == 2) { down = B | kDownDirect; cnt = wb.count; }
                        }
                    }
                }
                int x = npush;                    // wave prefix sum of the pushes
#pragma unroll
                for (int o = 1; o < kWave; o <<= 1) {
                    const int t = __shfl_up(x, o);
                    if (lane >= o) x += t;
                }
                tot = __builtin_amdgcn_readlane(x, kWave - 1);
                off = x - npush;
                if (k == 1 || top - k + tot <= kStack - kStackFree) break;
                k = k > 4 ? k / 4 : 1;
            }
            wave_sync();
            top -= k;
            for (int q = 0; q < npush; q++) W.stack[top + off + q] = child + q;
            top += tot;
            visited += __popcll(__ballot(B >= 0 && kind != 5 && c <= B));
            // ---- A's own lists
            if (MODE == 0) {
                const uint64_t m1 = __ballot(kind == 1);
                if (m1) {
                    const int pos = nm + __popcll(m1 & lt);
                    if (kind == 1 && pos < A.m2l_stride) mrow[pos] = B;
                    nm += __popcll(m1);
                    nm2l += __popcll(__ballot(kind == 1 && c < B));
                }
            }
            const bool direct = kind == 2;
            const uint64_t m2 = __ballot(direct);
            if (m2) {
                if (MODE == 0 && leaf) {
                    const int pos = np + __popcll(m2 & lt);
                    if (direct && pos < A.p2p_stride) prow[pos] = B;
                    if (direct) src += (unsigned)cnt;
                    np += __popcll(m2);
                }
                const uint64_t mo = __ballot(direct && c <= B);      // once per unordered pair
                np2p += __popcll(mo);
                if (MODE == 1) {
                    if (direct && c <= B) pbuf[npb + __popcll(mo & lt)] = make_int2(c, B);
                    npb += __popcll(mo);
                    if (npb > kCandBuf - kWave) flush_cand(pbuf, npb, lane, cls, A.cand, A.st);
                }
            }
            const bool todown = kind == 4 || (MODE == 0 && direct && !leaf);
            const uint64_t md = __ballot(todown);
            if (md) {
                if (MODE == 0) direct_down = direct_down || __any(direct);
                if (nd + __popcll(md) > kDownOwn) flush_down(A, xcd, W.down, nd, lane, seg_off, seg_n);
                if (todown) W.down[nd + __popcll(md & lt)] = down;
                nd += __popcll(md);
            }
        }
        // ---- publish: the children may start
        if (!leaf) {
            uint64_t h;
            const bool copied = MODE == 0 && !above && seg_off < 0 && nd + ni <= A.inl;
            uint32_t flags = (above || (ni > 0 && !copied) ? kHdrAbove : 0u) |
                             (direct_down || (copied && ni > 0) ? kHdrDirect : 0u);
            if (seg_off < 0 && nd <= A.inl) {
                const int all = copied ? nd + ni : nd;
                wave_sync();
                for (int q = lane; q < all; q += kWave)
                    st_relaxed(&A.space[(int64_t)c * A.inl + q],
                               W.down[q < nd ? q : kDownOwn + (q - nd)]);
                h = down_header(flags | kHdrInline, slack, all, 0u);
            } else {
                if (nd > 0) flush_down(A, xcd, W.down, nd, lane, seg_off, seg_n);
                if (seg_n & kDownLinked) flags |= kHdrLinked;
                h = down_header(flags, slack, seg_off < 0 ? 0 : seg_n & kDownCount,
                                seg_off < 0 ? 0u : (uint32_t)seg_off);
            }
            __atomic_signal_fence(__ATOMIC_SEQ_CST);
            __builtin_amdgcn_s_waitcnt(0);        // the entries are stored
            __atomic_signal_fence(__ATOMIC_SEQ_CST);
            if (lane == 0)
                __hip_atomic_store(&A.hdr[c], h, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        }
        if (MODE == 0) {
            if (leaf)
                for (int o = kWave / 2; o > 0; o >>= 1) src += __shfl_xor(src, o);
            if (lane == 0) {
                A.m2l_cnt[c] = nm;
                if (leaf) {
                    A.p2p_cnt[wa.entry] = np;
                    A.leaf_src[wa.entry] = src;
                    A.leaf_slack[wa.entry] = __int_as_float((int)(slack << 16));
                }
                if (nm > A.m2l_stride) latch_cap(A.st, ST_CAP_LISTS, nm);
                if (np > A.p2p_stride) latch_cap(A.st, ST_CAP_LISTS, np);
            }
            if (nm > kM2LListLDS) nlongm++;
            if (leaf && np > kP2PListLDS) nlongp++;
        }
        wave_sync();
    }
    if (MODE == 1) flush_cand(pbuf, npb, lane, cls, A.cand, A.st);
    if (lane == 0) {
        // the block's counts, added to its class's by the last wave
        atomicAdd(&s_visited, visited);
        atomicAdd(&s_m2l, nm2l);
        atomicAdd(&s_p2p, np2p);
        atomicAdd(&s_longm, nlongm);
        atomicAdd(&s_longp, nlongp);
        if (MODE == 0 && A.timing) {
            const unsigned long long busy = (unsigned long long)(clock64() - t_start);
            atomicAdd(&s_busy, busy);
            atomicMax(&s_busymax, busy);
        }
        if (atomicSub(&s_left, 1) == 1) {
            const unsigned long long v = atomicAdd(&s_visited, 0ull);
            const int m = atomicAdd(&s_m2l, 0), p = atomicAdd(&s_p2p, 0);
            const int lm = atomicAdd(&s_longm, 0), lp = atomicAdd(&s_longp, 0);
            if (v) atomicAdd((unsigned long long *)walk_ctr(A.ctr, cls, kCtrVisited), v);
            if (m) atomicAdd(walk_ctr(A.ctr, cls, kCtrM2L), m);
            if (p) atomicAdd(walk_ctr(A.ctr, cls, kCtrP2P), p);
            if (lm) atomicAdd(walk_ctr(A.ctr, cls, kCtrLongM2L), lm);
            if (lp) atomicAdd(walk_ctr(A.ctr, cls, kCtrLongP2P), lp);
            if (MODE == 0 && A.timing) {
                atomicAdd((unsigned long long *)walk_ctr(A.ctr, cls, kCtrBusy), atomicAdd(&s_busy, 0ull));
                atomicMax((unsigned long long *)walk_ctr(A.ctr, cls, kCtrBusyMax),
                          atomicAdd(&s_busymax, 0ull));
                atomicAdd(walk_ctr(A.ctr, cls, kCtrWaves), WPB);
            }
        }
    }
}

// Workgroups of a walk: as many as fit on the chip at once (`most`, if positive, limits
// them), one wave per cell at most, and a multiple of the classes, whose tickets each
// need a taker.
template <int MODE>
static int walk_grid(int64_t cell_cap, int most) {
    static std::atomic<int> cached[64];             // per device; any thread fills it in
    int dev = 0;
    (void)hipGetDevice(&dev);
    int g = dev >= 0 && dev < 64 ? cached[dev].load(std::memory_order_relaxed) : 0;
    if (g == 0) {
        int per_cu = 0, ncu = 0;
        if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, (const void *)k_walk<MODE>,
                                                         kWalkBlock, 0) != hipSuccess ||
            hipDeviceGetAttribute(&ncu, hipDeviceAttributeMultiprocessorCount, dev) !=
                hipSuccess ||
            per_cu < 1 || ncu < 1) {
            (void)hipGetLastError();
            per_cu = 2;
            ncu = 256;
        }
        g = per_cu * ncu;
        if (dev >= 0 && dev < 64) cached[dev].store(g, std::memory_order_relaxed);
    }
    int64_t want = (cell_cap + kWalkBlock / kWave - 1) / (kWalkBlock / kWave);
    if (want > g) want = g;
    if (most > 0 && want > most) want = most;
    want = want / kWalkClasses * kWalkClasses;
    return (int)(want < kWalkClasses ? kWalkClasses : want);
}

// most: most workgroups of the gravity walk (0: as many as fit)
hipError_t launch_walk(Workspace &ws, int mode, int ncs, int ncc_pre, int ncc_post, int most,
                       hipStream_t s, const ncorp_params *rcrit_prm) {
    RcritArgs R = {};
    if (rcrit_prm) R = rcrit_args(ws, *rcrit_prm);
    // the headers take the other walk's cell records, which each walk's own climb
    // rewrites before they are read again
    uint64_t *hdr = reinterpret_cast<uint64_t *>(mode == 0 ? ws.wc : ws.wg);
    int64_t gi = (ws.cell_cap + 255) / 256;
    gi = gi < 1 ? 1 : (gi > 1024 ? 1024 : gi);
    k_walk_init<<<(int)gi, 256, 0, s>>>(ws.st, ws.wq, hdr, ws.walk_ctr,
                                        (mode == 0 ? kWalkClasses : kWalkClasses + kCandRegions) *
                                            kCtrStride,
                                        mode, R, rcrit_prm ? 1 : 0);
    WalkArgs A = {};
    A.st = ws.st; A.wq = ws.wq; A.hdr = hdr; A.ctr = ws.walk_ctr;
    A.ncs = ncs; A.ncc_pre = ncc_pre; A.ncc_post = ncc_post;
    const ListSpace sp = list_space(ws.space_words, ws.queue_cap, ws.cell_cap);
    A.space = ws.space;
    A.visit_cap = ws.queue_cap;
    A.inl = sp.inl;
    A.shared0 = sp.shared0;
    A.shared_n = sp.shared_n;
    if (mode == 0) {
        A.cell = ws.wg;
        A.m2l_cnt = ws.m2l_cnt; A.m2l_seg = ws.m2l_seg; A.m2l_stride = ws.m2l_stride;
        A.p2p_cnt = ws.p2p_cnt; A.p2p_seg = ws.p2p_seg; A.p2p_stride = ws.p2p_stride;
        A.c_rmax = ws.c_rmax;
        A.leaf_slack = ws.leaf_slack;
        A.leaf_src = ws.ent_work;
        A.timing = ws.timing ? 1 : 0;
        k_walk<0><<<walk_grid<0>(ws.cell_cap, most), kWalkBlock, 0, s>>>(A);
    } else {
        A.cell = ws.wc;
        A.cand = cand_out(ws);
        k_walk<1><<<walk_grid<1>(ws.cell_cap, 0), kWalkBlock, 0, s>>>(A);
    }
    return hipGetLastError();
}

// directed moonlet interactions of the direct sums: per leaf, its moonlets times
// the moonlets of all its sources, minus the i == j terms
__global__ void k_count_inter(DevState *st, const int32_t *__restrict__ ent_cell,
                              const int32_t *__restrict__ c_count,
                              const int32_t *__restrict__ p2p_cnt,
                              const int32_t *__restrict__ p2p_seg, int stride,
                              const int32_t *__restrict__ m2l_cnt) {
    if (st->status & kSkipMask) return;
    const int K = st->nleaves;
    unsigned long long tot = 0;
    long long smax = 0;
    int lp = 0, lm = 0;
    for (int e = blockIdx.x * blockDim.x + threadIdx.x; e < K || e < st->ncells;
         e += gridDim.x * blockDim.x) {
        if (e < st->ncells) lm = m2l_cnt[e] > lm ? m2l_cnt[e] : lm;
        if (e >= K) continue;
        lp = p2p_cnt[e] > lp ? p2p_cnt[e] : lp;
        const int nt = c_count[ent_cell[e]];
        const int32_t *seg = p2p_seg + (int64_t)e * stride;
        long long srcs = 0;
        for (int q = 0; q < p2p_cnt[e]; q++) srcs += c_count[seg[q]];
        tot += (unsigned long long)(nt * srcs - nt);
        smax = srcs > smax ? srcs : smax;
    }
    for (int o = kWave / 2; o > 0; o >>= 1) {
        tot += __shfl_xor(tot, o);
        const int a = __shfl_xor(lp, o), b = __shfl_xor(lm, o);
        lp = a > lp ? a : lp;
        lm = b > lm ? b : lm;
        const long long c = __shfl_xor(smax, o);
        smax = c > smax ? c : smax;
    }
    if (threadIdx.x % kWave == 0) {
        if (tot) atomicAdd((unsigned long long *)&st->p2p_inter, tot);
        if (lp) atomicMax(&st->p2p_maxlist, lp);
        if (lm) atomicMax(&st->m2l_maxlist, lm);
        if (smax) atomicMax((unsigned long long *)&st->p2p_src_max, (unsigned long long)smax);
    }
}

__global__ void k_zero_inter(DevState *st) {
    if (threadIdx.x == 0 && blockIdx.x == 0) {
        st->p2p_inter = 0;
        st->m2l_maxlist = 0;
        st->p2p_maxlist = 0;
        st->p2p_src_max = 0;
    }
}

hipError_t launch_count_interactions(const Workspace &ws, hipStream_t s) {
    k_zero_inter<<<1, 64, 0, s>>>(ws.st);
    if (!ws.p2p_cnt) return hipGetLastError();
    k_count_inter<<<256, 256, 0, s>>>(ws.st, ws.ent_cell, ws.c_count, ws.p2p_cnt, ws.p2p_seg,
                                      ws.p2p_stride, ws.m2l_cnt);
    return hipGetLastError();
}

}  // namespace ncorp
