// Flat octree from Hilbert-sorted keys (Sect. 3.4.1, Sect. 3.4.6).
//
// A cell is a key prefix; it is split iff it holds more than s moonlets and is
// above the depth cap.  With sorted keys the level of each moonlet's leaf follows
// from one sliding window: the level-l cell containing moonlet i holds more than
// s moonlets iff some window [j, j+s] containing i has its two end keys sharing
// l leading digits.  Leaves are then compacted in moonlet order ("entries"), and
// every entry e emits the cells of levels [dv_e, L_e] it starts (dv_e = first
// level where its key differs from the previous moonlet's).  Counting those per
// level gives each cell's breadth-first index directly: cells are ordered by
// level, then by key prefix, so children of consecutive parents are contiguous --
// the ordering the paper's flat tree uses.  No per-level kernel launches.
//
// Bound by launches and dependent loads at every size: three passes over the moonlets
// (levels and counts; entries and cells; ranges), with a scan of the blocks' counts
// between the first two only where there are too many blocks for each to add them up.
// Counting and emitting by moonlet instead of by entry needs no pass between (eight
// launches before, of which the cells' had one block per 1024 leaves): 1e5 moonlets,
// s = 48: 43 -> 24 us, 1e6: 80 -> 62 us.
//
// Batched calls build a forest: moonlets of different disks share no cell (their
// common-prefix length counts as -1), each disk's first moonlet starts all levels
// from 0, so level 0 holds one root per non-empty disk, in disk order.
#include "ncorp_internal.h"

namespace ncorp {

constexpr int kTreeBlock = 1024;
constexpr int kNLev = kMaxDepth + 1;          // levels 0..21
constexpr int kNCol = kNLev + 1;              // and the leaves
// blocks of moonlets up to which the emitting pass adds up the counts itself
constexpr int kAddBlocks = 128;
static_assert(kNCol <= 32, "a column per lane of half a wave");

__device__ __forceinline__ int cpl_digits(uint64_t a, uint64_t b) {
    if (a == b) return kMaxDepth;
    return (__clzll((long long)(a ^ b)) - 1) / 3;   // keys use bits 0..62
}

// lanes of the wave below this one
__device__ __forceinline__ uint64_t lanemask_lt64() {
    uint32_t l = threadIdx.x % kWave;
    return l == 0 ? 0ull : (~0ull >> (64 - l));
}

// code: L (bits 0-7), dv (bits 8-15), leaf-start flag (bit 16).  Also the block's leaves
// (partials) and cells per level (lcount[block][level]), and the positions in tree order
// from the packed records of the key pass: one 32-byte record per moonlet instead of three
// scattered words, and with the scaled masses in it the whole record (pos4), which the
// gravity climb and the direct sums read.
__global__ void __launch_bounds__(kTreeBlock)
k_leaf_levels(const uint64_t *__restrict__ keys, const uint16_t *__restrict__ seg, int64_t n,
              int s, uint32_t *__restrict__ code, int32_t *__restrict__ partials,
              int32_t *__restrict__ lcount, const double4 *__restrict__ pack4,
              const uint32_t *__restrict__ idx, double *__restrict__ xs, double *__restrict__ ys,
              double *__restrict__ zs, double4 *__restrict__ pos4) {
    extern __shared__ uint64_t sk[];                 // keys [b0 - s, b0 + B + s)
    int32_t *sc = (int32_t *)(sk + kTreeBlock + 2 * s);   // c(j), j in [b0 - s, b0 + B)
    uint16_t *sd = (uint16_t *)(sc + kTreeBlock + s);      // disk ids, same span as sk
    __shared__ int32_t red[kTreeBlock / kWave][kNCol];
    const int64_t b0 = (int64_t)blockIdx.x * kTreeBlock;
    const int span = kTreeBlock + 2 * s;
    const int64_t i = b0 + threadIdx.x;
    const uint32_t from = i < n ? idx[i] : 0u;
    for (int k = threadIdx.x; k < span; k += kTreeBlock) {
        int64_t j = b0 - s + k;
        const bool in = j >= 0 && j < n;
        sk[k] = in ? keys[j] : 0ull;
        sd[k] = (in && seg) ? seg[j] : (uint16_t)0;
    }
    double4 p;
    if (i < n) p = pack4[from];
    __syncthreads();
    for (int k = threadIdx.x; k < kTreeBlock + s; k += kTreeBlock) {
        int64_t j = b0 - s + k;
        sc[k] = (j >= 0 && j + s < n && sd[k] == sd[k + s]) ? cpl_digits(sk[k], sk[k + s]) : -1;
    }
    __syncthreads();
    int start = 0, L = -1, dv = 1;
    if (i < n) {
        int M = -1;
        int jlo = (int)(i - s < 0 ? 0 : i - s);
        for (int64_t j = jlo; j <= i; j++) {
            int c = sc[j - (b0 - s)];
            M = c > M ? c : M;
        }
        L = M + 1 < kMaxDepth ? M + 1 : kMaxDepth;
        if (i == 0 || sd[threadIdx.x + s - 1] != sd[threadIdx.x + s]) dv = 0;
        else {
            uint64_t a = sk[threadIdx.x + s - 1], b = sk[threadIdx.x + s];
            dv = (a == b) ? kMaxDepth + 1 : cpl_digits(a, b) + 1;
        }
        start = dv <= L;
        code[i] = (uint32_t)L | ((uint32_t)dv << 8) | ((uint32_t)start << 16);
        xs[i] = p.x;
        ys[i] = p.y;
        zs[i] = p.z;
        if (pos4) pos4[i] = p;
    }
    const int w = threadIdx.x / kWave, lane = threadIdx.x % kWave;
    int32_t mine = 0;                                // lane l: cells of level l, then leaves
#pragma unroll
    for (int l = 0; l < kNLev; l++) {
        const int c = __popcll(__ballot(dv <= l && l <= L));
        if (lane == l) mine = c;
    }
    const int leaves = __popcll(__ballot(start));
    if (lane == kNLev) mine = leaves;
    if (lane < kNCol) red[w][lane] = mine;
    __syncthreads();
    if (threadIdx.x < kNCol) {
        int t = 0;
        for (int k = 0; k < kTreeBlock / kWave; k++) t += red[k][threadIdx.x];
        if (threadIdx.x < kNLev) lcount[(int64_t)blockIdx.x * kNLev + threadIdx.x] = t;
        else partials[blockIdx.x] = t;
    }
}

// One block per level and one for the leaves: exclusive scan of the blocks' counts in
// place, and the total.
__global__ void __launch_bounds__(256)
k_level_scan(int32_t *lcount, int32_t *partials, int nb, DevState *st) {
    __shared__ int32_t sh[256];
    const int l = blockIdx.x;
    int32_t *v = l < kNLev ? lcount + l : partials;
    const int step = l < kNLev ? kNLev : 1;
    int32_t carry = 0;
    for (int b0 = 0; b0 < nb; b0 += 256) {
        int b = b0 + threadIdx.x;
        int32_t x = b < nb ? v[(int64_t)b * step] : 0;
        sh[threadIdx.x] = x;
        __syncthreads();
        for (int o = 1; o < 256; o <<= 1) {
            int32_t t = threadIdx.x >= o ? sh[threadIdx.x - o] : 0;
            __syncthreads();
            sh[threadIdx.x] += t;
            __syncthreads();
        }
        if (b < nb) v[(int64_t)b * step] = carry + sh[threadIdx.x] - x;
        carry += sh[255];
        __syncthreads();
    }
    if (threadIdx.x == 0) {
        if (l < kNLev) st->level_count[l] = carry;
        else st->nleaves = carry;
    }
}

// Every leaf start becomes an entry and writes the cells it starts, with parent and
// first-child links.  ADD: each block adds up the blocks' counts before it and in all
// (kAddBlocks and fewer: 9 KB from L2, less than the launch of the scan); otherwise
// k_level_scan did.  Each block forms the level offsets from the level totals; block 0
// also publishes them with the cell count and depth (and latches an overflow of cell_cap).
template <bool ADD>
__global__ void __launch_bounds__(kTreeBlock)
k_emit_cells(const uint32_t *__restrict__ code, int64_t n, int nb,
             const uint64_t *__restrict__ keys, const int32_t *__restrict__ lcount,
             const int32_t *__restrict__ partials,
             DevState *st, int64_t cell_cap, int32_t *__restrict__ c_level,
             int32_t *__restrict__ c_first, int32_t *__restrict__ c_child,
             int32_t *__restrict__ c_nchild, int32_t *__restrict__ c_parent,
             int32_t *__restrict__ c_entry, uint64_t *__restrict__ c_prefix,
             int32_t *__restrict__ ent_cell, const uint16_t *__restrict__ seg,
             int32_t *__restrict__ disk_root) {
    __shared__ int32_t wcnt[kTreeBlock / kWave][kNCol];
    __shared__ uint64_t wmask[kTreeBlock / kWave][kNLev];
    __shared__ int32_t pre[kNCol], tot[kNCol], loff[kNLev];
    const int w = threadIdx.x / kWave, lane = threadIdx.x % kWave;
    const int64_t i = (int64_t)blockIdx.x * kTreeBlock + threadIdx.x;
    const uint32_t c = i < n ? code[i] : 0x100u;
    const int start = (c >> 16) & 1;
    const int L = start ? (int)(c & 255u) : -1, dv = (c >> 8) & 255u;
    const uint64_t key = start ? keys[i] : 0ull;
    if (ADD) {
        if (threadIdx.x < kNCol) pre[threadIdx.x] = tot[threadIdx.x] = 0;
        __syncthreads();
        const int col = threadIdx.x % 32;
        if (col < kNCol) {
            int32_t before = 0, all = 0;
            for (int b = threadIdx.x / 32; b < nb; b += kTreeBlock / 32) {
                const int32_t v = col < kNLev ? lcount[b * kNLev + col] : partials[b];
                all += v;
                if (b < (int)blockIdx.x) before += v;
            }
            if (before) atomicAdd(&pre[col], before);
            if (all) atomicAdd(&tot[col], all);
        }
    } else if (threadIdx.x < kNCol) {
        const int l = threadIdx.x;
        pre[l] = l < kNLev ? lcount[(int64_t)blockIdx.x * kNLev + l] : partials[blockIdx.x];
        tot[l] = l < kNLev ? st->level_count[l] : 0;
    }
    // the cells each wave starts, per level, and which lanes start them
    int32_t mine = 0;
#pragma unroll
    for (int l = 0; l < kNLev; l++) {
        const uint64_t m = __ballot(dv <= l && l <= L);
        if (lane == l) {
            mine = __popcll(m);
            wmask[w][l] = m;
        }
    }
    const uint64_t mstart = __ballot(start);
    if (lane == kNLev) mine = __popcll(mstart);
    if (lane < kNCol) wcnt[w][lane] = mine;
    __syncthreads();
    if (threadIdx.x < kNCol) {
        int32_t run = pre[threadIdx.x];              // counts before each wave
        for (int k = 0; k < kTreeBlock / kWave; k++) {
            int32_t t = wcnt[k][threadIdx.x];
            wcnt[k][threadIdx.x] = run;
            run += t;
        }
    }
    if (threadIdx.x == kTreeBlock - 1) {
        int32_t off = 0, maxl = 0;
        for (int l = 0; l < kNLev; l++) {
            loff[l] = off;
            off += tot[l];
            if (tot[l] > 0) maxl = l;
        }
        if (blockIdx.x == 0) {
            for (int l = 0; l < kNLev; l++) {
                st->level_off[l] = loff[l];
                if (ADD) st->level_count[l] = tot[l];
            }
            if (ADD) st->nleaves = tot[kNLev];
            st->level_off[kNLev] = off;
            st->ncells = off;
            st->maxlevel = maxl;
            if (off > cell_cap) {
                atomicOr(&st->status, (int32_t)ST_CAP_CELLS);
                atomicMax((unsigned long long *)&st->required, (unsigned long long)off);
                st->ncells = (int32_t)cell_cap;   // later passes only see what was written
            }
        }
    }
    __syncthreads();
    if (!start) return;
    const uint64_t lt = lanemask_lt64();
    const int e = wcnt[w][kNLev] + __popcll(mstart & lt);
    // exclusive count of level-l cell starts before this moonlet
    auto excl = [&](int l) { return wcnt[w][l] + __popcll(wmask[w][l] & lt); };
    for (int l = dv; l <= L; l++) {     // the levels this entry starts
        int64_t ci = (int64_t)loff[l] + excl(l);
        if (ci >= cell_cap) continue;
        c_level[ci] = l;
        c_first[ci] = (int32_t)i;
        c_entry[ci] = (int32_t)e;
        c_prefix[ci] = key >> (3 * (kMaxDepth - l));
        if (l == 0) disk_root[seg ? seg[i] : 0] = (int32_t)ci;
        if (l < L) {
            c_child[ci] = loff[l + 1] + excl(l + 1);
        } else {
            c_child[ci] = -1;
            c_nchild[ci] = 0;
            ent_cell[e] = (int32_t)ci;
        }
        int32_t par = -1;
        if (l >= 1) {
            if (l - 1 >= dv) par = loff[l - 1] + excl(l - 1);          // also started here
            else par = loff[l - 1] + excl(l - 1) - 1;                  // last start before
        }
        c_parent[ci] = par;
    }
}

// child counts, moonlet counts and leaf ranges: walk up while this cell (or its
// ancestor) is the last child; the next sibling then starts where it ends.  An
// overflowed tree is unusable: it exposes no cells or leaves to later passes.  Also
// clears the coordinate maximum that the next build's key pass (or a step's drift
// before it) accumulates into, and the first climb's arrival and leaf counters.
__global__ void k_cell_ranges(DevState *st, int64_t n,
                              const int32_t *__restrict__ c_first, const int32_t *__restrict__ c_child,
                              const int32_t *__restrict__ c_parent, const int32_t *__restrict__ c_entry,
                              int32_t *__restrict__ c_count, int32_t *__restrict__ c_nchild,
                              int32_t *__restrict__ c_nent, int32_t *__restrict__ c_arrive,
                              int32_t *__restrict__ climb_next) {
    const bool first = blockIdx.x == 0 && threadIdx.x == 0;
    if (first) st->max_abs = 0.0;
    if (blockIdx.x == 0)
        for (int t = threadIdx.x; t < kClimbClasses; t += blockDim.x) climb_next[t * kCtrStride] = 0;
    if (st->status & ST_CAP_CELLS) {
        if (first) {
            st->ncells = 0;
            st->nleaves = 0;
        }
        return;
    }
    const int nc = st->ncells, K = st->nleaves;
    for (int c = blockIdx.x * blockDim.x + threadIdx.x; c < nc; c += gridDim.x * blockDim.x) {
        c_arrive[c] = 0;
        int par = c_parent[c];
        bool last_child = par >= 0 && (c + 1 >= nc || c_parent[c + 1] != par);
        if (last_child) c_nchild[par] = c - c_child[par] + 1;
        // roots (parent -1) are siblings of each other: the next root starts where
        // a root ends, and the last root ends at n
        int x = c;
        for (int up = 0; up <= kMaxDepth + 1 && x >= 0; up++) {   // bounded by the depth cap
            int px = c_parent[x];
            if (x + 1 < nc && c_parent[x + 1] == px) break;
            x = px;
        }
        int end, eend;
        if (x < 0) { end = (int)n; eend = K; }
        else { end = c_first[x + 1]; eend = c_entry[x + 1]; }
        c_count[c] = end - c_first[c];
        c_nent[c] = eend - c_entry[c];
    }
}


hipError_t launch_build_tree(const Workspace &ws, int64_t n, int s, bool with_mus,
                             hipStream_t st) {
    int nb = (int)((n + kTreeBlock - 1) / kTreeBlock);
    size_t shmem = (size_t)(kTreeBlock + 2 * s) * sizeof(uint64_t) +
                   (size_t)(kTreeBlock + s) * sizeof(int32_t) +
                   (size_t)(kTreeBlock + 2 * s) * sizeof(uint16_t);
    const uint16_t *seg = ws.ndisks > 1 ? ws.seg : nullptr;
    int32_t *lcount = ws.cnt_a;   // nb x kNLev
    k_leaf_levels<<<nb, kTreeBlock, shmem, st>>>(ws.keys, seg, n, s, ws.code, ws.scan_part, lcount,
                                                 ws.pack4, ws.idx, ws.xs, ws.ys, ws.zs,
                                                 with_mus ? ws.vcol : nullptr);
    const bool add = nb <= kAddBlocks;
    if (!add) k_level_scan<<<kNCol, 256, 0, st>>>(lcount, ws.scan_part, nb, ws.st);
    auto emit = add ? k_emit_cells<true> : k_emit_cells<false>;
    emit<<<nb, kTreeBlock, 0, st>>>(ws.code, n, nb, ws.keys, lcount, ws.scan_part, ws.st,
                                    ws.cell_cap, ws.c_level, ws.c_first, ws.c_child, ws.c_nchild,
                                    ws.c_parent, ws.c_entry, ws.c_prefix, ws.ent_cell, seg,
                                    ws.disk_root);
    int g = (int)((ws.cell_cap + 255) / 256);
    if (g > 2048) g = 2048;
    k_cell_ranges<<<g, 256, 0, st>>>(ws.st, n, ws.c_first, ws.c_child, ws.c_parent, ws.c_entry,
                                     ws.c_count, ws.c_nchild, ws.c_nent, ws.c_arrive,
                                     ws.climb_next);
    return hipGetLastError();
}

}  // namespace ncorp
