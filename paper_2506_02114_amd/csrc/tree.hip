// Quadtree of the FMM (sec. 3.3, app. C.1), built on the device.
//
// Stars are sorted by their Morton key at the finest level (24 bits per axis),
// so the stars of any square of any level are one contiguous range of the
// sorted array.  The tree is then built level by level from the root: a node
// is divided into four children when the stars of its 3x3 block of
// same-level squares (the node and its neighbours) exceed nmax.  A divided
// node always gets all four children, so every square of a level inside the
// root is a node or lies inside a leaf of a coarser level; each node keeps its
// 3x3 neighbourhood as such references ("colleagues"), found from its
// parent's in O(1), and the block count and the interaction lists follow
// from them without searching the whole key array.
#include <algorithm>
#include <atomic>
#include <chrono>
#include <cmath>

#include "cubic.hpp"
#include "dev.hpp"

namespace mlm {

namespace {

constexpr int BLK = 256;
constexpr int ACTIVE_LEAVES = MAX_LEVELS - 1;   // (no tree has that level)
constexpr int COARSE_NODES = 16384;             // nodes that one workgroup numbers at most

// first node of each level
struct LevelStarts {
    int32_t lo[MAX_LEVELS];
};

inline unsigned nblocks(int64_t n, int b = BLK) { return (unsigned)((n + b - 1) / b); }

__global__ void k_keys(const double *__restrict__ x, const double *__restrict__ y, int32_t n,
                       double L0, double scale, uint64_t *__restrict__ key, int32_t *__restrict__ idx)
{
    int32_t s = blockIdx.x * blockDim.x + threadIdx.x;
    if (s >= n) return;
    key[s] = morton2(fine_cell(x[s], L0, scale), fine_cell(y[s], L0, scale));
    idx[s] = s;
}

__global__ void k_gather(const int32_t *__restrict__ idx, const double *__restrict__ x,
                         const double *__restrict__ y, const double *__restrict__ m, int32_t n,
                         double *__restrict__ sx, double *__restrict__ sy, double *__restrict__ sm)
{
    int32_t s = blockIdx.x * blockDim.x + threadIdx.x;
    if (s >= n) return;
    int32_t k = idx[s];
    sx[s] = x[k];
    sy[s] = y[k];
    sm[s] = m[k];
}

__global__ void k_root(uint64_t *code, int32_t *level, int32_t *parent)
{
    code[0] = 0;
    level[0] = 0;
    parent[0] = -1;
}

// star range of a node's square: a sub-range of its parent's
__device__ inline void node_stars(int64_t q, int lev, const uint64_t *__restrict__ code,
                                  const int32_t *__restrict__ parent, const uint64_t *__restrict__ keys, int32_t n,
                                  int32_t *slo, int32_t *shi)
{
    if (lev == 0) {
        slo[q] = 0;
        shi[q] = n;
        return;
    }
    const uint64_t c = code[q];
    const int sh = 2 * (KEY_BITS - lev);
    const int32_t pq = parent[q], a = slo[pq], b = shi[pq];
    int32_t s0, s1;
    two_bounds_u64(keys, a, b, c << sh, (c + 1) << sh, s0, s1);
    slo[q] = s0;
    shi[q] = s1;
}

__global__ void k_level(int64_t lo, int64_t hi, int lev, const uint64_t *__restrict__ code,
                        const int32_t *__restrict__ parent, const uint64_t *__restrict__ keys, int32_t n,
                        int32_t *slo, int32_t *shi)
{
    const int64_t q = lo + (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (q < hi) node_stars(q, lev, code, parent, keys, n, slo, shi);
}

// square (a, b) of level lev, one of the children of the parent-level
// reference pc: its own reference
__device__ inline int32_t child_ref(int32_t pc, uint32_t a, uint32_t b, const int32_t *__restrict__ child0)
{
    if (pc == -1) return -1;
    if (pc <= -2) return pc;
    const int32_t c0 = child0[pc];
    return c0 >= 0 ? c0 + (int32_t)((a & 1u) | ((b & 1u) << 1)) : -(pc + 2);
}

// colleagues of a node (from its parent's) and the star count of its 3x3 block
// (each step of the nine chains parent's colleague, child, star range is loaded
// for all of them before the next, on any index where there is nothing to load:
// the pass is bound by the latency of its loads)
__device__ inline int32_t node_block(int64_t q, int lev, const uint64_t *code, const int32_t *parent,
                                     const int32_t *child0, const int32_t *slo, const int32_t *shi,
                                     const uint64_t *__restrict__ keys, int32_t *coll)
{
    const uint64_t c = code[q];
    const int64_t i = compact_bits(c), j = compact_bits(c >> 1), side = 1ll << lev;
    const int sh = 2 * (KEY_BITS - lev);
    const int32_t *pc = coll + (lev > 0 ? (int64_t)parent[q] * 9 : 0);
    int32_t up[9], c0[9], ref[9], n[9];
#pragma unroll
    for (int e = 0; e < 9; ++e) {
        const int64_t a = i + e % 3 - 1, b = j + e / 3 - 1;
        const int k = (int)((b >> 1) - (j >> 1) + 1) * 3 + (int)((a >> 1) - (i >> 1) + 1);
        up[e] = pc[k];
        if (lev == 0 || a < 0 || b < 0 || a >= side || b >= side) up[e] = -1;
    }
#pragma unroll
    for (int e = 0; e < 9; ++e) c0[e] = child0[max(up[e], 0)];
#pragma unroll
    for (int e = 0; e < 9; ++e) {
        const uint32_t a = (uint32_t)(i + e % 3 - 1), b = (uint32_t)(j + e / 3 - 1);
        ref[e] = up[e] < 0 ? up[e] : c0[e] >= 0 ? c0[e] + (int32_t)((a & 1u) | ((b & 1u) << 1)) : -(up[e] + 2);
        if (lev == 0 && e == 4) ref[e] = (int32_t)q;
    }
#pragma unroll
    for (int e = 0; e < 9; ++e) n[e] = shi[max(ref[e], 0)] - slo[max(ref[e], 0)];
    int32_t blk = 0;
#pragma unroll
    for (int e = 0; e < 9; ++e) blk += ref[e] >= 0 ? n[e] : 0;
#pragma unroll
    for (int e = 0; e < 9; ++e)
        if (ref[e] <= -2) {
            int32_t s0, s1;
            ref_stars(ref[e], morton2((uint32_t)(i + e % 3 - 1), (uint32_t)(j + e / 3 - 1)), sh, slo, shi, keys, s0, s1);
            blk += s1 - s0;
        }
#pragma unroll
    for (int e = 0; e < 9; ++e) coll[q * 9 + e] = ref[e];
    return blk;
}

__global__ void k_block(int64_t lo, int64_t hi, int lev, int lmax, int nmax, const uint64_t *__restrict__ code,
                        const int32_t *__restrict__ parent, const int32_t *__restrict__ child0,
                        const int32_t *__restrict__ slo, const int32_t *__restrict__ shi,
                        const uint64_t *__restrict__ keys, int32_t *coll, int32_t *__restrict__ block,
                        int32_t *__restrict__ split)
{
    const int64_t q = lo + (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (q >= hi) return;
    const int32_t blk = node_block(q, lev, code, parent, child0, slo, shi, keys, coll);
    block[q] = blk;
    split[q - lo] = (blk > nmax && lev < lmax) ? 1 : 0;
}

// the children of a divided node at cb .. cb + 3, in Morton order
__device__ inline void emit_children(int64_t q, int64_t cb, bool split, uint64_t *code, int32_t *level,
                                     int32_t *parent, int32_t *child0, int32_t *leaf, int next_level)
{
    leaf[q] = split ? 0 : 1;
    child0[q] = split ? (int32_t)cb : -1;
    if (!split) return;
    const uint64_t c = code[q] << 2;
    for (int quad = 0; quad < 4; ++quad) {
        code[cb + quad] = c | (uint64_t)quad;
        parent[cb + quad] = (int32_t)q;
        level[cb + quad] = next_level;
    }
}

__global__ void k_emit(int64_t lo, int64_t hi, int64_t base, const int32_t *__restrict__ split,
                       const int32_t *__restrict__ offs, uint64_t *code, int32_t *level, int32_t *parent,
                       int32_t *child0, int32_t *leaf, int next_level)
{
    int64_t q = lo + (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (q >= hi) return;
    emit_children(q, base + 4 * (int64_t)offs[q - lo], split[q - lo] != 0, code, level, parent, child0, leaf, next_level);
}

__global__ void k_leaf_index(int64_t nnodes, const int32_t *__restrict__ leaf,
                             const int32_t *__restrict__ offs, int32_t *__restrict__ node_leaf,
                             int32_t *__restrict__ leaf_node)
{
    int64_t q = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (q >= nnodes) return;
    if (leaf[q]) {
        node_leaf[q] = offs[q];
        leaf_node[offs[q]] = (int32_t)q;
    } else {
        node_leaf[q] = -1;
    }
}

__global__ void k_zero_first(int64_t *p) { p[0] = 0; }

__global__ void k_zero_counts(int32_t *p, int n)
{
    if ((int)threadIdx.x < n) p[threadIdx.x] = 0;
}

// The check of the points of a deflection: the points read once (copied to the
// host and looked at there, 400,000 points took 0.6 ms of the call's 2.0).
constexpr int OUTSIDE_BLOCKS = 512;

// part[block]: the first coordinate of the block's share that is not within
// (-L0, L0), or n
__global__ __launch_bounds__(BLK) void k_outside(const double *__restrict__ z, int64_t n, double L0,
                                                 int64_t *__restrict__ part)
{
    __shared__ unsigned long long first;
    if (threadIdx.x == 0) first = (unsigned long long)n;
    __syncthreads();
    int64_t bad = n;
    for (int64_t i = (int64_t)blockIdx.x * BLK + threadIdx.x; i < n; i += (int64_t)gridDim.x * BLK)
        if (!(fabs(z[i]) < L0)) {
            bad = i;
            break;
        }
    if (bad < n) atomicMin(&first, (unsigned long long)bad);
    __syncthreads();
    if (threadIdx.x == 0) part[blockIdx.x] = (int64_t)first;
}

// the least of the parts to total_dev or the host
__global__ __launch_bounds__(64) void k_outside_first(const int64_t *__restrict__ part, int np, int64_t n,
                                                      int64_t *total_dev, int64_t *total_host, int64_t seq)
{
    int64_t m = n;
    for (int i = threadIdx.x; i < np; i += 64) m = min(m, part[i]);
    for (int d = 32; d; d >>= 1) m = min(m, (int64_t)__shfl_xor((long long)m, d, 64));
    if (threadIdx.x == 0) {
        if (total_dev) *total_dev = m;
        if (total_host) store_host_total(total_host, m, seq);
    }
}

// Which rows and columns of the lattice hit the widened map: a workgroup takes
// LAT_ROWS rows, a thread every BLK-th column of them.
constexpr int LAT_ROWS = 4;

__global__ __launch_bounds__(BLK) void k_lattice(CubicSearch S, LatticeBox *__restrict__ part)
{
    __shared__ LatticeBox B;
    if (threadIdx.x == 0) B = LatticeBox{LAT, -1, LAT, -1};
    __syncthreads();
    LatticeBox b{LAT, -1, LAT, -1};
    for (int j = blockIdx.x * LAT_ROWS; j < (int)(blockIdx.x + 1) * LAT_ROWS; ++j) {
        const double y = S.y(j);
        for (int i = threadIdx.x; i < LAT; i += BLK)
            if (S.hit(S.x(i), y)) {
                b.i0 = min(b.i0, i);
                b.i1 = max(b.i1, i);
                b.j0 = min(b.j0, j);
                b.j1 = max(b.j1, j);
            }
    }
    if (b.i1 >= 0) {
        atomicMin(&B.i0, b.i0);
        atomicMax(&B.i1, b.i1);
        atomicMin(&B.j0, b.j0);
        atomicMax(&B.j1, b.j1);
    }
    __syncthreads();
    if (threadIdx.x == 0) part[blockIdx.x] = B;
}

// the counts of the large-triangle lists, then the sequence number, to the host
__global__ __launch_bounds__(BIG_SHARDS) void k_publish_counts(const unsigned long long *__restrict__ count,
                                                               int64_t *host, int64_t seq)
{
    host[2 + threadIdx.x] = (int64_t)count[(size_t)threadIdx.x * BIG_STRIDE];
    __threadfence_system();
    __syncthreads();
    if (threadIdx.x == 0) __hip_atomic_store(host + 1, seq, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
}

// (dst: pinned host memory)
__global__ void k_copy_counts(const int32_t *__restrict__ src, int32_t *dst, int n)
{
    if ((int)threadIdx.x < n) dst[threadIdx.x] = src[threadIdx.x];
    __threadfence_system();
}

// The nodes of levels >= 2 whose square meets the rays' rectangle, listed level
// by level (level lev's from act[level_lo[lev]] on, in no particular order:
// nodes are evaluated independently) and counted in cnt[lev] (zeroed), the
// leaves among them in cnt[ACTIVE_LEAVES].  Lanes
// of a wavefront whose nodes share a level take one range of its list.
__global__ __launch_bounds__(BLK) void k_active(int64_t lo, int64_t hi, double L0, RayBox box,
                                                const uint64_t *__restrict__ code,
                                                const int32_t *__restrict__ level,
                                                const int32_t *__restrict__ leaf, LevelStarts starts,
                                                int32_t *__restrict__ act, int32_t *__restrict__ cnt)
{
    const int64_t q = lo + (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    const int lane = threadIdx.x & 63;
    const int lev = q < hi ? level[q] : -1;
    unsigned long long todo = __ballot(lev >= 0 && in_box(code[q], lev, L0, box));
    const unsigned long long leaves = todo & __ballot(lev >= 0 && leaf[q] != 0);
    if (lane == 0 && leaves) atomicAdd(cnt + ACTIVE_LEAVES, __popcll(leaves));
    while (todo) {
        const int lead = __ffsll(todo) - 1;
        const int l = __shfl(lev, lead, 64);
        const unsigned long long same = __ballot((todo >> lane & 1) && lev == l);
        int base = 0;
        if (lane == lead) base = atomicAdd(cnt + l, __popcll(same));
        base = __shfl(base, lead, 64);
        if (same >> lane & 1) act[starts.lo[l] + base + __popcll(same & ((1ull << lane) - 1ull))] = (int32_t)q;
        todo &= ~same;
    }
}

// Up to SORT_SMALL stars: keys, the stable sort by them and the gather in one
// workgroup, keys and indices in LDS: the same order as by the radix sort
// (20 launches, 65 us of kernels for 1000 stars; this takes 15).  A wavefront
// ranks its consecutive items round by round, lanes with the same digit found
// with ballots, as there.
constexpr int SORT_SMALL = 4096;
constexpr int WG = 1024;
constexpr int WG_WAVES = WG / 64;

__global__ __launch_bounds__(WG) void k_sort_small(const double *__restrict__ x, const double *__restrict__ y,
                                                   const double *__restrict__ m, int32_t n, double L0, double scale,
                                                   uint64_t *__restrict__ keys, double *__restrict__ sx,
                                                   double *__restrict__ sy, double *__restrict__ sm)
{
    __shared__ uint64_t key[2][SORT_SMALL];
    __shared__ uint16_t idx[2][SORT_SMALL];
    __shared__ int32_t cnt[WG_WAVES][256];   // a wavefront's items per digit, then where they go
    __shared__ int32_t part[4];
    const int t = threadIdx.x, lane = t & 63, wave = t >> 6;
    const unsigned long long lt = (1ull << lane) - 1ull;
    for (int i = t; i < n; i += WG) {
        key[0][i] = morton2(fine_cell(x[i], L0, scale), fine_cell(y[i], L0, scale));
        idx[0][i] = (uint16_t)i;
    }
    constexpr int ROUNDS = SORT_SMALL / WG;
    const int rounds = (n + WG - 1) / WG;
    int src = 0;
    for (int shift = 0; shift < 2 * KEY_BITS; shift += 8) {
        for (int d = lane; d < 256; d += 64) cnt[wave][d] = 0;
        __syncthreads();
        int dig[ROUNDS], rank[ROUNDS];
#pragma unroll
        for (int r = 0; r < ROUNDS; ++r) {
            if (r >= rounds) break;
            const int i = (wave * rounds + r) * 64 + lane;
            const bool valid = i < n;
            const int d = valid ? (int)((key[src][i] >> shift) & 0xff) : 0;
            unsigned long long same = __ballot(valid);
#pragma unroll
            for (int b = 0; b < 8; ++b) {
                const unsigned long long ones = __ballot(valid && ((d >> b) & 1));
                same &= ((d >> b) & 1) ? ones : ~ones;
            }
            dig[r] = d;
            rank[r] = __popcll(same & lt) + cnt[wave][d];
            __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
            __builtin_amdgcn_wave_barrier();
            if (valid && (same & lt) == 0) cnt[wave][d] += __popcll(same);
            __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
            __builtin_amdgcn_wave_barrier();
        }
        __syncthreads();
        // exclusive over (digit, wavefront): threads 0 .. 255 own a digit each
        int total = 0, incl = 0;
        if (t < 256) {
#pragma unroll
            for (int w = 0; w < WG_WAVES; ++w) total += cnt[w][t];
            incl = total;
#pragma unroll
            for (int d = 1; d < 64; d <<= 1) {
                const int o = __shfl_up(incl, d, 64);
                if (lane >= d) incl += o;
            }
            if (lane == 63) part[wave] = incl;
        }
        __syncthreads();
        if (t < 256) {
            int base = incl - total;
            for (int w = 0; w < wave; ++w) base += part[w];
#pragma unroll
            for (int w = 0; w < WG_WAVES; ++w) {
                const int c = cnt[w][t];
                cnt[w][t] = base;
                base += c;
            }
        }
        __syncthreads();
#pragma unroll
        for (int r = 0; r < ROUNDS; ++r) {
            if (r >= rounds) break;
            const int i = (wave * rounds + r) * 64 + lane;
            if (i < n) {
                const int pos = cnt[wave][dig[r]] + rank[r];
                key[src ^ 1][pos] = key[src][i];
                idx[src ^ 1][pos] = idx[src][i];
            }
        }
        src ^= 1;
        __syncthreads();
    }
    for (int i = t; i < n; i += WG) {
        const int k = idx[src][i];
        keys[i] = key[src][i];
        sx[i] = x[k];
        sy[i] = y[k];
        sm[i] = m[k];
    }
}

// the node arrays of a tree
struct NodeArrays {
    uint64_t *code;
    int32_t *level, *leaf, *slo, *shi, *block, *parent, *child0, *coll, *node_leaf, *leaf_node, *near_offs, *active;
};

// what k_coarse_tree tells the host
struct CoarseTree {
    int32_t level_hi[MAX_LEVELS];   // end of each level that it numbered
    int32_t active[MAX_LEVELS];     // listed nodes per level, listed leaves in ACTIVE_LEAVES
    int32_t nlevels, done, nleaves, near_total;
};

// exclusive scan of one value per thread over the workgroup; part: WG_WAVES
// LDS slots
__device__ inline int wg_excl_scan(int v, int *part, int &total)
{
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    int in_wave;
    const int e = wave_excl_scan(v, lane, in_wave);
    if (lane == 0) part[wave] = in_wave;
    __syncthreads();
    int before = 0;
    total = 0;
#pragma unroll
    for (int w = 0; w < WG_WAVES; ++w) {
        const int c = part[w];
        if (w < wave) before += c;
        total += c;
    }
    __syncthreads();
    return before + e;
}

// The levels of up to WG nodes, one after the other in one workgroup, a thread
// per node, as long as the next level surely fits `cap` nodes; and, where that
// was the whole tree, the lists and numbers of its nodes: the nodes that meet
// the rays' rectangle, the leaves, and the offsets of their star tables.  Such
// a level's time is the latency of its loads: level by level over the grid it
// took four launches and the host's wait for the count, some 25 us, and here it
// takes 7.  SMALL: the keys are searched in LDS.
template <bool SMALL>
__global__ __launch_bounds__(WG) void k_coarse_tree(NodeArrays A, const uint64_t *__restrict__ gkeys, int32_t n,
                                                    int lmax, int nmax, int32_t cap, double L0, RayBox box,
                                                    CoarseTree *host, int64_t *total_host, int64_t seq)
{
    __shared__ int part[WG_WAVES], first[MAX_LEVELS], count[MAX_LEVELS];
    __shared__ uint64_t lkeys[SMALL ? SORT_SMALL : 1];
    const int t = threadIdx.x, lane = t & 63;
    const uint64_t *keys = SMALL ? lkeys : gkeys;
    if (SMALL)
        for (int i = t; i < n; i += WG) lkeys[i] = gkeys[i];
    if (t == 0) {
        A.code[0] = 0;
        A.level[0] = 0;
        A.parent[0] = -1;
    }
    if (t < MAX_LEVELS) count[t] = 0;
    __syncthreads();
    int32_t lo = 0, hi = 1;
    int lev = 0;
    bool done = false;
    while (hi - lo <= WG && hi + 4 * (hi - lo) <= cap) {
        const int32_t q = lo + t;
        if (t == 0) {
            first[lev] = lo;
            host->level_hi[lev] = hi;
        }
        if (q < hi) node_stars(q, lev, A.code, A.parent, keys, n, A.slo, A.shi);
        __syncthreads();
        bool split = false;
        if (q < hi) {
            const int32_t blk = node_block(q, lev, A.code, A.parent, A.child0, A.slo, A.shi, keys, A.coll);
            A.block[q] = blk;
            split = blk > nmax && lev < lmax;
        }
        int nsplit;
        const int off = wg_excl_scan(split ? 1 : 0, part, nsplit);
        if (q < hi) emit_children(q, (int64_t)hi + 4 * off, split, A.code, A.level, A.parent, A.child0, A.leaf, lev + 1);
        __syncthreads();
        ++lev;
        lo = hi;
        hi += 4 * nsplit;
        if (nsplit == 0) {
            done = true;
            break;
        }
    }
    if (done) {
        int32_t leaf0 = 0, near0 = 0;
        for (int32_t base = 0; base < hi; base += WG) {
            const int32_t q = base + t;
            const bool valid = q < hi;
            const int l = valid ? A.level[q] : -1;
            const bool is_leaf = valid && A.leaf[q] != 0, boxed = valid && in_box(A.code[q], l, L0, box);
            int nleaf, nnear;
            const int lf = leaf0 + wg_excl_scan(is_leaf ? 1 : 0, part, nleaf);
            const int blk = is_leaf && boxed ? A.block[q] : 0;
            const int off = near0 + wg_excl_scan(blk, part, nnear);
            if (valid) A.node_leaf[q] = is_leaf ? lf : -1;
            if (is_leaf) {
                A.leaf_node[lf] = q;
                A.near_offs[lf] = off;
            }
            leaf0 += nleaf;
            near0 += nnear;
            unsigned long long todo = __ballot(boxed && l >= 2);
            const unsigned long long leaves = todo & __ballot(is_leaf);
            if (lane == 0 && leaves) atomicAdd(count + ACTIVE_LEAVES, __popcll(leaves));
            while (todo) {
                const int lead = __ffsll(todo) - 1;
                const int ll = __shfl(l, lead, 64);
                const unsigned long long same = __ballot((todo >> lane & 1) && l == ll);
                int at = 0;
                if (lane == lead) at = atomicAdd(count + ll, __popcll(same));
                at = __shfl(at, lead, 64);
                if (same >> lane & 1) A.active[first[ll] + at + __popcll(same & ((1ull << lane) - 1ull))] = q;
                todo &= ~same;
            }
        }
        __syncthreads();
        if (t < MAX_LEVELS) host->active[t] = count[t];
        if (t == 0) {
            host->nleaves = leaf0;
            host->near_total = near0;
        }
    }
    if (t == 0) {
        host->level_hi[lev] = hi;   // (the level that the grid goes on with, if there is one)
        host->nlevels = lev;
        host->done = done ? 1 : 0;
    }
    __threadfence_system();
    __syncthreads();
    if (t == 0) __hip_atomic_store(total_host + 1, seq, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
}

// interaction squares of the listed nodes of levels >= 2: the children of the
// parent's 3x3 block that are outside the node's own 3x3 block (27 of them),
// read from the parent's colleagues: a node (M2L), a part of a leaf (P2L from
// its stars in the square) or nothing.  One wavefront per node, a lane per
// child square (36, the 27 kept in lane order): a thread walking its node's
// squares one after the other spent the pass on the latency of their loads
// (43 us for 78k nodes).  All levels in one launch: listed.lo[lev] listed nodes
// come before those of level lev.
__global__ __launch_bounds__(BLK) void k_ilist(LevelStarts starts, LevelStarts listed, int nlevels,
                                               const int32_t *__restrict__ act, const uint64_t *__restrict__ code,
                                               const int32_t *__restrict__ parent,
                                               const int32_t *__restrict__ child0, const int32_t *__restrict__ slo,
                                               const int32_t *__restrict__ shi, const uint64_t *__restrict__ keys,
                                               const int32_t *__restrict__ coll, IEntry *__restrict__ list)
{
    const int lane = threadIdx.x & 63;
    const int k = __builtin_amdgcn_readfirstlane(blockIdx.x * (BLK / 64) + (threadIdx.x >> 6));
    int lev = 2;
    while (lev + 1 < nlevels && k >= listed.lo[lev + 1]) ++lev;
    const int sh = 2 * (KEY_BITS - lev);
    if (k >= listed.lo[nlevels]) return;
    const int64_t q = act[starts.lo[lev] + k - listed.lo[lev]];
    const uint64_t c = code[q];
    const int64_t i = compact_bits(c), j = compact_bits(c >> 1);
    const int32_t *pc = coll + (int64_t)parent[q] * 9;
    const int b = lane >> 2;   // parent's colleague, its child (lane & 3)
    const int64_t si = 2 * ((i >> 1) + b % 3 - 1) + (lane & 1), sj = 2 * ((j >> 1) + b / 3 - 1) + (lane >> 1 & 1);
    const int64_t dx = si - i, dy = sj - j;
    const bool keep = lane < 36 && !(dx >= -1 && dx <= 1 && dy >= -1 && dy <= 1);
    const int e = __popcll(__ballot(keep) & ((1ull << lane) - 1ull));
    if (!keep) return;
    IEntry en;
    en.off = (int32_t)((dx + 3) + 7 * (dy + 3));
    en.src = -2;
    en.slo = en.shi = 0;
    const int32_t ref = child_ref(pc[b], (uint32_t)si, (uint32_t)sj, child0);
    if (ref >= 0) {
        en.src = ref;
    } else if (ref <= -2) {
        int32_t s0, s1;
        ref_stars(ref, morton2((uint32_t)si, (uint32_t)sj), sh, slo, shi, keys, s0, s1);
        if (s1 > s0) {
            en.src = -1;
            en.slo = s0;
            en.shi = s1;
        }
    }
    list[q * NLIST + e] = en;
}

template <class T>
T *grow_keep(DevBuf &b, size_t used_elems, size_t need_elems, hipStream_t st)
{
    return static_cast<T *>(b.grow_keep(used_elems * sizeof(T), need_elems * sizeof(T), st));
}

void *scan_tmp(Workspace &ws, size_t bytes) { return ws.scan_tmp.reserve(bytes ? bytes : 1); }

// A scan's total, read back to the host: the scan stores it straight into a
// coherent pinned slot with a sequence number behind it, and the host spins
// until that number appears instead of synchronising the stream (whose
// wake-up would add its latency to every tree level and count).  After a
// short spin it blocks on the stream instead, which also reports any error
// of the queued work.  Inside a scratch arena (no pinned slot) the total goes
// to a scratch slot that is copied, after a synchronisation.
struct TotalSlot {
    int64_t *dev = nullptr, *host = nullptr;
    int64_t seq = 0;
};

TotalSlot total_slot(mlm_lens *lens)
{
    TotalSlot t;
    if (Arena *a = thread_arena()) {
        t.dev = static_cast<int64_t *>(a->take(sizeof(int64_t)));
        return t;
    }
    Workspace &ws = lens->ws;
    if (!ws.spin) ws.spin = static_cast<int64_t *>(coherent_pinned((2 + BIG_SHARDS) * sizeof(int64_t), ws.spin_cap, ws.spin_dev));
    t.host = ws.spin;
    t.seq = ++ws.spin_seq;
    return t;
}

int64_t read_total(const TotalSlot &t, hipStream_t st)
{
    if (t.dev) {
        int64_t v = 0;
        MLM_HIP(hipMemcpyAsync(&v, t.dev, sizeof v, hipMemcpyDeviceToHost, st));
        MLM_HIP(hipStreamSynchronize(st));
        return v;
    }
    const volatile int64_t *h = t.host;
    const auto t0 = std::chrono::steady_clock::now();
    for (int k = 1; h[1] != t.seq; ++k) {
        if ((k & 255) == 0 && std::chrono::steady_clock::now() - t0 > std::chrono::microseconds(200)) {
            MLM_HIP(hipStreamSynchronize(st));
            if (h[1] != t.seq) fail(MLM_EDEVICE, "a scan's total did not arrive");
            break;
        }
        __builtin_ia32_pause();
    }
    std::atomic_thread_fence(std::memory_order_acquire);
    return h[0];
}

// exclusive prefix sum of n int32 flags; returns the total
int64_t scan_total(mlm_lens *lens, const int32_t *in, int32_t *out, int64_t n, hipStream_t st)
{
    if (n == 0) return 0;
    const TotalSlot t = total_slot(lens);
    dev_scan_i32(in, out, n, false, scan_tmp(lens->ws, scan_tmp_bytes(n)), t.dev, t.host, t.seq, st);
    return read_total(t, st);
}

}  // namespace

int64_t scan_total_public(mlm_lens *lens, const int32_t *in, int32_t *out, int64_t n, hipStream_t st)
{
    return scan_total(lens, in, out, n, st);
}

// exclusive prefix sum of n int32 counts into n + 1 int64 offsets (the last
// one is the total, which is returned)
int64_t scan_i32_to_i64(mlm_lens *lens, const int32_t *in, int64_t *out, int64_t n, hipStream_t st)
{
    if (n == 0) return 0;
    const TotalSlot t = total_slot(lens);
    hipLaunchKernelGGL(k_zero_first, dim3(1), dim3(1), 0, st, out);
    dev_scan_i32_i64(in, out + 1, n, true, scan_tmp(lens->ws, scan_tmp_bytes(n)), t.dev, t.host, t.seq, st);
    return read_total(t, st);
}

int64_t scan_excl(mlm_lens *lens, const int32_t *in, int64_t *out, int64_t n, hipStream_t st)
{
    if (n == 0) return 0;
    const TotalSlot t = total_slot(lens);
    dev_scan_i32_i64(in, out, n, false, scan_tmp(lens->ws, scan_tmp_bytes(n)), t.dev, t.host, t.seq, st);
    return read_total(t, st);
}

// exclusive prefix sum of n int32 counts into n + 1 uint64 offsets; returns the total
int64_t scan_i32_to_u64(mlm_lens *lens, const int32_t *in, unsigned long long *out, int64_t n, hipStream_t st)
{
    return scan_i32_to_i64(lens, in, reinterpret_cast<int64_t *>(out), n, st);
}

bool read_big_counts(mlm_lens *lens, const BigList &bl, BigStarts &at, hipStream_t st)
{
    const TotalSlot t = total_slot(lens);   // (pinned: lists are not kept inside a scratch arena)
    hipLaunchKernelGGL(k_publish_counts, dim3(1), dim3(BIG_SHARDS), 0, st, bl.count, t.host, t.seq);
    (void)read_total(t, st);
    bool whole = true;
    at.lo[0] = 0;
    for (int k = 0; k < BIG_SHARDS; ++k) {
        at.lo[k + 1] = at.lo[k] + t.host[2 + k];
        whole = whole && t.host[2 + k] <= bl.cap;
    }
    return whole;
}

int64_t first_outside(mlm_lens *lens, const double *z, int64_t n, double L0, hipStream_t st)
{
    const int np = (int)std::min<int64_t>((n + BLK - 1) / BLK, OUTSIDE_BLOCKS);
    int64_t *part = static_cast<int64_t *>(lens->ws.search.reserve(OUTSIDE_BLOCKS * sizeof(int64_t)));
    const TotalSlot t = total_slot(lens);
    hipLaunchKernelGGL(k_outside, dim3(np), dim3(BLK), 0, st, z, n, L0, part);
    hipLaunchKernelGGL(k_outside_first, dim3(1), dim3(64), 0, st, part, np, n, t.dev, t.host, t.seq);
    return read_total(t, st);
}

LatticeBox search_lattice(const CubicSearch &S, Workspace &ws, hipStream_t st)
{
    constexpr int np = LAT / LAT_ROWS;
    static_assert(np * LAT_ROWS == LAT, "whole workgroups of rows");
    LatticeBox *part = static_cast<LatticeBox *>(ws.search.reserve(np * sizeof(LatticeBox)));
    hipLaunchKernelGGL(k_lattice, dim3(np), dim3(BLK), 0, st, S, part);
    std::vector<LatticeBox> h(np);
    MLM_HIP(hipMemcpyAsync(h.data(), part, np * sizeof(LatticeBox), hipMemcpyDeviceToHost, st));
    MLM_HIP(hipStreamSynchronize(st));
    LatticeBox B = h[0];
    for (const LatticeBox &b : h)
        B = LatticeBox{std::min(B.i0, b.i0), std::max(B.i1, b.i1), std::min(B.j0, b.j0), std::max(B.j1, b.j1)};
    return B;
}

void box_rays(Tree &T, const Region &R, int64_t vb0, int64_t vb1)
{
    // one cell and the rounding of the largest coordinate to spare
    const double e1 = R.d1 + 1e-12 * R.L0, e2 = R.d2 + 1e-12 * R.L0;
    T.boxed = true;
    T.box[0] = R.x0 - e1;
    T.box[1] = R.x0 + (double)(R.nr1 - 1) * R.d1 + e1;
    T.box[2] = R.y0 + (double)vb0 * R.d2 - e2;
    T.box[3] = R.y0 + (double)vb1 * R.d2 + e2;
}

RayBox ray_box(const Tree &T)
{
    if (!T.boxed) return RayBox{-HUGE_VAL, HUGE_VAL, -HUGE_VAL, HUGE_VAL};
    return RayBox{T.box[0], T.box[1], T.box[2], T.box[3]};
}

namespace {

// the nodes of levels >= 2 that the rays need, listed level by level (in the
// sort's input buffer, free by now, where it is large enough: it is unless
// leaves hold a star or two), their counts stored to the host before the total
// it next waits for, and the numbers of the leaves
void number_nodes(mlm_lens *lens, Tree &T, hipStream_t st)
{
    Workspace &ws = lens->ws;
    const size_t act_bytes = (size_t)(T.nnodes + MAX_LEVELS) * sizeof(int32_t);
    T.active = static_cast<int32_t *>(act_bytes <= ws.keys_in.cap ? ws.keys_in.p : ws.active.reserve(act_bytes));
    int32_t *cnt = T.active + T.nnodes;
    if (T.nlevels > 2) {
        const int64_t lo = T.level_lo[2], hi = T.nnodes;
        LevelStarts starts{};
        for (int lev = 0; lev < T.nlevels; ++lev) starts.lo[lev] = (int32_t)T.level_lo[lev];
        hipLaunchKernelGGL(k_zero_counts, dim3(1), dim3(64), 0, st, cnt, MAX_LEVELS);
        hipLaunchKernelGGL(k_active, dim3(nblocks(hi - lo)), dim3(BLK), 0, st, lo, hi, T.L0, ray_box(T), T.code,
                           T.level, T.leaf, starts, T.active, cnt);
    }
    const TotalSlot slot = total_slot(lens);
    int32_t *host_cnt = slot.host ? reinterpret_cast<int32_t *>(slot.host + 2) : nullptr;
    if (T.nlevels > 2 && host_cnt) hipLaunchKernelGGL(k_copy_counts, dim3(1), dim3(64), 0, st, cnt, host_cnt, MAX_LEVELS);
    int32_t *offs = static_cast<int32_t *>(ws.offs.reserve(T.nnodes * 4));
    T.node_leaf = static_cast<int32_t *>(ws.node_leaf.reserve(T.nnodes * 4));
    dev_scan_i32(T.leaf, offs, T.nnodes, false, scan_tmp(ws, scan_tmp_bytes(T.nnodes)), slot.dev, slot.host, slot.seq, st);
    T.nleaves = read_total(slot, st);
    T.leaf_node = static_cast<int32_t *>(ws.leaf_node.reserve(T.nleaves * 4));
    hipLaunchKernelGGL(k_leaf_index, dim3(nblocks(T.nnodes)), dim3(BLK), 0, st, T.nnodes, T.leaf, offs,
                       T.node_leaf, T.leaf_node);
    if (T.nlevels > 2) {
        if (host_cnt) {
            std::copy(host_cnt, host_cnt + MAX_LEVELS, T.nactive);
        } else {
            MLM_HIP(hipMemcpyAsync(T.nactive, cnt, sizeof T.nactive, hipMemcpyDeviceToHost, st));
            MLM_HIP(hipStreamSynchronize(st));
        }
    }
}

// interaction lists of the listed nodes
void list_interactions(Workspace &ws, Tree &T, hipStream_t st)
{
    T.nactive_leaves = T.nlevels > 2 ? T.nactive[ACTIVE_LEAVES] : T.nleaves;
    T.ilist = static_cast<IEntry *>(ws.ilist.reserve((size_t)T.nnodes * NLIST * sizeof(IEntry)));
    LevelStarts starts{}, listed{};
    for (int lev = 2; lev < T.nlevels; ++lev) {
        starts.lo[lev] = (int32_t)T.level_lo[lev];
        listed.lo[lev + 1] = listed.lo[lev] + T.nactive[lev];
    }
    const int32_t n = T.nlevels > 2 ? listed.lo[T.nlevels] : 0;
    if (n > 0)
        hipLaunchKernelGGL(k_ilist, dim3(nblocks(n, BLK / 64)), dim3(BLK), 0, st, starts, listed, T.nlevels, T.active,
                           T.code, T.parent, T.child0, T.slo, T.shi, T.keys, T.coll, T.ilist);
}

}  // namespace

void build_tree(mlm_lens *lens, const Region &R, const mlm_map_request &req, Tree &T, hipStream_t st)
{
    Workspace &ws = lens->ws;
    const int32_t n = (int32_t)lens->n;
    T.L0 = R.L0;
    T.L0_exp = R.L0_exp;
    T.nmax = req.leaf_max > 0 ? req.leaf_max : 32;
    T.lmax = (req.max_level > 0 && req.max_level < KEY_BITS) ? req.max_level : KEY_BITS;
    T.n = n;

    // 1. Morton keys of the stars at the finest level, radix sort, gather
    size_t nn = (size_t)(n > 0 ? n : 1);
    uint64_t *kin = static_cast<uint64_t *>(ws.keys_in.reserve(nn * 8));
    uint64_t *kout = static_cast<uint64_t *>(ws.keys.reserve(nn * 8));
    int32_t *iin = static_cast<int32_t *>(ws.idx_in.reserve(nn * 4));
    int32_t *iout = static_cast<int32_t *>(ws.idx.reserve(nn * 4));
    T.x = static_cast<double *>(ws.sx.reserve(nn * 8));
    T.y = static_cast<double *>(ws.sy.reserve(nn * 8));
    T.m = static_cast<double *>(ws.sm.reserve(nn * 8));
    T.keys = kout;
    if (n > 0) {
        double scale = std::ldexp(1.0, KEY_BITS - R.L0_exp);   // 2^24 / (2 L0)
        if (n <= SORT_SMALL) {
            hipLaunchKernelGGL(k_sort_small, dim3(1), dim3(WG), 0, st, lens->d_x, lens->d_y, lens->d_m, n, R.L0, scale,
                               kout, T.x, T.y, T.m);
        } else {
            hipLaunchKernelGGL(k_keys, dim3(nblocks(n)), dim3(BLK), 0, st, lens->d_x, lens->d_y, n, R.L0, scale, kin,
                               iin);
            radix_sort_pairs(kin, iin, kout, iout, n, 2 * KEY_BITS, scan_tmp(ws, radix_sort_tmp_bytes(n)), st);
            hipLaunchKernelGGL(k_gather, dim3(nblocks(n)), dim3(BLK), 0, st, iout, lens->d_x, lens->d_y, lens->d_m, n,
                               T.x, T.y, T.m);
        }
    }

    // 2. levels, top down
    T.level_lo.assign(1, 0);
    T.level_hi.assign(1, 1);
    size_t used = 0;
    int32_t *&coll = T.coll;   // 9 colleague references per node
    auto ensure = [&](size_t need) {
        T.code = grow_keep<uint64_t>(ws.code, used, need, st);
        T.level = grow_keep<int32_t>(ws.level, used, need, st);
        T.leaf = grow_keep<int32_t>(ws.leaf, used, need, st);
        T.slo = grow_keep<int32_t>(ws.slo, used, need, st);
        T.shi = grow_keep<int32_t>(ws.shi, used, need, st);
        T.block = grow_keep<int32_t>(ws.block, used, need, st);
        T.parent = grow_keep<int32_t>(ws.parent, used, need, st);
        T.child0 = grow_keep<int32_t>(ws.child0, used, need, st);
        coll = grow_keep<int32_t>(ws.coll, 9 * used, 9 * need, st);
    };
    int lev0 = 0;
    if (thread_arena()) {
        ensure(1024);
        hipLaunchKernelGGL(k_root, dim3(1), dim3(1), 0, st, T.code, T.level, T.parent);
        used = 1;
    } else {
        // the coarse levels, or all of a small tree, by one workgroup (not inside
        // a scratch arena, whose slices are sized by what a level needs)
        ensure(COARSE_NODES);
        const size_t bytes = (size_t)COARSE_NODES * sizeof(int32_t);
        T.node_leaf = static_cast<int32_t *>(ws.node_leaf.reserve(bytes));
        T.leaf_node = static_cast<int32_t *>(ws.leaf_node.reserve(bytes));
        T.near_offs = static_cast<int32_t *>(ws.near_offs.reserve(bytes));
        T.active = static_cast<int32_t *>(bytes <= ws.keys_in.cap ? ws.keys_in.p : ws.active.reserve(bytes));
        const NodeArrays A{T.code, T.level, T.leaf, T.slo, T.shi, T.block, T.parent, T.child0, coll,
                           T.node_leaf, T.leaf_node, T.near_offs, T.active};
        const TotalSlot slot = total_slot(lens);
        const CoarseTree *C = reinterpret_cast<const CoarseTree *>(slot.host + 2);
        static_assert(sizeof(CoarseTree) <= BIG_SHARDS * sizeof(int64_t), "room in the pinned slot");
        const auto k = n <= SORT_SMALL ? k_coarse_tree<true> : k_coarse_tree<false>;
        hipLaunchKernelGGL(k, dim3(1), dim3(WG), 0, st, A, T.keys, n, T.lmax, T.nmax, COARSE_NODES, T.L0, ray_box(T),
                           reinterpret_cast<CoarseTree *>(slot.host + 2), slot.host, slot.seq);
        (void)read_total(slot, st);
        T.level_hi.clear();
        T.level_lo.clear();
        const int nl = C->nlevels + (C->done ? 0 : 1);
        for (int lev = 0; lev < nl; ++lev) {
            T.level_lo.push_back(lev ? T.level_hi.back() : 0);
            T.level_hi.push_back(C->level_hi[lev]);
        }
        used = (size_t)T.level_hi.back();
        lev0 = C->nlevels;
        if (C->done) {
            T.nlevels = C->nlevels;
            T.nnodes = T.level_hi.back();
            T.nleaves = C->nleaves;
            T.near_total = C->near_total;
            T.near_numbered = true;
            std::copy(C->active, C->active + MAX_LEVELS, T.nactive);
        }
    }
    for (int lev = lev0; T.nlevels == 0; ++lev) {
        int64_t lo = T.level_lo[lev], hi = T.level_hi[lev], nl = hi - lo;
        int32_t *flags = static_cast<int32_t *>(ws.flags.reserve(nl * 4));
        int32_t *offs = static_cast<int32_t *>(ws.offs.reserve(nl * 4));
        hipLaunchKernelGGL(k_level, dim3(nblocks(nl)), dim3(BLK), 0, st, lo, hi, lev, T.code, T.parent, T.keys, n,
                           T.slo, T.shi);
        hipLaunchKernelGGL(k_block, dim3(nblocks(nl)), dim3(BLK), 0, st, lo, hi, lev, T.lmax, T.nmax, T.code,
                           T.parent, T.child0, T.slo, T.shi, T.keys, coll, T.block, flags);
        int64_t nsplit = scan_total(lens, flags, offs, nl, st);
        if (hi + 4 * nsplit > (int64_t)INT32_MAX) fail(MLM_ERANGE, "tree too large");
        ensure((size_t)(hi + 4 * nsplit));
        hipLaunchKernelGGL(k_emit, dim3(nblocks(nl)), dim3(BLK), 0, st, lo, hi, hi, flags, offs, T.code,
                           T.level, T.parent, T.child0, T.leaf, lev + 1);
        used = (size_t)(hi + 4 * nsplit);
        if (nsplit == 0) {
            T.nlevels = lev + 1;
            T.nnodes = hi;
            break;
        }
        T.level_lo.push_back(hi);
        T.level_hi.push_back(hi + 4 * nsplit);
    }
    if (!T.near_numbered) number_nodes(lens, T, st);
    list_interactions(ws, T, st);
}

}  // namespace mlm
