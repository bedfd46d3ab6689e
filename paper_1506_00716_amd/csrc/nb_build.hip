// nb_build.hip -- cluster-pair list construction on the GPU (gfx950).
//
// The paper's scheme (Section "SIMD parallelism"): place atoms on a grid in x
// and y, bin them in z, cut the z-ordered columns into clusters of exactly M
// atoms, and list every cluster pair that may contain atoms close enough to
// interact, with a buffer (r_list > r_cut) so the list can be reused over
// several steps.  The GPU additionally prunes the list (Section "Heterogeneous
// parallelization"); here the prune is an exact FP64 atom-pair test that also
// yields the list's exact atom-pair set.
//
// MI355X design: the whole build runs on the device with no host round trip.
//   1. k_bin          wrap into the box (integer image counts kept), xy column id
//   2. k_col_scan     per-system column offsets and group counts (one block; up to
//                     4096 columns it is a block of the next kernel)
//   3. k_scatter      counting-sort scatter of (z key, atom) into columns
//   4. k_col_sort     per-column bucket sort in LDS;
//      k_group_split  one wave per 8*M-atom chunk of a column: split 2 x 2 x 2
//                     (z, then y, then x halves) into an i-group of 8 clusters
//                     of M atoms; bounding boxes; staging of the new slots
//   5. k_search       one block per i-group: bounding-box culling against the
//                     clusters of the neighbouring columns, all periodic images;
//                     candidates sorted by (j-cluster, shift)
//                     and pruned at the atom level in FP32; explicit builds
//                     decide every atom pair exactly in the same pass (FP64
//                     where FP32 cannot), which gives the export masks
//   6. k_list_scan    CSR offsets of kept entries, work items and the transpose
//   7. k_list_write   compacted entries, FP32 shift vectors, work items
// k_prune computes the exact masks of a list that was built without them (asked
// for after a run of dynamics).
// Every step is deterministic (no order depends on atomics).
#include "nb_internal.h"

#include <type_traits>

#pragma clang fp contract(off)

namespace nbi {

namespace {

__device__ inline int floor_div(int a, int b) { return a >= 0 ? a / b : -((-a + b - 1) / b); }

__device__ inline double box_gap(double lo1, double hi1, double lo2, double hi2)
{
    double g = lo2 - hi1;
    double h = lo1 - hi2;
    double m = g > h ? g : h;
    return m > 0.0 ? m : 0.0;
}

// box fraction of a wrapped coordinate as a 32-bit key (non-finite -> 0)
// FP32 shift vector of a list entry in the force kernel's frame: j-group
// reference plus the periodic shift, minus the i-group reference (FP64, then
// rounded once)
template <class Box>
__device__ inline float4 entry_shift(const Box& d, const double rj[3], int sid, const double ri[3])
{
    const int s0 = sid % 5 - 2, s1 = (sid / 5) % 3 - 1, s2 = sid / 15 - 1;
    // the shift s0 a + s1 b + s2 c (rectangular: s L per dimension)
    const double tx = (s0 * d.box[0] + s1 * d.box_off[0]) + s2 * d.box_off[1];
    const double ty = s1 * d.box[1] + s2 * d.box_off[2];
    float4 S;
    S.x = (float)((rj[0] + tx) - ri[0]);
    S.y = (float)((rj[1] + ty) - ri[1]);
    S.z = (float)((rj[2] + s2 * d.box[2]) - ri[2]);
    S.w = 0.0f;
    return S;
}

__device__ inline unsigned int coord_key(double v, double inv)
{
    const double f = v * inv * 4294967296.0;
    if (!(f >= 0.0)) return 0u;
    if (f >= 4294967295.0) return 0xffffffffu;
    return (unsigned int)f;
}

// exclusive block scan of one int per thread (blockDim.x == 1024)
__device__ int block_exclusive_scan(int v, int* smem, int* total)
{
    const int tid = threadIdx.x;
    const int lane = tid & 63;
    const int wid = tid >> 6;
    int incl = v;
    for (int o = 1; o < 64; o <<= 1) {
        int t = __shfl_up(incl, o, 64);
        if (lane >= o) incl += t;
    }
    if (lane == 63) smem[wid] = incl;
    __syncthreads();
    if (wid == 0) {
        int w = lane < (int)(blockDim.x >> 6) ? smem[lane] : 0;
        int wi = w;
        for (int o = 1; o < 16; o <<= 1) {
            int t = __shfl_up(wi, o, 64);
            if (lane >= o) wi += t;
        }
        if (lane < 16) smem[16 + lane] = wi - w;
        if (lane == 15) smem[32] = wi;
    }
    __syncthreads();
    int res = incl - v + smem[16 + wid];
    *total = smem[32];
    __syncthreads();
    return res;
}

// Ascending sort of n <= NT distinct keys in LDS (16-byte aligned, room for n + 1)
// by rank: a wave counts, for 64 keys, those below each in a part of them (broadcast
// reads of two keys at a time, no barrier per stage; the parts make all waves work
// whatever n is), then every key moves to its rank.  rank: NT ints of scratch.
// With each key counted over all keys by one thread the sort took 4.3 to 5.0 us of
// a search block's 36.8 (a million atoms), now 2.7 to 3.0.
typedef unsigned long long nb_u64x2 __attribute__((ext_vector_type(2)));
template <int NT>
__device__ __forceinline__ void rank_sort_lds(unsigned long long* keys, int n, int* rank)
{
    const int wid = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63;
    if (threadIdx.x == 0) keys[n] = ~0ull;  // pad: above every key
    rank[threadIdx.x] = 0;
    __syncthreads();
    const int blocks = max(1, (n + 63) / 64), parts = (NT / 64) / blocks;
    const int part = wid / blocks, t = (wid % blocks) * 64 + lane;
    if (part < parts) {
        const int pairs = (n + 1) / 2, u0 = part * pairs / parts, u1 = (part + 1) * pairs / parts;
        const unsigned long long k = t < n ? keys[t] : 0ull;
        const nb_u64x2* kv = (const nb_u64x2*)keys;
        int r = 0;
#pragma unroll 4
        for (int u = u0; u < u1; ++u) {
            const nb_u64x2 ku = kv[u];
            r += (ku.x < k ? 1 : 0) + (ku.y < k ? 1 : 0);
        }
        atomicAdd(&rank[t], r);
    }
    const unsigned long long k = (int)threadIdx.x < n ? keys[threadIdx.x] : 0ull;
    __syncthreads();
    if ((int)threadIdx.x < n) keys[rank[threadIdx.x]] = k;
    __syncthreads();
}

// Ascending bitonic sort of keys[0..n) (n <= P, P a power of two), all
// comparators min-to-lower-index so the implicit +inf padding never moves.
__device__ __forceinline__ void bitonic_sort(unsigned long long* keys, int n, int P)
{
    const int nthr = blockDim.x;
    for (int k = 2; k <= P; k <<= 1) {
        for (int j = k >> 1; j > 0; j >>= 1) {
            for (int t = threadIdx.x; t < (P >> 1); t += nthr) {
                int i, p;
                if (j == (k >> 1)) {
                    i = (t / j) * k + (t % j);
                    p = i ^ (k - 1);
                } else {
                    i = (t / j) * 2 * j + (t % j);
                    p = i + j;
                }
                if (p < n) {
                    unsigned long long u = keys[i], w = keys[p];
                    if (u > w) {
                        keys[i] = w;
                        keys[p] = u;
                    }
                }
            }
            __syncthreads();
        }
    }
}

}  // namespace

// ---------------------------------------------------------------------------
// the build mode of a system: 0 = not rebuilt, 1 = rebuilt, 2 = first build
__device__ inline int build_mode(const int* flags, int sys, int first)
{
    return flags ? flags[sys] : (first ? 2 : 1);
}

// 0. clear the build counters, and the list-buffer guard: per block the largest
//    squared displacement since the previous build (mode 1), x recorded for the
//    next one.  status_clear: 1 = clear the status words too, 2 = all but the
//    fault flags of earlier steps (saturation, bad positions).  Inside md_step
//    the gather that ends the step before a rebuild does all of this instead
//    (the kernel is then not launched); the slot map is reset by k_bin.
__global__ __launch_bounds__(256) void k_build_clear(const SysDev* __restrict__ table, const int* flags,
                                                     int status_clear, int first)
{
    const int mode = build_mode(flags, blockIdx.y, first);
    if (mode == 0) return;
    const SysDev& d = table[blockIdx.y];
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (status_clear && i < ST_COUNT && !(status_clear == 2 && (i == ST_SATURATE || i == ST_BADPOS)))
        gst(&d.status[i], 0);
    if (i < d.n_cols) {
        gst(&d.col_count[i], 0);
        gst(&d.col_fill[i], 0);
    }
    if (i < d.max_groups) {
        gst(&d.cand_count[i], 0);
        gst(&d.cand_kept[i], 0);
        gst(&d.grp_w[i], 0);
    }
    if (i < d.max_groups * d.G) gst(&d.jfill[i], 0);
    // displacement partials: blocks [0, sys_blocks) stride over the atoms (the
    // same decomposition alone and in a batch); the others that the column scan
    // reads are 0 (the gather before a rebuild leaves more of them than this grid
    // has blocks)
    const int nb = sys_blocks(d.n_atoms), np = guard_partials(d);
    for (int k = nb + i; k < np; k += gridDim.x * blockDim.x) gst(&d.disp[k], 0.0);
    if ((int)blockIdx.x >= nb) return;
    __shared__ double sh[256];
    double m = 0.0;
    for (int a = blockIdx.x * blockDim.x + threadIdx.x; a < d.n_atoms; a += nb * blockDim.x) {
        double s2 = 0.0;
        for (int k = 0; k < 3; ++k) {
            const double x = gld(&d.x[3 * a + k]);
            if (mode == 1) {
                const double dd = x - gld(&d.x_build[3 * a + k]);
                s2 += dd * dd;
            }
            gst(&d.x_build[3 * a + k], x);
        }
        m = (s2 > m || s2 != s2) ? s2 : m;  // NaN wins
    }
    sh[threadIdx.x] = m;
    __syncthreads();
    for (int o = 128; o > 0; o >>= 1) {
        if ((int)threadIdx.x < o) {
            const double u = sh[threadIdx.x + o];
            if (u > sh[threadIdx.x] || u != u) sh[threadIdx.x] = u;
        }
        __syncthreads();
    }
    if (threadIdx.x == 0) d.disp[blockIdx.x] = sh[0];
}

// 1. wrap, column id, z key; column counts through a block-private LDS
//    histogram (device-scope atomics to one counter serialise)
constexpr int kHistLds = 4096;

__global__ __launch_bounds__(256) void k_bin(const SysDev* __restrict__ table, const int* flags)
{
    if (flags && !flags[blockIdx.y]) return;
    const SysDev& d = table[blockIdx.y];
    // every slot starts empty (the group split fills the real ones)
    const int slots = d.max_groups * d.G * d.M;
    for (int k = blockIdx.x * blockDim.x + threadIdx.x; k < slots; k += gridDim.x * blockDim.x)
        gst(&d.slot_atom[k], -1);
    __shared__ int hist[kHistLds];
    const bool priv = d.n_cols <= kHistLds;
    if (priv)
        for (int c = threadIdx.x; c < d.n_cols; c += blockDim.x) hist[c] = 0;
    __syncthreads();
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i < d.n_atoms) {
        double xw[3];
        bool finite = true;
        const double x0 = d.x[3 * i], x1 = d.x[3 * i + 1], x2 = d.x[3 * i + 2];
        int wl[3] = {0, 0, 0};
        // lattice counts in the order c, b, a: each component is reduced after
        // the higher lattice vectors were removed from it (rectangular: per
        // dimension)
        for (int k = 2; k >= 0; --k) {
            const double xk = k == 2 ? x2
                            : k == 1 ? x1 - (double)wl[2] * d.box_off[2]
                                     : (x0 - (double)wl[1] * d.box_off[0]) - (double)wl[2] * d.box_off[1];
            finite = finite && (fabs(xk) <= 1.7976931348623157e308);
            double t = floor(xk * d.invbox[k]);
            if (!(fabs(t) < 1e9)) t = 0.0;  // non-finite or absurd input: image 0
            int w = (int)t;
            double r = xk - t * d.box[k];
            if (r >= d.box[k]) {
                r -= d.box[k];
                w += 1;
            }
            if (r < 0.0) {
                r += d.box[k];
                w -= 1;
            }
            if (r >= d.box[k]) r = 0.0;  // r was -tiny: rounds to L; keep the image count, clamp
            xw[k] = r;
            wl[k] = w;
            d.atom_wrap[3 * i + k] = w;
        }
        const double fx = xw[0] * d.inv_cell[0], fy = xw[1] * d.inv_cell[1];
        int cx = (fx >= 0.0 && fx < 1e9) ? (int)fx : 0;  // non-finite input lands in column 0
        int cy = (fy >= 0.0 && fy < 1e9) ? (int)fy : 0;
        cx = cx < 0 ? 0 : (cx >= d.ncx ? d.ncx - 1 : cx);
        cy = cy < 0 ? 0 : (cy >= d.ncy ? d.ncy - 1 : cy);
        const int col = cx + d.ncx * cy;
        d.atom_col[i] = col;
        d.atom_zkey[i] = coord_key(xw[2], d.invbox[2]);
        if (!finite) atomicOr(&d.status[ST_BADPOS], 1);
        if (priv) atomicAdd(&hist[col], 1);
        else gatomic_add(&d.col_count[col], 1);
    }
    __syncthreads();
    if (priv)
        for (int c = threadIdx.x; c < d.n_cols; c += blockDim.x)
            if (hist[c]) gatomic_add(&d.col_count[c], hist[c]);
}

// 2. column offsets and group counts, and the list-buffer guard (one block of one
//    system)
template <int NT>
__device__ __forceinline__ void col_scan(const SysDev& d, int mode)
{
    __shared__ int smem[40];
    if (mode == 1) {
        // list-buffer guard: the largest displacement of this list lifetime
        // from the per-block partials (NaN wins), and whether it reached half
        // the buffer (the only way a pair could enter r_cut unlisted)
        __shared__ double shd[NT];
        double m = 0.0;
        const int np = guard_partials(d);
        for (int k = threadIdx.x; k < np; k += blockDim.x) {
            const double u = gld(&d.disp[k]);
            m = (u > m || u != u) ? u : m;
        }
        shd[threadIdx.x] = m;
        __syncthreads();
        for (int o = NT / 2; o > 0; o >>= 1) {
            if ((int)threadIdx.x < o) {
                const double u = shd[threadIdx.x + o];
                if (u > shd[threadIdx.x] || u != u) shd[threadIdx.x] = u;
            }
            __syncthreads();
        }
        if (threadIdx.x == 0) {
            const double mm = sqrt(shd[0]);
            if (mm > d.disp[kKeBlocks]) d.disp[kKeBlocks] = mm;
            if (!(2.0 * mm < d.buffer)) d.disp[kKeBlocks + 1] += 1.0;
        }
    }
    const int GM = d.G * d.M;
    int carry_a = 0, carry_g = 0;
    for (int base = 0; base < d.n_cols; base += NT) {
        const int c = base + threadIdx.x;
        const int cnt = c < d.n_cols ? gld(&d.col_count[c]) : 0;
        const int ng = (cnt + GM - 1) / GM;
        int tot_a, tot_g;
        int ea = block_exclusive_scan(cnt, smem, &tot_a);
        int eg = block_exclusive_scan(ng, smem, &tot_g);
        if (c < d.n_cols) {
            gst(&d.col_start[c], carry_a + ea);
            gst(&d.col_gstart[c], carry_g + eg);
        }
        carry_a += tot_a;
        carry_g += tot_g;
    }
    if (threadIdx.x == 0) {
        d.col_start[d.n_cols] = carry_a;
        d.col_gstart[d.n_cols] = carry_g;
        int ng = carry_g;
        if (ng > d.max_groups) {
            d.status[ST_OVERFLOW] = 1;
            atomicMax(&d.status[ST_NEED_GROUPS], ng);
            ng = d.max_groups;
        }
        d.n_groups[0] = ng;
    }
}

__global__ __launch_bounds__(1024) void k_col_scan(const SysDev* __restrict__ table, const int* flags, int first)
{
    const int mode = build_mode(flags, blockIdx.x, first);
    if (mode != 0) col_scan<1024>(table[blockIdx.x], mode);
}

// 3. scatter (z key, atom) into column segments: rank inside the block from an
//    LDS counter, one global reservation per (block, column); the per-column
//    sort makes the final order independent of the atomic order here.
//    SCAN (at most kHistLds columns): each block forms the column offsets from the
//    counts itself, and one more block does the column scan beside the others,
//    instead of a launch of its own before them (7.7 us for
//    both at 2744 atoms, 5.3 in one; 6.6 and 4.2 at 24000, 17.1 and 17.7 at a
//    million).
template <bool SCAN>
__global__ __launch_bounds__(256) void k_scatter(const SysDev* __restrict__ table, const int* flags, int first)
{
    const int mode = build_mode(flags, blockIdx.y, first);
    if (mode == 0) return;
    const SysDev& d = table[blockIdx.y];
    if (SCAN && blockIdx.x == gridDim.x - 1) {
        col_scan<256>(d, mode);
        return;
    }
    __shared__ int cnt[kHistLds];
    __shared__ int base[kHistLds];
    if ((int)(blockIdx.x * blockDim.x) >= d.n_atoms) return;
    const bool priv = d.n_cols <= kHistLds;
    if (priv)
        for (int c = threadIdx.x; c < d.n_cols; c += blockDim.x) {
            cnt[c] = 0;
            if (SCAN) base[c] = gld(&d.col_count[c]);
        }
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    const bool valid = i < d.n_atoms;
    const int col = valid ? gld(&d.atom_col[i]) : 0;
    const unsigned int zkey = valid ? gld(&d.atom_zkey[i]) : 0u;
    __syncthreads();
    int rank = 0;
    if (valid && priv) rank = atomicAdd(&cnt[col], 1);
    if (SCAN) {
        // exclusive prefix of the counts in place: a run of columns per thread
        __shared__ int wsum[4];
        const int run = (d.n_cols + 255) / 256, c0 = threadIdx.x * run, c1 = min(c0 + run, d.n_cols);
        int sum = 0;
        for (int c = c0; c < c1; ++c) sum += base[c];
        const int lane = threadIdx.x & 63, wid = threadIdx.x >> 6;
        int incl = sum;
        for (int o = 1; o < 64; o <<= 1) {
            const int t = __shfl_up(incl, o, 64);
            if (lane >= o) incl += t;
        }
        if (lane == 63) wsum[wid] = incl;
        __syncthreads();
        int at = incl - sum;
        for (int w = 0; w < wid; ++w) at += wsum[w];
        for (int c = c0; c < c1; ++c) {
            const int n = base[c];
            base[c] = at;
            at += n;
        }
    }
    __syncthreads();
    if (priv)
        for (int c = threadIdx.x; c < d.n_cols; c += blockDim.x)
            if (cnt[c]) base[c] = (SCAN ? base[c] : gld(&d.col_start[c])) + gatomic_add(&d.col_fill[c], cnt[c]);
    __syncthreads();
    if (valid) {
        const int pos = priv ? base[col] + rank : gld(&d.col_start[col]) + gatomic_add(&d.col_fill[col], 1);
        gst(&d.sort_key[pos], ((unsigned long long)zkey << 32) | (unsigned int)i);
    }
}

// 4a. sort of a column's n <= kSortLds (z key, atom) words into LDS by one block
//     of NT threads: counted into kSortBuckets buckets of the box height, placed
//     bucket by bucket, and ranked within the bucket (the keys are distinct: the
//     atom index is in the low word), so a key meets the few others at its height
//     instead of the whole column.  The
//     broadcast reads of a rank over the whole column bound it before: 172.7 us,
//     9.8 now, with a million atoms in long columns; 12.6 and 5.1 at 24000.
constexpr int kSortBuckets = 1024;

template <int NT>
__device__ __forceinline__ void sort_column(const unsigned long long* __restrict__ in, int n, unsigned long long* skeys,
                                            int* bucket)
{
    static_assert(kSortBuckets % NT == 0 || NT % kSortBuckets == 0, "buckets in runs");
    constexpr int kPer = (kSortLds + NT - 1) / NT, kRun = kSortBuckets / NT;
    __shared__ int wsum[NT / 64];
    unsigned long long key[kPer];
    int r[kPer];
    for (int c = threadIdx.x; c < kSortBuckets; c += NT) bucket[c] = 0;
#pragma unroll
    for (int k = 0; k < kPer; ++k) {
        if (k * NT >= n) break;
        const int t = k * NT + (int)threadIdx.x;
        key[k] = t < n ? gld(&in[t]) : ~0ull;
    }
    __syncthreads();
#pragma unroll
    for (int k = 0; k < kPer; ++k) {
        if (k * NT >= n) break;
        if (k * NT + (int)threadIdx.x < n) r[k] = atomicAdd(&bucket[key[k] >> 54], 1);
    }
    __syncthreads();
    // exclusive prefix of the bucket counts, in place
    int cnt[kRun], sum = 0;
#pragma unroll
    for (int u = 0; u < kRun; ++u) {
        cnt[u] = bucket[threadIdx.x * kRun + u];
        sum += cnt[u];
    }
    const int lane = threadIdx.x & 63, wid = threadIdx.x >> 6;
    int incl = sum;
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) {
        const int t = __shfl_up(incl, o, 64);
        if (lane >= o) incl += t;
    }
    if (lane == 63) wsum[wid] = incl;
    __syncthreads();
    int at = incl - sum;
#pragma unroll
    for (int w = 0; w < NT / 64 - 1; ++w) at += w < wid ? wsum[w] : 0;
#pragma unroll
    for (int u = 0; u < kRun; ++u) {
        bucket[threadIdx.x * kRun + u] = at;
        at += cnt[u];
    }
    __syncthreads();
#pragma unroll
    for (int k = 0; k < kPer; ++k) {
        if (k * NT >= n) break;
        if (k * NT + (int)threadIdx.x < n) skeys[bucket[key[k] >> 54] + r[k]] = key[k];
    }
    __syncthreads();
#pragma unroll
    for (int k = 0; k < kPer; ++k) {
        if (k * NT >= n) break;
        if (k * NT + (int)threadIdx.x < n) {
            const int b = (int)(key[k] >> 54);
            const int lo = bucket[b], hi = b + 1 < kSortBuckets ? bucket[b + 1] : n;
            int rank = lo;
            for (int u = lo; u < hi; ++u) rank += skeys[u] < key[k] ? 1 : 0;
            r[k] = rank;
        }
    }
    __syncthreads();
#pragma unroll
    for (int k = 0; k < kPer; ++k) {
        if (k * NT >= n) break;
        if (k * NT + (int)threadIdx.x < n) skeys[r[k]] = key[k];
    }
    __syncthreads();
}

// 4a. one block per column: the sort into sort_out, and each group's column and share
//     of the sorted keys.  Columns past kSortLds keys are sorted in place in HBM by a
//     bitonic network.
constexpr int kSortThreads = 512;

__global__ __launch_bounds__(kSortThreads) void k_col_sort(const SysDev* __restrict__ table, const int* flags)
{
    if (flags && !flags[blockIdx.y]) return;
    const SysDev& d = table[blockIdx.y];
    const int col = blockIdx.x;
    if (col >= d.n_cols) return;
    const int n = gld(&d.col_count[col]);
    const int base = gld(&d.col_start[col]);
    const int GM = d.G * d.M;
    const int g_begin = gld(&d.col_gstart[col]);
    const int n_grp = min((n + GM - 1) / GM, d.max_groups - g_begin);
    for (int t = threadIdx.x; t < n_grp; t += kSortThreads) {
        gst(&d.grp_col[g_begin + t], col);
        gst(&d.grp_range[g_begin + t], make_int2(base + t * GM, min(GM, n - t * GM)));
    }
    if (n <= kSortLds) {
        __shared__ unsigned long long skeys[kSortLds];
        __shared__ int bucket[kSortBuckets];
        sort_column<kSortThreads>(d.sort_key + base, n, skeys, bucket);
        for (int t = threadIdx.x; t < n; t += kSortThreads) gst(&d.sort_out[base + t], skeys[t]);
    } else {
        if (threadIdx.x == 0) d.status[ST_BIGCOL] = 1;
        int P = 1;
        while (P < n) P <<= 1;
        bitonic_sort(d.sort_key + base, n, P);  // block-coherent in HBM
        __syncthreads();
        for (int t = threadIdx.x; t < n; t += kSortThreads) gst(&d.sort_out[base + t], gld(&d.sort_key[base + t]));
    }
}

// LDS written by some lanes of a wave, read by others
__device__ __forceinline__ void wave_lds_sync()
{
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// 4b. one wave per i-group: the 2x2x2 split of its chunk of up to 8*M atoms (in z
//     order) into 8 clusters of M atoms, its slots and bounding boxes.  The halves'
//     ranks compare 64-bit keys (coordinate, atom) read two at a time from LDS, in
//     loops of fixed length (absent atoms: above every key): 13.9 us with the keys'
//     words read one by one over the atoms present, 6.1 now (24000 atoms, of which
//     a launch and three round trips are about 5; a million atoms 54.4 and 44.8).
//     Sorting and splitting in one kernel measured no gain (9.9 us for both at 2744
//     atoms, 8.5 in one; 11.2 and 11.7 at 24000), and spreads the groups of long
//     columns over fewer CUs.
// (one wave per block: the groups are independent and spread over all CUs)
__global__ __launch_bounds__(64) void k_group_split(const SysDev* __restrict__ table, const int* flags)
{
    if (flags && !flags[blockIdx.y]) return;
    const SysDev& d = table[blockIdx.y];
    __shared__ __align__(16) unsigned long long rank_key[64];
    __shared__ int place[64];
    const int gg = blockIdx.x, lane = threadIdx.x;
    // the group's key range (written by the column sort) is loaded together with
    // the group count (gg < max_groups: in bounds either way)
    const int ng_now = gld(&d.n_groups[0]);
    const int2 rg = gld(&d.grp_range[min(gg, d.max_groups - 1)]);
    if (gg >= ng_now) return;
    const int cnt = rg.y;
    const unsigned long long key = lane < cnt ? gld(&d.sort_out[rg.x + lane]) : 0ull;
    const int M = d.M, G = d.G, GM = G * M, H = 4 * M;
    // every load of the lane's atom at once (positions, image counts, the
    // staging's parameters); the original position and image counts go to the
    // slot arrays below
    double xo[3] = {0.0, 0.0, 0.0}, u[3] = {0.0, 0.0, 0.0};
    double qv = 0.0, sgv = 0.0, epv = 0.0;
    int wo[3] = {0, 0, 0};
    const int idx = (int)(key & 0xffffffffull);
    const bool have = lane < cnt;
    unsigned int kx = 0, ky = 0;
    if (have) {
        for (int c = 0; c < 3; ++c) {
            xo[c] = gld(&d.x[3 * idx + c]);
            wo[c] = gld(&d.atom_wrap[3 * idx + c]);
        }
        qv = gld(&d.q[idx]);
        if (d.lj == 1) {
            sgv = gld(&d.sig[idx]);
            epv = gld(&d.eps[idx]);
        }
        wrapped_pos(d, xo, wo, u);
        // integer rank keys (a strict total order with the atom index, also for
        // non-finite input)
        kx = coord_key(u[0], d.invbox[0]);
        ky = coord_key(u[1], d.invbox[1]);
    }
    typedef unsigned long long u64x2 __attribute__((ext_vector_type(2)));
    // z half by position in the z order, y half by rank in the z half, x half by
    // rank in the y half (the upper y half's keys above the lower's)
    const int zh = lane >= H ? 1 : 0, lo = have ? zh * H : 0, in_half = min(cnt, lo + H) - lo;
    const u64x2* half = (const u64x2*)&rank_key[lo];
    const unsigned long long yme = ((unsigned long long)ky << 32) | (unsigned int)idx;
    rank_key[lane] = have ? yme : ~0ull;
    if (lane < GM) place[lane] = -1;
    wave_lds_sync();
    int yr = 0;
#pragma unroll 4
    for (int m = 0; m < H / 2; ++m) {
        const u64x2 v = half[m];
        yr += (v.x < yme ? 1 : 0) + (v.y < yme ? 1 : 0);
    }
    const int yh = yr >= 2 * M ? 1 : 0;
    const unsigned long long xme = ((unsigned long long)yh << 63) | ((unsigned long long)kx << 31) | (unsigned int)idx;
    wave_lds_sync();
    rank_key[lane] = have ? xme : ~0ull;
    wave_lds_sync();
    int xr = 0;
#pragma unroll 4
    for (int m = 0; m < H / 2; ++m) {
        const u64x2 v = half[m];
        xr += (v.x < xme ? 1 : 0) + (v.y < xme ? 1 : 0);
    }
    xr -= yh ? min(2 * M, in_half) : 0;
    const int xh = xr >= M ? 1 : 0;
    if (have) place[(zh * 4 + yh * 2 + xh) * M + (xr - xh * M)] = lane;
    wave_lds_sync();
    // every atom to the lane of its slot in the group (lane = cluster * M + place)
    const int src = lane < GM ? place[lane] : -1;
    const bool real = src >= 0;
    const int from = real ? src : lane;
    const int at = __shfl(idx, from, 64);
    for (int c = 0; c < 3; ++c) {
        xo[c] = __shfl(xo[c], from, 64);
        wo[c] = __shfl(wo[c], from, 64);
        u[c] = __shfl(u[c], from, 64);
    }
    qv = __shfl(qv, from, 64);
    if (d.lj == 1) {
        sgv = __shfl(sgv, from, 64);
        epv = __shfl(epv, from, 64);
    }
    const int slot = gg * GM + lane;
    if (real) {
        gst(&d.slot_atom[slot], at);
        for (int c = 0; c < 3; ++c) {
            gst(&d.slot_wrap[3 * slot + c], wo[c]);
            gst(&d.slot_x[3 * slot + c], xo[c]);
        }
    }
    // bounding boxes: min/max over the M lanes of each cluster, then over all
    double lo3[3], hi3[3];
    for (int k = 0; k < 3; ++k) {
        lo3[k] = real ? u[k] : 1e300;
        hi3[k] = real ? u[k] : -1e300;
    }
    const unsigned long long rb = __ballot(real);
    for (int o = 1; o < M; o <<= 1)
        for (int k = 0; k < 3; ++k) {
            lo3[k] = fmin(lo3[k], __shfl_xor(lo3[k], o, 64));
            hi3[k] = fmax(hi3[k], __shfl_xor(hi3[k], o, 64));
        }
    if (lane < GM && (lane % M) == 0) {
        const int ci = gg * G + lane / M;
        const unsigned long long cm = (M >= 64) ? ~0ull : (((1ull << M) - 1ull) << lane);
        gst(&d.cl_nreal[ci], (int)__popcll(rb & cm));
        for (int c = 0; c < 3; ++c) {
            gst(&d.cl_bb[6 * ci + c], lo3[c]);
            gst(&d.cl_bb[6 * ci + 3 + c], hi3[c]);
        }
    }
    for (int o = M; o < 64; o <<= 1)
        for (int k = 0; k < 3; ++k) {
            lo3[k] = fmin(lo3[k], __shfl_xor(lo3[k], o, 64));
            hi3[k] = fmax(hi3[k], __shfl_xor(hi3[k], o, 64));
        }
    double ref[3];
    for (int c = 0; c < 3; ++c) ref[c] = 0.5 * (lo3[c] + hi3[c]);
    if (lane == 0)
        for (int c = 0; c < 3; ++c) {
            gst(&d.gr_bb[6 * gg + c], lo3[c]);
            gst(&d.gr_bb[6 * gg + 3 + c], hi3[c]);
            gst(&d.gr_ref[3 * gg + c], ref[c]);
        }
    // stage the group's slots at these positions (the force kernel's frame; the
    // same arithmetic as every other staging)
    if (lane < GM) {
        float4 p = pad_pos(slot);
        float2 l = make_float2(0.f, 0.f);
        if (real) {
            // u is the wrapped position of stage_pos (FP64, no contraction), so
            // (float)(u - ref) is the staged value
            p.x = (float)(u[0] - ref[0]);
            p.y = (float)(u[1] - ref[1]);
            p.z = (float)(u[2] - ref[2]);
            p.w = (float)(qv * (double)d.qscale);
            if (d.lj == 1) {
                l.x = (float)(0.5 * sgv);
                l.y = (float)(2.0 * sqrt(epv));
            }
        }
        gst(&d.xq[slot], p);
        if (d.lj == 1) gst(&d.ljs[slot], l);
    }
}

// 5. bounding-box search: one block of 8 waves per i-group; the waves share
//    out the column cells within reach; a wave tests a column's groups by their
//    boxes and the 8 j-clusters of a group in reach against the 8 i-clusters at once (lane = j * 8 + i-cluster), so the
//    byte j of the ballot is that j-cluster's i-cluster mask.  Candidates are
//    appended in any order, then sorted by (j-cluster, shift) so the list is
//    canonical (deterministic) and j-ordered for cache locality.  Each
//    candidate's mask is then pruned at the atom level in FP32 (below).
constexpr int kCandLds = 4096;
// Waves of a search block: 8, so that two blocks share a CU (their LDS and
// registers fill it); 16 where the launch has no more blocks than the GPU has CUs,
// so that a second block per CU would find no work (2,744 atoms 18.9 us
// against 21.0; an explicit build of 3,001 27.6 against 30.9, of 11,873 32 against 37).
// At 24,000 atoms (some 380 blocks) the second block per CU is worth more.
constexpr int kSearchWaves = 8, kSearchWavesFew = 16, kSearchFew = 256;
constexpr int kPruneXj = 2048;  // shifted j-atoms staged per chunk of candidates

// v with lane k replaced by the scalar x (v_writelane; clang has no builtin for the
// intrinsic, which the compiler then knows to keep clear of the SGPR hazards that an
// asm statement would have to)
extern "C" __device__ int nb_amdgcn_writelane(int x, int k, int v) __asm("llvm.amdgcn.writelane.i32");
__device__ __forceinline__ int lane_write(int x, int k, int v) { return nb_amdgcn_writelane(x, k, v); }

// Whether atom pair (i-slot si, j-slot sj) of a list entry with shift sid is in
// the exact pair set, in FP64 from the original positions: the minimum image as
// the set's definition takes it (the nearest multiples of c, b, a removed from
// z, y, x in that order; per dimension in a rectangular box), which must be this
// entry's image, and r^2 < r_list^2; inrc: also r^2 < r_cut^2.
__device__ __forceinline__ bool exact_pair(const SysDev& d, int si, int sj, int sid, bool& inrc)
{
    double e[3];
    int dw[3];
    for (int q = 0; q < 3; ++q) {
        e[q] = gld(&d.slot_x[3 * (size_t)sj + q]) - gld(&d.slot_x[3 * (size_t)si + q]);
        dw[q] = gld(&d.slot_wrap[3 * (size_t)sj + q]) - gld(&d.slot_wrap[3 * (size_t)si + q]);
    }
    const int s0 = sid % 5 - 2, s1 = (sid / 5) % 3 - 1, s2 = sid / 15 - 1;
    const double k2 = rint(e[2] * d.invbox[2]);
    const double e0 = e[0] - k2 * d.box_off[1], e1 = e[1] - k2 * d.box_off[2], z = e[2] - k2 * d.box[2];
    const double k1 = rint(e1 * d.invbox[1]);
    const double f0 = e0 - k1 * d.box_off[0], y = e1 - k1 * d.box[1];
    const double k0 = rint(f0 * d.invbox[0]);
    const double x = f0 - k0 * d.box[0];
    const bool own = (dw[0] - (int)k0 == s0) && (dw[1] - (int)k1 == s1) && (dw[2] - (int)k2 == s2);
    const double t = x * x + y * y;
    const double r2 = t + z * z;
    const bool bit = own && (r2 < d.rlist2);
    inrc = bit && (r2 < d.rcut2);
    return bit;
}

// Half-width of the band around r2c (r_list^2 or r_cut^2) in which an FP32 r^2
// of the search's frame does not decide whether the exact r^2 is below r2c.
// The frame's coordinates differ from the exact ones by at most 2^-24 (E + r)
// per component (E: the largest coordinate magnitudes that were rounded, i and
// j side added; r: the difference's own rounding), so r by sqrt(3) times that,
// and the sum of squares adds 3 roundings; the bound is doubled (which also covers
// its own FP32 arithmetic and the rounding of r2c).
__device__ __forceinline__ float exact_band(float r2c, float E)
{
    const float u = 1.0f / 16777216.0f, r = sqrtf(r2c);
    return 2.0f * (2.0f * r * 1.7320508f * u * (E + 1.01f * r) + 4.0f * u * r2c);
}

// EXACT: every atom pair of the kept candidates is decided as in the exact pair
// set (the masks go to cand_mask, the pairs within r_cut are counted); otherwise
// the FP32-pruned candidates are the list.  TRIC: some system of the launch has
// a triclinic box (the rectangular-only variant leaves that search out)
// M8: every system of the launch has 8-atom clusters (the cluster size a
// compile-time constant: the code for other sizes, and the scalar registers it
// holds, drop out of the variant)
//
// The exact decision rides on the FP32 prune: a pair whose FP32 r^2 lies outside
// the band above is decided by it (a pair within r_list has one image only, the
// entry's, so no image test is needed), and the few inside the band (about 1 in
// 10^4 cluster pairs) by FP64.  An exact prune of its own, testing every pair of
// every candidate in FP64, was the longest kernel of a build (104 us at 24,000
// atoms, 3.45 ms at 1,000,000); with the decision here a list build and force
// call takes 234 against 329 us and 3.20 against 6.31 ms.  A candidate is checked
// against the bands once, by the least distance of any of its r^2 to a radius, and
// so no ballots for both edges of both bands at every cluster pair (1188 us at
// 1,000,000 atoms).  There the kernel issues vector instructions 80 % of the time, so
// a cluster pair's 12 (17 with two differences and selects for the mask words) and a
// candidate's own (prefetched without a branch, the mask pointer held) set the time:
// 949 us against 1012.
template <bool TRIC, bool M8, bool EXACT, int W>
__global__ __launch_bounds__(64 * W, 4) void k_search(const SysDev* __restrict__ table, const int* flags)
{
    if (flags && !flags[blockIdx.y]) return;
    const SysDev& d = table[blockIdx.y];
    const int gi = blockIdx.x;
    if (gi >= d.n_groups[0]) return;
    const int wid = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int lane = threadIdx.x & 63;
    __shared__ __align__(16) unsigned long long keys_lds[kCandLds];
    __shared__ double ibb[kGroup][6];
    __shared__ float4 ixq[64];      // the group's staged i-atoms (slot order)
    __shared__ float4 xjs[kPruneXj];
    __shared__ int inr_s[kGroup];   // real atoms per i-cluster
    __shared__ int count_s, kept_s, kw_s;
    __shared__ int rc_s, ei_s, ej_s;  // (EXACT) pairs within r_cut; float bits of E's i and j parts
    const int G = d.G;
    const int M = M8 ? 8 : d.M;
    if (threadIdx.x < kGroup * 6) ibb[threadIdx.x / 6][threadIdx.x % 6] = d.cl_bb[6 * (gi * G) + threadIdx.x];
    if (threadIdx.x < G * M) ixq[threadIdx.x] = d.xq[(size_t)gi * G * M + threadIdx.x];
    if (threadIdx.x < kGroup) inr_s[threadIdx.x] = d.cl_nreal[gi * G + threadIdx.x];
    if (threadIdx.x == 0) {
        count_s = 0;
        kept_s = 0;
        kw_s = 0;
        rc_s = 0;
        ei_s = 0;
        ej_s = 0;
    }
    const double rl = d.rbb;
    const double rl2 = rl * rl;
    double gb[6];
    for (int k = 0; k < 6; ++k) gb[k] = d.gr_bb[6 * gi + k];
    const int ci0 = gi * G;
    const int ng_tot = d.n_groups[0];
    const int cap = d.cand_cap;
    // the group's column (unwrapped cell coordinates of the search start there)
    const int colg = gld(&d.grp_col[gi]);
    const int cxi = colg % d.ncx, cyi = colg / d.ncx;
    // keys past the LDS array are staged in the group's own candidate region
    // (8 bytes each)
    unsigned long long* gkeys = (unsigned long long*)(d.cand + (size_t)gi * cap);
    bool finite = true;
    for (int k = 0; k < 6; ++k) finite = finite && (fabs(gb[k]) < 1e9);
    __syncthreads();
    // this lane's i-cluster and its box
    const int g = lane & 7, jj = lane >> 3;
    double ib[6];
    for (int k = 0; k < 6; ++k) ib[k] = ibb[g][k];
    if (finite) {
        const int ci = ci0 + g;
        // Test the 8 clusters of group gj at once (lane = j * 8 + i-cluster),
        // with the j offset (ox, oy) in x and y and each z image t of tmask (z
        // shift t - 1, offset (t - 1) c_z).  The group owns the pair in its own
        // column (no x/y shift) with the z shift +1, or without a z shift with
        // cj >= ci (cj == ci: the cluster with itself).  An empty cluster's box is
        // out of reach of everything.
        double bn[6];
        auto load_group = [&](int gj) {
            const double* bb = d.cl_bb + 6 * ((size_t)gj * G + jj);
            for (int k = 0; k < 6; ++k) bn[k] = gld(bb + k);
        };
        auto test_group = [&](int gj, int sx, int sy, bool own_col, unsigned int tmask, double ox, double oy) {
            const int cj = gj * G + jj;
            const double fx = box_gap(ib[0], ib[3], bn[0] + ox, bn[3] + ox);
            const double fy = box_gap(ib[1], ib[4], bn[1] + oy, bn[4] + oy);
            const double fxy = fx * fx + fy * fy;
            for (int t = 0; t < 3; ++t) {
                if (!((tmask >> t) & 1u)) continue;
                const double zoff = (t - 1) * d.box[2];
                const double fz = box_gap(ib[2], ib[5], bn[2] + zoff, bn[5] + zoff);
                const int sid = shift_id(sx, sy, t - 1);
                const bool owns = !own_col || t == 2 || (t == 1 && cj >= ci);
                const unsigned long long bal = __ballot(owns && fxy + fz * fz < rl2);
                if (bal == 0ull) continue;
                // byte jj of the ballot: the i-cluster mask of j-cluster cj
                const unsigned long long nz = __ballot(g == 0 && ((bal >> (8 * jj)) & 255ull) != 0ull);
                const int n = __popcll(nz);
                int base = 0;
                if (lane == 0) base = atomicAdd(&count_s, n);  // LDS atomic
                base = __shfl(base, 0, 64);
                if ((nz >> lane) & 1ull) {
                    const int pos = base + __popcll(nz & ((1ull << lane) - 1ull));
                    const unsigned long long im = (bal >> (8 * jj)) & 255ull;
                    // appended into LDS; only keys past the LDS array go to HBM
                    const unsigned long long key =
                        ((unsigned long long)cj << 16) | ((unsigned long long)sid << 8) | im;
                    if (pos < min(cap, kCandLds)) keys_lds[pos] = key;
                    else if (pos < cap) gst(gkeys + pos, key);
                }
            }
        };
        // Half list by half-space, the same share for every group: in unwrapped
        // cell coordinates (periodic images included) the group owns its pairs
        // with the columns above it in y, with those above it in x in its own
        // row, and in its own column as above.  Seen from the other cluster a
        // pair has the opposite offset, so every cluster pair and shift is
        // listed once.  The cell coordinates count lattice images, not
        // distances, so the rule holds in triclinic boxes too.
        //
        // The cells in reach are worked out one per lane (the same in every
        // wave), with their columns' groups; wave w takes every W-th of the
        // non-empty ones from the w-th on.  A wave tests up to 64 groups of a
        // column by their boxes, one per lane, and only the groups in reach by
        // their clusters (all clusters of every column tested, as before, the
        // scan took 28 us per block in a 21.5 nm box against 11.6 in 6.2 nm).
        int taken = 0;  // non-empty cells so far
        auto scan_cells = [&](bool in_cell, int sx, int sy, bool own, unsigned int tmask, int col, double xo,
                              double yo) {
            int g0 = 0, g1 = 0;
            if (in_cell) {
                g0 = gld(&d.col_gstart[col]);
                g1 = min(gld(&d.col_gstart[col + 1]), ng_tot);
            }
            const unsigned long long cells = __ballot(g0 < g1);
            unsigned long long mine = __ballot(
                g0 < g1 && ((taken + __popcll(cells & ((1ull << lane) - 1ull))) & (W - 1)) == wid);
            taken += __popcll(cells);
            while (mine) {
                const int l = __builtin_ctzll(mine);
                mine &= mine - 1ull;
                const int c0 = __builtin_amdgcn_readlane(g0, l), c1 = __builtin_amdgcn_readlane(g1, l);
                const int csx = __builtin_amdgcn_readlane(sx, l), csy = __builtin_amdgcn_readlane(sy, l);
                const bool cown = __builtin_amdgcn_readlane(own ? 1 : 0, l) != 0;
                const double ox = csx * d.box[0] + (TRIC ? csy * d.box_off[0] + xo : 0.0);
                const double oy = csy * d.box[1] + (TRIC ? yo : 0.0);
                for (int cb = c0; cb < c1; cb += 64) {
                    double q[6];
                    const double* bb = d.gr_bb + 6 * (size_t)min(cb + lane, c1 - 1);
                    for (int k = 0; k < 6; ++k) q[k] = gld(bb + k);
                    const double fx = box_gap(gb[0], gb[3], q[0] + ox, q[3] + ox);
                    const double fy = box_gap(gb[1], gb[4], q[1] + oy, q[4] + oy);
                    const double fxy = fx * fx + fy * fy;
                    unsigned int tm = 0u;
                    for (int t = 0; t < 3; ++t) {
                        const double zoff = (t - 1) * d.box[2];
                        const double fz = box_gap(gb[2], gb[5], q[2] + zoff, q[5] + zoff);
                        const bool owns = !cown || t == 2 || (t == 1 && cb + lane >= gi);
                        if (((tmask >> t) & 1u) && owns && fxy + fz * fz < rl2) tm |= 1u << t;
                    }
                    unsigned long long hit = __ballot(cb + lane < c1 && tm != 0u);
                    if (hit) load_group(cb + __builtin_ctzll(hit));
                    while (hit) {
                        const int h = __builtin_ctzll(hit);
                        hit &= hit - 1ull;
                        test_group(cb + h, csx, csy, cown, (unsigned int)__builtin_amdgcn_readlane((int)tm, h), ox, oy);
                        if (hit) load_group(cb + __builtin_ctzll(hit));
                    }
                }
            }
        };
        if (!TRIC || !d.tric) {
            // gb lies in [0, L) and r_list < L/2, so the ranges span at most [-n, 2n)
            const int cx0 = max(-d.ncx, (int)floor((gb[0] - rl) * d.inv_cell[0]));
            const int cx1 = min(2 * d.ncx - 1, (int)floor((gb[3] + rl) * d.inv_cell[0]));
            const int cy0 = max(-d.ncy, (int)floor((gb[1] - rl) * d.inv_cell[1]));
            const int cy1 = min(2 * d.ncy - 1, (int)floor((gb[4] + rl) * d.inv_cell[1]));
            const int nxc = cx1 - cx0 + 1;
            const int ncell = nxc * (cy1 - cy0 + 1);
            // the (up to 3) periodic z images in reach: j images occupy [zoff, zoff + L)
            unsigned int tmask = 0u;
            for (int t = 0; t < 3; ++t) {
                const double zoff = (t - 1) * d.box[2];
                if (!(gb[2] - rl >= zoff + d.box[2] || gb[5] + rl < zoff)) tmask |= 1u << t;
            }
            for (int base = 0; base < ncell; base += 64) {
                const int cell = base + lane;
                const int cy = cy0 + cell / nxc, cx = cx0 + cell % nxc;
                const int dcy = cy - cyi, dcx = cx - cxi;
                const bool own = dcy == 0 && dcx == 0;
                const int sy = floor_div(cy, d.ncy), sx = floor_div(cx, d.ncx);
                const int cyw = cy - sy * d.ncy, cxw = cx - sx * d.ncx;
                const double ylo = cyw * d.cell[1] + sy * d.box[1];
                const double gy = box_gap(gb[1], gb[4], ylo, ylo + d.cell[1]);
                const double xlo = cxw * d.cell[0] + sx * d.box[0];
                const double gx = box_gap(gb[0], gb[3], xlo, xlo + d.cell[0]);
                const bool in = cell < ncell && (dcy > 0 || (dcy == 0 && dcx >= 0)) && gx * gx + gy * gy < rl2;
                scan_cells(in, sx, sy, own, tmask, in ? cxw + d.ncx * cyw : 0, 0.0, 0.0);
            }
        } else {
            // triclinic: the j-image with lattice shift (sx, sy, sz) of column
            // (cxw, cyw) is offset by sx a + sy b + sz c, so each z image moves the
            // cells in x and y (sz c_x, sz c_y) and each y image moves a row in x
            // (sy b_x); per z image the rows in reach, per row its cells
            const int nxc = (int)floor((gb[3] - gb[0] + 2.0 * rl) * d.inv_cell[0]) + 2;
            for (int t = 0; t < 3; ++t) {
                const int sz = t - 1;
                const double zoff = sz * d.box[2];
                if (gb[2] - rl >= zoff + d.box[2] || gb[5] + rl < zoff) continue;
                const double cxo = sz * d.box_off[1], cyo = sz * d.box_off[2];
                const int cy0 = (int)floor((gb[1] - rl - cyo) * d.inv_cell[1]);
                const int cy1 = (int)floor((gb[4] + rl - cyo) * d.inv_cell[1]);
                const int ncell = nxc * (cy1 - cy0 + 1);
                for (int base = 0; base < ncell; base += 64) {
                    const int cell = base + lane;
                    const int cy = cy0 + cell / nxc;
                    const int sy = floor_div(cy, d.ncy);
                    const int cyw = cy - sy * d.ncy;
                    const double xo = sy * d.box_off[0] + cxo;  // this row's image offset in x (without sx)
                    const int cx = (int)floor((gb[0] - rl - xo) * d.inv_cell[0]) + cell % nxc;
                    const int dcy = cy - cyi, dcx = cx - cxi;
                    const bool own = dcy == 0 && dcx == 0;
                    const int sx = floor_div(cx, d.ncx);
                    const int cxw = cx - sx * d.ncx;
                    const double ylo = cyw * d.cell[1] + sy * d.box[1] + cyo;
                    const double gy = box_gap(gb[1], gb[4], ylo, ylo + d.cell[1]);
                    const double xlo = cxw * d.cell[0] + sx * d.box[0] + xo;
                    const double gx = box_gap(gb[0], gb[3], xlo, xlo + d.cell[0]);
                    // (the own column's pairs with the z shift -1 are owned from the other side)
                    const bool in = cell < ncell && cx <= (int)floor((gb[3] + rl - xo) * d.inv_cell[0]) &&
                                    (dcy > 0 || (dcy == 0 && dcx >= 0)) && !(own && sz < 0) &&
                                    gx * gx + gy * gy < rl2;
                    scan_cells(in, sx, sy, own, 1u << t, in ? cxw + d.ncx * cyw : 0, cxo, cyo);
                }
            }
        }
    }
    __syncthreads();
    const int count = count_s;
    const int n = min(count, cap);
    int P = 1;
    while (P < n) P <<= 1;
    // sorted in LDS when they fit, else in place in HBM (each branch with its
    // own address space, so LDS accesses are not flat ones)
    const bool in_lds = n <= kCandLds;
    if (in_lds) {
        // the keys are distinct (one per j-cluster and shift)
        if (n <= 64 * W) rank_sort_lds<64 * W>(keys_lds, n, (int*)xjs);
        else bitonic_sort(keys_lds, n, P);
    } else {
        for (int t = threadIdx.x; t < kCandLds; t += blockDim.x) gst(gkeys + t, keys_lds[t]);
        __syncthreads();
        bitonic_sort(gkeys, n, P);
    }
    __syncthreads();
    // keys -> candidate words, in chunks (in place: a chunk's keys are read
    // before its words are written).  The i-cluster mask of each candidate is
    // pruned in the force kernel's FP32 frame (the positions staged at this
    // build, the entry's FP32 shift vector): a bit stays if the cluster pair has
    // an atom pair within r_list (1 + 2^-14), a margin far above that frame's
    // rounding, so every cluster pair the exact FP64 test keeps is kept.
    //  (a) one thread per (candidate, j-atom): the shifted j-atoms of the chunk
    //      into LDS (w = 1 for a real atom), all loads in flight together;
    //  (b) one wave per candidate: pair p = k*64 + lane of the group's
    //      8*M*M pairs is (i-cluster p/(M*M), i-atom (p/M) mod M, j-atom p mod M),
    //      as in the exact prune's mask words, so each pair costs a difference,
    //      r^2 and a compare.
    const int LM = (M == 8) ? 3 : (M == 4) ? 2 : 0;  // M is 1, 4 or 8
    const int MM = M * M;
    const int K = (kGroup * MM + 63) / 64;  // 64-pair words per cluster pair
    const float rlp = d.rl2_prune;
    // (the group's reference as the split forms it, without a load)
    const double ri[3] = {0.5 * (gb[0] + gb[3]), 0.5 * (gb[1] + gb[4]), 0.5 * (gb[2] + gb[5])};
    // this lane's i-atom of word k (registers)
    float4 xr[8];
#pragma unroll
    for (int k = 0; k < 8; ++k) {
        const int p = k * 64 + lane;
        xr[k] = (k < K && p < kGroup * MM) ? ixq[p >> LM] : make_float4(0.f, 0.f, 0.f, 0.f);
    }
    const unsigned long long segm = (MM >= 64) ? ~0ull : ((1ull << MM) - 1ull);
    const unsigned long long tri8 = __ballot((lane >> 3) < (lane & 7));    // M = 8: a < b
    const unsigned long long offd8 = __ballot((lane >> 3) != (lane & 7));  // a != b
    // a wave's kept candidates and their weight (wave-uniform), added to the
    // group's totals once at the end
    int kept_w = 0, kw_w = 0;
    int rc_w = 0;  // (EXACT) the wave's pairs within r_cut
    // (loaded here: after the stores in the loop the compiler would load the
    // pointer again for every candidate, and wait)
    unsigned long long* cmask = EXACT ? d.cand_mask + (size_t)gi * cap * K : nullptr;
    if (EXACT) asm volatile("" : "+s"(cmask));
    if (EXACT && threadIdx.x < G * M && (int)(threadIdx.x & (M - 1)) < inr_s[threadIdx.x >> LM]) {
        const float4 p = ixq[threadIdx.x];
        atomicMax(&ei_s, __float_as_int(fmaxf(fabsf(p.x), fmaxf(fabsf(p.y), fabsf(p.z)))));
    }
    for (int t0 = 0; t0 < n; t0 += kPruneXj / M) {
        const int cnt = min(n - t0, kPruneXj / M);
        // the chunk's keys are read from LDS only (keys sorted in HBM are
        // copied into the then unused key array first), so no read below
        // waits on the stores of the candidate words
        int k0 = t0;
        if (!in_lds) {
            for (int q = threadIdx.x; q < cnt; q += blockDim.x) keys_lds[q] = gld(gkeys + t0 + q);
            __syncthreads();
            k0 = 0;
        }
        // (a) a fixed number of items per thread with clamped indices: all their
        //     loads are issued first, then the shifts are formed
        constexpr int kU = kPruneXj / (64 * W);
        float4 xjv[kU];
        double rjv[kU][3];
        int nrv[kU], sidv[kU];
#pragma unroll
        for (int u = 0; u < kU; ++u) {
            const int qc = min((int)threadIdx.x + u * 64 * W, cnt * M - 1);
            const unsigned long long kv = keys_lds[k0 + (qc >> LM)];
            const int cj = (int)(kv >> 16), gj = cj / G;
            sidv[u] = (int)((kv >> 8) & 255ull);
            xjv[u] = gld(&d.xq[(size_t)cj * M + (qc & (M - 1))]);
            nrv[u] = gld(&d.cl_nreal[cj]);
            for (int c = 0; c < 3; ++c) rjv[u][c] = gld(&d.gr_ref[3 * gj + c]);
        }
        float ej = 0.0f;
#pragma unroll
        for (int u = 0; u < kU; ++u) {
            const int q = threadIdx.x + u * 64 * W;
            const float4 S = entry_shift(d, rjv[u], sidv[u], ri);
            const bool real = (q & (M - 1)) < nrv[u];
            const float4 p = make_float4(xjv[u].x + S.x, xjv[u].y + S.y, xjv[u].z + S.z, real ? 1.0f : 0.0f);
            if (q < cnt * M) xjs[q] = p;
            if (EXACT && real && q < cnt * M)
                ej = fmaxf(ej, fmaxf(fabsf(xjv[u].x) + fabsf(S.x) + fabsf(p.x),
                                     fmaxf(fabsf(xjv[u].y) + fabsf(S.y) + fabsf(p.y),
                                           fabsf(xjv[u].z) + fabsf(S.z) + fabsf(p.z))));
        }
        if (EXACT) {
            // (values >= 0: their bits order as they do)
            int m = __float_as_int(ej);
            m = max(m, __builtin_amdgcn_update_dpp(0, m, 0x111, 0xF, 0xF, true));  // row_shr 1, 2, 4, 8:
            m = max(m, __builtin_amdgcn_update_dpp(0, m, 0x112, 0xF, 0xF, true));  // lane 15 of a row
            m = max(m, __builtin_amdgcn_update_dpp(0, m, 0x114, 0xF, 0xF, true));  // has the row's
            m = max(m, __builtin_amdgcn_update_dpp(0, m, 0x118, 0xF, 0xF, true));
            if ((lane & 15) == 15) atomicMax(&ej_s, m);  // (a NaN position: fmaxf drops it)
        }
        __syncthreads();
        // (EXACT) an FP32 r^2 within band of either squared radius decides nothing
        // (the wider band of the two, r_list's, for both).  r^2 is formed less the
        // middle of the two, which lie at -half and +half then: one difference tells
        // the distance to the nearer, and the first FMA takes the middle for free.
        const float mid = (float)(0.5 * (d.rlist2 + d.rcut2)), half = (float)(0.5 * (d.rlist2 - d.rcut2));
        const float bandw =
            EXACT ? exact_band((float)d.rlist2, __int_as_float(ei_s) + __int_as_float(ej_s)) : 0.0f;
        // (b) the next candidate's key and j-atoms are read while this one is tested
        unsigned long long kv_n = 0ull;
        float4 xj_n = make_float4(0.f, 0.f, 0.f, 0.f);
        if (wid < cnt) {
            kv_n = keys_lds[k0 + wid];
            xj_n = xjs[wid * M + (lane & (M - 1))];
        }
        // the wave's q-th candidate of the chunk is recorded by lane q mod 64;
        // its word (and the j-cluster count) is written with the wave's others
        // once 64 are recorded or the chunk ends: one store for them all
        int rec_n = 0, rec_c0 = wid;  // recorded so far, the first of them
        int rec_cj = 0, rec_w = 0;
        auto write_recorded = [&]() {
            if (lane < rec_n) {
                gst(&d.cand[(size_t)gi * cap + t0 + rec_c0 + lane * W], make_int2(rec_cj, rec_w));
                // the list's entries per j-cluster (the transpose's counts)
                if (((rec_w >> 8) & 255) != 0) gatomic_add(&d.jfill[rec_cj], 1);
            }
            rec_c0 += rec_n * W;
            rec_n = 0;
        };
        for (int c = wid; c < cnt; c += W) {
            // key = cj << 16 | sid << 8 | imask (the same for the whole wave)
            const unsigned long long kv = kv_n;
            const float4 xj = xj_n;
            // (past the last one the chunk's last again, unused)
            const int cn = min(c + W, cnt - 1);
            kv_n = keys_lds[k0 + cn];
            xj_n = xjs[cn * M + (lane & (M - 1))];
            const int cj = __builtin_amdgcn_readfirstlane((int)(kv >> 16));
            const int sid = __builtin_amdgcn_readfirstlane((int)((kv >> 8) & 255ull));
            const unsigned int im = (unsigned int)__builtin_amdgcn_readfirstlane((int)(kv & 255ull));
            // a cluster with itself: at zero shift each pair once (a < b), with
            // one of its images every pair but a == b (an atom and its own image,
            // never within r_list; for a padding slot no distance would tell)
            const int gself = cj - ci0;
            const bool once = sid == kShiftZero;
            unsigned int keep = 0u;
            // (EXACT) lane k: word k of the candidate's atom-pair mask; its pairs
            // within r_cut; the least distance of this lane's r^2 to a radius
            int wlo = 0, whi = 0, nrc = 0;
            float near = 1e30f;
            auto word = [&](int k, float dx, float dy, float dz, unsigned long long on) {
                const float t = fmaf(dz, dz, fmaf(dy, dy, fmaf(dx, dx, -mid)));
                // (the lesser of two values >= 0; 0, so undecided, if one is NaN)
                near = __builtin_amdgcn_fmed3f(near, fabsf(fabsf(t) - half), 0.0f);
                const unsigned long long lo = __ballot(t < half) & on;
                wlo = lane_write((int)lo, k, wlo);
                whi = lane_write((int)(lo >> 32), k, whi);
                nrc += __popcll(__ballot(t < -half) & on);
            };
            if (M == 8) {
                // word g = i-cluster g, lanes (a, b) (padding slots lie out of
                // reach of every other slot)
                auto clusters = [&](auto self) {
#pragma unroll
                    for (int g = 0; g < kGroup; ++g) {
                        if (!((im >> g) & 1u)) continue;
                        const unsigned long long on = !self.value || g != gself ? ~0ull : once ? tri8 : offd8;
                        const float dx = xr[g].x - xj.x, dy = xr[g].y - xj.y, dz = xr[g].z - xj.z;
                        if (EXACT) word(g, dx, dy, dz, on);
                        else if (__ballot(fmaf(dz, dz, fmaf(dy, dy, dx * dx)) < rlp) & on) keep |= 1u << g;
                    }
                };
                if ((unsigned int)gself < (unsigned int)kGroup)
                    clusters(std::true_type{});
                else
                    clusters(std::false_type{});
            } else {
#pragma unroll
            for (int k = 0; k < 8; ++k) {
                if (k >= K) break;
                // i-clusters of word k, and its lanes that hold a pair to test
                const int glo = (k * 64) >> (2 * LM), ghi = min(kGroup - 1, (k * 64 + 63) >> (2 * LM));
                unsigned long long on = 0ull;
                for (int g = glo; g <= ghi; ++g) {
                    if (!((im >> g) & 1u)) continue;
                    unsigned long long sg = segm << ((g * MM) & 63);
                    if (g == gself) {
                        const int a = ((k * 64 + lane) >> LM) & (M - 1), b = lane & (M - 1);
                        sg &= __ballot(once ? a < b : a != b);
                    }
                    on |= sg;
                }
                if (on == 0ull) continue;
                const float dx = xr[k].x - xj.x, dy = xr[k].y - xj.y, dz = xr[k].z - xj.z;
                if (EXACT) {
                    word(k, dx, dy, dz, on);
                    continue;
                }
                const unsigned long long hit = __ballot(fmaf(dz, dz, fmaf(dy, dy, dx * dx)) < rlp) & on;
                for (int g = glo; g <= ghi; ++g)
                    if (hit & (segm << ((g * MM) & 63))) keep |= 1u << g;
            }
            }
            if (EXACT) {
                unsigned long long wv = (unsigned long long)(unsigned int)whi << 32 | (unsigned int)wlo;
                // with an undecided pair: all of its pairs in FP64
                if (__ballot(near <= bandw)) {
                    nrc = 0;
                    for (int k = 0; k < K; ++k) {
                        const int p = k * 64 + lane, g = p / MM, a = (p >> LM) & (M - 1), b = lane & (M - 1);
                        bool bit = false, inrc = false;
                        if (g < kGroup && ((im >> g) & 1u) && a < inr_s[g] && xj.w != 0.0f &&
                            !(g == gself && once && a >= b))
                            bit = exact_pair(d, gi * G * M + (p >> LM), cj * M + b, sid, inrc);
                        const unsigned long long w = __ballot(bit);
                        wv = lane == k ? w : wv;
                        nrc += __popcll(__ballot(inrc));
                    }
                }
                if (lane < K) gst(cmask + (size_t)(t0 + c) * K + lane, wv);
                // the i-clusters with a pair left (lanes past the words hold none)
                if (M == 8) {
                    keep = (unsigned int)__ballot(wv != 0ull);
                } else {
                    const int k0 = lane < kGroup ? (lane * MM) >> 6 : 0;
                    const unsigned long long w = __shfl(wv, k0, 64);
                    keep = (unsigned int)__ballot(lane < kGroup && (w & (segm << ((lane * MM) & 63))) != 0ull);
                }
                rc_w += nrc;
            }
            if (keep) {
                kept_w += 1;
                kw_w += entry_weight(M, keep);
            }
            rec_cj = lane_write(cj, rec_n, rec_cj);
            rec_w = lane_write(sid | (int)(keep << 8), rec_n, rec_w);
            if (++rec_n == 64) write_recorded();
        }
        write_recorded();
        __syncthreads();
    }
    if (lane == 0 && kept_w > 0) {
        atomicAdd(&kept_s, kept_w);  // LDS atomics
        atomicAdd(&kw_s, kw_w);
    }
    if (EXACT && lane == 0 && rc_w > 0) atomicAdd(&rc_s, rc_w);
    __syncthreads();
    if (threadIdx.x == 0) {
        d.cand_count[gi] = count;
        d.cand_kept[gi] = kept_s;
        d.grp_w[gi] = kw_s;
        d.grp_rc[gi] = rc_s;
        if (count > cap) {
            d.status[ST_OVERFLOW] = 1;
            atomicMax(&d.status[ST_NEED_CAND], count);
        }
    }
}

// Exact FP64 atom-pair masks of a list built without them (refinement for
// export and statistics): kPruneBlocks blocks of 4 waves per i-group, waves
// stride over the group's candidates, one atom pair per lane.  The candidate's
// i-cluster mask (the one the force list was written from) is left as it is; its
// word takes the pairs-within-r_cut count.
constexpr int kPruneBlocks = 8;

__global__ __launch_bounds__(256) void k_prune(const SysDev* __restrict__ table)
{
    const SysDev& d = table[blockIdx.y];
    const int gi = blockIdx.x / kPruneBlocks;
    if (gi >= d.n_groups[0]) return;
    const int wid = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int wg = (blockIdx.x % kPruneBlocks) * 4 + wid;
    const int lane = threadIdx.x & 63;
    const int M = d.M, G = d.G, MM = M * M, GM = G * M;
    const int ncand = min(d.cand_count[gi], d.cand_cap);
    const int words = d.mask_words;  // <= 8: G * M * M / 64 rounded up, M <= 8
    // the group's i-atoms (<= 64 slots), shared by the block's 4 waves; a
    // padding slot has atom -1
    __shared__ double ix[64][3];
    __shared__ int iw[64][3];
    __shared__ int ireal[64];
    if (threadIdx.x < GM) {
        const int sa = gi * GM + threadIdx.x;
        const bool real = d.slot_atom[sa] >= 0;
        ireal[threadIdx.x] = real ? 1 : 0;
        for (int q = 0; q < 3; ++q) {
            ix[threadIdx.x][q] = real ? d.slot_x[3 * sa + q] : 0.0;
            iw[threadIdx.x][q] = real ? d.slot_wrap[3 * sa + q] : 0;
        }
    }
    __syncthreads();
    if (wg >= ncand) return;
    // word p, lane l is pair (k, a, b) with p*64 + l = k*M*M + a*M + b: its
    // i-atom is group slot (p*64 + l) / M, its j-atom b is the same in every word
    const int b = lane % M;
    const double box0 = d.box[0], box1 = d.box[1], box2 = d.box[2];
    const double off0 = d.box_off[0], off1 = d.box_off[1], off2 = d.box_off[2];  // b_x, c_x, c_y
    const double ib0 = d.invbox[0], ib1 = d.invbox[1], ib2 = d.invbox[2];
    const double rl2 = d.rlist2, rc2 = d.rcut2;
    // software pipeline: the next candidate and its j-atom are loaded while the
    // current one is tested
    int2 cd_n = d.cand[(size_t)gi * d.cand_cap + wg];
    int sb_n = cd_n.x * M + b;
    int jat_n = d.slot_atom[sb_n];
    double xb_n[3] = {d.slot_x[3 * sb_n], d.slot_x[3 * sb_n + 1], d.slot_x[3 * sb_n + 2]};
    int wb_n[3] = {d.slot_wrap[3 * sb_n], d.slot_wrap[3 * sb_n + 1], d.slot_wrap[3 * sb_n + 2]};
    for (int c = wg; c < ncand; c += kPruneBlocks * 4) {
        const size_t ce = (size_t)gi * d.cand_cap + c;
        const int2 cd = cd_n;
        const bool jreal = jat_n >= 0;
        const double xb[3] = {xb_n[0], xb_n[1], xb_n[2]};
        const int wb[3] = {wb_n[0], wb_n[1], wb_n[2]};
        if (c + kPruneBlocks * 4 < ncand) {
            cd_n = d.cand[ce + kPruneBlocks * 4];
            sb_n = cd_n.x * M + b;
            jat_n = d.slot_atom[sb_n];
            for (int q = 0; q < 3; ++q) {
                xb_n[q] = d.slot_x[3 * sb_n + q];
                wb_n[q] = d.slot_wrap[3 * sb_n + q];
            }
        }
        const int cj = cd.x;
        const int sid = cd.y & 255;
        const unsigned int im = (unsigned int)(cd.y >> 8) & 255u;
        const int s0 = sid % 5 - 2, s1 = (sid / 5) % 3 - 1, s2 = sid / 15 - 1;
        int nrc = 0;
        for (int p = 0; p < words; ++p) {
            // i-clusters covered by this 64-pair word: [p*64/MM, (p*64+63)/MM]
            const int k_lo = (p * 64) / MM, k_hi = min(G - 1, (p * 64 + 63) / MM);
            const unsigned int wmask = ((2u << k_hi) - 1u) & ~((1u << k_lo) - 1u);
            if (!(im & wmask)) {  // no listed i-cluster in this word
                if (lane == 0) d.cand_mask[ce * words + p] = 0ull;
                continue;
            }
            const int pi = p * 64 + lane;
            const int k = pi / MM, a = (pi / M) % M, ia = min(pi / M, 63);
            bool bit = false, inrc = false;
            if (jreal && k < G && ((im >> k) & 1u) && ireal[ia] &&
                !(gi * G + k == cj && sid == kShiftZero && a >= b)) {
                // the minimum image as the pair-set definition takes it: the
                // nearest multiples of c, b, a removed from z, y, x in that
                // order (per dimension in a rectangular box)
                double e0 = xb[0] - ix[ia][0], e1 = xb[1] - ix[ia][1], e2 = xb[2] - ix[ia][2];
                const double k2 = rint(e2 * ib2);
                e0 = e0 - k2 * off1;
                e1 = e1 - k2 * off2;
                e2 = e2 - k2 * box2;
                const double k1 = rint(e1 * ib1);
                e0 = e0 - k1 * off0;
                e1 = e1 - k1 * box1;
                const double k0 = rint(e0 * ib0);
                e0 = e0 - k0 * box0;
                const bool own = (wb[0] - iw[ia][0] - (int)k0 == s0) && (wb[1] - iw[ia][1] - (int)k1 == s1) &&
                                 (wb[2] - iw[ia][2] - (int)k2 == s2);
                const double t = e0 * e0 + e1 * e1;
                const double r2 = t + e2 * e2;
                bit = own && (r2 < rl2);
                inrc = bit && (r2 < rc2);
            }
            nrc += __popcll(__ballot(inrc));
            const unsigned long long w = __ballot(bit);
            if (lane == 0) d.cand_mask[ce * words + p] = w;
        }
        if (lane == 0) d.cand[ce] = make_int2(cj, (cd.y & 0xffff) | (min(nrc, 4095) << 16));
    }
}

// kept candidates and pairs within r_cut per i-group after that (one wave per group)
__global__ __launch_bounds__(256) void k_count_kept(const SysDev* __restrict__ table)
{
    const SysDev& d = table[blockIdx.y];
    const int wid = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int lane = threadIdx.x & 63;
    const int gi = blockIdx.x * 4 + wid;
    if (gi >= d.n_groups[0]) return;
    const int ncand = min(d.cand_count[gi], d.cand_cap);
    int kept = 0, nrc = 0, kw = 0;
    for (int cb = 0; cb < ncand; cb += 64) {
        const int c = cb + lane;
        int2 cd = make_int2(0, 0);
        if (c < ncand) cd = d.cand[(size_t)gi * d.cand_cap + c];
        const int y = cd.y;
        const bool kp = ((y >> 8) & 255) != 0;
        kept += __popcll(__ballot(kp));
        if (kp) kw += entry_weight(d.M, (unsigned int)(y >> 8));
        nrc += (y >> 16) & 4095;
    }
    for (int o = 32; o > 0; o >>= 1) {
        nrc += __shfl_xor(nrc, o, 64);
        kw += __shfl_xor(kw, o, 64);
    }
    if (lane == 0) {
        d.cand_kept[gi] = kept;
        d.grp_w[gi] = kw;
        d.grp_rc[gi] = nrc;
    }
}

// 6. CSR offsets of kept entries and work items (block (system, 0)), and of the
//    transpose: per j-cluster, the rows of the entries that name it (blocks (system,
//    1 ..), kScanSlice clusters each, every block summing the counts before its own;
//    the counts come from the search or the exact prune, and the list writer counts
//    them down to place the entries).  One block for all of it took 152 us at a
//    million atoms, latency over latency; 16.8
//    now (24000 atoms: 7.3 and 4.8).  item_prefix (one system
//    only): the prefix {0, items} the force kernel reads; seen (one system, may be
//    NULL): the build's verdict for the host {seq, items, capacity exceeded}.
constexpr int kScanSlice = 8 * 1024;

__global__ __launch_bounds__(1024) void k_list_scan(const SysDev* __restrict__ table, const int* flags,
                                                     int* item_prefix, unsigned long long* seen, unsigned int seq)
{
    if (flags && !flags[blockIdx.x]) return;
    const SysDev& d = table[blockIdx.x];
    __shared__ int smem[40];
    const int ng = gld(&d.n_groups[0]);
    const int over0 = gld(&d.status[ST_OVERFLOW]);  // (groups or candidates, by the kernels before)
    if (blockIdx.y > 0) {
        // (8 clusters per thread, one group's: 32 bytes)
        const int ncl = ng * d.G, first = ((int)blockIdx.y - 1) * kScanSlice, c = first + 8 * (int)threadIdx.x;
        if (first >= ncl) {
            if (ncl == 0 && blockIdx.y == 1 && threadIdx.x == 0) d.jstart[0] = 0;
            return;
        }
        int4 v0 = make_int4(0, 0, 0, 0), v1 = v0;
        if (c < ncl) {
            v0 = gld((const int4*)&d.jfill[c]);
            v1 = gld((const int4*)&d.jfill[c + 4]);
        }
        int before = 0, carry, tot;
#pragma unroll 4
        for (int k = 4 * (int)threadIdx.x; k < first; k += 4 * 1024) {
            const int4 v = gld((const int4*)&d.jfill[k]);
            before += (v.x + v.y) + (v.z + v.w);
        }
        if (first > 0)
            block_exclusive_scan(before, smem, &carry);
        else
            carry = 0;
        const int sum = ((v0.x + v0.y) + (v0.z + v0.w)) + ((v1.x + v1.y) + (v1.z + v1.w));
        const int at = carry + block_exclusive_scan(sum, smem, &tot);
        if (c < ncl) {
            int4 s0, s1;
            s0.x = at;
            s0.y = s0.x + v0.x;
            s0.z = s0.y + v0.y;
            s0.w = s0.z + v0.z;
            s1.x = s0.w + v0.w;
            s1.y = s1.x + v1.x;
            s1.z = s1.y + v1.y;
            s1.w = s1.z + v1.z;
            gst((int4*)&d.jstart[c], s0);
            gst((int4*)&d.jstart[c + 4], s1);
        }
        if (threadIdx.x == 0 && first + kScanSlice >= ncl) d.jstart[ncl] = carry + tot;
        return;
    }
    const int W = d.item_w;
    // (4 groups per thread and round; the last quad's loads stay within the arrays'
    // padding to 256 bytes)
    int carry_e = 0, carry_i = 0;
    for (int base = 0; base < ng; base += 4 * 1024) {
        const int g = base + 4 * (int)threadIdx.x;
        int4 kv = make_int4(0, 0, 0, 0), wv = kv;
        if (g < ng) {
            kv = gld((const int4*)&d.cand_kept[g]);
            wv = gld((const int4*)&d.grp_w[g]);
        }
        const int kept[4] = {kv.x, kv.y, kv.z, kv.w}, w[4] = {wv.x, wv.y, wv.z, wv.w};
        int se = 0, si = 0, te, ti;
#pragma unroll
        for (int u = 0; u < 4; ++u)
            if (g + u < ng) {
                se += kept[u];
                si += (w[u] + W - 1) / W;
            }
        int ee = carry_e + block_exclusive_scan(se, smem, &te);
        int ei = carry_i + block_exclusive_scan(si, smem, &ti);
#pragma unroll
        for (int u = 0; u < 4; ++u)
            if (g + u < ng) {
                gst(&d.ent_start[g + u], ee);
                gst(&d.item_start[g + u], ei);
                ee += kept[u];
                ei += (w[u] + W - 1) / W;
            }
        carry_e += te;
        carry_i += ti;
    }
    if (threadIdx.x == 0) {
        d.ent_start[ng] = carry_e;
        d.item_start[ng] = carry_i;
        int ne = carry_e, ni = carry_i;
        if (ne > d.ent_cap) {
            d.status[ST_OVERFLOW] = 1;
            atomicMax(&d.status[ST_NEED_ENT], ne);
        }
        if (ni > d.item_cap) {
            d.status[ST_OVERFLOW] = 1;
            atomicMax(&d.status[ST_NEED_ITEM], ni);
        }
        const bool over = ne > d.ent_cap || ni > d.item_cap, any = over || over0 != 0;
        d.n_ent[0] = over ? ~0 : any ? ~ne : ne;
        d.n_items[0] = over ? 0 : ni;
        if (item_prefix) {
            item_prefix[0] = 0;
            item_prefix[1] = over ? 0 : ni;
        }
        d.status[ST_ITEMS] = ni;
        if (seen)
            __hip_atomic_store(seen, (any ? 1ull << 63 : 0ull) | (unsigned long long)(unsigned int)ni << 32 | seq,
                               __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
    }
}

// Inclusive sum over the wave by DPP row moves and broadcasts
__device__ __forceinline__ int wave_scan(int v)
{
    v += __builtin_amdgcn_update_dpp(0, v, 0x111, 0xF, 0xF, true);  // row_shr 1, 2, 4, 8
    v += __builtin_amdgcn_update_dpp(0, v, 0x112, 0xF, 0xF, true);
    v += __builtin_amdgcn_update_dpp(0, v, 0x114, 0xF, 0xF, true);
    v += __builtin_amdgcn_update_dpp(0, v, 0x118, 0xF, 0xF, true);
    v += __builtin_amdgcn_update_dpp(0, v, 0x142, 0xA, 0xF, false);  // row_bcast 15 into rows 1, 3
    v += __builtin_amdgcn_update_dpp(0, v, 0x143, 0xC, 0xF, false);  // row_bcast 31 into rows 2, 3
    return v;
}

// 7. compacted entries, shift vectors and work items: one block per i-group, a
//    candidate per thread.  Bound by its chain of round trips: everything that
//    depends on the group alone, and the first candidates, is loaded in one.  (With
//    a wave per group, its 64 candidates at a time one after the other, the group's
//    values behind two early exits and 64-bit divisions, the kernel took 9.1 us at
//    24,389 atoms and 7.5 at 2,744, now 4.9 and 3.9; 38.6 at 1,000,000, now 37.6.)
__global__ __launch_bounds__(256) void k_list_write(const SysDev* __restrict__ table, const int* flags)
{
    if (flags && !flags[blockIdx.y]) return;
    const SysDev& d = table[blockIdx.y];
    const int wid = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int lane = threadIdx.x & 63;
    if ((int)blockIdx.x >= d.max_groups) return;
    const int gi = blockIdx.x;
    const int *jstart = d.jstart, *nreal = d.cl_nreal;
    const double* gr_ref = d.gr_ref;
    int* jfill = d.jfill;
    int2* ent = d.ent;
    float4* entS = d.ent_S;
    int4* items = d.items;
    struct {
        double box[3], box_off[3];
    } bx;
    for (int k = 0; k < 3; ++k) {
        bx.box[k] = d.box[k];
        bx.box_off[k] = d.box_off[k];
    }
    const int G = d.G, M = d.M, W = d.item_w, cap = d.cand_cap;
    const int2* cand = d.cand + (size_t)gi * cap;
    const int ng = gld(d.n_groups), ne = gld(d.n_ent), nc = gld(&d.cand_count[gi]);
    const int e0 = gld(&d.ent_start[gi]), e1 = gld(&d.ent_start[gi + 1]);
    const int it0 = gld(&d.item_start[gi]), it1 = gld(&d.item_start[gi + 1]), wg = gld(&d.grp_w[gi]);
    const double ri[3] = {gld(&gr_ref[3 * gi]), gld(&gr_ref[3 * gi + 1]), gld(&gr_ref[3 * gi + 2])};
    int2 cd = gld(&cand[min((int)threadIdx.x, cap - 1)]);
    __shared__ int tot[2][4];
    if (gi >= ng) return;
    if (ne == 0 || ne == ~0) return;  // empty list, or overflow: list unusable
    const int ncand = min(nc, cap);
    const int nit = it1 - it0;
    // the group's weight wg is cut into its nit = ceil(wg / W) items at the
    // points floor(k wg / nit), so its items weigh the same (not nit - 1 of W
    // and a remainder); when those points lie closer together than an entry
    // can weigh, at the multiples of W instead
    const bool even = nit > 0 && wg / nit >= (M == 8 ? kEntWMax : 1);
    const bool small = (long long)wg * (nit + 1) < 0x7fffffffll;  // (the products below fit 32 bits)
    int pos = e0, wpos = 0;  // entries and weight before these 256 candidates
    for (int cb = 0, par = 0; cb < ncand; cb += 256, par ^= 1) {
        const int c = cb + (int)threadIdx.x;
        if (cb > 0) cd = gld(&cand[min(c, cap - 1)]);
        const bool keep = c < ncand && ((cd.y >> 8) & 255) != 0;
        // the entry's place and weight range [P, P + w) among the group's kept
        // entries, counted together (the weight of 256 is below 2^16)
        const int w = keep ? entry_weight(M, (unsigned int)(cd.y >> 8)) : 0;
        const int inc = wave_scan(w | (keep ? 1 << 16 : 0));
        if (lane == 63) tot[par][wid] = inc;
        __syncthreads();
        int before = 0, all = 0;
        for (int u = 0; u < 4; ++u) {
            const int t = tot[par][u];
            before += u < wid ? t : 0;
            all += t;
        }
        if (keep) {
            const int P = wpos + ((before + inc) & 0xffff) - w;
            const int e = pos + ((before + inc) >> 16) - 1;
            const int cj = cd.x, sid = cd.y & 255, gj = cj / G;
            // the row of this entry's j-force partial, carried in the shift
            // vector's w word: the j-cluster's rows are contiguous; the order
            // inside them depends on atomics, and the gather's int64
            // fixed-point sums do not depend on it
            const int left = gatomic_add(&jfill[cj], -1), row0 = gld(&jstart[cj]), nr = gld(&nreal[cj]);
            const double rj[3] = {gld(&gr_ref[3 * gj]), gld(&gr_ref[3 * gj + 1]), gld(&gr_ref[3 * gj + 2])};
            // meta: shift id, the i-clusters to evaluate (all the build kept,
            // until a dynamic prune narrows them), j real atoms, the build's
            // i-clusters
            gst(&ent[e], make_int2(cj, (cd.y & 0xffff) | (nr << kMetaNreal) | (((cd.y >> 8) & 255) << kMetaOuter)));
            float4 S = entry_shift(bx, rj, sid, ri);
            S.w = __int_as_float(row0 + left - 1);
            gst(&entS[e], S);
            // the entry whose range holds item k's point starts work item k:
            // {group, first entry, end, its j-cluster} (the force kernel loads
            // the first j-atoms with the item).  The points lie at least an
            // entry's weight apart, so a range holds at most one; the end is
            // the next item's first entry
            int k;
            bool starts;
            if (!even) {
                k = (P + W - 1) / W;
                starts = k * W < P + w;
            } else if (small) {
                k = (int)((unsigned int)(P * nit + wg - 1) / (unsigned int)wg);  // the first point >= P
                starts = k < nit && (int)((unsigned int)(k * wg) / (unsigned int)nit) < P + w;
            } else {
                k = (int)(((long long)P * nit + wg - 1) / wg);
                starts = k < nit && ((long long)k * wg) / nit < P + w;
            }
            if (starts) {
                int* item = (int*)&items[it0 + k];
                gst(item, gi);
                gst(item + 1, e);
                gst(item + 3, cj);
                if (k > 0) gst(item - 2, e);  // .z of item k - 1
                if (k == nit - 1) gst(item + 2, e1);
            }
        }
        pos += all >> 16;
        wpos += all & 0xffff;
    }
}

__global__ void k_clear_status(const SysDev* __restrict__ table, int keep_faults)
{
    const SysDev& d = table[blockIdx.x];
    const int t = threadIdx.x;
    if (t < ST_COUNT && !(keep_faults && (t == ST_SATURATE || t == ST_BADPOS))) d.status[t] = 0;
}

hipError_t launch_clear_status(const SysDev* table, int n_sys, hipStream_t s, bool keep_faults)
{
    hipLaunchKernelGGL(k_clear_status, dim3(n_sys), dim3(64), 0, s, table, keep_faults ? 1 : 0);
    return hipGetLastError();
}

template <int W>
static auto pick_search(const Bounds& b, bool exact)
{
    return b.any_tric ? (b.all_m8 ? (exact ? k_search<true, true, true, W> : k_search<true, true, false, W>)
                                  : (exact ? k_search<true, false, true, W> : k_search<true, false, false, W>))
                      : (b.all_m8 ? (exact ? k_search<false, true, true, W> : k_search<false, true, false, W>)
                                  : (exact ? k_search<false, false, true, W> : k_search<false, false, false, W>));
}

hipError_t launch_build(const SysDev* table, int n_sys, const Bounds& b, const int* flags, hipStream_t s,
                        bool exact, int status_clear, int* item_prefix, bool first, bool cleared,
                        unsigned long long* seen, unsigned int seq)
{
    const int clear_n = max(max(b.max_cols, b.max_groups * kGroup), (int)ST_COUNT);
    // enough blocks for the clears and for the displacement partials
    const int atom_b = min(kKeBlocks, max(1, (b.max_atoms + 255) / 256));
    const int fst = first ? 1 : 0;
    if (!cleared)
        hipLaunchKernelGGL(k_build_clear, dim3(max((clear_n + 255) / 256, atom_b), n_sys), dim3(256), 0, s, table,
                           flags, status_clear, fst);
    hipLaunchKernelGGL(k_bin, dim3((b.max_atoms + 255) / 256, n_sys), dim3(256), 0, s, table, flags);
    if (b.max_cols <= kHistLds) {
        hipLaunchKernelGGL(k_scatter<true>, dim3((b.max_atoms + 255) / 256 + 1, n_sys), dim3(256), 0, s, table, flags,
                           fst);
    } else {
        hipLaunchKernelGGL(k_col_scan, dim3(n_sys), dim3(1024), 0, s, table, flags, fst);
        hipLaunchKernelGGL(k_scatter<false>, dim3((b.max_atoms + 255) / 256, n_sys), dim3(256), 0, s, table, flags,
                           fst);
    }
    hipLaunchKernelGGL(k_col_sort, dim3(b.max_cols, n_sys), dim3(kSortThreads), 0, s, table, flags);
    hipLaunchKernelGGL(k_group_split, dim3(b.max_groups, n_sys), dim3(64), 0, s, table, flags);
    const bool few = b.max_groups * n_sys <= kSearchFew;
    auto search = few ? pick_search<kSearchWavesFew>(b, exact) : pick_search<kSearchWaves>(b, exact);
    hipLaunchKernelGGL(search, dim3(b.max_groups, n_sys), dim3(64 * (few ? kSearchWavesFew : kSearchWaves)), 0, s,
                       table, flags);
    const int slices = (b.max_groups * kGroup + kScanSlice - 1) / kScanSlice;
    hipLaunchKernelGGL(k_list_scan, dim3(n_sys, 1 + slices), dim3(1024), 0, s, table, flags, n_sys == 1 ? item_prefix : nullptr,
                       n_sys == 1 ? seen : nullptr, seq);
    hipLaunchKernelGGL(k_list_write, dim3(b.max_groups, n_sys), dim3(256), 0, s, table, flags);
    return hipGetLastError();
}

hipError_t launch_refine(const SysDev* table, int n_sys, const Bounds& b, hipStream_t s)
{
    hipLaunchKernelGGL(k_prune, dim3(b.max_groups * kPruneBlocks, n_sys), dim3(256), 0, s, table);
    hipLaunchKernelGGL(k_count_kept, dim3((b.max_groups + 3) / 4, n_sys), dim3(256), 0, s, table);
    return hipGetLastError();
}

// OR of the members' overflow / saturation flags into out[0..1]
__global__ void k_ens_status(const SysDev* __restrict__ table, int n_sys, int* out)
{
    int ov = 0, sat = 0;
    for (int i = threadIdx.x; i < n_sys; i += blockDim.x) {
        ov |= table[i].status[ST_OVERFLOW];
        sat |= table[i].status[ST_SATURATE] | table[i].status[ST_BADPOS];
    }
    if (ov) atomicOr(&out[0], 1);
    if (sat) atomicOr(&out[1], 1);
}

__global__ void k_zero_ints(int* p, int n)
{
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n) p[i] = 0;
}

hipError_t launch_ens_status(const SysDev* table, int n_sys, int* out, hipStream_t s)
{
    hipLaunchKernelGGL(k_zero_ints, dim3(1), dim3(64), 0, s, out, 2);
    hipLaunchKernelGGL(k_ens_status, dim3(1), dim3(256), 0, s, table, n_sys, out);
    return hipGetLastError();
}

}  // namespace nbi
