// nb_internal.h -- device data layout and launch helpers of libnb (gfx950).
//
// One system lives in one caller-provided arena.  Its descriptor (SysDev) is a
// plain struct of sizes, model constants and device pointers into the arena; a
// copy sits at the start of the arena so that kernels can read it, and batched
// launches read an array of such descriptors (one per member system).
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>
#include <stddef.h>

namespace nbi {

constexpr int kWave = 64;
constexpr int kGroup = 8;            // clusters per i-group (2 x 2 x 2 split of a column chunk)
// periodic shift (sx, sy, sz) of a list entry: sx a + sy b + sz c, sx in -2..2
// (a skewed box's rows can reach two a-images), sy, sz in -1..1
__host__ __device__ constexpr int shift_id(int sx, int sy, int sz) { return (sx + 2) + 5 * (sy + 1) + 15 * (sz + 1); }
constexpr int kShiftZero = shift_id(0, 0, 0);
constexpr int kSortLds = 4096;       // column keys sorted in LDS (larger columns sort in HBM)
constexpr int kTraceCap = 1024;      // device energy-trace ring rows
constexpr int kEoutAt = 64;          // the status words, padded to this; eout follows,
constexpr int kStatusBytes = 192;    // and the trace ring after that (one copy returns them)
constexpr int kKeBlocks = 4096;      // max blocks of the per-system partial sums (kinetic energy, max|F|)
constexpr int kEnerPart = 8;         // per-item partials: E_lj, E_c, W_xx, W_yy, W_zz, W_xy, W_xz, W_yz
constexpr int kEwTab = 256;          // cubic intervals of the Ewald tables on [0, r_cut]
constexpr int kEwTabN = kEwTab + 1;  // plus one interval past r_cut: an FP32 r that rounds to r_cut reads a valid one

// List entry meta word: bits 0-7 shift id, 8-15 the i-clusters the force
// kernel evaluates (after a dynamic prune: those with a pair within r_inner),
// 16-19 real atoms of the j-cluster, 20-27 the i-clusters the build listed.
constexpr int kMetaInner = 8;
constexpr int kMetaNreal = 16;
constexpr int kMetaOuter = 20;

// Work items of the force kernel cut by cost.  With 8-atom clusters a list
// entry costs a fixed part (its loads, the j-force reduction and store: about
// 3.5 times the cost of one listed cluster pair, measured per item on MI355X)
// plus a part per i-cluster it lists: weight kEntW0 + kEntW1 popcount(mask).
// A group's kept entries, in list order, cover consecutive weight ranges
// [P, P + w); an entry whose range holds a multiple of the item weight W starts
// an item, so a group has ceil(total / W) items of about equal cost.  Other
// cluster sizes weigh every entry 1 (items of jtile entries).
constexpr int kEntW0 = 7;
constexpr int kEntW1 = 2;
constexpr int kEntWMax = kEntW0 + kEntW1 * kGroup;
constexpr int kEntWNom = 16;  // jtile counts nominal entries of this weight
__host__ __device__ inline int entry_weight(int M, unsigned int im)
{
    return M == 8 ? kEntW0 + kEntW1 * __builtin_popcount(im & 255u) : 1;
}
__host__ __device__ inline int item_weight(int M, int jtile)
{
    return M == 8 ? (jtile * kEntWNom > kEntWMax ? jtile * kEntWNom : kEntWMax) : jtile;
}
// items for ent entries in n_groups groups, at most
__host__ __device__ inline double item_bound(int M, int jtile, double ent, int n_groups)
{
    return ent * (M == 8 ? kEntWMax : 1) / item_weight(M, jtile) + n_groups;
}

// global-address-space loads (the pointers live in a descriptor, so the compiler
// would otherwise emit flat loads); vector types go through ext_vector_type
// because aggregate copies would drop the address space
typedef float nb_v4f __attribute__((ext_vector_type(4)));
typedef float nb_v2f __attribute__((ext_vector_type(2)));
typedef double nb_v2d __attribute__((ext_vector_type(2)));
typedef int nb_v2i __attribute__((ext_vector_type(2)));
typedef int nb_v4i __attribute__((ext_vector_type(4)));
#define NB_GLOBAL __attribute__((address_space(1)))

__device__ __forceinline__ float4 gld(const float4* p)
{
    const nb_v4f v = *(const NB_GLOBAL nb_v4f*)p;
    return make_float4(v.x, v.y, v.z, v.w);
}
__device__ __forceinline__ float2 gld(const float2* p)
{
    const nb_v2f v = *(const NB_GLOBAL nb_v2f*)p;
    return make_float2(v.x, v.y);
}
__device__ __forceinline__ double2 gld(const double2* p)
{
    const nb_v2d v = *(const NB_GLOBAL nb_v2d*)p;
    return make_double2(v.x, v.y);
}
__device__ __forceinline__ int2 gld(const int2* p)
{
    const nb_v2i v = *(const NB_GLOBAL nb_v2i*)p;
    return make_int2(v.x, v.y);
}
__device__ __forceinline__ int4 gld(const int4* p)
{
    const nb_v4i v = *(const NB_GLOBAL nb_v4i*)p;
    return make_int4(v.x, v.y, v.z, v.w);
}
// scalars (int, float, double, 64-bit words)
template <class T>
__device__ __forceinline__ T gld(const T* p)
{
    return *(const NB_GLOBAL T*)p;
}
template <class T>
__device__ __forceinline__ void gst(T* p, T v)
{
    *(NB_GLOBAL T*)p = v;
}
__device__ __forceinline__ void gst(int2* p, int2 v) { *(NB_GLOBAL nb_v2i*)p = nb_v2i{v.x, v.y}; }
__device__ __forceinline__ void gst(double2* p, double2 v) { *(NB_GLOBAL nb_v2d*)p = nb_v2d{v.x, v.y}; }
__device__ __forceinline__ void gst(int4* p, int4 v) { *(NB_GLOBAL nb_v4i*)p = nb_v4i{v.x, v.y, v.z, v.w}; }
__device__ __forceinline__ void gst(float4* p, float4 v) { *(NB_GLOBAL nb_v4f*)p = nb_v4f{v.x, v.y, v.z, v.w}; }
__device__ __forceinline__ void gst(float2* p, float2 v) { *(NB_GLOBAL nb_v2f*)p = nb_v2f{v.x, v.y}; }
// a wave-uniform base plus a lane's 32-bit byte offset (a scalar base register
// and a vector offset in the instruction, no 64-bit vector arithmetic)
__device__ __forceinline__ float4 gld4(const void* base, unsigned int off)
{
    const nb_v4f v = *(const NB_GLOBAL nb_v4f*)((const NB_GLOBAL char*)base + off);
    return make_float4(v.x, v.y, v.z, v.w);
}
__device__ __forceinline__ float2 gld2(const void* base, unsigned int off)
{
    const nb_v2f v = *(const NB_GLOBAL nb_v2f*)((const NB_GLOBAL char*)base + off);
    return make_float2(v.x, v.y);
}
__device__ __forceinline__ void gst1(void* base, unsigned int off, float v)
{
    *(NB_GLOBAL float*)((NB_GLOBAL char*)base + off) = v;
}
// device-scope integer add in the global address space (a flat atomic would
// also count against the LDS wait counter)
__device__ __forceinline__ int gatomic_add(int* p, int v)
{
    return __hip_atomic_fetch_add((NB_GLOBAL int*)p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// Blocks per system for per-atom loops: a function of the system alone, so the
// kinetic-energy partial sums decompose the same way alone and in a batch.
__device__ inline int sys_blocks(int n_atoms)
{
    int b = (n_atoms + 255) / 256;
    return b > kKeBlocks ? kKeBlocks : (b < 1 ? 1 : b);
}


// status word indices
enum { ST_OVERFLOW = 0, ST_NEED_CAND = 1, ST_NEED_ENT = 2, ST_NEED_ITEM = 3, ST_NEED_GROUPS = 4,
       ST_SATURATE = 5, ST_BIGCOL = 6, ST_BADPOS = 7, ST_ITEMS = 8, ST_COUNT = 9 };  // ST_ITEMS: work items of the build

struct SysDev {
    // ---- what the pair kernel reads for every work item, in four cache lines --
    // (its waves start with these loads, so they are kept together)
    int4* items;          // [item_cap] {group, e0, e1, j-cluster of entry e0}
    float4* ew_tab;       // [kEwTabN] cubic coefficients of q(r) = erfc(beta r) + 2 beta r/sqrt(pi) exp(-beta^2 r^2)
    float4* xq;           // [max_slots] local x,y,z, scaled charge
    int2* ent;            // [ent_cap] {cj, sid | imask<<8 | nreal(cj)<<16}
    float4* ent_S;        // [ent_cap] shift vector (FP32); w: the row of the entry's j-partial (int bits)
    // force partials, summed by the gather
    float* jpart;         // [ent_cap*M*3] j-atom forces of each entry
    float* ipart;         // [item_cap*G*M*3] i-atom forces of each work item
    float2* ljs;          // [max_slots] sigma/2, 2 sqrt(eps)
    // model (FP32 pair arithmetic)
    float rc2;
    float ew_tinv;                  // kEwTab / r_cut
    float c6x6, c12x12, c6, c12;    // single-type LJ
    float krf2, krf, crf;           // 2 k_rf, k_rf, c_rf
    float rin2;                     // r_inner^2 (dynamic pruning in the force kernel; 0: off)
    float ew_shift;                 // erfc(beta rc)/rc (0 without shift)
    float lj_shift;                 // single type: c12/rc^12 - c6/rc^6
    float irc6, irc12;              // 1/rc^6, 1/rc^12 (LB shift)
    int pot_shift;
    float4* ew_etab;      // [kEwTabN] cubic coefficients of e(r) = erfc(beta r) (energies)
    float* epart;         // [item_cap*kEnerPart]
    // ---- sizes -------------------------------------------------------
    int n_atoms;
    int M;              // cluster size
    int G;              // clusters per group (kGroup)
    int ncx, ncy;       // coarse columns
    int n_cols;
    int max_groups;
    int cand_cap;       // candidates per group
    int ent_cap;        // entries (total)
    int item_cap;       // work items (total)
    int jtile;          // entries per work item (nominal entries with 8-atom clusters)
    int item_w;         // weight per work item: item_weight(M, jtile)
    int mask_words;     // u64 words of atom masks per entry (G*M*M/64 rounded up)
    int coulomb, lj, fp32_reduce;
    // ---- geometry (FP64) ---------------------------------------------
    double box[3], invbox[3];
    double box_off[3];  // triclinic b_x, c_x, c_y (a = (box0,0,0), b = (b_x,box1,0), c = (c_x,c_y,box2))
    int tric;           // box_off not all zero
    double cell[2], inv_cell[2];
    double rlist2;      // exact pair criterion r^2 < rlist2
    double rcut2;       // FP64 r_cut^2 (list statistics only)
    double rbb;         // bounding-box search radius (r_list + margin)
    // ---- model ----------------------------------------------------------
    float rl2_prune;                // r_list^2 (1 + 2^-14): the search's FP32 atom-pair prune
    int prune_on;                   // dynamic pruning configured
    double prune_half;              // (r_inner - r_cut) / 2: the prune interval's displacement guard
    float qscale;                   // sqrt(1/(4 pi eps0 eps_r))
    double fx_scale, fx_inv;        // fixed-point 2^bits, 2^-bits
    float fx_lim;                   // max |partial| representable
    // ---- per-atom inputs (device copies, original order) ----------------
    const double* q;      // [N]
    const double* sig;    // [N] (LB)
    const double* eps;    // [N] (LB)
    const double* mass;   // [N]
    // ---- caller state (set per call) -----------------------------------
    const double* x;      // [N,3]
    double* v;            // [N,3]
    float* f;             // [N,3]
    // ---- binning -------------------------------------------------------
    int* atom_col;        // [N]
    int* atom_wrap;       // [N,3]
    unsigned int* atom_zkey; // [N]
    int* col_count;       // [n_cols]
    int* col_fill;        // [n_cols]
    int* col_start;       // [n_cols+1]
    int* col_gstart;      // [n_cols+1]
    unsigned long long* sort_key; // [N] (z key, atom) words in column segments, unsorted
    unsigned long long* sort_out; // [N] the same, sorted within each column
    // ---- slots (cluster order) ----------------------------------------
    int* slot_atom;       // [max_slots] original atom or -1
    int* slot_wrap;       // [max_slots*3]
    double* slot_x;       // [max_slots*3] original FP64 positions at build (exact prune)
    // ---- clusters and groups -------------------------------------------
    int* n_groups;        // [1]
    int* cl_nreal;        // [max_groups*G]
    double* cl_bb;        // [max_groups*G*6] lo.xyz, hi.xyz (wrapped frame)
    double* gr_ref;       // [max_groups*3]
    double* gr_bb;        // [max_groups*6]
    int* grp_col;         // [max_groups] column of each group
    int2* grp_range;      // [max_groups] each group's atoms: {first sorted key, count}
    // ---- candidates ------------------------------------------------------
    int* cand_count;      // [max_groups]
    int2* cand;           // [max_groups*cand_cap] {cj, sid | imask<<8}
    unsigned long long* cand_mask; // [max_groups*cand_cap*mask_words]
    int* cand_kept;       // [max_groups]
    int* grp_rc;          // [max_groups] atom pairs within r_cut at build (statistics)
    int* grp_w;           // [max_groups] weight of the kept entries (work-item cutting)
    // ---- list ------------------------------------------------------------
    int* ent_start;       // [max_groups+1]
    int* item_start;      // [max_groups+1]
    // ---- transpose of the list (a j-cluster's rows of partials) ----------
    int* jstart;          // [max_groups*G+1] entries that list each cluster as j (CSR)
    int* jfill;           // [max_groups*G] their counts, counted down as the list is written
    int* n_items;         // [1]
    int* n_ent;           // [1] entries written; ~ of it if a capacity was exceeded
    // ---- reductions and outputs -----------------------------------------
    double* ke_part;      // [kKeBlocks]
    double* eout;         // [16]: E_lj, E_c, Xi xx,yy,zz,xy,xz,yz, KE; kEoutAt bytes after status
    double* trace;        // [kTraceCap*5], kStatusBytes after status
    double* fmax_part;    // [kKeBlocks]
    int* status;          // [ST_COUNT]
    double* x_build;      // [N,3] positions at the last list build
    double* x_bak;        // [N,3] x, v at the last full step before a rebuild step
    double* v_bak;        //       (restored if that rebuild runs out of capacity)
    double* disp;         // [kKeBlocks] per-block max displacement^2; [kKeBlocks..+2): max, violations
    double* x_prune;      // [N,3] positions at the last dynamic prune (or build)
    double* pg_part;      // [2 kKeBlocks + 2]: two buffers of per-block max displacement^2 of a
                          // prune interval, then the statistics {max displacement, violations}
    double buffer;        // r_list - r_cut
    int* stats;           // [8] scratch for statistics
    // pair export scratch
    long long* exp_count; // [max_groups+1]
    // ---- reciprocal-space Ewald (PME), NULL without it -------------------
    const float* pme_f;   // [N,3] reciprocal-space forces, added by the gather
    const double* pme_e;  // [8] reciprocal + self + background energy, Xi xx,yy,zz,xy,xz,yz
};

// The list-buffer guard's partials: every kernel that measures a list lifetime leaves
// this many (a gather's blocks have 4 clusters each, or more; an atom loop has fewer
// blocks), zero where it has nothing, and the column scan reads them all
__host__ __device__ inline int guard_partials(const SysDev& d)
{
    const int n = d.max_groups * (kGroup / 4);
    return n > kKeBlocks ? kKeBlocks : n;
}

// Smooth particle-mesh Ewald of one system: a K0 x K1 x K2 grid along the
// lattice vectors a, b, c, cardinal B-splines of order `order`.
struct PmeDev {
    int n_atoms;
    int K[3];
    int H2;                // K2/2 + 1 half-complex points along c
    int order;
    int solve_blocks;      // blocks of the solve (rows of energy partials)
    double rec[6];         // a* = (rec0, rec1, rec2), b* = (0, rec3, rec4), c* = (0, 0, rec5)
    double fel;            // 1/(4 pi eps0 eps_r)
    double beta, vol;
    double pi2_b2;         // pi^2 / beta^2
    const double* q;       // [N] charges (the system's device copy)
    int col_cap;           // atoms a column bucket holds (twice the mean occupancy + 16)
    int* col_count;        // [K0*K1] atoms per (base_a, base_b) grid column; all zero between evaluations
    double2* bkt_w;        // [K0*K1][col_cap][2] each column's bucket of atoms (any order within
                           // it): offsets {w_a, w_b}, {w_c, q}
    int* bkt_c;            // [K0*K1][col_cap] their base points along c
    int* ovf_count;        // [1] atoms past their column's bucket; zero between evaluations
    int* ovf_list;         // [N] those atoms (any order)
    int4* atom_base;       // [N] spline base points (a, b, c) and column
    double2* atom_w;       // [N][2] spline offsets {w_a, w_b}, {w_c, q}
    double* conv;          // [K0*K1*K2] potential grid (theta_rec * Q)
    double2* cgrid;        // [H2][K0][K1] transforms in place, one plane per h_c
    double* bmod;          // [K0+K1+K2] |b(m)|^2 of each dimension
    double* gtab;          // [H2][K0][K1] influence function G(m) on the half-complex grid
    double2* tw;           // [K0+K1+K2] (cos, sin)(2 pi j / K) of each dimension
    double* epart;         // [solve_blocks*8] energy and virial partials of the a pass
    double* qsum;          // [2] sum q, sum q^2
    double* eout;          // [8] E_recip + E_self + E_background, Xi xx,yy,zz,xy,xz,yz
    float* frec;           // [N,3] reciprocal-space forces
};

// A position moved into the primary cell by its integer lattice counts w
// (x - w_a a - w_b b - w_c c), FP64 without contraction, components in the
// order ((x - w_a a_x) - w_b b_x) - w_c c_x, (y - w_b b_y) - w_c c_y,
// z - w_c c_z (for a rectangular box: x - w L per dimension).
__device__ __forceinline__ void wrapped_pos(const SysDev& d, const double x[3], const int w[3], double u[3])
{
#pragma clang fp contract(off)
    u[0] = ((x[0] - (double)w[0] * d.box[0]) - (double)w[1] * d.box_off[0]) - (double)w[2] * d.box_off[1];
    u[1] = (x[1] - (double)w[1] * d.box[1]) - (double)w[2] * d.box_off[2];
    u[2] = x[2] - (double)w[2] * d.box[2];
}

// Group-local FP32 coordinates of a position: its wrapped position minus the
// group's reference point in FP64, rounded once.  Every kernel that stages
// positions uses it, so a slot's staged value does not depend on which kernel
// wrote it.
__device__ __forceinline__ void stage_pos(const SysDev& d, const double x[3], const int w[3], const double ref[3],
                                          float4& p)
{
#pragma clang fp contract(off)
    double u[3];
    wrapped_pos(d, x, w, u);
    p.x = (float)(u[0] - ref[0]);
    p.y = (float)(u[1] - ref[1]);
    p.z = (float)(u[2] - ref[2]);
}

// Staged position of a padding slot: out of reach of every atom and of every
// other padding slot (two slots differ by at least 1e9 nm in x or y), so the
// cut-off tests of the pair kernel and of the search drop its pairs by
// themselves and need no lane masks of real atoms (but the pair of a slot with
// its own image in an entry of a cluster with itself has to be masked).
__device__ __forceinline__ float4 pad_pos(int slot)
{
    return make_float4(1e9f * (float)(1 + (slot & 4095)), 1e9f * (float)(1 + (slot >> 12)), 0.0f, 0.0f);
}

// ---- launch entry points (implemented in the .hip files) ------------------
// All take a device array of `n_sys` descriptors and the per-launch grid bounds
// the host knows statically (max over members).
struct Bounds {
    int max_atoms;
    int max_cols;
    int max_groups;
    int max_slots;
    int total_slots;  // of all members
    int max_ent;    // largest entry capacity of the members
    bool any_tric;  // some member has a triclinic box
    bool all_m8;    // every member has 8-atom clusters
};

// the whole list build with its transpose, after the list-buffer guard (the
// largest displacement since the previous build, then x recorded for the next
// one).  The search prunes every candidate at the atom level in FP32 (the force
// kernel's frame).  exact: then the FP64 atom-pair prune (export-ready masks)
// decides the list; otherwise the FP32 result is the list (masks left undefined
// until launch_refine).  item_prefix: also the prefix over the systems of their
// work-item counts.  flags (per system, NULL = the one system): 0 = skip, 1 =
// rebuild, 2 = first build (x only recorded); without flags, first says which.
// cleared: the gather before it already cleared the counters and status words
// and took the list-buffer guard's partials (md_step's rebuilds).  seen (one
// system): a word in pinned host memory that receives {seq, work items | 1 << 31 if a
// capacity was exceeded} when that is known
hipError_t launch_build(const SysDev* table, int n_sys, const Bounds& b, const int* flags, hipStream_t s,
                        bool exact, int status_clear = 0, int* item_prefix = nullptr, bool first = false,
                        bool cleared = false, unsigned long long* seen = nullptr, unsigned int seq = 0);
// exact masks (cand_mask) and pair counts for a list built without them, from
// the stored build positions; the force list itself is not touched
hipError_t launch_refine(const SysDev* table, int n_sys, const Bounds& b, hipStream_t s);
hipError_t launch_ens_status(const SysDev* table, int n_sys, int* out, hipStream_t s);
// flags (per system, NULL = every system): 0 = skip that system; clear_status:
// also every status word, as launch_clear_status would before it
hipError_t launch_stage(const SysDev* table, int n_sys, const Bounds& b, hipStream_t s,
                        const int* flags = nullptr, bool clear_status = false);
// mode 0: x, v -> x_bak, v_bak of every system; mode 1: back again
hipError_t launch_state_copy(const SysDev* table, int n_sys, const Bounds& b, int mode, hipStream_t s);
// A block per item where a launch has about as many items as the GPU has SIMDs, or
// fewer: forces of 2,700 atoms 15.0 us a call against 17.2, of 6,000 with Ewald 18.1
// against 22, of 8,500 with reaction field (1,030 items) 18.8 against 21.6; of 10,000
// (1,210) 20.5 against 19.5, of 8,500 with Ewald (1,370) 23.4 against 23.1.
constexpr int kSplitItems = 1150, kSplitNever = 1 << 24;
// Items past which 4 waves per SIMD on 256 CUs, 4096, do not take all at once (a uniform
// liquid's are counted a few per cent too high): 26,000 atoms (4,190) 31.7 us a call
// with 4 waves and 32.2 with 5, 28,000 (4,510) 37.1 and 34.8, 30,000 38.7 and 35.5,
// 50,000 49.4 and 48.3, 80,000 66.6 and 63.5.
constexpr int kManyItems = 4400;
// which of the forms above a plain launch of that many items takes
inline int force_form(int few_items) { return few_items <= kSplitItems ? 0 : few_items > kManyItems ? 2 : 1; }
// prune: the force pass also prunes every entry's i-cluster mask to r_inner
// (from the build's mask), and later passes evaluate the pruned mask.
// max_blocks > 0 caps the persistent grid (its waves loop over the work items).
// red_row >= 0 (one system): without energies and pruning an extra block writes
// the previous energy pass's energy row as launch_energy_reduce(table, 1, red_row,
// true, red_step) would; with pruning, red_row = prune_guard_arg(...), extra blocks
// do what launch_prune_guard_k(table, n_atoms, 1, cur, fold) would
hipError_t launch_force(const SysDev* table, int n_sys, const int* item_prefix, int M, int coulomb,
                        int lj, bool ener, int max_blocks, int total_item_cap, hipStream_t s, bool prune = false,
                        int red_row = -1, double red_step = 0.0, int few_items = kSplitNever);
// few_items: about the items of the launch, split_items summed over its systems; up
// to kSplitItems of them are worked on by a block each.  built: the items of the last
// build that the host has heard of (0: none).  The estimate from the mean density
// stands where it is higher: it is what the lines above were measured with, and holds
// where no build has run; a droplet's items are many times as many (24,389 atoms in a
// box of 4 times their edge, Ewald: 6,490 items, 49.6 us a call and 63.9 by the estimate)
int split_items(int M, int jtile, double n_rho_r3, int built);
// dynamic-prune guard of one system: check = 1: the largest displacement since
// x_prune into partial buffer cur; then x_prune = x.  fold: first fold the
// previous interval's partials (buffer 1 - cur) into the statistics
int prune_guard_arg(int n_atoms, int cur, int fold);
hipError_t launch_prune_guard_k(const SysDev* table, int n_atoms, int check, int cur, int fold, hipStream_t s);
// the force gather; ener (one system): a block of it also forms the energy row as
// launch_energy_reduce(table, 1, trace_row, false, step_value) does
hipError_t launch_finalize(const SysDev* table, int n_sys, const Bounds& b, bool fp32, hipStream_t s,
                           const int* flags = nullptr, bool ener = false, int trace_row = -1,
                           double step_value = 0.0);
// words of the device to pinned host memory (visible once the stream is waited for)
hipError_t launch_page_out(const int* from, int* pinned, int words, hipStream_t s);
hipError_t launch_energy_reduce(const SysDev* table, int n_sys, int trace_row, bool with_ke,
                                double step_value, hipStream_t s);
hipError_t launch_kick_drift(const SysDev* table, int n_sys, const Bounds& b, double dt, hipStream_t s);
hipError_t launch_item_prefix(const SysDev* table, int n_sys, int* item_prefix, hipStream_t s,
                              const int* flags = nullptr);
// fused plain-step kernels: kick + drift + staging; gather + kick (+ kinetic energy)
hipError_t launch_kick_drift_stage(const SysDev* table, int n_sys, const Bounds& b, double dt, hipStream_t s);
// next: 0 = gather + half-kick; 1 = and the next step's half-kick + drift, and
// the list build's clears and buffer-guard partials (a rebuild follows);
// 2 = and also the staging of the new positions (no list rebuild due).
// open: the first positions of a run (no half-kick closes a step; next 1 or 2);
// held: nothing moves and no force is stored if the list ran out of capacity
hipError_t launch_gather_kick(const SysDev* table, int n_sys, const Bounds& b, double dt, bool ke, hipStream_t s,
                              int next = 0, bool open = false, bool held = false);
// relaxation of one system: the force gather with the largest |F|^2 per block
// (kKeBlocks partials at most), and the move with its staging (see the kernel)
hipError_t launch_gather_fmax(const SysDev* table, const Bounds& b, hipStream_t s);
hipError_t launch_minimize_move(const SysDev* table, const Bounds& b, double max_disp, double f_tol, int it, int* done,
                                unsigned long long* seen, hipStream_t s);
// PME: twiddles, spline moduli and charge sums (after the charges are on the
// device); then per evaluation the spread, transforms, solve and gather of the
// positions x (device FP64 [N,3]) into p.frec, and with ener the energy and
// virial into p.eout
int pme_solve_blocks(int K1, int H2);
hipError_t launch_pme_setup(const PmeDev& p, hipStream_t s);
hipError_t launch_pme(const PmeDev& p, const double* x, bool ener, hipStream_t s);
// keep_faults: leave the saturation / bad-position flags of earlier steps set
// (clears inside a multi-step call); otherwise every flag is cleared
hipError_t launch_clear_status(const SysDev* table, int n_sys, hipStream_t s, bool keep_faults = false);

// Per-system energy/virial (and kinetic energy) from the per-item partials, in
// a fixed order: FP64 (V64r) or FP32 (V32).  Xi = -1/2 sum r_ij (x) F_ij.
// One block of 256 threads per system: thread t sums items t, t + 256, ... (two
// 16-byte loads per item, all of a thread's loads issued before its sums), then
// each wave sums its lanes with a fixed shuffle tree and the four wave totals
// are added in wave order -- the same decomposition alone and in a batch.
// The wave's trees of the eight values are one: each exchange sends half of the
// values that a lane still holds and keeps the other half, so 10 exchanges do for 48.
template <class T>
__device__ __forceinline__ T wave_tree_sum(T v)
{
    for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o, 64);
    return v;
}

// v[0..7] summed over the wave; the total of value lane / 8 is returned
template <class T>
__device__ __forceinline__ T wave_tree_sum8(const T v[8])
{
    const int lane = threadIdx.x & 63;
    T a[4], b[2];
    const bool h32 = lane & 32, h16 = lane & 16, h8 = lane & 8;
#pragma unroll
    for (int j = 0; j < 4; ++j) a[j] = (h32 ? v[4 + j] : v[j]) + __shfl_xor(h32 ? v[j] : v[4 + j], 32, 64);
#pragma unroll
    for (int j = 0; j < 2; ++j) b[j] = (h16 ? a[2 + j] : a[j]) + __shfl_xor(h16 ? a[j] : a[2 + j], 16, 64);
    T c = (h8 ? b[1] : b[0]) + __shfl_xor(h8 ? b[0] : b[1], 8, 64);
    for (int o = 4; o > 0; o >>= 1) c += __shfl_xor(c, o, 64);
    return c;
}

template <class T>
__device__ inline void energy_reduce_block(const SysDev& d, int n, int with_ke, T out[kEnerPart + 1])
{
    static_assert(kEnerPart == 8, "values per item");
    __shared__ T sh[4][kEnerPart + 1];
    T acc[kEnerPart], ke = T(0);
    for (int k = 0; k < kEnerPart; ++k) acc[k] = T(0);
    const nb_v4f* ep = (const nb_v4f*)d.epart;
    constexpr int kU = 4;
    for (int i0 = threadIdx.x; i0 < n; i0 += 256 * kU) {
        nb_v4f lo[kU], hi[kU];
#pragma unroll
        for (int u = 0; u < kU; ++u) {
            const int i = min(i0 + 256 * u, n - 1);  // (rows past the end are loaded, dropped)
            lo[u] = *(const NB_GLOBAL nb_v4f*)&ep[2 * i];
            hi[u] = *(const NB_GLOBAL nb_v4f*)&ep[2 * i + 1];
        }
#pragma unroll
        for (int u = 0; u < kU; ++u) {
            if (i0 + 256 * u >= n) break;
            acc[0] += T(lo[u].x); acc[1] += T(lo[u].y); acc[2] += T(lo[u].z); acc[3] += T(lo[u].w);
            acc[4] += T(hi[u].x); acc[5] += T(hi[u].y); acc[6] += T(hi[u].z); acc[7] += T(hi[u].w);
        }
    }
    const int wid = threadIdx.x >> 6, lane = threadIdx.x & 63;
    if (with_ke) {
        const int np = min(kKeBlocks, (d.max_groups * kGroup + 3) / 4);  // (a partial per 4 clusters at most)
        for (int i = threadIdx.x; i < np; i += 256) ke += T(gld(&d.ke_part[i]));
        ke = wave_tree_sum(ke);
    }
    const T w = wave_tree_sum8(acc);
    if ((lane & 7) == 0) sh[wid][lane >> 3] = w;
    if (lane == 0) sh[wid][kEnerPart] = ke;
    __syncthreads();
    for (int k = 0; k <= kEnerPart; ++k) out[k] = (sh[0][k] + sh[1][k]) + (sh[2][k] + sh[3][k]);
}

// The energy row of one system, by one block of 256 threads: the reduction
// above, then eout (E_lj, E_coul, the virial -1/2 sum r (x) F, the
// reciprocal-space terms when PME is on, E_kin) and, for trace_row >= 0, the
// trace ring row {step, E_lj, E_coul, E_kin, E_tot}.  Run by its own kernel, by an
// extra block of the next step's pair kernel or by one of the force gather (the
// same arithmetic).
__device__ inline void energy_reduce_system(const SysDev& d, int trace_row, int with_ke, double step_value)
{
    const int n = d.n_items[0];
    double out[kEnerPart + 1];
    if (d.fp32_reduce) {
        float o[kEnerPart + 1];
        energy_reduce_block<float>(d, n, with_ke, o);
        for (int k = 0; k <= kEnerPart; ++k) out[k] = o[k];
    } else {
        energy_reduce_block<double>(d, n, with_ke, out);
    }
    if (threadIdx.x == 0) {
        d.eout[0] = out[0];
        d.eout[1] = out[1];
        for (int k = 2; k < kEnerPart; ++k) d.eout[k] = -0.5 * out[k];
        if (d.pme_e) {
            // reciprocal space, self and background terms of the Ewald sum
            d.eout[1] += d.pme_e[0];
            for (int k = 2; k < kEnerPart; ++k) d.eout[k] += d.pme_e[k - 1];
            out[1] = d.eout[1];
        }
        if (with_ke) d.eout[8] = out[kEnerPart];
        if (trace_row >= 0) {
            double* t = d.trace + (size_t)(trace_row % kTraceCap) * 5;
            t[0] = step_value;
            t[1] = out[0];
            t[2] = out[1];
            t[3] = with_ke ? out[kEnerPart] : 0.0;
            t[4] = out[0] + out[1] + t[3];
        }
    }
}

// max over n >= 0 per-block partials (NaN wins), by all threads of a 256-thread
// block; every thread gets the result
__device__ inline double block_max_partials(const double* p, int n, double* sh)
{
    double m = 0.0;
    for (int k = threadIdx.x; k < n; k += 256) {
        const double u = p[k];
        m = (u > m || u != u) ? u : m;
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
    const double r = sh[0];
    __syncthreads();
    return r;
}

// Dynamic-prune guard of one system, run at the end of every prune
// interval (check = 1) and when a list is built afresh (check = 0): per block
// the largest squared displacement since x_prune (the positions at the last
// prune) into partial buffer `cur`, then x_prune = x.  Block 0 first folds the
// previous interval's partials (buffer 1 - cur, complete since that launch
// ended) into the interval statistics: the largest displacement, and the
// intervals in which it reached (r_inner - r_cut)/2 -- the only way a cluster
// pair pruned at the interval's start could have had a pair inside r_cut.
// Block blockIdx.x of nb, 256 threads; sh: 256 doubles of LDS.  At the end of an
// interval it runs in front of the pair work of the pass that prunes (a launch of
// its own before that pass took 4.6 us at 17,576 atoms).
__device__ inline void prune_guard_block(const SysDev& d, int nb, int check, int cur, int fold, double* sh)
{
    if (fold && blockIdx.x == 0) {
        const double m2 = block_max_partials(d.pg_part + (1 - cur) * kKeBlocks, nb, sh);
        if (threadIdx.x == 0) {
            const double mm = sqrt(m2);
            double* st = d.pg_part + 2 * kKeBlocks;
            if (mm > st[0] || mm != mm) st[0] = mm;
            if (!(mm < d.prune_half)) st[1] += 1.0;
        }
    }
    double m = 0.0;
    for (int a = blockIdx.x * blockDim.x + threadIdx.x; a < d.n_atoms; a += nb * blockDim.x) {
        double s2 = 0.0;
        for (int k = 0; k < 3; ++k) {
            const double x = gld(&d.x[3 * a + k]);
            if (check) {
                const double dd = x - gld(&d.x_prune[3 * a + k]);
                s2 += dd * dd;
            }
            gst(&d.x_prune[3 * a + k], x);
        }
        m = (s2 > m || s2 != s2) ? s2 : m;  // NaN wins
    }
    if (!check) return;
    sh[threadIdx.x] = m;
    __syncthreads();
    for (int o = 128; o > 0; o >>= 1) {
        if ((int)threadIdx.x < o) {
            const double u = sh[threadIdx.x + o];
            if (u > sh[threadIdx.x] || u != u) sh[threadIdx.x] = u;
        }
        __syncthreads();
    }
    if (threadIdx.x == 0) d.pg_part[cur * kKeBlocks + blockIdx.x] = sh[0];
}

}  // namespace nbi
