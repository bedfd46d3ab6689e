// nb_force.hip -- the cluster-pair non-bonded kernel (gfx950, wave64).
//
// The paper's kernel (Section "SIMD parallelism") keeps the atoms of an
// i-cluster in registers and, for each listed j-cluster, evaluates all M x N
// atom pairs without reloading particle data; its GPU variant groups 8
// clusters so each loaded j-cluster serves several i-clusters.  Newton's third
// law is used: every listed pair is evaluated once and the j-atoms receive the
// opposite force.
//
// MI355X mapping.  One wave64 processes one work item = (i-group of 8
// clusters, a run of `jtile` list entries).  Lane l handles pair (a, b) =
// ((l / M) % M, l % M) of entry (l / M^2), so for M = 8 a wave evaluates one
// full 8 x 8 cluster pair per instruction, for M = 4 four entries at once and
// for M = 1 (plain Verlet list) 64 entries at once.  The 8 i-clusters of the
// group sit in registers (lane holds i-atom a of each), their forces
// accumulate in registers over the whole item; each entry's j-forces are
// summed over the a-lanes with cross-lane shuffles once per entry (amortised
// over up to 8 i-clusters).  The kernel issues no atomics: each entry stores
// its j-atom forces and each item its i-atom forces as partials, and the
// gather kernel sums an atom's partials (int64 fixed point, so the result is
// independent of order and bitwise reproducible; FP32 in the V32 variant).
// Device-scope atomics from many waves to the same atom serialise at the
// memory side on this GPU, which is why they are avoided.  Pair arithmetic is
// FP32 on group-local coordinates; Ewald's force factor q(r) and, for
// energies, erfc(beta r) come from cubic tables in LDS (the same force table
// in every pass).
#include "nb_internal.h"

#include <algorithm>


namespace nbi {

namespace {


// keep a wave-uniform constant in an SGPR for the whole item (no re-loads inside
// the unrolled i-cluster loop)
__device__ __forceinline__ float pin(float v)
{
    asm volatile("" : "+s"(v));
    return v;
}

// the same for a wave-uniform base pointer
template <class T>
__device__ __forceinline__ T* pinp(T* p)
{
    asm volatile("" : "+s"(p));
    return p;
}

// lane ^ D exchange: DPP for 1, 2, 8; ds_swizzle for 4, 16; ds_bpermute for 32
template <int D>
__device__ __forceinline__ float xshfl(float v)
{
    const int i = __float_as_int(v);
    int r;
    // (bound_ctrl set, so that a following add takes the move as its operand)
    if (D == 1) r = __builtin_amdgcn_update_dpp(0, i, 0xB1, 0xF, 0xF, true);        // quad_perm [1,0,3,2]
    else if (D == 2) r = __builtin_amdgcn_update_dpp(0, i, 0x4E, 0xF, 0xF, true);   // quad_perm [2,3,0,1]
    else if (D == 8) r = __builtin_amdgcn_update_dpp(0, i, 0x128, 0xF, 0xF, true);  // row_ror:8
    else if (D == 4) r = __builtin_amdgcn_ds_swizzle(i, 0x101F);               // xor 4 in 32 lanes
    else if (D == 16) r = __builtin_amdgcn_ds_swizzle(i, 0x401F);              // xor 16 in 32 lanes
    else r = __shfl_xor(i, D, 64);
    return __int_as_float(r);
}

// Sum (x, y, z) over the 2^L lanes lane ^ (S * m), m < 2^L, splitting the
// components across lanes so the butterfly moves one value per step instead of
// three: L = 2 takes 3 exchanges (not 6).  Returns the total of component `comp`
// (0 x, 1 y, 2 z) held by this lane; `own` marks one lane per component.
template <int S, int L>
__device__ __forceinline__ float reduce3(float x, float y, float z, int idx, int& comp, bool& own)
{
    if (L == 2) {
        const bool lo = idx < 2;
        const float r1 = xshfl<2 * S>(lo ? z : x);
        const float r2 = xshfl<2 * S>(y);
        if (lo) {
            x += r1;
            y += r2;
        } else {
            z += r1;
        }
        const float snd = idx == 0 ? y : (idx == 1 ? x : z);
        float v = idx == 0 ? x : (idx == 1 ? y : z);
        v += xshfl<S>(snd);
        comp = idx == 0 ? 0 : (idx == 1 ? 1 : 2);
        own = idx <= 2;
        return v;
    } else {
        comp = -1;  // no reduction: the lane holds all three
        own = true;
        return 0.0f;
    }
}

__device__ __forceinline__ float wave_sum(float v)
{
    v += xshfl<1>(v);
    v += xshfl<2>(v);
    v += xshfl<4>(v);
    v += xshfl<8>(v);
    v += xshfl<16>(v);
    v += xshfl<32>(v);
    return v;
}

constexpr int kGuardLds = 256 * sizeof(double) / sizeof(float4);  // a prune guard block's LDS

constexpr int ilog2(int v) { return v <= 1 ? 0 : 1 + ilog2(v / 2); }

// Sum (x, y, z) over the 8 lanes lane ^ (8 m) (the a-lanes of an 8 x 8 cluster
// pair): the tree x[a] + x[a ^ 4], then a ^ 2, then a ^ 1, with the half and row
// exchanges done by VALU lane swaps that reduce two registers each.  The total of component 0 ends in lanes 0-15 (b = lane mod 8, twice), 2
// in 16-31 and 48-63, 1 in 32-47.
__device__ __forceinline__ float reduce8(float x, float y, float z)
{
    typedef unsigned int u2 __attribute__((ext_vector_type(2)));
    u2 p = __builtin_amdgcn_permlane32_swap(__float_as_uint(x), __float_as_uint(y), false, false);
    const float xy = __uint_as_float(p.x) + __uint_as_float(p.y);  // x in lanes 0-31, y in 32-63
    p = __builtin_amdgcn_permlane32_swap(__float_as_uint(z), __float_as_uint(z), false, false);
    const float zz = __uint_as_float(p.x) + __uint_as_float(p.y);
    p = __builtin_amdgcn_permlane16_swap(__float_as_uint(xy), __float_as_uint(zz), false, false);
    const float v = __uint_as_float(p.x) + __uint_as_float(p.y);  // rows x, z, y, z
    return v + xshfl<8>(v);
}

// Sum over the 8 lanes of equal lane / 8 (the b-lanes), valid in lanes with
// b < 4: the tree b ^ 4, b ^ 2, b ^ 1 by DPP row moves
__device__ __forceinline__ float sum_b(float v)
{
    v += __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), 0x104, 0xF, 0xF, true));  // row_shl:4
    v += xshfl<2>(v);
    return v + xshfl<1>(v);
}

// a + b rounded by itself (never fused with the product that made b)
__device__ __forceinline__ float add_rn(float a, float b)
{
#pragma clang fp contract(off)
    return a + b;
}

__device__ __forceinline__ int lane_read(int v, int k) { return __builtin_amdgcn_readlane(v, k); }
__device__ __forceinline__ float lane_read(float v, int k)
{
    return __int_as_float(__builtin_amdgcn_readlane(__float_as_int(v), k));
}

// What a force sum over x starts from: +0, or NaN for a coordinate that is not
// finite.  No pair of such an atom is within r_cut, so nothing else would carry it to
// the gather, which reports it.  (An FMA in the place of the move.)
__device__ __forceinline__ float zero_of(float x) { return __builtin_fmaf(0.0f, x, 0.0f); }

// What the pair arithmetic leaves for the energies
struct Pair {
    float rinv, rinv6, c6, c12, w;  // (c6, c12 with LJ == 1; w, kt with COUL == 2)
    int kt;
};

// The force on i over the vector from j, of a pair inside r_cut.  qq: charge product;
// li, lj: LJ parameters (LJ == 1); c6x6, c12x12: 6 C6 and 12 C12 (LJ == 0).  Ewald's
// q(r) from the cubic table: F_coul = qq q(r) r_ij / r^3
template <int COUL, int LJ>
__device__ __forceinline__ float pair_factor(float r2, float qq, float2 li, float2 lj, float c6x6, float c12x12,
                                             float krf2, const float4* tab, float ew_tinv, Pair& p)
{
    const float rinv = __builtin_amdgcn_rsqf(r2);
    const float rinv2 = rinv * rinv;
    const float rinv6 = rinv2 * rinv2 * rinv2;
    p.rinv = rinv;
    p.rinv6 = rinv6;
    float fl;
    if (LJ == 1) {
        const float sg = li.x + lj.x;
        const float ep = li.y * lj.y;
        const float s2 = sg * sg;
        const float s6 = s2 * s2 * s2;
        p.c6 = ep * s6;
        p.c12 = p.c6 * s6;
        fl = (12.0f * p.c12 * rinv6 - 6.0f * p.c6) * rinv6;
    } else {
        fl = fmaf(c12x12, rinv6, -c6x6) * rinv6;
    }
    if (COUL == 2) {
        const float rs = r2 * rinv * ew_tinv;
        p.kt = (int)rs;  // <= kEwTab: the tables have one interval past r_cut
        p.w = __builtin_amdgcn_fractf(rs);
        const float4 cf = tab[p.kt];
        const float qv = fmaf(fmaf(fmaf(cf.w, p.w, cf.z), p.w, cf.y), p.w, cf.x);
        return fmaf(qq * qv, rinv, fl) * rinv2;
    }
    const float fs = fl * rinv2;
    return COUL == 1 ? fmaf(qq, fmaf(rinv, rinv2, -krf2), fs) : fs;
}

// The system of work item it: the last one whose first item (first) is not past it.
// pre: the first items of up to 64 systems, one per lane; of more systems 64 are left
// by halving (halved down to one, the interval took a scalar round trip per step)
__device__ __forceinline__ int item_system(const int* item_prefix, int n_sys, int it, int pre, int lane, int& first)
{
    first = 0;
    if (n_sys == 1) return 0;
    int lo = 0, hi = n_sys - 1, p = pre;
    if (hi >= 64) {
        while (hi - lo >= 64) {
            const int mid = (lo + hi + 1) >> 1;
            if (item_prefix[mid] <= it) lo = mid; else hi = mid - 1;
        }
        p = gld(&item_prefix[min(lo + lane, hi)]);
    }
    const int u = __popcll(__builtin_amdgcn_ballot_w64(lane <= hi - lo && p <= it)) - 1;
    first = lane_read(p, u);
    return lo + u;
}

}  // namespace

// 8-atom clusters: one wave per work item, one 8 x 8 cluster pair per
// instruction.
//
// The kernel is bound by instruction issue: per entry about 30 VALU
// instructions per evaluated cluster pair plus a fixed part, which this form
// keeps small:
//  - the list words of (up to) 64 entries sit one per lane and are read with
//    v_readlane, so the entry's j-cluster, masks, shift and row are scalars:
//    its addresses are scalar arithmetic and no list load waits in the loop;
//  - padding slots lie out of reach of everything (pad_pos), so a cluster
//    pair's lanes are those with r < r_cut, taken as the execution mask: no
//    masks of real atoms, no selects, and only those lanes read the Ewald
//    table.  Only an entry of a cluster with itself masks lanes (SELF);
//  - the j-forces are summed over the a-lanes by VALU lane swaps (8
//    instructions, no LDS), the i-forces by DPP adds, and every lane stores the
//    component that it holds (lanes with the same one store the same value).
// The form before it (entry words and masks in vector registers, a butterfly
// through the LDS unit, selects) issued 82.2 M VALU, 32.0 M SALU and 3.6 M LDS
// instructions on 200,003 atoms with Ewald where this one issues 69.9, 28.2 and
// 1.7 M; with the descriptor read in one batch (below) it takes 123 us there
// against 147, 23.7 against 25.8 us at 24,389 atoms, and 12.7 against 14.6 us at
// 2,700 atoms with reaction field.  The sums, their order and so the forces are
// the same.
//
// WAVES: waves per SIMD that the registers leave room for (1: as it comes).  The
// plain Ewald pass takes 99 registers, 4 waves, and 96 for 5: better for a launch of
// more items than 4 waves per SIMD take at once (200,003 atoms 118.0 us against
// 126.4), not for one that they take (24,389 atoms, 3,890 items, 24.6 against 24.1).
// The Ewald tables are loaded in a branch of their own with the item, so that their
// registers (up to 40) are free again before the i-atoms need them: kept over two
// branches they counted against the whole kernel (120 registers for the plain pass),
// and row by row they cost a round trip each (energies of 3,001 atoms 23.7 us, now 21.4).
template <int COUL, int LJ, bool ENER, bool PRUNE, int WAVES = 1>
__global__ __launch_bounds__(256, WAVES) void k_force8(const SysDev* __restrict__ table, int n_sys,
                                                const int* __restrict__ item_prefix, int red_row, double red_step)
{
    constexpr int M = 8;
    constexpr int G = kGroup;
    // the kernel arguments in one scalar round trip, then the item count
    // together with the first system's descriptor lines (read again, from the
    // scalar cache, where the item's values are taken)
    int grid = (int)gridDim.x;
    asm volatile("" : "+s"(n_sys), "+s"(red_row), "+s"(grid));
    const int total = item_prefix[n_sys];
    {
        const int w0 = ((const int*)table)[0], w1 = ((const int*)table)[16], w2 = ((const int*)table)[32];
        asm volatile("" ::"s"(w0), "s"(w1), "s"(w2), "s"(total));
    }
    const int lane = threadIdx.x & 63;
    const int a = lane >> 3, b = lane & 7;
    const int wid = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    // the lanes of a cluster with itself: at zero shift each pair once (a < b),
    // with one of its images all but a slot and its own image
    const unsigned long long once = __builtin_amdgcn_ballot_w64(a < b), offd = __builtin_amdgcn_ballot_w64(a != b);

    constexpr bool TAB = (COUL == 2);
    constexpr bool ETAB = TAB && ENER;
    constexpr int kTabU = (kEwTabN + 63) / 64;
    __shared__ float4 tab_lds[TAB ? 4 * kTabU * 64 : PRUNE ? kGuardLds : 1];
    __shared__ float4 etab_lds[ETAB ? 4 * kTabU * 64 : 1];
    double* guard_lds = (double*)tab_lds;

    // XCD-aware order, as in k_force
    int pair0 = 0;  // the first pair block
    if constexpr (!ENER && !PRUNE) {
        if (red_row >= 0) {
            if (blockIdx.x < 8) {
                if (blockIdx.x == 0) energy_reduce_system(table[0], red_row, 1, red_step);
                return;
            }
            pair0 = 8;
        }
    }
    if constexpr (PRUNE) {
        if (red_row >= 0) {
            // the prune guard's blocks: red_row = buffer | fold << 1 | blocks << 2
            const int nb = red_row >> 2;
            if ((int)blockIdx.x < nb) prune_guard_block(table[0], nb, 1, red_row & 1, red_row & 2, guard_lds);
            pair0 = (nb + 7) / 8 * 8;
            if ((int)blockIdx.x < pair0) return;
        }
    }
    const int bx = (int)blockIdx.x - pair0;
    const int xcd = bx % 8;
    const int bj = bx / 8;
    const int per_xcd = (grid - pair0) / 8;
    const int chunk = (total + 7) / 8;
    const int it_end = min(total, (xcd + 1) * chunk);
    const int nwave = per_xcd * 4;
    float4* tab = tab_lds + (TAB ? wid * kTabU * 64 : 0);
    float4* etab = etab_lds + (ETAB ? wid * kTabU * 64 : 0);
    int tab_sys = -1;
    // byte offsets of this lane's store in a row of j-partials (its component
    // after reduce8) and in an i-cluster's partials (component b, lanes b < 3)
    const int row16 = lane >> 4;
    unsigned int joff = (unsigned int)(b * 3 + (row16 == 0 ? 0 : row16 == 2 ? 1 : 2)) * 4u;
    unsigned int aoff = a * sizeof(float4);
    unsigned int boff = b * sizeof(float4);
    const unsigned int ioff = (unsigned int)(a * 3 + b) * 4u;

    // (launches of up to 64 systems) their first items, one per lane
    const int pre = n_sys > 1 ? gld(&item_prefix[min(lane, n_sys - 1)]) : 0;
    for (int it = xcd * chunk + bj * 4 + wid; it < it_end; it += nwave) {
        int first;
        const int s = item_system(item_prefix, n_sys, it, pre, lane, first);
        const SysDev& d = table[s];
        // Everything the item needs from the descriptor, loaded together (one
        // scalar round trip) and kept in SGPRs: only what this variant uses (a
        // pinned value is never dropped by the compiler).  Pinned one by one,
        // each load waited for the one before it, ten round trips per item.
        constexpr bool LJ1 = LJ == 0;  // one LJ type
        const int4* items = d.items;
        const float4* xq = d.xq;
        const int2* ent = d.ent;
        const float4* entS = d.ent_S;
        char* jpart = (char*)d.jpart;
        float* ipart = d.ipart;
        float rc2 = d.rc2;
        const float4* ewt = TAB ? d.ew_tab : nullptr;
        const float4* ewe = ETAB ? d.ew_etab : nullptr;
        const float2* ljs = LJ == 1 ? d.ljs : nullptr;
        float c6x6 = LJ1 ? d.c6x6 : 0.f, c12x12 = LJ1 ? d.c12x12 : 0.f;
        float c6 = (LJ1 && ENER) ? d.c6 : 0.f, c12 = (LJ1 && ENER) ? d.c12 : 0.f;
        float krf2 = COUL == 1 ? d.krf2 : 0.f;
        float krf = (COUL == 1 && ENER) ? d.krf : 0.f, crf = (COUL == 1 && ENER) ? d.crf : 0.f;
        float ew_tinv = TAB ? d.ew_tinv : 0.f, ew_shift = ETAB ? d.ew_shift : 0.f;
        float rin2 = PRUNE ? d.rin2 : 0.f;
        int pot_shift = ENER ? d.pot_shift : 0;
        float lj_shift = (ENER && LJ1) ? d.lj_shift : 0.f;
        float irc6 = (ENER && !LJ1) ? d.irc6 : 0.f, irc12 = (ENER && !LJ1) ? d.irc12 : 0.f;
        float* epart = ENER ? d.epart : nullptr;
        asm volatile("" : "+s"(items), "+s"(xq), "+s"(ent), "+s"(entS), "+s"(jpart), "+s"(ipart), "+s"(rc2),
                     "+s"(ewt), "+s"(ljs), "+s"(c6x6), "+s"(c12x12), "+s"(krf2), "+s"(ew_tinv), "+s"(rin2));
        if (ENER)
            asm volatile("" : "+s"(ewe), "+s"(c6), "+s"(c12), "+s"(krf), "+s"(crf), "+s"(ew_shift), "+s"(pot_shift),
                         "+s"(lj_shift), "+s"(irc6), "+s"(irc12), "+s"(epart));
        // the tables (when the wave needs new ones) and the item in one memory round
        // trip, all rows in flight before the i-atoms need the registers
        const int li = it - first;
        int4 item;
        if (!TAB || s == tab_sys) {
            item = gld(&items[li]);
        } else {
            float4 tv[kTabU], te[ETAB ? kTabU : 1];
#pragma unroll
            for (int u = 0; u < kTabU; ++u) {
                tv[u] = gld(&ewt[min(lane + 64 * u, kEwTabN - 1)]);
                if (ETAB) te[u] = gld(&ewe[min(lane + 64 * u, kEwTabN - 1)]);
            }
            item = gld(&items[li]);
#pragma unroll
            for (int u = 0; u < kTabU; ++u) {
                tab[lane + 64 * u] = tv[u];
                if (ETAB) etab[lane + 64 * u] = te[u];
            }
            // LDS accesses of one wave complete in order; the fence keeps the
            // compiler from moving the table reads above these writes
            __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
            __builtin_amdgcn_wave_barrier();
            __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
            tab_sys = s;
        }
        const int gi = __builtin_amdgcn_readfirstlane(item.x), e0 = __builtin_amdgcn_readfirstlane(item.y),
                  e1 = __builtin_amdgcn_readfirstlane(item.z);
        int cj_n = __builtin_amdgcn_readfirstlane(item.w);

        // 6 C6 in a vector register: the LJ FMA takes one scalar operand only
        float c6v = 0.f;
        if (LJ1) asm volatile("v_mov_b32 %0, %1" : "=v"(c6v) : "s"(c6x6));

        // (kept as 32-bit offsets here, so that the loads take a scalar base)
        asm volatile("" : "+v"(aoff), "+v"(boff));
        float4 xi[G];
        float2 lji[G];
#pragma unroll
        for (int g = 0; g < G; ++g) {
            xi[g] = gld4(xq + (size_t)gi * (G * M), aoff + g * M * sizeof(float4));
            if (LJ == 1) lji[g] = gld2(ljs + (size_t)gi * (G * M), aoff / 2 + g * M * sizeof(float2));
        }
        float fix[G], fiy[G], fiz[G];
#pragma unroll
        for (int g = 0; g < G; ++g) {
            fix[g] = zero_of(xi[g].x);
            fiy[g] = zero_of(xi[g].y);
            fiz[g] = zero_of(xi[g].z);
        }
        float elj = 0.f, ec = 0.f, wxx = 0.f, wyy = 0.f, wzz = 0.f, wxy = 0.f, wxz = 0.f, wyz = 0.f;

        // the previous entry's j-partial, stored one entry late: after the wait
        // for the prefetched j-atoms and before the next prefetch
        char* pend_p = nullptr;
        float pend_v = 0.0f;
        // the list words of entries [c0, c0 + 64), one per lane, and the j-atoms
        // of the next entry
        int2 enl = gld(&ent[min(e0 + lane, e1 - 1)]);
        float4 Sl = gld(&entS[min(e0 + lane, e1 - 1)]);
        float4 xj_n = gld4(xq + (size_t)cj_n * M, boff);
        float2 ljj_n = make_float2(0.f, 0.f);
        if (LJ == 1) ljj_n = gld2(ljs + (size_t)cj_n * M, boff / 2);
        for (int c0 = e0; c0 < e1; c0 += 64) {
          if (c0 > e0) {
              // (items of more than 64 entries: the next 64 list words)
              enl = gld(&ent[min(c0 + lane, e1 - 1)]);
              Sl = gld(&entS[min(c0 + lane, e1 - 1)]);
          }
          // the entries to evaluate: those that a dynamic prune left i-clusters
          // (all until then, and in a pass that prunes).  An entry without any
          // had no pair inside r_inner >= r_cut in the pass that pruned it, which
          // left zeros in its row.
          unsigned long long todo =
              __builtin_amdgcn_ballot_w64(lane < e1 - c0 && (PRUNE || ((enl.y >> kMetaInner) & 255) != 0));
          int k = (int)__builtin_ctzll(todo | 1ull << 63);
          if (c0 > e0 || k > 0) {
              // (the first j-atoms loaded are those of the item's first entry)
              cj_n = lane_read(enl.x, k);
              xj_n = gld4(xq + (size_t)cj_n * M, boff);
              if (LJ == 1) ljj_n = gld2(ljs + (size_t)cj_n * M, boff / 2);
          }
          while (todo) {
            // (kept as 32-bit offsets here, so that the accesses below take a
            // scalar base)
            asm volatile("" : "+v"(boff), "+v"(joff));
            const int cj = cj_n;
            const unsigned int meta = (unsigned int)lane_read(enl.y, k);
            const int jrow = lane_read(__float_as_int(Sl.w), k);
            const int e = c0 + k;
            float4 xj = xj_n;
            const float2 ljj = ljj_n;
            xj.x += lane_read(Sl.x, k);
            xj.y += lane_read(Sl.y, k);
            xj.z += lane_read(Sl.z, k);
            __builtin_amdgcn_sched_barrier(0);
            if (pend_p) gst1(pend_p, joff, pend_v);
            // the next entry's j-atoms (after the last of the 64 those of lane
            // 63's entry, unused), always issued
            todo &= todo - 1ull;
            k = (int)__builtin_ctzll(todo | 1ull << 63);
            cj_n = lane_read(enl.x, k);
            xj_n = gld4(xq + (size_t)cj_n * M, boff);
            if (LJ == 1) ljj_n = gld2(ljs + (size_t)cj_n * M, boff / 2);
            const unsigned int im = (meta >> (PRUNE ? kMetaOuter : kMetaInner)) & 255u;
            unsigned int pin_m = 0u;  // (pruning) i-clusters with a pair within r_inner
            float fjx = zero_of(xj.x), fjy = zero_of(xj.y), fjz = zero_of(xj.z);
            // the i-cluster that is the entry's j-cluster (none if not in 0..7)
            const int gs = cj - gi * G;
            const unsigned long long selfm = (meta & 255u) == (unsigned int)kShiftZero ? once : offd;
#pragma unroll
            for (int g = 0; g < G; ++g) {
                if (!((im >> g) & 1u)) continue;
                const float dx = xi[g].x - xj.x;
                const float dy = xi[g].y - xj.y;
                const float dz = xi[g].z - xj.z;
                const float r2 = dx * dx + dy * dy + dz * dz;
                const unsigned long long onm = g == gs ? selfm : ~0ull;
                if (PRUNE)
                    if (__builtin_amdgcn_ballot_w64(r2 < rin2) & onm) pin_m |= 1u << g;
                if (__builtin_amdgcn_inverse_ballot_w64(__builtin_amdgcn_ballot_w64(r2 < rc2) & onm)) {
                    Pair p;
                    const float qq = xi[g].w * xj.w;
                    const float fs = pair_factor<COUL, LJ>(r2, qq, LJ == 1 ? lji[g] : make_float2(0.f, 0.f), ljj, c6v,
                                                           c12x12, krf2, tab, ew_tinv, p);
                    float vc = 0.f;
                    if (ENER) {
                        if (LJ == 0) {
                            p.c6 = c6;
                            p.c12 = c12;
                        }
                        if (COUL == 1) vc = qq * (p.rinv + krf * r2 - crf);
                        if (COUL == 2) {
                            // erfc(beta r) from the second table
                            const float4 ce = etab[p.kt];
                            const float ev = fmaf(fmaf(fmaf(ce.w, p.w, ce.z), p.w, ce.y), p.w, ce.x);
                            vc = qq * fmaf(ev, p.rinv, -ew_shift);
                        }
                    }
                    const float tx = fs * dx, ty = fs * dy, tz = fs * dz;
                    fix[g] += tx;
                    fiy[g] += ty;
                    fiz[g] += tz;
                    fjx -= tx;
                    fjy -= ty;
                    fjz -= tz;
                    if (ENER) {
                        float vl = (p.c12 * p.rinv6 - p.c6) * p.rinv6;
                        if (pot_shift) vl = add_rn(vl, LJ == 1 ? -fmaf(p.c12, irc12, -(p.c6 * irc6)) : -lj_shift);
                        elj = add_rn(elj, vl);
                        ec = add_rn(ec, vc);
                        wxx += tx * dx;
                        wyy += ty * dy;
                        wzz += tz * dz;
                        wxy += tx * dy;
                        wxz += tx * dz;
                        wyz += ty * dz;
                    }
                }
        }
            // this entry's j-partial (summed per atom by the gather; an entry
            // without any pair inside r_cut gives zeros)
            pend_v = reduce8(fjx, fjy, fjz);
            pend_p = jpart + (size_t)jrow * (M * 3 * sizeof(float));
            if (PRUNE && lane == 0)
                gst((int*)&ent[e] + 1, (int)((meta & ~(255u << kMetaInner)) | (pin_m << kMetaInner)));
          }
        }
        if (pend_p) gst1(pend_p, joff, pend_v);  // the item's last entry
        // i-forces: sum over b, stored as this item's partial
        char* ip = (char*)(ipart + (size_t)li * (G * M * 3));
        float v[G];
#pragma unroll
        for (int g = 0; g < G; ++g) {
            const float x = sum_b(fix[g]), y = sum_b(fiy[g]), z = sum_b(fiz[g]);
            v[g] = b == 0 ? x : b == 1 ? y : z;
        }
        if (b < 3) {
#pragma unroll
            for (int g = 0; g < G; ++g) gst1(ip, ioff + g * M * 3 * sizeof(float), v[g]);
        }
        if (ENER) {
            const float v0 = wave_sum(elj), v1 = wave_sum(ec), v2 = wave_sum(wxx), v3 = wave_sum(wyy),
                        v4 = wave_sum(wzz), v5 = wave_sum(wxy), v6 = wave_sum(wxz), v7 = wave_sum(wyz);
            if (lane == 0) {
                float* o = epart + (size_t)li * kEnerPart;
                o[0] = v0; o[1] = v1; o[2] = v2; o[3] = v3;
                o[4] = v4; o[5] = v5; o[6] = v6; o[7] = v7;
            }
        }
    }
}

// The same work with a block of 4 waves per item, for launches of few items
// (split_items): there a wave has a SIMD to itself and the launch lasts as long as one
// item, of which the entries' instructions are half.  The sums are those of k_force8,
// term by term:
//  - an entry's j-forces are its own, so wave w takes every 4th entry, and leaves the
//    pairs' force factors (0 outside r_cut) and the shifted j-atoms in LDS;
//  - an i-cluster's forces are summed over the entries in order, so after a barrier
//    wave w sums those of i-clusters 2w and 2w + 1 from the factors (6 instructions
//    for a cluster pair).
// An item reaches from the entry that holds its cut to the one that holds the next, so
// beyond its first entry it weighs less than kSplitWeight: that bounds its entries (by
// the least weight of one) and its cluster pairs (an entry of all kGroup i-clusters has
// the most for its weight).
constexpr int kSplitWeight = 256, kSplitEnt = 32, kSplitPairs = 97 + kGroup - 1;
static_assert(1 + (kSplitWeight - 1) / (kEntW0 + kEntW1) <= kSplitEnt, "an item's entries exceed their LDS");
static_assert(kGroup + (kSplitWeight - 1) * kGroup / kEntWMax <= kSplitPairs - (kGroup - 1),
              "an item's cluster pairs exceed their LDS (an entry may write kGroup factors from its first)");
static_assert(kSplitEnt == 32, "the scan over the entries covers 32 lanes");
template <int COUL, int LJ>
__global__ __launch_bounds__(256, 4) void k_force8_split(const SysDev* __restrict__ table, int n_sys,
                                                         const int* __restrict__ item_prefix, int red_row,
                                                         double red_step)
{
    constexpr int M = 8;
    constexpr int G = kGroup;
    constexpr bool TAB = COUL == 2, LJ1 = LJ == 0;
    int grid = (int)gridDim.x;
    asm volatile("" : "+s"(n_sys), "+s"(red_row), "+s"(grid));
    const int total = item_prefix[n_sys];
    {
        const int w0 = ((const int*)table)[0], w1 = ((const int*)table)[16], w2 = ((const int*)table)[32];
        asm volatile("" ::"s"(w0), "s"(w1), "s"(w2), "s"(total));
    }
    const int lane = threadIdx.x & 63;
    const int a = lane >> 3, b = lane & 7;
    const int wid = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const unsigned long long once = __builtin_amdgcn_ballot_w64(a < b), offd = __builtin_amdgcn_ballot_w64(a != b);
    __shared__ float fsl[kSplitPairs][64];
    __shared__ float4 xjl[kSplitEnt][M];
    __shared__ float4 tab[TAB ? kEwTabN : 1];
    int pair0 = 0;
    if (red_row >= 0) {
        if (blockIdx.x < 8) {
            if (blockIdx.x == 0) energy_reduce_system(table[0], red_row, 1, red_step);
            return;
        }
        pair0 = 8;
    }
    // XCD-aware order, as in k_force
    const int bx = (int)blockIdx.x - pair0;
    const int xcd = bx % 8;
    const int per_xcd = (grid - pair0) / 8;
    const int chunk = (total + 7) / 8;
    const int it_end = min(total, (xcd + 1) * chunk);
    const int row16 = lane >> 4;
    unsigned int joff = (unsigned int)(b * 3 + (row16 == 0 ? 0 : row16 == 2 ? 1 : 2)) * 4u;
    unsigned int aoff = a * sizeof(float4), boff = b * sizeof(float4);
    const unsigned int ioff = (unsigned int)(a * 3 + b) * 4u;
    const int pre = n_sys > 1 ? gld(&item_prefix[min(lane, n_sys - 1)]) : 0;
    int tab_sys = -1;

    for (int it = xcd * chunk + bx / 8; it < it_end; it += per_xcd) {
        int first;
        const int s = item_system(item_prefix, n_sys, it, pre, lane, first);
        const SysDev& d = table[s];
        // (the descriptor's values in one scalar round trip, as in k_force8)
        const int4* items = d.items;
        const float4* xq = d.xq;
        const int2* ent = d.ent;
        const float4* entS = d.ent_S;
        char* jpart = (char*)d.jpart;
        float* ipart = d.ipart;
        float rc2 = d.rc2;
        const float4* ewt = TAB ? d.ew_tab : nullptr;
        const float2* ljs = LJ1 ? nullptr : d.ljs;
        float c6x6 = LJ1 ? d.c6x6 : 0.f, c12x12 = LJ1 ? d.c12x12 : 0.f;
        float krf2 = COUL == 1 ? d.krf2 : 0.f, ew_tinv = TAB ? d.ew_tinv : 0.f;
        asm volatile("" : "+s"(items), "+s"(xq), "+s"(ent), "+s"(entS), "+s"(jpart), "+s"(ipart), "+s"(rc2),
                     "+s"(ewt), "+s"(ljs), "+s"(c6x6), "+s"(c12x12), "+s"(krf2), "+s"(ew_tinv));
        // (every wave's reads of the item before are done)
        if (tab_sys >= 0) __syncthreads();
        const int4 item = gld(&items[it - first]);
        if (TAB && s != tab_sys) {
            // (rows in flight with the item; read after the barrier below)
            const int t = threadIdx.x;
            const float4 v0 = gld(&ewt[t]), v1 = gld(&ewt[kEwTabN - 1]);
            tab[t] = v0;
            if (t == 0) tab[kEwTabN - 1] = v1;
        }
        const int gi = __builtin_amdgcn_readfirstlane(item.x), e0 = __builtin_amdgcn_readfirstlane(item.y),
                  e1 = __builtin_amdgcn_readfirstlane(item.z);
        float c6v = 0.f;
        if (LJ1) asm volatile("v_mov_b32 %0, %1" : "=v"(c6v) : "s"(c6x6));
        asm volatile("" : "+v"(aoff), "+v"(boff));
        float4 xi[G];
        float2 lji[G];
#pragma unroll
        for (int g = 0; g < G; ++g) {
            xi[g] = gld4(xq + (size_t)gi * (G * M), aoff + g * M * sizeof(float4));
            if (LJ == 1) lji[g] = gld2(ljs + (size_t)gi * (G * M), aoff / 2 + g * M * sizeof(float2));
        }
        // the item's list words, one entry per lane
        const int2 enl = gld(&ent[min(e0 + lane, e1 - 1)]);
        const float4 Sl = gld(&entS[min(e0 + lane, e1 - 1)]);
        const int iml = lane < min(e1 - e0, kSplitEnt) ? (enl.y >> kMetaInner) & 255 : 0;
        // the place of an entry's first factor: the cluster pairs before it (32 lanes)
        int slot = __popc(iml);
        const int own = slot;
        slot += __builtin_amdgcn_update_dpp(0, slot, 0x111, 0xF, 0xF, true);  // row_shr 1, 2, 4, 8
        slot += __builtin_amdgcn_update_dpp(0, slot, 0x112, 0xF, 0xF, true);
        slot += __builtin_amdgcn_update_dpp(0, slot, 0x114, 0xF, 0xF, true);
        slot += __builtin_amdgcn_update_dpp(0, slot, 0x118, 0xF, 0xF, true);
        const int row0 = lane_read(slot, 15);
        slot += (row16 == 1 ? row0 : 0) - own;
        // this wave's entries: every 4th of those with i-clusters
        const unsigned long long todo = __builtin_amdgcn_ballot_w64(iml != 0);
        const int rank = __popcll(todo & ((1ull << lane) - 1ull));
        unsigned long long mine = __builtin_amdgcn_ballot_w64(iml != 0 && (rank & 3) == wid);
        int k = (int)__builtin_ctzll(mine | 1ull << 63);
        float4 xj_n = gld4(xq + (size_t)lane_read(enl.x, k) * M, boff);
        float2 ljj_n = make_float2(0.f, 0.f);
        if (LJ == 1) ljj_n = gld2(ljs + (size_t)lane_read(enl.x, k) * M, boff / 2);
        if (TAB && s != tab_sys) __syncthreads();
        tab_sys = s;
        while (mine) {
            asm volatile("" : "+v"(boff), "+v"(joff));
            const int cj = lane_read(enl.x, k);
            const unsigned int meta = (unsigned int)lane_read(enl.y, k);
            const int jrow = lane_read(__float_as_int(Sl.w), k);
            float* fo = &fsl[0][0] + lane + min(lane_read(slot, k), kSplitPairs - G) * 64;
            float4 xj = xj_n;
            const float2 ljj = ljj_n;
            xj.x += lane_read(Sl.x, k);
            xj.y += lane_read(Sl.y, k);
            xj.z += lane_read(Sl.z, k);
            if (lane < M) xjl[k][lane] = xj;
            mine &= mine - 1ull;
            k = (int)__builtin_ctzll(mine | 1ull << 63);
            xj_n = gld4(xq + (size_t)lane_read(enl.x, k) * M, boff);
            if (LJ == 1) ljj_n = gld2(ljs + (size_t)lane_read(enl.x, k) * M, boff / 2);
            const unsigned int im = (meta >> kMetaInner) & 255u;
            float fjx = zero_of(xj.x), fjy = zero_of(xj.y), fjz = zero_of(xj.z);
            const int gs = cj - gi * G;
            const unsigned long long selfm = (meta & 255u) == (unsigned int)kShiftZero ? once : offd;
#pragma unroll
            for (int g = 0; g < G; ++g) {
                if (!((im >> g) & 1u)) continue;
                const float dx = xi[g].x - xj.x;
                const float dy = xi[g].y - xj.y;
                const float dz = xi[g].z - xj.z;
                const float r2 = dx * dx + dy * dy + dz * dz;
                const unsigned long long onm = g == gs ? selfm : ~0ull;
                float fs = 0.f;
                if (__builtin_amdgcn_inverse_ballot_w64(__builtin_amdgcn_ballot_w64(r2 < rc2) & onm)) {
                    Pair p;
                    fs = pair_factor<COUL, LJ>(r2, xi[g].w * xj.w, LJ == 1 ? lji[g] : make_float2(0.f, 0.f), ljj, c6v,
                                               c12x12, krf2, tab, ew_tinv, p);
                    fjx = fmaf(-dx, fs, fjx);
                    fjy = fmaf(-dy, fs, fjy);
                    fjz = fmaf(-dz, fs, fjz);
                }
                *fo = fs;
                fo += 64;
            }
            gst1(jpart + (size_t)jrow * (M * 3 * sizeof(float)), joff, reduce8(fjx, fjy, fjz));
        }
        __syncthreads();
        char* ip = (char*)(ipart + (size_t)(it - first) * (G * M * 3));
#pragma unroll
        for (int h = 0; h < 2; ++h) {
            const int g = 2 * wid + h;
            const float4 x = gld4(xq + (size_t)gi * (G * M), aoff + (unsigned int)g * (M * sizeof(float4)));
            const int from = slot + __popc(iml & ((1 << g) - 1));
            unsigned long long on = __builtin_amdgcn_ballot_w64(((iml >> g) & 1) != 0);
            float fx = zero_of(x.x), fy = zero_of(x.y), fz = zero_of(x.z);
            // (read an entry ahead)
            const auto read = [&](int e, float& f, float4& xj) {
                f = fsl[min(lane_read(from, e), kSplitPairs - 1)][lane];
                xj = xjl[e & (kSplitEnt - 1)][b];
            };
            float f0, f1;
            float4 x0, x1;
            int q = (int)__builtin_ctzll(on | 1ull << 63);
            read(q, f0, x0);
            while (on) {
                on &= on - 1ull;
                q = (int)__builtin_ctzll(on | 1ull << 63);
                read(q, f1, x1);
                fx = fmaf(x.x - x0.x, f0, fx);
                fy = fmaf(x.y - x0.y, f0, fy);
                fz = fmaf(x.z - x0.z, f0, fz);
                f0 = f1;
                x0 = x1;
            }
            const float sx = sum_b(fx), sy = sum_b(fy), sz = sum_b(fz);
            if (b < 3) gst1(ip, ioff + g * M * 3 * sizeof(float), b == 0 ? sx : b == 1 ? sy : sz);
        }
    }
}

// PRUNE: the pass evaluates each entry's build mask and stores the mask pruned
// to r_inner (a separate variant, so the plain pass carries none of it)
//
// red_row >= 0 (one system, force-only passes without pruning): the grid has
// 8 blocks in front of the pair work (one per XCD, dispatched first); block 0
// writes the previous energy pass's energy row (trace row red_row, step
// red_step) with the kinetic energy while the pair blocks run.  That pass's
// partials are complete, this pass writes none of them, and no list build has
// run in between, so the row is the one the energy-reduction kernel would
// write, and its launch is saved.  A pass that prunes has the prune guard's blocks
// there (prune_guard_arg): they read x and write what no pair block reads.
//
// Clusters of 4 and 1 atoms (8-atom clusters: k_force8)
template <int M, int COUL, int LJ, bool ENER, bool PRUNE>
__global__ __launch_bounds__(256) void k_force(const SysDev* __restrict__ table, int n_sys,
                                               const int* __restrict__ item_prefix, int red_row,
                                               double red_step)
{
    constexpr bool prune = PRUNE;
    constexpr int MM = M * M;
    constexpr int E = 64 / MM;
    constexpr int G = kGroup;
    constexpr int LM = ilog2(M);
    const int lane = threadIdx.x & 63;
    const int esub = lane / MM;
    const int a = (lane / M) % M;
    const int b = lane % M;
    const int wid = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);

    // Ewald tables: the force table (every pass) and, with energies, the erfc
    // table; one private copy per wave, reloaded when the wave moves to an
    // item of another system
    constexpr bool TAB = (COUL == 2);
    constexpr bool ETAB = TAB && ENER;
    // per wave kTabU * 64 rows: every lane writes each of its kTabU rows (the
    // rows past the table repeat its last interval and are never read)
    constexpr int kTabU = (kEwTabN + 63) / 64;
    __shared__ float4 tab_lds[TAB ? 4 * kTabU * 64 : PRUNE ? kGuardLds : 1];
    __shared__ float4 etab_lds[ETAB ? 4 * kTabU * 64 : 1];
    double* guard_lds = (double*)tab_lds;

    // XCD-aware order: blocks are dispatched round-robin over the 8 XCDs
    // (XCD = block id mod 8).  Give each XCD a contiguous eighth of the items
    // (items of nearby i-groups share j-clusters in that XCD's L2) and spread
    // it over that XCD's blocks, so all XCDs work whatever the item count.
    int pair0 = 0;  // the first pair block
    if constexpr (!ENER && !PRUNE) {
        if (red_row >= 0) {
            if (blockIdx.x < 8) {
                if (blockIdx.x == 0) energy_reduce_system(table[0], red_row, 1, red_step);
                return;
            }
            pair0 = 8;
        }
    }
    if constexpr (PRUNE) {
        if (red_row >= 0) {
            // the prune guard's blocks: red_row = buffer | fold << 1 | blocks << 2
            const int nb = red_row >> 2;
            if ((int)blockIdx.x < nb) prune_guard_block(table[0], nb, 1, red_row & 1, red_row & 2, guard_lds);
            pair0 = (nb + 7) / 8 * 8;
            if ((int)blockIdx.x < pair0) return;
        }
    }
    const int total = item_prefix[n_sys];
    const int bx = (int)blockIdx.x - pair0;  // (bx mod 8 is still the block's XCD)
    const int xcd = bx % 8;
    const int bj = bx / 8;
    const int per_xcd = ((int)gridDim.x - pair0) / 8;  // the pair blocks are a multiple of 8
    const int chunk = (total + 7) / 8;
    const int it_end = min(total, (xcd + 1) * chunk);
    const int nwave = per_xcd * 4;
    float4* tab = tab_lds + (TAB ? wid * kTabU * 64 : 0);
    float4* etab = etab_lds + (ETAB ? wid * kTabU * 64 : 0);
    int tab_sys = -1;

    for (int it = xcd * chunk + bj * 4 + wid; it < it_end; it += nwave) {
        int s = 0;
        if (n_sys > 1) {
            int lo = 0, hi = n_sys - 1;
            while (lo < hi) {
                const int mid = (lo + hi + 1) >> 1;
                if (item_prefix[mid] <= it) lo = mid; else hi = mid - 1;
            }
            s = lo;
        }
        s = __builtin_amdgcn_readfirstlane(s);
        const SysDev& d = table[s];
        // the table (when the wave needs a new one) and the work item are
        // loaded in one memory round trip, then the i-atoms, cluster sizes,
        // first entries and first j-atoms (through the item's j-cluster)
        // together: a fixed number of unconditional loads per lane, so none is
        // moved behind a branch.  With per-atom LJ parameters the variant is
        // short of registers for the table in flight: it loads one row per
        // lane at a time (its waves take several items each in the large
        // systems it serves, and refill only for another system), and so do the
        // energy passes (the rare ones) for both their tables
        constexpr bool TAB1 = TAB && LJ == 0 && !ENER;
        const bool fill = TAB && s != tab_sys;
        float4 tv[TAB1 ? kTabU : 1];
        if (TAB1 && fill) {
#pragma unroll
            for (int u = 0; u < kTabU; ++u) tv[u] = gld(&d.ew_tab[min(lane + 64 * u, kEwTabN - 1)]);
        }
        const int li = n_sys > 1 ? it - item_prefix[s] : it;  // item_prefix[0] = 0
        const int4 item = gld(&d.items[li]);
        if (fill) {
            if (TAB1) {
#pragma unroll
                for (int u = 0; u < kTabU; ++u) tab[lane + 64 * u] = tv[u];
            } else {
                for (int k = lane; k < kEwTabN; k += 64) tab[k] = gld(&d.ew_tab[k]);
            }
            if (ETAB)
                for (int k = lane; k < kEwTabN; k += 64) etab[k] = gld(&d.ew_etab[k]);
            // LDS accesses of one wave complete in order; the fence keeps the
            // compiler from moving the table reads above these writes
            __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
            __builtin_amdgcn_wave_barrier();
            __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
            tab_sys = s;
        }
        const int gi = item.x, e0 = item.y, e1 = item.z;

        // model constants, one SGPR each for the item; only those this variant
        // uses are loaded (a pinned value is never dropped by the compiler)
        const float rc2 = pin(d.rc2);
        const float rmask2 = __int_as_float(__builtin_amdgcn_readfirstlane(__float_as_int(0.5f * d.rc2)));
        constexpr bool LJ1 = LJ == 0;                  // one LJ type
        const float c6 = (LJ1 && ENER) ? pin(d.c6) : 0.f, c12 = (LJ1 && ENER) ? pin(d.c12) : 0.f;
        const float c6x6 = LJ1 ? pin(d.c6x6) : 0.f, c12x12 = LJ1 ? pin(d.c12x12) : 0.f;
        // 6 C6 in a vector register: the LJ FMA takes one scalar operand only
        float c6v = 0.f;
        if (LJ1) asm volatile("v_mov_b32 %0, %1" : "=v"(c6v) : "s"(c6x6));
        const float krf = (COUL == 1 && ENER) ? pin(d.krf) : 0.f, crf = (COUL == 1 && ENER) ? pin(d.crf) : 0.f;
        const float krf2 = COUL == 1 ? pin(d.krf2) : 0.f;
        const float ew_tinv = TAB ? pin(d.ew_tinv) : 0.f;
        // dynamic pruning (a pass that prunes evaluates the build's i-cluster
        // mask and keeps, per entry, the i-clusters with a pair within r_inner)
        const float rin2 = prune ? pin(d.rin2) : 0.f;

        float4 xi[G];
        float2 lji[G];
        unsigned int ireal = 0, iany = 0;
#pragma unroll
        for (int g = 0; g < G; ++g) {
            const int slot = (gi * G + g) * M + a;
            xi[g] = gld(&d.xq[slot]);
            if (LJ == 1) lji[g] = gld(&d.ljs[slot]);
        }
        // the group's 8 cluster sizes (32-byte aligned)
        const int4 nr03 = gld((const int4*)&d.cl_nreal[gi * G]);
        const int4 nr47 = gld((const int4*)&d.cl_nreal[gi * G + 4]);
        float fix[G], fiy[G], fiz[G];
#pragma unroll
        for (int g = 0; g < G; ++g) fix[g] = fiy[g] = fiz[g] = 0.0f;
        float elj = 0.f, ec = 0.f, wxx = 0.f, wyy = 0.f, wzz = 0.f, wxy = 0.f, wxz = 0.f, wyz = 0.f;

        // software pipeline, two stages deep: the list data of the entry after
        // next and the j-atoms of the next entry are in flight while the current
        // entry is evaluated, so no load waits on another load inside the loop
        const int2* ent = pinp(d.ent);
        const float4* entS = pinp(d.ent_S);
        const float4* xq = pinp(d.xq);
        const float2* ljs = pinp(d.ljs);
        float* jpart = pinp(d.jpart);
        int* entw = PRUNE ? pinp((int*)d.ent) : nullptr;
        int2 en_n, en_nn;
        float4 S_n, xj_n;
        float2 ljj_n = make_float2(0.f, 0.f);
        {
            const int e = min(e0 + esub, e1 - 1);
            en_n = gld(&ent[e]);
            S_n = gld(&entS[e]);
            en_nn = gld(&ent[min(e0 + E + esub, e1 - 1)]);
            xj_n = gld(&xq[en_n.x * M + b]);
            if (LJ == 1) ljj_n = gld(&ljs[en_n.x * M + b]);
        }
        // ireal: per lane, the i-clusters whose atom a is real
        {
            const int nrg[G] = {nr03.x, nr03.y, nr03.z, nr03.w, nr47.x, nr47.y, nr47.z, nr47.w};
#pragma unroll
            for (int g = 0; g < G; ++g) {
                if (a < nrg[g]) ireal |= 1u << g;
                if (nrg[g] > 0) iany |= 1u << g;
            }
            iany = __builtin_amdgcn_readfirstlane(iany);
        }
        bool pend = false;  // a j-partial of the previous entry waits to be stored
        float* pend_p = jpart;
        float pend_x = 0.f, pend_y = 0.f, pend_z = 0.f;
        bool pend_m = false;  // (pruning) its pruned meta word, stored with it
        int* pend_mp = entw;
        int pend_mv = 0;
        for (int eb = e0; eb < e1; eb += E) {
            const int e = eb + esub;
            const bool valid = e < e1;
            const int2 en = en_n;
            const float4 S = S_n;
            float4 xj = xj_n;
            const float2 ljj = ljj_n;
            // this entry's data and the next entry's j-cluster are used first, so
            // the wait for the prefetched loads comes before this iteration's store
            int cj_next = en_nn.x;
            asm volatile("" : "+v"(cj_next));  // materialised (waited for) here
            xj.x += S.x;
            xj.y += S.y;
            xj.z += S.z;
            __builtin_amdgcn_sched_barrier(0);
            // the previous entry's j-partial, stored one entry late: issued after
            // that wait and before this iteration's prefetch, so no wait for a
            // prefetch also waits for a store issued after it
            if (pend) {
                if (LM == 0) {
                    gst(pend_p, pend_x);
                    gst(pend_p + 1, pend_y);
                    gst(pend_p + 2, pend_z);
                } else {
                    gst(pend_p, pend_x);
                }
            }
            if (pend_m) gst(pend_mp, pend_mv);
            // issued on every iteration (indices clamped to the item's last
            // entry; the last iteration's loads go unused): with a fixed number
            // of loads per iteration the compiler waits for the current entry's
            // data only, not for the prefetch just issued
            en_n = en_nn;
            S_n = gld(&entS[min(eb + E + esub, e1 - 1)]);
            xj_n = gld(&xq[cj_next * M + b]);
            if (LJ == 1) ljj_n = gld(&ljs[cj_next * M + b]);
            en_nn = gld(&ent[min(eb + 2 * E + esub, e1 - 1)]);
            // row of this entry's j-partial (the shift vector's w word)
            const int jrow = __float_as_int(S.w);
            const int cj = en.x;
            const unsigned int meta = (unsigned int)en.y;
            const int sid = meta & 255u;
            const unsigned int im = (meta >> (prune ? kMetaOuter : kMetaInner)) & 255u;
            const int nrj = (meta >> kMetaNreal) & 15u;
            unsigned int pin_m = 0u;  // (pruning) i-clusters with a pair within r_inner
            const bool jreal = valid && (b < nrj);
            // i-clusters this lane interacts with in this entry; the entry of a
            // cluster with itself (zero shift) counts each pair once (a < b)
            const int gself = (sid == kShiftZero) ? (cj - gi * G) : -1;
            unsigned int act = jreal ? (im & ireal) : 0u;
            if (gself >= 0 && gself < G && a >= b) act &= ~(1u << gself);
            float fjx = 0.f, fjy = 0.f, fjz = 0.f;
#pragma unroll
            for (int g = 0; g < G; ++g) {
                // lanes of this cluster pair that hold a pair to evaluate, as a
                // wave mask: the tests below stay scalar
                const unsigned long long onm = __builtin_amdgcn_ballot_w64(((act >> g) & 1u) != 0u);
                if (onm == 0ull) continue;
                const float dx = xi[g].x - xj.x;
                const float dy = xi[g].y - xj.y;
                const float dz = xi[g].z - xj.z;
                const float r2 = dx * dx + dy * dy + dz * dz;
                if (prune && ((act >> g) & 1u) && r2 < rin2) pin_m |= 1u << g;
                const unsigned long long cm = __builtin_amdgcn_ballot_w64(r2 < rc2) & onm;
                if (cm == 0ull) continue;  // listed cluster pair with no pair inside r_cut now
                const bool c = __builtin_amdgcn_inverse_ballot_w64(cm);
                // lanes without a pair get r^2 = r_cut^2 / 2: finite, and a table
                // index inside the table (their result is discarded below)
                const float r2s = c ? r2 : rmask2;
                const float rinv = __builtin_amdgcn_rsqf(r2s);
                const float rinv2 = rinv * rinv;
                const float rinv6 = rinv2 * rinv2 * rinv2;
                float c6p, c12p, fl;
                if (LJ == 1) {
                    const float sg = lji[g].x + ljj.x;
                    const float ep = lji[g].y * ljj.y;
                    const float s2 = sg * sg;
                    const float s6 = s2 * s2 * s2;
                    c6p = ep * s6;
                    c12p = c6p * s6;
                    fl = (12.0f * c12p * rinv6 - 6.0f * c6p) * rinv6;
                } else {
                    c6p = c6;
                    c12p = c12;
                    fl = fmaf(c12x12, rinv6, -c6v) * rinv6;
                }
                float fs = fl * rinv2;
                float vc = 0.f;
                const float qq = xi[g].w * xj.w;
                if (COUL == 1) {
                    fs += qq * (rinv * rinv2 - krf2);
                    if (ENER) vc = qq * (rinv + krf * r2s - crf);
                } else if (COUL == 2) {
                    // q(r) from the cubic table: F_coul = qq q(r) r_ij / r^3;
                    // energies: erfc(beta r) from the second table
                    const float r = r2s * rinv;
                    const float rs = r * ew_tinv;
                    const int k = (int)rs;  // <= kEwTab: the tables have one interval past r_cut
                    const float w = __builtin_amdgcn_fractf(rs);
                    const float4 cf = tab[k];
                    const float qv = fmaf(fmaf(fmaf(cf.w, w, cf.z), w, cf.y), w, cf.x);
                    fs = fmaf(qq * qv, rinv, fl) * rinv2;
                    if (ENER) {
                        const float4 ce = etab[k];
                        const float ev = fmaf(fmaf(fmaf(ce.w, w, ce.z), w, ce.y), w, ce.x);
                        vc = qq * fmaf(ev, rinv, -d.ew_shift);
                    }
                }
                fs = c ? fs : 0.0f;
                const float tx = fs * dx, ty = fs * dy, tz = fs * dz;
                fix[g] += tx;
                fiy[g] += ty;
                fiz[g] += tz;
                fjx -= tx;
                fjy -= ty;
                fjz -= tz;
                if (ENER) {
                    float vl = (c12p * rinv6 - c6p) * rinv6;
                    if (d.pot_shift) vl -= (LJ == 1) ? (c12p * d.irc12 - c6p * d.irc6) : d.lj_shift;
                    elj += c ? vl : 0.0f;
                    ec += c ? vc : 0.0f;
                    wxx += tx * dx;
                    wyy += ty * dy;
                    wzz += tz * dz;
                    wxy += tx * dy;
                    wxz += tx * dz;
                    wyz += ty * dz;
                }
            }
            // j-forces: sum over the a-lanes of each (entry, b), one component per
            // lane, this entry's partial (summed per atom by the gather; an entry
            // without any pair inside r_cut gives zeros), stored at the next entry
            {
                float* jp = jpart + ((size_t)jrow * M + b) * 3;
                if (LM == 0) {
                    pend = valid;
                    pend_p = jp;
                    pend_x = fjx;
                    pend_y = fjy;
                    pend_z = fjz;
                } else {
                    int comp;
                    bool own;
                    pend_x = reduce3<M, LM>(fjx, fjy, fjz, a, comp, own);
                    pend = valid && own;
                    pend_p = jp + comp;
                }
            }
            if (prune) {
                // the entry's pruned mask, one lane per entry (the OR over the
                // entry's lanes)
                for (int o = 1; o < MM; o <<= 1) pin_m |= (unsigned int)__shfl_xor((int)pin_m, o, 64);
                pend_m = valid && (lane % MM) == 0;
                pend_mp = entw + 2 * (size_t)e + 1;
                pend_mv = (int)((meta & ~(255u << kMetaInner)) | (pin_m << kMetaInner));
            }
        }
        if (pend) {  // the item's last entry
            gst(pend_p, pend_x);
            if (LM == 0) {
                gst(pend_p + 1, pend_y);
                gst(pend_p + 2, pend_z);
            }
        }
        if (pend_m) gst(pend_mp, pend_mv);
        // i-forces: sum over b (3-component butterfly), then over the entries of
        // the wave; stored as this item's partial
        float* ip = d.ipart + (size_t)li * (G * M * 3);
#pragma unroll
        for (int g = 0; g < G; ++g) {
            if (!((iany >> g) & 1u)) continue;
            if (LM == 0) {
                float x = fix[g], y = fiy[g], z = fiz[g];
#pragma unroll
                for (int m = 1; m < 64; m <<= 1) {
                    x += __shfl_xor(x, m, 64);
                    y += __shfl_xor(y, m, 64);
                    z += __shfl_xor(z, m, 64);
                }
                if (lane == 0) {
                    gst(ip + g * 3, x);
                    gst(ip + g * 3 + 1, y);
                    gst(ip + g * 3 + 2, z);
                }
            } else {
                int comp;
                bool own;
                float v = reduce3<1, LM>(fix[g], fiy[g], fiz[g], b, comp, own);
                if (E >= 2) v += xshfl<MM>(v);
                if (E >= 4) v += xshfl<2 * MM>(v);
                if (own && esub == 0) gst(ip + (g * M + a) * 3 + comp, v);
            }
        }
        if (ENER) {
            const float v0 = wave_sum(elj), v1 = wave_sum(ec), v2 = wave_sum(wxx), v3 = wave_sum(wyy),
                        v4 = wave_sum(wzz), v5 = wave_sum(wxy), v6 = wave_sum(wxz), v7 = wave_sum(wyz);
            if (lane == 0) {
                float* o = d.epart + (size_t)li * kEnerPart;
                o[0] = v0; o[1] = v1; o[2] = v2; o[3] = v3;
                o[4] = v4; o[5] = v5; o[6] = v6; o[7] = v7;
            }
        }
    }
}

// ---- dispatch table (the C++ analogue of the paper's kernel function table) ----
typedef void (*ForceFn)(const SysDev*, int, const int*, int, double);

template <int M, int C, int L>
static ForceFn pick(bool ener, bool prune)
{
    if constexpr (M == 8) {
        if (prune) return ener ? k_force8<C, L, true, true> : k_force8<C, L, false, true>;
        return ener ? k_force8<C, L, true, false> : k_force8<C, L, false, false>;
    } else {
        if (prune) return ener ? k_force<M, C, L, true, true> : k_force<M, C, L, false, true>;
        return ener ? k_force<M, C, L, true, false> : k_force<M, C, L, false, false>;
    }
}

template <int M>
static ForceFn pick_m(int coul, int lj, bool ener, bool prune)
{
    switch (coul * 2 + lj) {
    case 0: return pick<M, 0, 0>(ener, prune);
    case 1: return pick<M, 0, 1>(ener, prune);
    case 2: return pick<M, 1, 0>(ener, prune);
    case 3: return pick<M, 1, 1>(ener, prune);
    case 4: return pick<M, 2, 0>(ener, prune);
    default: return pick<M, 2, 1>(ener, prune);
    }
}

static ForceFn pick_split(int coul, int lj)
{
    switch (coul * 2 + lj) {
    case 0: return k_force8_split<0, 0>;
    case 1: return k_force8_split<0, 1>;
    case 2: return k_force8_split<1, 0>;
    case 3: return k_force8_split<1, 1>;
    case 4: return k_force8_split<2, 0>;
    default: return k_force8_split<2, 1>;
    }
}

int split_items(int M, int jtile, double n_rho_r3, int built)
{
    if (M != 8 || item_weight(M, jtile) > kSplitWeight) return kSplitNever;
    return (int)std::min(std::max(0.31 * n_rho_r3 / item_weight(M, jtile), (double)built), (double)kSplitNever);
}

hipError_t launch_force(const SysDev* table, int n_sys, const int* item_prefix, int M, int coulomb,
                        int lj, bool ener, int max_blocks, int total_item_cap, hipStream_t s, bool prune,
                        int red_row, double red_step, int few_items)
{
    if (red_row >= 0 && (n_sys != 1 || (ener && !prune))) return hipErrorInvalidValue;
    ForceFn fn;
    if (M == 8) fn = pick_m<8>(coulomb, lj, ener, prune);
    else if (M == 4) fn = pick_m<4>(coulomb, lj, ener, prune);
    else if (M == 1) fn = pick_m<1>(coulomb, lj, ener, prune);
    else return hipErrorInvalidValue;
    // persistent grid: up to one wave per work item (4096 blocks at most), more
    // than the CUs hold at once: on the 1M-atom slab one resident round of
    // blocks (1024) is 4 % slower.  max_blocks > 0 caps it (a multiple of 8 so
    // the XCD-aware block remap in the kernel is a bijection)
    const int form = force_form(few_items);
    const bool split = M == 8 && !ener && !prune && form == 0;
    if (split) fn = pick_split(coulomb, lj);
    else if (M == 8 && coulomb == 2 && lj == 0 && !ener && !prune && form == 2)
        fn = k_force8<2, 0, false, false, 5>;
    int blocks = split ? total_item_cap : (total_item_cap + 3) / 4;
    if (blocks > 4096) blocks = 4096;
    if (max_blocks > 0 && blocks > max_blocks) blocks = max_blocks;
    if (blocks < 8) blocks = 8;
    blocks = (blocks + 7) / 8 * 8;
    // the energy row's block, and 7 that exit; the prune guard's blocks
    if (red_row >= 0) blocks += prune ? ((red_row >> 2) + 7) / 8 * 8 : 8;
    hipLaunchKernelGGL(fn, dim3(blocks), dim3(256), 0, s, table, n_sys, item_prefix, red_row, red_step);
    return hipGetLastError();
}

}  // namespace nbi
