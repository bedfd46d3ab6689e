// nb_step.hip -- per-step kernels around the force kernel (gfx950):
// position staging, force gather, FP64 energy/virial/kinetic reductions,
// velocity Verlet, and the steepest-descent relaxation step.
//
// Positions and velocities stay FP64 in HBM; the force kernel sees FP32
// coordinates relative to each i-group's reference point (its bounding-box
// centre), so FP32 rounding is set by the group size (< 1 nm), not by the box.
#include "nb_internal.h"

namespace nbi {

// FP64 master x -> FP32 group-local SoA (+ scaled charge, LB parameters);
// flags (per system, NULL = every system): 0 = skip.  clear: block 0 also
// clears the status words (no kernel before it in the stream is still running,
// and this one writes none)
__global__ __launch_bounds__(256) void k_stage(const SysDev* __restrict__ table, const int* flags, int clear)
{
    if (flags && !flags[blockIdx.y]) return;
    const SysDev& d = table[blockIdx.y];
    if (clear && blockIdx.x == 0 && threadIdx.x < ST_COUNT) d.status[threadIdx.x] = 0;
    const int slot = blockIdx.x * blockDim.x + threadIdx.x;
    const int GM = d.G * d.M;
    if (slot >= d.n_groups[0] * GM) return;
    const int a = d.slot_atom[slot];
    const int g = slot / GM;
    float4 p = pad_pos(slot);
    float2 l = make_float2(0.f, 0.f);
    if (a >= 0) {
        const double xa[3] = {d.x[3 * a], d.x[3 * a + 1], d.x[3 * a + 2]};
        const int wa[3] = {d.slot_wrap[3 * slot], d.slot_wrap[3 * slot + 1], d.slot_wrap[3 * slot + 2]};
        const double ref[3] = {d.gr_ref[3 * g], d.gr_ref[3 * g + 1], d.gr_ref[3 * g + 2]};
        stage_pos(d, xa, wa, ref, p);
        p.w = (float)(d.q[a] * (double)d.qscale);
        if (d.lj == 1) {
            l.x = (float)(0.5 * d.sig[a]);
            l.y = (float)(2.0 * sqrt(d.eps[a]));
        }
    }
    d.xq[slot] = p;
    if (d.lj == 1) d.ljs[slot] = l;
}

__device__ __forceinline__ long long to_fixed(float v, double scale)
{
    // v * scale rounded to an integer: 1.5 * 2^52 puts the integer in the low
    // mantissa bits for |v * scale| < 2^51.
    const double t = fma((double)v, scale, 6755399441055744.0);
    return __double_as_longlong(t) - 0x4338000000000000LL;
}

// one block per system (the energy pass's trace row, see energy_reduce_system)
__global__ __launch_bounds__(256) void k_energy_reduce(const SysDev* __restrict__ table,
                                                       int trace_row, int with_ke, double step_value)
{
    energy_reduce_system(table[blockIdx.x], trace_row, with_ke, step_value);
}


// v += dt/2 F/m ; x += dt v  (every velocity-Verlet update in this file is
// written with explicit FMAs, so fused and separate kernels agree bitwise)
__global__ __launch_bounds__(256) void k_kick_drift(const SysDev* __restrict__ table, double dt)
{
    const SysDev& d = table[blockIdx.y];
    const int nb = sys_blocks(d.n_atoms);
    if ((int)blockIdx.x >= nb) return;
    const int stride = nb * blockDim.x;
    double* x = (double*)d.x;
    for (int i = blockIdx.x * blockDim.x + threadIdx.x; i < d.n_atoms; i += stride) {
        const double h = 0.5 * dt / d.mass[i];
        for (int k = 0; k < 3; ++k) {
            const double v = fma(h, (double)d.f[3 * i + k], d.v[3 * i + k]);
            d.v[3 * i + k] = v;
            x[3 * i + k] = fma(dt, v, x[3 * i + k]);
        }
    }
}

// List-buffer guard (Verlet displacement criterion): at each rebuild, the
// largest displacement since the previous build; a pair can only have entered
// r_cut unlisted if two atoms moved by >= (r_list - r_cut)/2 each.

__device__ double block_max_partials(const double* p, int n)
{
    __shared__ double sh[256];
    return block_max_partials(p, n, sh);
}

// (as a kernel of its own where no pruning force pass follows)
__global__ __launch_bounds__(256) void k_prune_guard(const SysDev* __restrict__ table, int check, int cur,
                                                     int fold)
{
    __shared__ double sh[256];
    prune_guard_block(table[0], gridDim.x, check, cur, fold, sh);
}

// Steepest descent of one system: x += max_disp * F / max|F| (the largest move is
// max_disp), and the staging of the new positions, per slot.  max|F|^2 comes from
// the n_part partials that the force gather left.  A step that finds max|F| < f_tol
// (or NaN) sets done and moves nothing, nor does any step after it, so the host can
// enqueue ahead and look later: it follows through *seen, a word in pinned host
// memory {steps done, 1 + the step that converged or 0}.  (With a kernel of its own
// for max|F|, another for the staging, and the flag copied back and waited for in
// every iteration, an iteration of 24,000 atoms took 87 us.)
__global__ __launch_bounds__(256) void k_minimize_move(const SysDev* __restrict__ table, double max_disp, double f_tol,
                                                       int n_part, int it, int* done, unsigned long long* seen)
{
    const SysDev& d = table[0];
    // (one read per block: block 0 may set it meanwhile)
    __shared__ int done_s;
    if (threadIdx.x == 0) done_s = gld(done);
    __syncthreads();
    const int done0 = done_s;
    int stop = done0;
    double fm = 0.0;
    if (!stop) {
        fm = sqrt(block_max_partials(d.fmax_part, n_part));
        if (!(fm >= f_tol)) stop = it + 1;
    }
    if (blockIdx.x == 0 && threadIdx.x == 0) {
        if (stop && !done0) gst(done, stop);
        // (one word: no order between two stores to keep)
        __hip_atomic_store(seen, ((unsigned long long)stop << 32) | (unsigned int)(it + 1), __ATOMIC_RELAXED,
                           __HIP_MEMORY_SCOPE_SYSTEM);
    }
    if (stop) return;
    const int slot = blockIdx.x * blockDim.x + threadIdx.x;
    const int GM = d.G * d.M;
    if (slot >= d.n_groups[0] * GM) return;
    const int a = gld(&d.slot_atom[slot]);
    if (a < 0) return;  // padding slots keep their staged values
    const double s = max_disp / fm;
    double* x = (double*)d.x;
    double xn[3];
    int wa[3];
    double ref[3];
    const int g = slot / GM;
    for (int k = 0; k < 3; ++k) {
        xn[k] = fma(s, (double)gld(&d.f[3 * a + k]), gld(&x[3 * a + k]));
        wa[k] = gld(&d.slot_wrap[3 * slot + k]);
        ref[k] = gld(&d.gr_ref[3 * g + k]);
    }
    for (int k = 0; k < 3; ++k) gst(&x[3 * a + k], xn[k]);
    float4 p;
    stage_pos(d, xn, wa, ref, p);
    p.w = (float)(gld(&d.q[a]) * (double)d.qscale);
    gst(&d.xq[slot], p);
}

// prefix over member systems of their work-item counts (one wave, 64 systems at a
// time: one by one, each count waited for the one before, 8 us for 20 systems); a
// system with flag 0 contributes no items
__global__ __launch_bounds__(64) void k_item_prefix(const SysDev* __restrict__ table, int n_sys, int* prefix,
                                                    const int* flags)
{
    const int lane = threadIdx.x;
    int carry = 0;
    if (lane == 0) prefix[0] = 0;
    for (int s0 = 0; s0 < n_sys; s0 += 64) {
        const int s = s0 + lane;
        const bool on = s < n_sys && (!flags || flags[s] != 0);
        int incl = on ? gld(table[s].n_items) : 0;
        for (int o = 1; o < 64; o <<= 1) {
            const int t = __shfl_up(incl, o, 64);
            if (lane >= o) incl += t;
        }
        if (s < n_sys) prefix[s + 1] = carry + incl;
        carry += __shfl(incl, 63, 64);
    }
}

// mode 0: x, v -> x_bak, v_bak (every atom); mode 1: back again
__global__ __launch_bounds__(256) void k_state_copy(const SysDev* __restrict__ table, int mode)
{
    const SysDev& d = table[blockIdx.y];
    const int n3 = 3 * d.n_atoms;
    double* x = (double*)d.x;
    for (int i = blockIdx.x * blockDim.x + threadIdx.x; i < n3; i += gridDim.x * blockDim.x) {
        if (mode == 0) {
            gst(&d.x_bak[i], gld(&x[i]));
            gst(&d.v_bak[i], gld(&d.v[i]));
        } else {
            gst(&x[i], gld(&d.x_bak[i]));
            gst(&d.v[i], gld(&d.v_bak[i]));
        }
    }
}

// ---- fused per-slot step kernels (plain steps without a list rebuild) --------
// Every real atom owns exactly one slot, so per-atom updates can run in cluster
// order and the FP64 arithmetic is the same as in k_kick_drift.

// v += dt/2 F/m ; x += dt v ; stage the new x into the group-local FP32 SoA
__global__ __launch_bounds__(256) void k_kick_drift_stage(const SysDev* __restrict__ table, double dt)
{
    const SysDev& d = table[blockIdx.y];
    const int slot = blockIdx.x * blockDim.x + threadIdx.x;
    const int GM = d.G * d.M;
    if (slot >= d.n_groups[0] * GM) return;
    const int a = d.slot_atom[slot];
    if (a < 0) return;  // padding slots keep their staged values
    const int g = slot / GM;
    double* x = (double*)d.x;
    const double h = 0.5 * dt / d.mass[a];
    double xn[3];
    for (int k = 0; k < 3; ++k) {
        const double v = fma(h, (double)d.f[3 * a + k], d.v[3 * a + k]);
        d.v[3 * a + k] = v;
        xn[k] = fma(dt, v, x[3 * a + k]);
        x[3 * a + k] = xn[k];
    }
    float4 p;
    {
        const int wa[3] = {d.slot_wrap[3 * slot], d.slot_wrap[3 * slot + 1], d.slot_wrap[3 * slot + 2]};
        const double ref[3] = {d.gr_ref[3 * g], d.gr_ref[3 * g + 1], d.gr_ref[3 * g + 2]};
        stage_pos(d, xn, wa, ref, p);
    }
    p.w = (float)(d.q[a] * (double)d.qscale);
    d.xq[slot] = p;
}

// Force gather: an atom's force is the sum of its i-partials (one per work item
// of its group) and its j-partials (one per list entry with its cluster as j;
// the force kernel writes them in rows grouped by j-cluster, so a cluster's
// j-partials are contiguous).  V64r sums in int64 fixed point (exact, so the
// result does not depend on the order: bitwise reproducible); V32 sums in FP32.
// The force goes to the caller's f[N,3] in original atom order; with KICK the
// velocity half-kick v += dt/2 F/m follows (plus kinetic-energy partials), fusing
// the end of a velocity-Verlet step.
//
// R lanes share an atom's rows: a wave's lane (r, a) handles its atom a and every
// R-th row, then the rows are summed with shuffles.  Small launches take R = 64/M (a
// wave per cluster), bound by latency; large ones R = 2 (WIDE), where a wave per
// cluster finishes 8 atoms with 64 lanes and shuffles int64 sums: its FP64 work and
// not memory was the bound (ensemble of 20 systems 42.2 us a step, 20.6 now;
// 1,000,000 atoms 123 and 76.8, where the 350 MB of partials take about 70).
//
// Kinetic-energy partial p covers 4 clusters (p, p + nb, ...): a block of one-cluster
// waves, or one wave of R = 2 (32 slots), with the same sums in the same order, so
// the energies do not depend on R, and the count depends only on the system: they
// are the same alone and in a batch.
__device__ inline int cluster_blocks(int n_clusters)
{
    int b = (n_clusters + 3) / 4;
    return b > kKeBlocks ? kKeBlocks : (b < 1 ? 1 : b);
}

// NEXT (with KICK): 0 = stop after the half-kick; 1 = also the next step's
// half-kick and drift (v += dt/2 F/m, x += dt v: the same FP64 operations as
// k_kick_drift), keeping the full-step x, v in x_bak, v_bak, and the work of
// the list build's first kernel (a rebuild follows: its counters and status
// words cleared, the list-buffer guard's largest squared displacement since the
// last build per block, x recorded for the next one); 2 = half-kick, drift and
// the staging of the new x (as k_kick_drift_stage).  open: the forces of a run's
// first positions, with no step to close: only the next step's half-kick and drift
// (NEXT 1 or 2).  held: a list that ran out of capacity moves nothing, x, v and f
// stay as they are (the host has enqueued past a rebuild whose verdict it does not
// know yet; see md_step).
// FMAX (without KICK): also the largest |F|^2 per block into fmax_part (NaN wins)
// WIDE (all systems of 8-atom clusters): R = 2
// ENER (one system, without KICK): block 0 forms the energy row from the pair
// kernel's partials meanwhile (a kernel of its own after the gather took 6 to 8 us)
//
// The kernel is a chain of memory round trips: the descriptor (every field that it
// needs in one batch, pinned), then the counts with the first cluster's row ranges
// and slots, then rows and atom data; nothing else waits on a load (with fields and
// staging data loaded where they are used 5.6 us at 2,744 atoms, now 4.4, of which
// the launch is about 2.5).
template <bool KICK, bool FMAX, int NEXT, bool WIDE, bool ENER = false>
__global__ __launch_bounds__(256) void k_gather(const SysDev* __restrict__ table, double dt, int ke, int open,
                                                int held, const int* flags, int ener_row, double ener_step)
{
    if (flags && !flags[blockIdx.y]) return;  // (only the force-only gather takes flags)
    const SysDev& d = table[blockIdx.y];
    if (ENER && blockIdx.x == 0) {
        energy_reduce_system(d, ener_row, 0, ener_step);
        return;
    }
    const int bx = (int)blockIdx.x - (ENER ? 1 : 0);
    const int *n_groups_p = d.n_groups, *n_items_p = d.n_items, *n_ent_p = d.n_ent;
    const int *nreal_p = d.cl_nreal, *item_start = d.item_start, *jstart = d.jstart, *slot_atom = d.slot_atom;
    const float *ipart = d.ipart, *jpart = d.jpart, *pme_f = d.pme_f;
    float* fp = d.f;
    const int M = WIDE ? 8 : d.M;
    const int max_slots = d.max_groups * kGroup * M;
    const bool f32 = d.fp32_reduce != 0;
    const float lim = d.fx_lim;
    const double sc = d.fx_scale, fx_inv = d.fx_inv;
    const double* mass_p = KICK ? d.mass : nullptr;
    double *xp = KICK ? (double*)d.x : nullptr, *vp = KICK ? d.v : nullptr;
    const int* wrap_p = NEXT == 2 ? d.slot_wrap : nullptr;
    const double *ref_p = NEXT == 2 ? d.gr_ref : nullptr, *q_p = NEXT == 2 ? d.q : nullptr;
    float4* xq = NEXT == 2 ? d.xq : nullptr;
    asm volatile("" ::"s"(n_groups_p), "s"(n_items_p), "s"(n_ent_p), "s"(nreal_p), "s"(item_start), "s"(jstart),
                 "s"(slot_atom), "s"(ipart), "s"(jpart), "s"(pme_f), "s"(fp), "s"(mass_p), "s"(xp), "s"(vp),
                 "s"(wrap_p), "s"(ref_p), "s"(q_p), "s"(xq), "s"(lim), "s"(sc), "s"(fx_inv));
    if (NEXT == 1) {
        // the build's counters and status words (all but the fault flags of
        // earlier steps); none of them is read before the build
        const int t = bx * blockDim.x + threadIdx.x, ts = gridDim.x * blockDim.x;
        for (int i = t; i < d.n_cols; i += ts) {
            gst(&d.col_count[i], 0);
            gst(&d.col_fill[i], 0);
        }
        for (int i = t; i < d.max_groups; i += ts) {
            gst(&d.cand_count[i], 0);
            gst(&d.cand_kept[i], 0);
            gst(&d.grp_w[i], 0);
        }
        for (int i = t; i < d.max_groups * d.G; i += ts) gst(&d.jfill[i], 0);
        if (t < ST_COUNT && t != ST_SATURATE && t != ST_BADPOS) gst(&d.status[t], 0);
        // guard partials past this grid
        if (bx == 0)
            for (int k = gridDim.x + threadIdx.x; k < guard_partials(d); k += blockDim.x) gst(&d.disp[k], 0.0);
    }
    const int wid = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int lane = threadIdx.x & 63;
    const int R = WIDE ? 2 : 64 / M, A = 64 / R;  // lanes per atom, slots per wave
    const int a = lane & (A - 1), r = lane / A;
    const int LM = M == 8 ? 3 : M == 4 ? 2 : 0;
    // the wave's slots, and of the lane's slot: its cluster's size, row ranges and
    // atom, and the frame of the staging
    const int w0 = (bx * 4 + wid) * A;
    int nr_l, it0, it1, js0, js1, atom_l;
    int wa[3];
    double ref[3];
    auto load_slot = [&](int base) {
        const int slot = min(base + a, max_slots - 1), cl = slot >> LM, g = cl / kGroup;
        nr_l = gld(&nreal_p[cl]);
        it0 = gld(&item_start[g]);
        it1 = gld(&item_start[g + 1]);
        js0 = gld(&jstart[cl]);
        js1 = gld(&jstart[cl + 1]);
        atom_l = gld(&slot_atom[slot]);
        if (NEXT == 2)
            for (int c = 0; c < 3; ++c) {
                wa[c] = gld(&wrap_p[3 * slot + c]);
                ref[c] = gld(&ref_p[3 * g + c]);
            }
    };
    // (in bounds whatever the counts, which are loaded together with them)
    load_slot(w0);
    // partial rows written by the force kernel: a list whose build ran out of
    // capacity has none (its offsets may point past the partial arrays, so the
    // row ranges below are clamped to what exists)
    const int n_it = gld(n_items_p), ent_w = __builtin_amdgcn_readfirstlane(gld(n_ent_p));
    const int n_en = ent_w ^ (ent_w >> 31);  // (~ of it marks a capacity exceeded)
    const int n_cl = __builtin_amdgcn_readfirstlane(gld(n_groups_p)) * kGroup;
    const int nb = cluster_blocks(n_cl);           // kinetic-energy partials
    const int stride = nb * 4 * M;                 // slots per pass of all waves
    const int part = WIDE ? bx * 4 + wid : bx;
    const bool idle = WIDE ? bx * 4 >= nb : bx >= nb;  // (the whole block)
    if (idle) {
        if (KICK && ke && (WIDE ? threadIdx.x < 4 : threadIdx.x == 0)) {
            const int p = WIDE ? bx * 4 + (int)threadIdx.x : bx;
            if (p < kKeBlocks) gst(&d.ke_part[p], 0.0);
        }
        if (NEXT == 1 && threadIdx.x == 0) gst(&d.disp[bx], 0.0);
        if (FMAX && threadIdx.x == 0) gst(&d.fmax_part[bx], 0.0);
        return;
    }
    bool bad = false;
    double kin = 0.0;
    // the largest squared displacement since the last build (NEXT 1) or squared
    // force (FMAX)
    double disp_m = 0.0;
    // (a wave of the last block may have no partial of its own)
    const int end = (!WIDE || part < nb) && !(KICK && held && ent_w < 0) ? n_cl * M : 0;
    for (int base = w0; base < end; base += stride) {
        // No branch or conditional load sits between the loads of a round trip, so
        // none waits on another.  Empty clusters (no partials are written for
        // them) and padding lanes get empty row ranges and no atom.
        if (base != w0) load_slot(base);
        const int slot = min(base + a, max_slots - 1), k = (slot >> LM) % kGroup, as = slot & (M - 1);
        const bool real = base + a < n_cl * M && as < nr_l;
        const int t0 = min(it0, n_it), t1 = real ? max(t0, min(it1, n_it)) : t0;
        const int j0 = min(js0, n_en), j1 = real ? max(j0, min(js1, n_en)) : j0;
        const bool fin = (r == 0) && real;
        const int atom = fin ? atom_l : -1;
        // the atom data are loaded for every lane (a clamped index), used by
        // the finishing lanes only
        const int ac = atom >= 0 ? atom : 0;
        double m = 1.0, v0[3] = {0.0, 0.0, 0.0}, x0[3] = {0.0, 0.0, 0.0}, xb[3] = {0.0, 0.0, 0.0}, qa = 0.0;
        if (KICK) {
            m = gld(&mass_p[ac]);
            for (int c = 0; c < 3; ++c) v0[c] = gld(&vp[3 * ac + c]);
            if (NEXT != 0)
                for (int c = 0; c < 3; ++c) x0[c] = gld(&xp[3 * ac + c]);
            if (NEXT == 1)
                for (int c = 0; c < 3; ++c) xb[c] = gld(&d.x_build[3 * ac + c]);
            if (NEXT == 2) qa = gld(&q_p[ac]);
        }
        float pf[3] = {0.f, 0.f, 0.f};
        if (pme_f)
            for (int c = 0; c < 3; ++c) pf[c] = gld(&pme_f[3 * ac + c]);
        long long sx = 0, sy = 0, sz = 0;
        float fx = 0.f, fy = 0.f, fz = 0.f;
        // one row space over the atom's i-partials, then its j-partials; rows go
        // in batches of kB per lane whose loads are all issued before any of them
        // is summed
        constexpr int kB = WIDE ? 8 : 4;
        const int ni = t1 - t0, nrow = ni + (j1 - j0);
        const size_t istride = (size_t)kGroup * M * 3;
        const float* ipl = ipart + (size_t)t0 * istride + ((size_t)k * M + as) * 3;
        const float* jpl = jpart + ((size_t)j0 * M + as) * 3;
        const size_t jstr = (size_t)M * 3;
        auto rows = [&](auto add) {
            for (int q0 = r; q0 < nrow; q0 += kB * R) {
                float v[kB][3];
#pragma unroll
                for (int u = 0; u < kB; ++u) {
                    // rows past the end read row q0 (loaded unconditionally, dropped)
                    const int qu = q0 + u * R, q = qu < nrow ? qu : q0;
                    const float* pr = q < ni ? ipl + (size_t)q * istride : jpl + (size_t)(q - ni) * jstr;
                    for (int c = 0; c < 3; ++c) {
                        const float w = gld(pr + c);
                        v[u][c] = qu < nrow ? w : 0.0f;
                    }
                }
                __builtin_amdgcn_sched_barrier(0);  // all loads of the batch first
#pragma unroll
                for (int u = 0; u < kB; ++u) add(v[u]);
            }
        };
        auto add_fixed = [&](const float w[3]) {
            bad = bad || !(fabsf(w[0]) < lim) || !(fabsf(w[1]) < lim) || !(fabsf(w[2]) < lim);
            sx += to_fixed(w[0], sc);
            sy += to_fixed(w[1], sc);
            sz += to_fixed(w[2], sc);
        };
        auto add_f32 = [&](const float w[3]) {
            fx += w[0];
            fy += w[1];
            fz += w[2];
        };
        if (f32)
            rows(add_f32);
        else
            rows(add_fixed);
        for (int o = A; o < 64; o <<= 1) {
            if (f32) {
                fx += __shfl_xor(fx, o, 64);
                fy += __shfl_xor(fy, o, 64);
                fz += __shfl_xor(fz, o, 64);
            } else {
                sx += __shfl_xor(sx, o, 64);
                sy += __shfl_xor(sy, o, 64);
                sz += __shfl_xor(sz, o, 64);
            }
        }
        if (atom >= 0) {
            // the reciprocal-space force of the atom joins the same sum
            if (pme_f) {
                if (f32)
                    add_f32(pf);
                else
                    add_fixed(pf);
            }
            float F[3];
            if (f32) {
                F[0] = fx;
                F[1] = fy;
                F[2] = fz;
                bad = bad || !(fabsf(fx) <= 3.4e38f) || !(fabsf(fy) <= 3.4e38f) || !(fabsf(fz) <= 3.4e38f);
            } else {
                F[0] = (float)((double)sx * fx_inv);
                F[1] = (float)((double)sy * fx_inv);
                F[2] = (float)((double)sz * fx_inv);
            }
            for (int c = 0; c < 3; ++c) gst(&fp[3 * atom + c], F[c]);
            if (KICK) {
                const double h = 0.5 * dt / m;
                double s2 = 0.0;
                double vn[3];
                for (int c = 0; c < 3; ++c) {
                    vn[c] = open ? v0[c] : fma(h, (double)F[c], v0[c]);
                    s2 += vn[c] * vn[c];
                }
                kin += 0.5 * m * s2;
                if (NEXT == 0) {
                    for (int c = 0; c < 3; ++c) gst(&vp[3 * atom + c], vn[c]);
                } else {
                    double xn[3];
                    if (NEXT == 1)  // a rebuild step follows: keep the full step
                        for (int c = 0; c < 3; ++c) {
                            gst(&d.x_bak[3 * atom + c], x0[c]);
                            gst(&d.v_bak[3 * atom + c], vn[c]);
                        }
                    for (int c = 0; c < 3; ++c) {
                        const double v2 = fma(h, (double)F[c], vn[c]);
                        gst(&vp[3 * atom + c], v2);
                        xn[c] = fma(dt, v2, x0[c]);
                        gst(&xp[3 * atom + c], xn[c]);
                    }
                    if (NEXT == 1) {  // (the same operations as k_build_clear)
                        double s2 = 0.0;
                        for (int c = 0; c < 3; ++c) {
                            const double dd = xn[c] - xb[c];
                            s2 += dd * dd;
                            gst(&d.x_build[3 * atom + c], xn[c]);
                        }
                        disp_m = (s2 > disp_m || s2 != s2) ? s2 : disp_m;  // NaN wins
                    }
                    if (NEXT == 2) {
                        float4 p;
                        stage_pos(d, xn, wa, ref, p);
                        p.w = (float)(qa * (double)d.qscale);
                        gst(&xq[slot], p);
                    }
                }
            } else if (FMAX) {
                const double fx = F[0], fy = F[1], fz = F[2];
                const double f2 = fma(fz, fz, fma(fy, fy, fx * fx));
                disp_m = (f2 > disp_m || f2 != f2) ? f2 : disp_m;  // NaN wins
            }
        }
    }
    if (bad) atomicOr(&d.status[ST_SATURATE], 1);
    __shared__ double sh[4];
    if (NEXT == 1 || FMAX) {
        // over the block (NaN wins)
        for (int o = 1; o < 64; o <<= 1) {
            const double u = __shfl_xor(disp_m, o, 64);
            disp_m = (u > disp_m || u != u) ? u : disp_m;
        }
        __shared__ double shd[4];
        if (lane == 0) shd[wid] = disp_m;
        __syncthreads();
        if (threadIdx.x == 0) {
            double mm = shd[0];
            for (int w = 1; w < 4; ++w) mm = (shd[w] > mm || shd[w] != shd[w]) ? shd[w] : mm;
            if (FMAX) gst(&d.fmax_part[bx], mm);
            else gst(&d.disp[bx], mm);
        }
    }
    if (!(KICK && ke)) return;
    // kinetic-energy partials in fixed order: the atoms of a cluster, then the four
    // clusters in pairs
    for (int o = 1; o < 64; o <<= 1) kin += __shfl_xor(kin, o, 64);
    if (WIDE) {
        if (lane == 0 && part < kKeBlocks) gst(&d.ke_part[part], kin);
        return;
    }
    if (lane == 0) sh[wid] = kin;
    __syncthreads();
    if (threadIdx.x == 0) gst(&d.ke_part[bx], (sh[0] + sh[1]) + (sh[2] + sh[3]));
}

static int atom_blocks(int max_atoms)
{
    int b = (max_atoms + 255) / 256;
    if (b > kKeBlocks) b = kKeBlocks;
    return b < 1 ? 1 : b;
}

hipError_t launch_stage(const SysDev* table, int n_sys, const Bounds& b, hipStream_t s, const int* flags,
                        bool clear_status)
{
    hipLaunchKernelGGL(k_stage, dim3((b.max_slots + 255) / 256, n_sys), dim3(256), 0, s, table, flags,
                       clear_status ? 1 : 0);
    return hipGetLastError();
}

hipError_t launch_state_copy(const SysDev* table, int n_sys, const Bounds& b, int mode, hipStream_t s)
{
    const int blocks = min(kKeBlocks, max(1, (3 * b.max_atoms + 255) / 256));
    hipLaunchKernelGGL(k_state_copy, dim3(blocks, n_sys), dim3(256), 0, s, table, mode);
    return hipGetLastError();
}

// R = 64/M and R = 2 (us): 4.4 and 4.8 at 2,744 atoms, 7.25 and 7.1 at 17,576, 7.4 and
// 6.9 at 24,389, 16.8 and 13.9 at 200,003, 94 and 77 at 1,000,000
constexpr int kWideSlots = 16384;
static bool gather_wide(const Bounds& b) { return b.all_m8 && b.total_slots > kWideSlots; }

static int gather_blocks(const Bounds& b)
{
    const int ncl = b.max_groups * kGroup;
    const int parts = max(1, min(kKeBlocks, (ncl + 3) / 4));
    return gather_wide(b) ? (parts + 3) / 4 : parts;
}

template <bool KICK, bool FMAX, int NEXT, bool ENER = false>
static void launch_gather(const SysDev* table, int n_sys, const Bounds& b, double dt, bool ke, bool open, bool held,
                          const int* flags, hipStream_t s, int ener_row = -1, double ener_step = 0.0)
{
    hipLaunchKernelGGL((gather_wide(b) ? k_gather<KICK, FMAX, NEXT, true, ENER>
                                       : k_gather<KICK, FMAX, NEXT, false, ENER>),
                       dim3(gather_blocks(b) + (ENER ? 1 : 0), n_sys), dim3(256), 0, s, table, dt, ke ? 1 : 0,
                       open ? 1 : 0, held ? 1 : 0, flags, ener_row, ener_step);
}

hipError_t launch_finalize(const SysDev* table, int n_sys, const Bounds& b, bool fp32, hipStream_t s,
                           const int* flags, bool ener, int trace_row, double step_value)
{
    (void)fp32;
    if (ener)
        launch_gather<false, false, 0, true>(table, n_sys, b, 0.0, false, false, false, flags, s, trace_row, step_value);
    else
        launch_gather<false, false, 0>(table, n_sys, b, 0.0, false, false, false, flags, s);
    return hipGetLastError();
}

// (a copy engine's or blit kernel's 192 bytes took 4.2 us and a longer call)
__global__ __launch_bounds__(64) void k_page_out(const int* __restrict__ from, int* pinned, int words)
{
    for (int k = threadIdx.x; k < words; k += 64)
        __hip_atomic_store(&pinned[k], gld(&from[k]), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
}

hipError_t launch_page_out(const int* from, int* pinned, int words, hipStream_t s)
{
    hipLaunchKernelGGL(k_page_out, dim3(1), dim3(64), 0, s, from, pinned, words);
    return hipGetLastError();
}

hipError_t launch_energy_reduce(const SysDev* table, int n_sys, int trace_row, bool with_ke,
                                double step_value, hipStream_t s)
{
    hipLaunchKernelGGL(k_energy_reduce, dim3(n_sys), dim3(256), 0, s, table, trace_row,
                       with_ke ? 1 : 0, step_value);
    return hipGetLastError();
}

hipError_t launch_kick_drift(const SysDev* table, int n_sys, const Bounds& b, double dt, hipStream_t s)
{
    hipLaunchKernelGGL(k_kick_drift, dim3(atom_blocks(b.max_atoms), n_sys), dim3(256), 0, s, table, dt);
    return hipGetLastError();
}

hipError_t launch_kick_drift_stage(const SysDev* table, int n_sys, const Bounds& b, double dt, hipStream_t s)
{
    hipLaunchKernelGGL(k_kick_drift_stage, dim3((b.max_slots + 255) / 256, n_sys), dim3(256), 0, s, table, dt);
    return hipGetLastError();
}

hipError_t launch_gather_kick(const SysDev* table, int n_sys, const Bounds& b, double dt, bool ke, hipStream_t s,
                              int next, bool open, bool held)
{
    if (next == 2)
        launch_gather<true, false, 2>(table, n_sys, b, dt, ke, open, held, nullptr, s);
    else if (next == 1)
        launch_gather<true, false, 1>(table, n_sys, b, dt, ke, open, held, nullptr, s);
    else
        launch_gather<true, false, 0>(table, n_sys, b, dt, ke, open, held, nullptr, s);
    return hipGetLastError();
}

hipError_t launch_item_prefix(const SysDev* table, int n_sys, int* item_prefix, hipStream_t s, const int* flags)
{
    hipLaunchKernelGGL(k_item_prefix, dim3(1), dim3(64), 0, s, table, n_sys, item_prefix, flags);
    return hipGetLastError();
}

hipError_t launch_prune_guard_k(const SysDev* table, int n_atoms, int check, int cur, int fold, hipStream_t s)
{
    hipLaunchKernelGGL(k_prune_guard, dim3(atom_blocks(n_atoms)), dim3(256), 0, s, table, check, cur, fold);
    return hipGetLastError();
}

int prune_guard_arg(int n_atoms, int cur, int fold)
{
    return cur | (fold ? 2 : 0) | atom_blocks(n_atoms) << 2;
}

hipError_t launch_gather_fmax(const SysDev* table, const Bounds& b, hipStream_t s)
{
    launch_gather<false, true, 0>(table, 1, b, 0.0, false, false, false, nullptr, s);
    return hipGetLastError();
}

hipError_t launch_minimize_move(const SysDev* table, const Bounds& b, double max_disp, double f_tol, int it, int* done,
                                unsigned long long* seen, hipStream_t s)
{
    hipLaunchKernelGGL(k_minimize_move, dim3((b.max_slots + 255) / 256), dim3(256), 0, s, table, max_disp, f_tol,
                       gather_blocks(b), it, done, seen);
    return hipGetLastError();
}

}  // namespace nbi
