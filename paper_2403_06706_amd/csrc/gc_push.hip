// gc_push.hip -- the hot path: advance particles by a chunk of steps.
//
// One particle per lane.  Its state is loaded into registers once per launch,
// advanced for n_steps steps of the third-order predictor-corrector (Eqs. 5-6)
// with hard-sphere scattering (Eqs. 9-10), and stored once.  Each step makes
// two trilinear gathers of the 12 field components (at X^n and at X*), a third
// one on bootstrap steps (injection and after a collision).
#include <hip/hip_runtime.h>

#include "gc_device.h"
#include "gc_launch.h"
#include "gc_step.h"

namespace gc {

// Forms of the push (bitwise identical in their results):
//   kFormLane   one lane per particle; a cell's nodes stay in its registers, so the loads of
//               a gather are made on a change of cell only, all in flight at once;
//   kFormTail   the same, below the tail threshold (the steps are counted apart);
//   kFormPair   two lanes per particle, six components each, else as the next; counted
//               as kFormTail;
//   kFormQuad   four lanes per particle (an aligned quad), FP32 and FP64 fields: each lane
//               keeps and interpolates three of the twelve components, the quad shares the
//               results, all four run the rest of the step on identical values, lane gl = 0
//               writes.
enum { kFormLane = 0, kFormTail = 1, kFormQuad = 2, kFormPair = 3 };
template <int FORM> constexpr uint32_t kGroup = FORM == kFormQuad ? 4 : FORM == kFormPair ? 2 : 1;   // lanes per particle
template <int FDT, int G> struct FormCell { using type = GroupCell<FDT, G>; };
template <int FDT> struct FormCell<FDT, 1> { using type = LaneCell<FDT>; };
template <int FDT, int MODE> constexpr bool kHasQuad = MODE != 2 && FDT != GC_F16;

// MODE 0: the reduced equations, no rebirth, centres at rest.  MODE 1: also
// rebirth and scattering in the wind frame (Sect. 3 and 3.3); a separate
// instantiation because the out-of-line rebirth raises the register count of
// the FP32 forms.  MODE 2: also the full Eqs. 1-2 (the extra node array is
// gathered with the field's stencil at each evaluation; no quad form).
// TAME: the field is tame (FieldDev::tame), so the gathers skip their
// finiteness test (compiled out; a run-time branch around it measured slower,
// and in the quad form no faster than the test).
template <int PREC, int FDT, int MODE, int FORM = kFormLane, bool TAME = false>
__device__ __forceinline__ uint32_t advance_slot(const PushArgs &a, uint32_t slot, uint32_t gl = 0) {
    constexpr bool EXT = MODE >= 1;
    constexpr bool FULL = MODE == 2;
    using R = typename PrecT<PREC>::R;
    using A = typename PrecT<PREC>::A;
    constexpr bool kKahan = PrecT<PREC>::kKahan;
    // The particle of this slot is read from sr at ls and written to st at
    // slot: the same place, or (a reorder's permutation applied by the push)
    // its place in the other state buffer.  In place, a stopped particle costs
    // one load.  Moved, every field of the step is loaded at once, one round
    // trip after the permutation's.  What only rare events or the final store
    // need (id, ensemble index, global index, birth) is read there.
    const SoA &st = a.st, &sr = a.src;
    const bool moved = a.perm != nullptr;
    const uint32_t ls = moved ? a.perm[slot] : slot;
    if (!moved && sr.status[ls] != GC_ACTIVE) return 0;
    uint32_t status = sr.status[ls], flags = sr.flags[ls], k = sr.k[ls], step0 = sr.step[ls];
    uint32_t eidx = sr.ens[ls];
    double r0 = sr.r[ls], th0 = sr.th[ls], ph0 = sr.ph[ls], u0 = sr.u[ls], t0 = sr.t[ls];
    double fr0 = sr.fr[ls], fth0 = sr.fth[ls], fph0 = sr.fph[ls], fu0 = sr.fu[ls];
    double mu0 = sr.mu[ls], dtp0 = sr.dtp[ls], s0 = sr.s[ls], ell0 = sr.ell[ls];
    double cr0 = 0, cth0 = 0, cph0 = 0, cu0 = 0, ct0 = 0;
    if (kKahan) { cr0 = sr.cr[ls]; cth0 = sr.cth[ls]; cph0 = sr.cph[ls]; cu0 = sr.cu[ls]; ct0 = sr.ct[ls]; }
    // The empty statements below take every loaded value, so the loads are all
    // issued before the status test (else the compiler issues the status load
    // alone, and the others after its round trip).
#define GC_LOADED(x) asm volatile("" : "+v"(x))
    GC_LOADED(status); GC_LOADED(flags); GC_LOADED(k); GC_LOADED(step0); GC_LOADED(eidx);
    GC_LOADED(r0); GC_LOADED(th0); GC_LOADED(ph0); GC_LOADED(u0); GC_LOADED(t0);
    GC_LOADED(fr0); GC_LOADED(fth0); GC_LOADED(fph0); GC_LOADED(fu0);
    GC_LOADED(mu0); GC_LOADED(dtp0); GC_LOADED(s0); GC_LOADED(ell0);
    if (kKahan) { GC_LOADED(cr0); GC_LOADED(cth0); GC_LOADED(cph0); GC_LOADED(cu0); GC_LOADED(ct0); }
#undef GC_LOADED
    // (moved: every slot is active, a reorder puts the active particles first)
    if (status != GC_ACTIVE) return 0;
    eidx = min(eidx, (uint32_t)(kMaxEnsembles - 1));
    const EnsDev &e = a.ens[eidx];
    A X0 = (A)r0, X1 = (A)th0, X2 = (A)ph0, X3 = (A)u0;
    A T = (A)t0;
    A c0 = (A)cr0, c1 = (A)cth0, c2 = (A)cph0, c3 = (A)cu0, cT = (A)ct0;
    R fp0 = (R)fr0, fp1 = (R)fth0, fp2 = (R)fph0, fp3 = (R)fu0;
    R mu = (R)mu0, s = (R)s0, ell = (R)ell0;
    const R qm = (R)e.qm, iqm = (R)e.iqm;
    const bool drift_free = e.drift_free != 0;
    const bool scatter = e.lambda > 0.0;
    const R vw = EXT ? (R)e.v_wind : (R)0;          // > 0: scattering centres move with the wind
    const R h = (R)a.dt;
    const double r_in = e.r_in, r_out = e.r_out, th_lo = a.f.th_lo, th_hi = a.f.th_hi;
    // Steps to take: the stop step (max_steps, tested after a step) may come first.
    uint32_t todo = (uint32_t)a.n_steps;
    uint32_t at_end = GC_ACTIVE;                    // status after todo steps
    if (e.max_steps > 0) {
        const int64_t left = max(e.max_steps - (int64_t)step0, (int64_t)1);
        if (left <= (int64_t)todo) { todo = (uint32_t)left; at_end = GC_FINISHED; }
    }
    // Step ratio of the first step; every later one follows a step of size h (or
    // a bootstrap, whose ratio is 1).
    R tau = (R)dtp0 == h ? (R)1 : h * rcp_nr((R)dtp0);
    // Resident cells: 96 registers of nodes per lane for FP32 fields, 48 FP16, 192
    // FP64, and 168, 96 and 336 with the extra array of the full equations; a half in
    // the pair form and a quarter in the quad form.
    // Bound when every gather loaded its stencil: vector issue 0.70 and the gather
    // paths (TA/TD) 0.68/0.73 busy, both evaluations of a step loading 24 x 16 bytes a
    // lane (FP64 fields 48).  An electron crosses a cell in about ten steps, so now some
    // lanes of a wavefront load at X*, and seldom any at X^n.  Per 64-step launch (FP64
    // on an FP32 256x128x256 field): 2^20 electrons 2.40 -> 1.91 ms, 1,000 reborn
    // electrons in the quad form 2.09 -> 1.71 us a step; 300,007 in FP32 arithmetic 0.61
    // -> 0.39 ms; full equations, 150,000: 0.88 -> 0.72 ms.
    using Cell = typename FormCell<FDT, kGroup<FORM>>::type;
    CellPos<R> at;
    Cell cell;
    [[maybe_unused]] typename std::conditional<FULL, LaneCell<FDT, 9>, NoCell>::type xcell;
    // move to a point; false where it cannot be evaluated
    auto seek = [&](R x, R t, R p) -> bool { return cell_seek<FDT, R>(a.f, x, t, p, gl, at, cell, a.fx, xcell); };
    // the components there (and those of the extra array); false for a non-finite one
    auto value = [&](R g[12]) -> bool {
        cell.template value<0, 12, R>(a.f, at, gl, g);
        return TAME || finite_sum<12>(g);
    };
    auto xvalue = [&](R xg[12]) -> bool {
        if constexpr (FULL) {
            xcell.template value<0, 9, R>(a.fx, at, gl, xg);
            return finite_sum<9>(xg);
        }
        return true;
    };

    // A bootstrap step needs a third evaluation, F^{n-1} at X^n - dt F^n.  A lane
    // that bootstraps makes it at the X^n site of the next turn of the loop (its
    // own step ends one turn later than the others'): in the same turn, every
    // bootstrap would cost its wavefront an evaluation.  F^n and its speed are
    // kept in Fb and vpb until then.
    constexpr uint32_t kBack = GC_FLAG_PENDING << 1;   // internal: this lane is about to evaluate F^{n-1}
    static_assert(kBack < (1u << GC_FLAG_GEN_SHIFT), "flag bit in use");
    R Fb[4] = {0, 0, 0, 0}, vpb = 0;
    uint32_t done = 0;                              // steps taken
    do {
        // Rare events (collision, bootstrap, drift-free electrons, exit,
        // rebirth) stand in branches that the compiler places out of line: a
        // lone wavefront waits for its instructions after every taken branch.
        // A point that cannot be evaluated only marks the step as bad; what
        // follows runs on arbitrary values and is not committed.
        R Fn[4], Fs[4], vpn, vps;
        R px = (R)X0, pth = (R)X1, pph = (R)X2, pu = (R)X3;
        auto rhs_at = [&](R ir, R is, R u, R g[12], R xg[12], R F[4], R &vp) {
            if constexpr (FULL) gc_rhs_at<R, true>(ir, is, u, mu, qm, iqm, drift_free, g, F, vp, xg);
            else gc_rhs_at<R>(ir, is, u, mu, qm, iqm, drift_free, g, F, vp);
            if (EXT) vp = path_speed<R>(vp, g, vw);
        };
        if (rare((flags & kBack) != 0)) {
            // backward Euler start (Sect. 2.2)
            px = (R)X0 - h * Fb[0]; pth = (R)X1 - h * Fb[1]; pph = (R)X2 - h * Fb[2]; pu = (R)X3 - h * Fb[3];
        }
        bool bad = !seek(px, pth, pph);
        if (rare((flags & GC_FLAG_PENDING) != 0)) {
            // collision k+1 (Eqs. 9-10) at X^n: |p| kept, new pitch cosine and free path
            const CollisionDraw d = draw_collision(sr.id[ls], k + 1, flags >> GC_FLAG_GEN_SHIFT, e.seed, e.ensemble,
                                                   e.scatter_law, e.lambda);
            R g[12];
            if constexpr (TAME) cell.template value<0, 3, R>(a.f, at, gl, g);   // B alone
            else if (!bad) bad = !value(g);
            if (!bad) {
                const R mun = (R)d.mun;
                const R B = sqrt(g[0] * g[0] + g[1] * g[1] + g[2] * g[2]);
                R p2 = pu * pu + (R)2 * mu * B;                  // (p/m)^2, kept in the inertial frame
                R un;
                if (EXT && vw > (R)0) wind_collision<R>(pu, mu, B, g[0], vw, mun, un, p2);
                else un = mun * sqrt(p2);
                X3 = (A)un;
                c3 = 0;
                pu = (R)X3;
                mu = p2 * ((R)1 - mun * mun) / ((R)2 * B);
                ell = (R)d.ell;
                s = 0;
                k += 1;
                flags = (flags | GC_FLAG_BOOTSTRAP) & ~GC_FLAG_PENDING;
                if (a.log_depth > 0 && k <= (uint32_t)a.log_depth && gl == 0)
                    a.log[(size_t)sr.gid[ls] * a.log_depth + (k - 1)] = step0 + done;
            }
        }
        {   // X^n (or X^{n-1} of a bootstrap)
            const R ir = rcp_nr(px), is = rcp_nr(sin_0_pi(pth));
            R g[12], xg[12];
            bad |= !xvalue(xg);
            bad |= !value(g);
            rhs_at(ir, is, pu, g, xg, Fn, vpn);
        }
        bool go = true;
        if (rare((flags & GC_FLAG_BOOTSTRAP) != 0 && !bad)) {
            if (!(flags & kBack)) {
                Fb[0] = Fn[0]; Fb[1] = Fn[1]; Fb[2] = Fn[2]; Fb[3] = Fn[3];
                vpb = vpn;
                flags |= kBack;
                go = false;
            } else {
                fp0 = Fn[0]; fp1 = Fn[1]; fp2 = Fn[2]; fp3 = Fn[3];
                Fn[0] = Fb[0]; Fn[1] = Fb[1]; Fn[2] = Fb[2]; Fn[3] = Fb[3];
                vpn = vpb;
                tau = (R)1;
                flags &= ~(uint32_t)(GC_FLAG_BOOTSTRAP | kBack);
            }
        }
        if (go) {
            {   // predictor X*, Eq. 5
                const R wn = (R)1 + (R)0.5 * tau, wq = (R)0.5 * tau;
                const R d0 = h * (wn * Fn[0] - wq * fp0), d1 = h * (wn * Fn[1] - wq * fp1);
                const R d2 = h * (wn * Fn[2] - wq * fp2), d3 = h * (wn * Fn[3] - wq * fp3);
                if (kKahan) {
                    px = (R)(X0 + (d0 - c0)); pth = (R)(X1 + (d1 - c1)); pph = (R)(X2 + (d2 - c2)); pu = (R)(X3 + (d3 - c3));
                } else {
                    px = (R)(X0 + (A)d0); pth = (R)(X1 + (A)d1); pph = (R)(X2 + (A)d2); pu = (R)(X3 + (A)d3);
                }
                bad |= !seek(px, pth, pph);
                // 1/r and 1/sin(th) while a new cell's nodes are on their way (the empty
                // statement keeps the compiler from moving them to their use)
                R ir = rcp_nr(px), is = rcp_nr(sin_0_pi(pth));
                asm volatile("" : "+v"(ir), "+v"(is));
                R g[12], xg[12];
                bad |= !xvalue(xg);
                bad |= !value(g);
                rhs_at(ir, is, pu, g, xg, Fs, vps);
            }
            if (rare(bad)) {
                status = GC_NONFINITE;
                todo = 0;
            } else {
                // corrector, Eq. 6: dt/(6(1+tau)) [(1+tau)(3+tau) F^n + (3+2 tau) F* - tau^2 F^{n-1}]
                R cf = h * (R)(1.0 / 12.0);
                if (rare(tau != (R)1)) cf = h * rcp_nr((R)6 * ((R)1 + tau));
                const R an = ((R)1 + tau) * ((R)3 + tau), as = (R)3 + (R)2 * tau, ap = tau * tau;
                const R e0 = cf * (an * Fn[0] + as * Fs[0] - ap * fp0);
                const R e1 = cf * (an * Fn[1] + as * Fs[1] - ap * fp1);
                const R e2 = cf * (an * Fn[2] + as * Fs[2] - ap * fp2);
                const R e3 = cf * (an * Fn[3] + as * Fs[3] - ap * fp3);
                tau = (R)1;
                // path along the field line over the step (trapezoid of |v_par|), Eq. 9
                const R s1 = s + (R)0.5 * (fabs(vpn) + fabs(vps)) * h;
                s = scatter ? s1 : s;
                flags |= scatter && s >= ell ? (uint32_t)GC_FLAG_PENDING : 0u;
                if (kKahan) {
                    kahan_add(X0, c0, (A)e0); kahan_add(X1, c1, (A)e1);
                    kahan_add(X2, c2, (A)e2); kahan_add(X3, c3, (A)e3);
                    kahan_add(T, cT, (A)h);
                } else {
                    X0 += (A)e0; X1 += (A)e1; X2 += (A)e2; X3 += (A)e3;
                    T += (A)a.dt;
                }
                fp0 = Fn[0]; fp1 = Fn[1]; fp2 = Fn[2]; fp3 = Fn[3];
                done += 1;
                const double r = (double)X0, th = (double)X1;
                const bool inside = r >= r_in && r <= r_out && th >= th_lo && th <= th_hi;   // false for non-finite r, th
                if (rare(!(inside && isfinite(X2) && isfinite(X3)))) {
                    if (!(isfinite(X0) && isfinite(X1) && isfinite(X2) && isfinite(X3))) {
                        status = GC_NONFINITE;
                        todo = 0;
                    } else if (!EXT || (int64_t)(step0 + done) >= e.rebirth_steps) {
                        status = GC_EXITED;
                        todo = 0;
                    } else {
                        // rebirth (continuous injection, Sect. 3): the next generation starts
                        // from the injection state with its own generator stream
                        const uint32_t gen = (flags >> GC_FLAG_GEN_SHIFT) + 1;
                        const BirthState b = rebirth_state<FDT>(a.fdev, a.ens + eidx, sr.id[ls], gen);
                        at = CellPos<R>();           // another cell: the nodes need not be kept over the call
                        cell.drop();
                        if constexpr (FULL) xcell.drop();
                        X0 = (A)b.r; X1 = (A)b.th; X2 = (A)b.ph; X3 = (A)b.u;
                        c0 = 0; c1 = 0; c2 = 0; c3 = 0; cT = 0; T = 0;
                        fp0 = 0; fp1 = 0; fp2 = 0; fp3 = 0;
                        mu = (R)b.mu; s = 0; ell = (R)b.ell;
                        k = 0;
                        flags = GC_FLAG_BOOTSTRAP | (gen << GC_FLAG_GEN_SHIFT);
                        if (gl == 0) {
                            st.birth[slot] = step0 + done;
                            if (a.log_depth > 0) {
                                uint32_t *row = a.log + (size_t)sr.gid[ls] * a.log_depth;
                                for (int j = 0; j < a.log_depth; ++j) row[j] = 0xFFFFFFFFu;
                            }
                        }
                        if (b.status != GC_ACTIVE) {
                            status = b.status;
                            todo = 0;
                        }
                    }
                }
            }
        }
    } while (done < todo);
    if (gl != 0) return 0;
    if (status == GC_ACTIVE) status = at_end;
    st.r[slot] = (double)X0; st.th[slot] = (double)X1; st.ph[slot] = (double)X2; st.u[slot] = (double)X3;
    if (kKahan) {
        st.cr[slot] = (double)c0; st.cth[slot] = (double)c1; st.cph[slot] = (double)c2;
        st.cu[slot] = (double)c3; st.ct[slot] = (double)cT;
    }
    st.t[slot] = (double)T;
    st.fr[slot] = (double)fp0; st.fth[slot] = (double)fp1; st.fph[slot] = (double)fp2; st.fu[slot] = (double)fp3;
    st.mu[slot] = (double)mu; st.s[slot] = (double)s; st.ell[slot] = (double)ell;
    // step size of the last step; 0 for a generation that has not taken one
    const uint32_t flags0 = sr.flags[ls];
    const bool reborn = EXT && (flags >> GC_FLAG_GEN_SHIFT) != (flags0 >> GC_FLAG_GEN_SHIFT);
    const bool fresh = reborn && st.birth[slot] == step0 + done;
    st.dtp[slot] = fresh ? 0.0 : done > 0 ? (double)h : (double)(R)sr.dtp[ls];
    st.k[slot] = k; st.status[slot] = status; st.step[slot] = step0 + done;
    if (moved) {
        st.id[slot] = sr.id[ls]; st.ens[slot] = sr.ens[ls]; st.gid[slot] = sr.gid[ls];
        if (!reborn) st.birth[slot] = sr.birth[ls];
    }
    st.flags[slot] = flags & ~kBack;
    return done;
}

// Grid form: one slot per G lanes.  Workgroups are dispatched round-robin over
// the 8 XCDs.  Only the first ceil(G n_active / blockDim) workgroups have work
// (active particles fill a prefix of the slots after reordering); the remap
// gives each XCD a contiguous range of that prefix, so that (with cell-sorted
// slots) its L2 holds the field cells of its own particles, and every XCD gets
// an equal share however small the active prefix is.
template <int PREC, int FDT, int MODE, int FORM, bool TAME = false>
__device__ __forceinline__ void push_grid(const PushArgs &a) {
    constexpr uint32_t G = kGroup<FORM>;
    const uint32_t n = *a.n_active;
    const uint32_t per_block = blockDim.x / G;                // particles per workgroup
    const uint32_t nb = (n + per_block - 1) / per_block, b = blockIdx.x;
    if (b >= nb) return;
    const uint32_t q = nb >> 3, rem = nb & 7u, xcd = b & 7u, pos = b >> 3;
    const uint32_t lb = (xcd < rem ? xcd * (q + 1) : rem * (q + 1) + (xcd - rem) * q) + pos;
    const uint32_t slot = lb * per_block + threadIdx.x / G;
    uint32_t taken = 0;
    if (slot < n) taken = advance_slot<PREC, FDT, MODE, FORM, TAME>(a, slot, threadIdx.x % G);
    count_steps(a, taken);
}

// One lane per particle: at most 256 registers (two wavefronts per SIMD); the
// larger cells of FP64 fields and of the full equations take the 512 of one.
template <int FDT, int MODE> constexpr int kLaneWaves = MODE == 2 || FDT == GC_F64 ? 1 : 2;

template <int PREC, int FDT, int MODE, bool TAME>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(kLaneWaves<FDT, MODE>))) void k_push(PushArgs a) {
    push_grid<PREC, FDT, MODE, kFormLane, TAME>(a);
}

// For fewer active particles than fill the machine (tail_lanes): a wavefront's
// step time is then its chain of instructions and memory round trips; the quad
// form spreads the particles over four times as many wavefronts (and compute
// units) and interpolates a quarter of the values per lane.
template <int PREC, int FDT, int MODE, bool TAME>
__global__ __launch_bounds__(256) void k_push_quad(PushArgs a) {
    push_grid<PREC, FDT, MODE, kFormQuad, TAME>(a);
}

// The same for a few more particles, two lanes each.  512 steps of 20,011 electrons
// in FP64 on the 256x128x256 FP32 field 1.46 -> 1.21 ms: two thirds of the values
// converted, and half of the products, per lane of what was one wavefront.
template <int PREC, int FDT, int MODE, bool TAME>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(2))) void k_push_pair(PushArgs a) {
    push_grid<PREC, FDT, MODE, kFormPair, TAME>(a);
}

// Persistent forms: a fixed grid pulls tiles of consecutive slots from an
// atomic counter until the tiles run out (every workgroup reaches the exit).
// A tile holds a.tile particles, fewer when the live prefix would not give
// every workgroup a tile (down to one particle per thread, or per quad), so
// that a thinning population stays spread over the machine instead of
// queueing behind few workgroups.
//
// With a tail threshold T = a.tail > 0 each chunk launches the one-lane kernel
// and the quad kernel in turn, and the live count on the device (written by the
// reorder) selects the one that works, the other returning at once: the quad
// form below quad_limit.  The choice is made on the device so that a captured
// graph follows the count without a host read-back.  Steps are counted per form
// (a.steps_done + form), the one-lane form's below T under kFormTail.
template <int PREC, int FDT, int MODE, int FORM, bool TAME = false>
__device__ __forceinline__ void push_persistent(const PushArgs &a) {
    __shared__ uint32_t s_tile;
    const uint32_t n = *a.n_active;
    const uint32_t T = a.tail;
    const uint32_t quad = quad_limit(T, PREC == GC_PREC_F64, FDT, MODE == 2);
    if (FORM == kFormQuad ? n >= quad : n < quad) return;
    constexpr uint32_t G = kGroup<FORM>;
    const uint32_t per = blockDim.x / G;                       // particles per workgroup round
    const uint32_t share = ((n + gridDim.x - 1) / gridDim.x + per - 1) / per * per;
    const uint32_t tile = min(max((uint32_t)a.tile, per), max(per, share));
    const uint32_t ntiles = (n + tile - 1) / tile;
    uint32_t taken = 0;
    for (;;) {
        if (threadIdx.x == 0) s_tile = atomicAdd(a.queue, 1u);
        __syncthreads();
        const uint32_t t = s_tile;
        __syncthreads();
        if (t >= ntiles) break;
        const uint32_t end = min(n, (t + 1) * tile);
        for (uint32_t slot = t * tile + threadIdx.x / G; slot < end; slot += per)
            taken += advance_slot<PREC, FDT, MODE, FORM, TAME>(a, slot, threadIdx.x % G);
    }
    count_steps(a.steps_done + (FORM == kFormLane && n < T ? kFormTail : FORM), taken);
}

template <int PREC, int FDT, int MODE, bool TAME>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(kLaneWaves<FDT, MODE>)))
void k_push_persistent(PushArgs a) {
    push_persistent<PREC, FDT, MODE, kFormLane, TAME>(a);
}

template <int PREC, int FDT, int MODE, bool TAME>
__global__ __launch_bounds__(256) void k_push_persistent_quad(PushArgs a) {
    push_persistent<PREC, FDT, MODE, kFormQuad, TAME>(a);
}

template <int PREC, int FDT, int MODE, bool TAME>
static hipError_t launch_rt(const PushArgs &a, int block, bool persistent, int form, int grid_blocks, hipStream_t s,
                           LaunchEvents ev) {
    constexpr bool kQuad = kHasQuad<FDT, MODE>;
    if (persistent) {
        const bool quad = kQuad && a.tail > 0;
        launch_timed((k_push_persistent<PREC, FDT, MODE, TAME>), dim3(grid_blocks), dim3(block), s, ev.start,
                     quad ? nullptr : ev.stop, a);
        if constexpr (kQuad)
            if (quad)   // 256-thread workgroups (64 particles per round), as the grid quad form
                launch_timed((k_push_persistent_quad<PREC, FDT, MODE, TAME>), dim3((uint32_t)grid_blocks * block / 256),
                             dim3(256), s, nullptr, ev.stop, a);
        return hipGetLastError();
    }
    const uint32_t nb = (a.n_slots + block - 1) / block;
    if (nb == 0) {
        if (ev.start) (void)hipEventRecord(ev.start, s);
        if (ev.stop) (void)hipEventRecord(ev.stop, s);
        return hipGetLastError();
    }
    if constexpr (kQuad) {
        if (form == kFormPair) {
            const uint32_t pb = (2 * a.n_slots + 255) / 256;
            launch_timed((k_push_pair<PREC, FDT, MODE, TAME>), dim3(pb), dim3(256), s, ev.start, ev.stop, a);
            return hipGetLastError();
        }
        if (form == kFormQuad) {
            // 256-thread workgroups whatever the block size (64 particles each;
            // measured faster for this form than 64 threads)
            const uint32_t qb = (4 * a.n_slots + 255) / 256;
            launch_timed((k_push_quad<PREC, FDT, MODE, TAME>), dim3(qb), dim3(256), s, ev.start, ev.stop, a);
            return hipGetLastError();
        }
    }
    launch_timed((k_push<PREC, FDT, MODE, TAME>), dim3(nb), dim3(block), s, ev.start, ev.stop, a);
    return hipGetLastError();
}

// The tame instantiations (FieldDev::tame) for the reduced equations; the
// full equations test every gather (their extra node array is not scanned).
template <int PREC, int FDT, int MODE>
static hipError_t launch_r(const PushArgs &a, int block, bool persistent, int form, int grid_blocks, hipStream_t s,
                           LaunchEvents ev) {
    if constexpr (MODE != 2)
        if (a.f.tame) return launch_rt<PREC, FDT, MODE, true>(a, block, persistent, form, grid_blocks, s, ev);
    return launch_rt<PREC, FDT, MODE, false>(a, block, persistent, form, grid_blocks, s, ev);
}

template <int PREC, int FDT>
static hipError_t launch_t(const PushArgs &a, int block, bool persistent, int form, int grid_blocks, hipStream_t s,
                           LaunchEvents ev) {
    switch (a.mode) {
        case 0: return launch_r<PREC, FDT, 0>(a, block, persistent, form, grid_blocks, s, ev);
        case 1: return launch_r<PREC, FDT, 1>(a, block, persistent, form, grid_blocks, s, ev);
        default: return launch_r<PREC, FDT, 2>(a, block, persistent, form, grid_blocks, s, ev);
    }
}

template <int PREC>
static hipError_t launch_p(const PushArgs &a, int block, bool persistent, int form, int grid_blocks, hipStream_t s,
                           LaunchEvents ev) {
    switch (a.f.dtype) {
        case GC_F64: return launch_t<PREC, GC_F64>(a, block, persistent, form, grid_blocks, s, ev);
        case GC_F32: return launch_t<PREC, GC_F32>(a, block, persistent, form, grid_blocks, s, ev);
        case GC_F16: return launch_t<PREC, GC_F16>(a, block, persistent, form, grid_blocks, s, ev);
    }
    return hipErrorInvalidValue;
}

hipError_t launch_push(const PushArgs &a, int precision, int block, bool persistent, int form, int grid_blocks,
                       hipStream_t s, LaunchEvents ev) {
    switch (precision) {
        case GC_PREC_F64: return launch_p<GC_PREC_F64>(a, block, persistent, form, grid_blocks, s, ev);
        case GC_PREC_F32_ACC64: return launch_p<GC_PREC_F32_ACC64>(a, block, persistent, form, grid_blocks, s, ev);
        case GC_PREC_F32_KAHAN: return launch_p<GC_PREC_F32_KAHAN>(a, block, persistent, form, grid_blocks, s, ev);
    }
    return hipErrorInvalidValue;
}

}  // namespace gc
