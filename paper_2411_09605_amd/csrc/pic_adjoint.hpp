// Device code of the adjoint (reverse-mode derivative) of an ESEC2 run, 1D-1V
// electrostatic, for the loss J = lw * sum_{n=1..N} W_E^n (W_E of section 5.1) with
// respect to the parameters of the initial condition.
//
// Reverse of one step n (state n -> n+1), with x*, v*, x^{n+1/2} and Gamma recomputed
// from the stored state of step n and the fields the forward pass B of that step built
// and kept (E*, E-bar, E^{n+1}):
//
//   R1: per particle, the adjoint of v-dagger from the adjoint of v^{n+1} through
//       v^{n+1} = Gamma v-dagger and Gamma = sqrt(1 + 2 num / den) (eq. (opt_solution);
//       a fallback particle has the constant Gamma = 1); deposit dt * vdagger_bar at
//       x^{n+1/2} into G1 (the adjoint of the averaged field E-bar).
//   R2: every workgroup forms the adjoint of E^{n+1} (from step n+1, the loss term
//       lw h E^{n+1} and G1 / 2) and from it the adjoint of the centred current,
//       jbar2 = -dt (lambda - mean lambda) (Ampere update with its mean removed); per
//       particle, the adjoints of x^{n+1/2}, v*, x^{n+1} and the predictor gather;
//       deposit dt/2 * vstar_bar at x* into G2 (the adjoint of E*).
//   R3: every workgroup forms jbar1 = -dt/2 (G2 - mean G2); per particle, the adjoints
//       of x* and of the predictor deposit; write the adjoint of (x^n, v^n).  The lead
//       workgroup stores the adjoint of E^n = lambda' + G1 / 2 + G2 for step n - 1; every
//       workgroup clears its share of the other parity's G2 (of G1 in R2).
//
// Gathers and deposits are the forward's (same stencils); their derivatives with
// respect to the particle position use the derivative of the B-spline weights.
#pragma once

#include "pic_device.hpp"

namespace pic {

constexpr int kAdjMaxModes = 16;
// Rows of the grids kept per forward step: E^n | j^{n,*} | j^{*,n+1/2} | E* | E-bar | E^{n+1}.
constexpr int kSaveRows = 6;

struct AdjParams {
    int32_t n_modes;
    int32_t nparam;        // n_modes + 2 (amplitudes, beam speed, beam spread)
    double k[kAdjMaxModes], alpha[kAdjMaxModes];
    double v_beam, v_spread;
    double lbw;            // loss_bar * lw * h: weight of E^{n+1} in the adjoint of E^{n+1}
};

struct AdjWork {
    double *ax, *av;       // [N_p] adjoint of the particle state
    double *lam[2];        // [N_g] adjoint of E^{n+1} from the later steps (by parity)
    double *G1[2], *G2[2]; // [nrep][N_g] deposits of R1, R2 (by parity, replicated)
    double *rhobar;        // [N_g] Gauss solve of the final lambda (see k_adj_rhobar)
    double *gpart;         // [nblocks][nparam] per-workgroup gradient partial sums
};

// Derivative of the B-spline weights with respect to x / h, on the stencil's nodes (first
// unchanged), from the particle's offset.
template <int ORDER> __device__ __forceinline__ Stencil<ORDER> dstencil_at(const Pos &p)
{
    Stencil<ORDER> s;
    if constexpr (ORDER == 2) {
        s.first = (int)(p.n - 1);
        s.w[0] = p.d - 0.5;
        s.w[1] = -2.0 * p.d;
        s.w[2] = 0.5 + p.d;
    } else {
        s.first = (int)p.n;
        s.w[0] = -1.0;
        s.w[1] = 1.0;
    }
    return s;
}

// Gamma and its branch: ok = the root is real (no fallback).  num2 = 2 num is formed as in
// the forward pass, but from a recomputed state that agrees with the forward run only to
// rounding (see adj_particle), and Gamma takes the whole quotient and root where the forward
// pass uses a Taylor series for small corrections: a particle whose radicand is within
// rounding of zero could take the other branch than in the forward run (the tests compare the
// fallback counts of the two; they agree).
// The derivative needs 1 / den and 1 / (2 Gamma) too, so the reciprocal and the reciprocal
// root are refined themselves (two Newton steps; Goldschmidt's iteration) and the quotient and
// the root are corrected with them, in place of three divisions and a square root (with the
// loop's other changes STAGE 4 21.9 -> 18.8 us, see k_adj_reverse).
__device__ __forceinline__ double adj_gamma(double num2, double den, double &rho, double &rden,
                                            double &half_inv, bool &ok)
{
    double y = __builtin_amdgcn_rcp(den);
    y = fma(y, fma(-den, y, 1.0), y);
    y = fma(y, fma(-den, y, 1.0), y);
    rden = y;
    rho = num2 * y;
    rho = fma(fma(-rho, den, num2), y, rho);
    if (__any(den < 1e-280)) {
        asm volatile("");              // (not to be computed beside the usual quotient)
        if (den < 1e-280) {
            rden = 1.0 / den;
            rho = num2 / den;
        }
    }
    const double rr = 1.0 + rho;
    ok = rr >= 0.0 && isfinite(rr);
    const double s = __builtin_amdgcn_rsq(rr);
    double root = rr * s, half = 0.5 * s;
    double e = fma(-half, root, 0.5);
    root = fma(root, e, root);
    half = fma(half, e, half);
    root = fma(fma(-root, root, rr), half, root);
    e = fma(-half, root, 0.5);
    half_inv = fma(half, e, half);     // 1 / (2 Gamma)
    if (!(rr > 0.0)) {
        root = 0.0;
        half_inv = 0.5 / root;         // (as the division by Gamma = 0 gives)
    }
    return ok ? root : 1.0;
}

// Everything a reverse pass needs about one particle.  STAGE 1: the adjoint of the
// averaged-field gather (ebar_b); 2: also the adjoint of the predictor gather (ehat_b)
// and the partial adjoints of x, v; 3: the complete adjoint of (x^n, v^n).
template <int ORDER, int STAGE>
struct AdjOut {
    Stencil<ORDER> ss, sh;
    Slots<ORDER> ns, nh;
    double ebar_b, ehat_b, xb, vb;
};

// A particle's place, its stencil and the stencil's slots.
template <int ORDER>
__device__ __forceinline__ Pos adj_place(Stencil<ORDER> &st, Slots<ORDER> &sl, double s, double scale, int ng)
{
    Pos p = locate<ORDER>(s, scale, 0.0);
    int b = (int)first_slot<ORDER>(p);
    if (first_slot<ORDER>(p) > (unsigned)(ng + 2 * kGhost - ORDER - 1))
        b = far_slot<ORDER>(p, ng);
    st = stencil_at<ORDER>(p);
#pragma unroll
    for (int k = 0; k <= ORDER; ++k)
        sl.n[k] = b + k;
    return p;
}

// es, eb: predictor and averaged fields; lt, g2: the adjoint of E^{n+1} and the deposits of
// R2, with their means (ghost-padded LDS tiles).  The current adjoints are affine in them,
// jbar2 = -dt (lt - mean) and jbar1 = -dt/2 (G2 - mean), and a spline's weights sum to one
// (those of its derivative to zero), so the gathers take lt and G2 themselves and the particle
// applies the rest: no second round over the grid.
// x, v: state n; axp, avp: adjoint of state n+1; q: w_p / h.
template <int ORDER, int STAGE>
__device__ __forceinline__ AdjOut<ORDER, STAGE> adj_particle(const Run &r, double x, double v,
                                                            double axp, double avp, double q,
                                                            const double *es, const double *eb,
                                                            const double *lt, double mean_l,
                                                            const double *g2, double mean_g)
{
    AdjOut<ORDER, STAGE> o;
    // forward recompute: the quantities of pass A / pass B, equal to theirs up to rounding
    // (the gathers here take the stencil weights, the passes the cell polynomials of
    // gather_poly; the derivative needs the weights anyway)
    const Pos ps = adj_place<ORDER>(o.ss, o.ns, fma(r.hdt, v, x), r.inv_h, r.ng);      // x*
    const double vs = fma(r.hdt, gather1<ORDER>(es, o.ss, o.ns), v);
    const double x1 = fma(r.dt, vs, x);
    const Pos ph = adj_place<ORDER>(o.sh, o.nh, x + x1, r.hinv_h, r.ng);               // x^{n+1/2}
    const double vd = fma(r.dt, gather1<ORDER>(eb, o.sh, o.nh), v);
    // num2 = 2 num = a2 b with a2 = 2 v* - (vd + v), b = vd - v
    const double a2 = fma(2.0, vs, -(vd + v)), b = vd - v;
    const double num2 = fma(a2, b, 0.0), den = fma(vd, vd, 0.0);
    double rho, rden, half_inv;
    bool ok;
    const double gam = adj_gamma(num2, den, rho, rden, half_inv, ok);

    // v^{n+1} = Gamma vd
    double vdb = gam * avp;
    const double gb = avp * vd;
    double numb = 0.0, denb = 0.0;              // adjoints of num2 and den
    if (ok) {
        numb = gb * half_inv * rden;
        denb = -rho * numb;
    }
    const double ab = numb * b, bb = numb * a2;  // adjoints of a2 and b
    double vsb = 2.0 * ab;
    vdb += -ab + bb + 2.0 * vd * denb;
    double vb = -ab - bb + vdb;                 // vd = v + dt Ebar_p
    o.ebar_b = r.dt * vdb;
    o.ehat_b = 0.0;
    o.xb = 0.0;
    o.vb = vb;
    if constexpr (STAGE >= 2) {
        // x^{n+1/2}: averaged-field gather and centred deposit
        const Stencil<ORDER> dh = dstencil_at<ORDER>(ph);
        const double xhb = r.inv_h * (o.ebar_b * gather1<ORDER>(eb, dh, o.nh)
                                      - r.dt * q * vs * gather1<ORDER>(lt, dh, o.nh));
        vsb = fma(-r.dt * q, gather1<ORDER>(lt, o.sh, o.nh) - mean_l, vsb);
        double x1b = axp + 0.5 * xhb;            // x^{n+1} = wrap(x1): a translation
        double xb = 0.5 * xhb + x1b;             // x1 = x + dt v*
        vsb = fma(r.dt, x1b, vsb);
        vb += vsb;                               // v* = v + dt/2 E-hat
        o.ehat_b = r.hdt * vsb;
        o.xb = xb;
        o.vb = vb;
        if constexpr (STAGE >= 3) {
            // x*: predictor gather and predictor deposit
            const Stencil<ORDER> ds = dstencil_at<ORDER>(ps);
            const double xsb = r.inv_h * (o.ehat_b * gather1<ORDER>(es, ds, o.ns)
                                          - r.hdt * q * v * gather1<ORDER>(g2, ds, o.ns));
            vb = fma(-r.hdt * q, gather1<ORDER>(g2, o.ss, o.ns) - mean_g, vb);
            o.xb = xb + xsb;
            o.vb = fma(r.hdt, xsb, vb);
        }
    }
    return o;
}

// The replica of the grid-adjoint deposits a workgroup adds into (replica stride ng).
__device__ __forceinline__ double *g_slot(double *G, int nrep, int ng)
{
    return G + (size_t)(blockIdx.x % nrep) * ng;
}

// LDS of the reverse passes: es | eb | lt | G2-or-deposit tile (tw each), and for the fused
// pass (STAGE 4) the previous step's es | eb | deposit tile (tw each).
__host__ __device__ constexpr size_t adj_lds_doubles(int tw, int stage)
{
    return stage == 4 ? 7 * (size_t)tw : 4 * (size_t)tw;
}

// Node i's value into its slot of a tile and the slots of its periodic images.
__device__ __forceinline__ void tile_put(double *t, int i, double v, int ng, int tw)
{
    t[kGhost + i] = v;
    if (i < kGhost)
        for (int s = i + kGhost + ng; s < tw; s += ng)
            t[s] = v;
    if (i >= ng - kGhost)
        for (int s = i + kGhost - ng; s >= 0; s -= ng)
            t[s] = v;
}

// A lane's batch of the reverse passes: the state, its adjoint and (STAGE 4) the state of
// the step before.
template <int STAGE> struct AdjBatch {
    double x, v, ax, av, xm, vm;
    __device__ __forceinline__ void load(const double *X, const double *V, const AdjWork &aw,
                                         const double *Xm, const double *Vm, int64_t start, int64_t p1)
    {
        const BatchAddr a(start, p1, 64);
        const unsigned o = a.off(threadIdx.x & 63, 0);
        x = (X + a.b0)[o];
        v = (V + a.b0)[o];
        ax = (aw.ax + a.b0)[o];
        av = (aw.av + a.b0)[o];
        if constexpr (STAGE == 4) {
            xm = (Xm + a.b0)[o];
            vm = (Vm + a.b0)[o];
        }
    }
};

// Reverse pass of step n.  STAGE 1, 2, 3 as described at the top; STAGE 4 is R3 of step n
// fused with R1 of step n - 1: with the adjoint of (x^n, v^n) just computed, the same
// thread recomputes step n - 1 of its particle (Xm, Vm, grids gm) and deposits its
// E-bar adjoint into the other parity's G1.  G1 and G2 have nrep replicas.
//
// What bounds it at 1e6 particles: each pass has about four batches per wavefront, so the
// round trips before and inside the loop.  The prologue is one round of loads (the fields the
// forward pass B built for step n, and n - 1, and the grid adjoints), one barrier for the
// tiles, their ghosts and the means; the next batch loads while the current one is processed
// (beside the recompute, 1e6 particles x 256 cells: STAGE 4 21.9 -> 18.8 us, STAGE 2 13.3 ->
// 12.2; the shortest 21.2 -> 17.0 and 12.7 -> 10.9).  STAGE 4's floor is the 64 B per particle
// it moves, 10 us; its 400 vector instructions per particle and wavefront take as long.  Doing
// its two forward steps together, stage by stage, costs registers that the recompute beside it
// needs (6.20 -> 6.23 ms for the sweep).
template <int ORDER, int STAGE>
__global__ __launch_bounds__(1024) __attribute__((amdgpu_waves_per_eu(4)))
void k_adj_reverse(Run r, AdjWork aw, AdjParams ap, int q, const double *__restrict__ X,
                   const double *__restrict__ V, const double *__restrict__ g,
                   const double *__restrict__ Xm, const double *__restrict__ Vm,
                   const double *__restrict__ gm)
{
    extern __shared__ double smem[];
    __shared__ double red[kRedSize];
    __shared__ int wctr;
    const int ng = r.ng, tw = r.tw, nrep = r.nrep;
    const unsigned nt = nthreads();
    const int64_t p0 = (int64_t)blockIdx.x * r.chunk;
    const int64_t p1 = min(r.np, p0 + r.chunk);
    // wavefronts claim batches of 64 particles (the counter is set before the barrier below)
    WaveBatches<1> wb(batch_order(p0, 64, false, blockIdx.x, r.nblocks, r.np, false), &wctr, nt);
    wb.reset();
    double *es = smem, *eb = es + tw, *lt = eb + tw, *t4 = lt + tw;
    double *esm = t4 + tw, *ebm = esm + tw, *tm = ebm + tw;   // STAGE 4
    double *dt_tile = STAGE == 4 ? tm : t4;                   // the deposit
    //   lt = lambda + lbw E^{n+1} + G1 / 2 (the adjoint of E^{n+1}); t4 = G2 (STAGE >= 3)
    double m[2] = {0.0, 0.0};
    AdjBatch<STAGE> cur, nxt;
    int64_t bcur = wb.first();
    bool loaded = false;
    for (int base = 0; base < ng; base += (int)nt) {
        const int i = base + (int)threadIdx.x, j = min(i, ng - 1);
        double fe = 0.0, fb = 0.0, fem = 0.0, fbm = 0.0, e1 = 0.0, lam = 0.0, g1 = 0.0, g2 = 0.0;
        double a1[STAGE >= 2 ? kMaxRep : 1] = {}, a2[STAGE >= 3 ? kMaxRep : 1] = {};
        if (__builtin_amdgcn_readfirstlane(i) < ng) {        // (the wavefront has nodes)
            fe = g[3 * ng + j];
            fb = g[4 * ng + j];
            if constexpr (STAGE == 4) {
                fem = gm[3 * ng + j];
                fbm = gm[4 * ng + j];
            }
            if constexpr (STAGE >= 2) {
                e1 = g[5 * ng + j];
                lam = aw.lam[q][j];
#pragma unroll
                for (int k = 0; k < kMaxRep; ++k) {
                    a1[k] = (aw.G1[q] + (size_t)min(k, nrep - 1) * ng)[j];
                    if constexpr (STAGE >= 3)
                        a2[k] = (aw.G2[q] + (size_t)min(k, nrep - 1) * ng)[j];
                }
            }
        }
        if (!loaded) {
            // the first particles, behind the first round of grid loads
            cur.load(X, V, aw, Xm, Vm, bcur, p1);
            if constexpr (STAGE != 3)
                tile_zero(dt_tile, tw, nt);
            loaded = true;
        }
        if (i < ng) {
            tile_put(es, i, fe, ng, tw);
            tile_put(eb, i, fb, ng, tw);
            if constexpr (STAGE == 4) {
                tile_put(esm, i, fem, ng, tw);
                tile_put(ebm, i, fbm, ng, tw);
            }
            if constexpr (STAGE >= 2) {
                g1 = a1[0];
#pragma unroll
                for (int k = 1; k < kMaxRep; ++k)
                    g1 += k < nrep ? a1[k] : 0.0;
                const double l = fma(ap.lbw, e1, lam) + 0.5 * g1;
                tile_put(lt, i, l, ng, tw);
                m[0] += l;
                if constexpr (STAGE >= 3) {
                    g2 = a2[0];
#pragma unroll
                    for (int k = 1; k < kMaxRep; ++k)
                        g2 += k < nrep ? a2[k] : 0.0;
                    tile_put(t4, i, g2, ng, tw);
                    m[1] += g2;
                    // adjoint of E^n for step n - 1
                    if (blockIdx.x == 0)
                        aw.lam[q ^ 1][i] = l + 0.5 * g1 + g2;
                }
            }
        }
    }
    // the next reverse step deposits into the other parity's G1 (R2, in the pass after this)
    // and G2 (cleared by R3): every workgroup clears its share
    if constexpr (STAGE == 2)
        rep_zero_part(aw.G1[q ^ 1], ng, nrep, ng, blockIdx.x, r.nblocks, nt);
    if constexpr (STAGE >= 3)
        rep_zero_part(aw.G2[q ^ 1], ng, nrep, ng, blockIdx.x, r.nblocks, nt);
    double mean_l = 0.0, mean_g2 = 0.0;
    if constexpr (STAGE >= 2)
        wave_partials<0u>(m, red);
    lds_barrier();
    if constexpr (STAGE >= 2) {
        mean_l = read_lane(wave_total(red, 0, nt >> 6), 0) * r.inv_ng;
        mean_g2 = read_lane(wave_total(red, 1, nt >> 6), 0) * r.inv_ng;
    }

    Depo<ORDER, 1, 3> dep;          // adjoint values: FP64 atomics (no fixed-point scale)
    while (batch_begins(bcur, p1)) {
        const int64_t bnxt = wb.claim(), p = bcur + (threadIdx.x & 63);
        const bool valid = p < p1;
        double w = r.wu;
        if (r.w)
            w = r.w[min(p, p1 - 1)];
        nxt.load(X, V, aw, Xm, Vm, bnxt, p1);          // the last one is discarded
        const double qp = w * r.qs;
        const AdjOut<ORDER, STAGE == 4 ? 3 : STAGE> o = adj_particle<ORDER, STAGE == 4 ? 3 : STAGE>(
            r, cur.x, cur.v, cur.ax, cur.av, qp, es, eb, lt, mean_l, t4, mean_g2);
        if (valid) {
            if constexpr (STAGE == 1) {
                const double c[1] = {o.ebar_b};
                dep.add(dt_tile, tw, ng, o.sh, c);
            } else if constexpr (STAGE == 2) {
                const double c[1] = {o.ehat_b};
                dep.add(dt_tile, tw, ng, o.ss, c);
            } else {
                aw.ax[p] = o.xb;
                aw.av[p] = o.vb;
                if constexpr (STAGE == 4) {
                    const AdjOut<ORDER, 1> o1 = adj_particle<ORDER, 1>(
                        r, cur.xm, cur.vm, o.xb, o.vb, qp, esm, ebm, lt, mean_l, t4, mean_g2);
                    const double c[1] = {o1.ebar_b};
                    dep.add(dt_tile, tw, ng, o1.sh, c);
                }
            }
        }
        cur = nxt;
        bcur = bnxt;
    }
    if constexpr (STAGE != 3) {
        lds_barrier();
        double *G = STAGE == 1 ? aw.G1[q] : (STAGE == 2 ? aw.G2[q] : aw.G1[q ^ 1]);
        tile_flush(dt_tile, g_slot(G, nrep, ng), 1, ng, tw);
    }
}

// Recompute of nsteps steps of the forward run, from its state (X, V) into (Xo, Vo), state
// j + 1 at Xo + j np, in one launch: with the fields of every step kept (g: kSaveRows rows of
// N_g per step, E* and E-bar among them) no step waits for another particle's, so a lane keeps
// its U particles in registers from state to state and only writes them.  The coefficients and
// the particle's arithmetic are those of pass B, so the states are the forward run's bit for
// bit; nothing is deposited.  (A launch of pass B's kind per step took 9.7 us a step; the two
// segments of a 100-step gradient of 1e6 particles, 256 cells: 6.24 -> 5.83 ms forward and
// backward.)
// What bounds it is a lane's chain of four particles and the 16 MB a step writes.  The segment
// the sweep waits for first has the chip to itself: whole workgroups.  The others run beside
// the reverse passes, whose 16 wavefronts of 96 registers leave a CU room for four of 128: one
// workgroup of four wavefronts per CU, for the whole segment.  (Eight wavefronts and ten steps
// a launch 5.93 ms, sixteen and five 5.94-6.15, four and ten 5.88; two particles per lane
// 5.88-5.93.)  Both shapes were chosen there: with fewer particles the first segment's launch
// leaves CUs idle (5e4: 13 workgroups), and on grids beyond about 1070 cells two buffers no longer
// fit a CU beside a reverse workgroup; a step is faster than with a launch of its own all the
// same (backward of 40 steps, 5e4 x 256 1345 -> 715 us, 1e6 x 1200 2920 -> 2000).
// LDS: nbuf buffers of the coefficients of E* and E-bar ([2][(ORDER + 1) tw] each).  With two,
// the next step's node values load while the particles of the present one are pushed, and a
// step has one barrier.
constexpr int kRecUnroll = 4, kRecBlocks = 256;
constexpr int kRecThreadsAlone = 1024, kRecThreadsBeside = 256;

template <int ORDER> __host__ __device__ constexpr size_t recompute_lds_doubles(int tw, int nbuf)
{
    return (size_t)nbuf * 2 * (ORDER + 1) * tw;
}

// The node values of coefficient slot threadIdx.x of both fields.  (Two slots per thread in
// flight would spill beside four particles: 5.62 against 5.59 ms.)
template <int ORDER> struct RecNodes {
    double e[2][ORDER + 1];
    __device__ __forceinline__ void load_slot(const double *g, int s, int ng)
    {
#pragma unroll
        for (int j = 0; j <= ORDER; ++j) {
            int i = wrap_ghost(s - kGhost, ng) + j;
            i -= i >= ng ? ng : 0;
            e[0][j] = g[3 * ng + i];
            e[1][j] = g[4 * ng + i];
        }
    }
    __device__ __forceinline__ void fill_slot(double *ct, int s, int tw) const
    {
#pragma unroll
        for (int f = 0; f < 2; ++f)
            coefs<ORDER>(ct + f * (ORDER + 1) * tw + (ORDER + 1) * s, e[f]);
    }
    __device__ __forceinline__ void load(const double *g, int ng, int tw)
    {
        if ((int)threadIdx.x < tw - ORDER)
            load_slot(g, threadIdx.x, ng);
    }
    // The coefficients from the values loaded, and those of the slots beyond.
    __device__ __forceinline__ void fill(double *ct, const double *g, int ng, int tw, unsigned nt)
    {
        if ((int)threadIdx.x < tw - ORDER)
            fill_slot(ct, threadIdx.x, tw);
        for (int s = (int)(threadIdx.x + nt); s < tw - ORDER; s += nt) {
            load_slot(g, s, ng);
            fill_slot(ct, s, tw);
        }
    }
};

template <int ORDER>
__global__ __launch_bounds__(1024) __attribute__((amdgpu_waves_per_eu(4)))
void k_adj_recompute(Run r, const double *__restrict__ g, int nsteps, int nbuf,
                     const double *__restrict__ X, const double *__restrict__ V, double *Xo, double *Vo)
{
    constexpr int U = kRecUnroll;
    extern __shared__ double smem[];
    const int ng = r.ng, tw = r.tw;
    const unsigned nt = nthreads(), lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    const int64_t span = (int64_t)nt * U;
    const size_t row = (size_t)kSaveRows * ng, buf = 2 * (size_t)(ORDER + 1) * tw;
    const Run q = reload(kernarg_run());
    RecNodes<ORDER> nodes;
    for (int64_t base = blockIdx.x * span; base < r.np; base += gridDim.x * span) {
        const int64_t b = base + 64 * U * (int64_t)wave;
        PBatch<U, 1> cur;
        nodes.load(g, ng, tw);
        load_batch(cur, X, V, r.vstride, nullptr, 0.0, b, r.np);
        bool valid[U];
#pragma unroll
        for (int u = 0; u < U; ++u)
            valid[u] = b + 64 * u + lane < r.np;
        lds_barrier();                  // (the tiles of the particles before are done with)
        nodes.fill(smem, g, ng, tw, nt);
        for (int s = 0; s < nsteps; ++s) {
            const double *gn = g + (s + 1) * row, *cts = smem + (nbuf == 2 && (s & 1) ? buf : 0);
            lds_barrier();
            if (s + 1 < nsteps)
                nodes.load(gn, ng, tw);
            double vs[U][1], x1[U], vd[U][1], gam[U], vn[U][1], xw[U];
            Pos pos[U];
            Cell<ORDER> c[U];
            int fb = 0;
            half_steps<ORDER, 1, false, U>(q, cur.x, cur.v, cts, nullptr, vs, x1);
            mid_points<ORDER, U>(pos, cur.x, x1, q);
            cells_at<ORDER, U>(c, pos, ng);
#pragma unroll
            for (int u = 0; u < U; ++u)
                dagger_es<1>(vd[u], cur.v[u], vs[u], gather_poly<ORDER>(cts + (ORDER + 1) * tw, c[u]), q);
            gamma_all<1, U>(gam, vs, vd, cur.v, valid, fb);
#pragma unroll
            for (int u = 0; u < U; ++u)
                vn[u][0] = gam[u] * vd[u][0];
            wrap_all<U>(xw, x1, q);
            store_all<1, U>(xw, vn, valid, Xo + s * r.np, Vo + s * r.np, b, r.vstride);
#pragma unroll
            for (int u = 0; u < U; ++u) {
                cur.x[u] = xw[u];
                cur.v[u][0] = vn[u][0];
            }
            if (s + 1 < nsteps) {
                if (nbuf == 1)
                    lds_barrier();
                nodes.fill(smem + (nbuf == 2 && !(s & 1) ? buf : 0), gn, ng, tw, nt);
            }
        }
    }
}

// Inverse-CDF positions for the density 1 + sum_m alpha_m cos(k_m x) on [0, L): Newton
// on x + sum_m (alpha_m / k_m) sin(k_m x) = u L from x = u L, to 1e-15 L; velocities
// v_b s_p + v_s g_p.
__global__ __launch_bounds__(1024) void k_adj_sample(Run r, AdjParams ap, const double *__restrict__ U,
                                                     const double *__restrict__ S,
                                                     const double *__restrict__ Gn, double *X,
                                                     double *V)
{
    for (int64_t p = (int64_t)blockIdx.x * nthreads() + threadIdx.x; p < r.np;
         p += (int64_t)gridDim.x * nthreads()) {
        const double target = U[p] * r.L;
        double x = target;
        for (int it = 0; it < 60 && ap.n_modes > 0; ++it) {
            double f = x - target, d = 1.0;
            for (int m = 0; m < ap.n_modes; ++m) {
                double sn, cs;
                sincos(ap.k[m] * x, &sn, &cs);
                f += ap.alpha[m] / ap.k[m] * sn;
                d += ap.alpha[m] * cs;
            }
            const double step = f / d;
            x -= step;
            if (fabs(step) < 1e-15 * r.L)
                break;
        }
        if (x >= r.L)
            x -= r.L;
        if (x < 0.0)
            x += r.L;
        X[p] = x;
        V[p] = fma(ap.v_beam, S[p], ap.v_spread * Gn[p]);
    }
}

// rhobar = Gauss solve of lambda^0 (one workgroup): the Gauss map rho -> E is a real
// circulant whose eigenvalues 1 / (i k_m) are imaginary, so its transpose is its
// negative and the adjoint of rho is -rhobar.
__global__ __launch_bounds__(1024) void k_adj_rhobar(Run r, Work wk, AdjWork aw, int q)
{
    extern __shared__ double smem[];
    Work t = wk;
    t.J2[0] = aw.lam[q];
    t.E = aw.rhobar;
    Run r1 = r;
    r1.nrep = 1;
    gauss_body(r1, t, smem);
}

// Per workgroup: the adjoint of x^0 gets the Gauss start's term, then the partial sums
// of the gradient: amplitudes (implicit differentiation of the inverse CDF:
// dx/dalpha_m = -sin(k_m x) / (k_m (1 + sum_j alpha_j cos(k_j x)))), beam speed
// (sum vbar s), beam spread (sum vbar g).
template <int ORDER>
__global__ __launch_bounds__(1024) void k_adj_grad(Run r, AdjWork aw, AdjParams ap,
                                                   const double *__restrict__ X0,
                                                   const double *__restrict__ S,
                                                   const double *__restrict__ Gn)
{
    extern __shared__ double smem[];
    __shared__ double red[kRedSize];
    const int ng = r.ng, tw = r.tw;
    double *rb = smem;
    for (int i = threadIdx.x; i < ng; i += nthreads())
        rb[kGhost + i] = -aw.rhobar[i];
    __syncthreads();
    ghost_fill(rb, 1, ng, tw);
    __syncthreads();
    // (the loops over the modes are unrolled, so the sums stay in registers: 66 -> 48 us at 1e6
    // particles and 8 modes, with the sine and the cosine from one call)
    double acc[kAdjMaxModes], acc_v = 0.0, acc_s = 0.0;
#pragma unroll
    for (int m = 0; m < kAdjMaxModes; ++m)
        acc[m] = 0.0;
    const int64_t p0 = (int64_t)blockIdx.x * r.chunk;
    const int64_t p1 = min(r.np, p0 + r.chunk);
    for (int64_t p = p0 + threadIdx.x; p < p1; p += nthreads()) {
        const double x = X0[p];
        const double q = (r.w ? r.w[p] : r.wu) * r.qs;
        const Stencil<ORDER> s = stencil_at<ORDER>(locate<ORDER>(x, r.inv_h, 0.0));
        const Slots<ORDER> n = slots_of<ORDER>(s, ng);
        const Stencil<ORDER> d = dstencil_at<ORDER>(locate<ORDER>(x, r.inv_h, 0.0));
        const double xb = aw.ax[p] + q * r.inv_h * gather1<ORDER>(rb, d, n);
        double dens = 1.0, sn[kAdjMaxModes];
#pragma unroll
        for (int m = 0; m < kAdjMaxModes; ++m)
            if (m < ap.n_modes) {
                double cs;
                sincos(ap.k[m] * x, &sn[m], &cs);
                dens += ap.alpha[m] * cs;
            }
#pragma unroll
        for (int m = 0; m < kAdjMaxModes; ++m)
            if (m < ap.n_modes)
                acc[m] -= xb * sn[m] / (ap.k[m] * dens);
        acc_v = fma(aw.av[p], S[p], acc_v);
        acc_s = fma(aw.av[p], Gn[p], acc_s);
    }
    auto put = [&](int m, double v) {
        const double t = block_sum(v, red);
        if (threadIdx.x == 0)
            aw.gpart[(size_t)blockIdx.x * ap.nparam + m] = t;
    };
#pragma unroll
    for (int m = 0; m < kAdjMaxModes; ++m)
        if (m < ap.n_modes)
            put(m, acc[m]);
    put(ap.n_modes, acc_v);
    put(ap.n_modes + 1, acc_s);
}

// Gradient = sum of the workgroup partials in workgroup order (one workgroup).
__global__ void k_adj_grad_final(AdjWork aw, int nblocks, int nparam, double *grad)
{
    __shared__ double red[kRedSize];
    for (int m = 0; m < nparam; ++m) {
        double s = 0.0;
        for (int b = threadIdx.x; b < nblocks; b += nthreads())
            s += aw.gpart[(size_t)b * nparam + m];
        s = block_sum(s, red);
        if (threadIdx.x == 0)
            grad[m] = s;
    }
}

// J = lw * sum_{n=1..N} W_E^n from the record ring (one workgroup, fixed order).
__global__ void k_adj_loss(Work wk, int rec_cap, int64_t nsteps, double lw, double *loss)
{
    __shared__ double red[kRedSize];
    double s = 0.0;
    for (int64_t n = 1 + threadIdx.x; n <= nsteps; n += nthreads())
        s += wk.rec[n % rec_cap].field_e;
    s = block_sum(s, red);
    if (threadIdx.x == 0)
        *loss = lw * s;
}

}  // namespace pic
