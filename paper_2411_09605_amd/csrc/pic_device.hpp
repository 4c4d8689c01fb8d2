// Device code of the explicit energy-conserving PIC step for gfx950 (CDNA4).
//
// Particle state is a structure of FP64 arrays (x[N_p], v[nv][N_p]) streamed from HBM
// with one lane per particle; the 1D grid (a few hundred nodes) lives in LDS for the
// whole pass.  One step of ESEC2 / EMEC(LI) (eq. (good_translation), (EMbasic)) is two
// kernel launches:
//
//   pass A: every workgroup builds the predictor fields E* (B*) in LDS from E^n (B^n)
//           and the predictor current j^{n,*}; per particle x* = x + dt/2 v, gather at
//           x*, v*, x^{n+1}, x^{n+1/2} = (x^n + x^{n+1}) / 2, deposit w v* at x^{n+1/2}
//           into an LDS tile; the tile is added to the global current with FP64 atomics
//   pass B: every workgroup rebuilds E* (bit-identically) and builds E^{n+1} (B^{n+1})
//           and the averaged fields from the centred current (Ampere / Crank-Nicolson);
//           per particle it recomputes x*, v*, x^{n+1/2}, gathers the averaged fields at
//           x^{n+1/2}, forms v-dagger and Gamma (eq. (opt_solution)) with the fallback,
//           writes x^{n+1} (wrapped) and v^{n+1}, and - because x*_{n+1} = x^{n+1} +
//           dt/2 v^{n+1} is then known - deposits the NEXT step's predictor current
//           w v^{n+1} at x*_{n+1}; the last workgroup stores E^{n+1} (B^{n+1}) and W_E, W_B
//
// The grid work is tiny (N_g nodes) and is repeated by every workgroup in its prologue,
// which costs a few microseconds of L2 reads and saves the single-workgroup kernels and
// the grid-wide synchronisation they would need.  Fields and currents are double
// buffered by step parity.  The particle state is read twice and written once per step
// (48 B per particle in 1D-1V, 96 B in 1D-3V).  Recomputing v* in pass B instead of
// storing it keeps the deposit in pass A and the gather in pass B at exactly the same
// x^{n+1/2} (the code is compiled without FP contraction), which is what the energy
// identity of eq. (exp_econs_simple) needs.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include "pic_types.hpp"

namespace pic {

// Particles whose loads each thread issues together before computing on them, per pass (more
// loads in flight against fewer waves per SIMD from the extra registers).  The register windows
// (Depo kinds 1 and 2) move less often if a lane's next particle is 64 further on rather than in
// the wavefront's next batch, a thousand on: with three components too they take two (EMEC(LI)
// 2e6 x 256, one and two particles: wavefront window 128 and 109 us a step, thread window on
// sorted particles 153 and 126).
template <int NV, int DEP> constexpr int kUnrollA = NV == 1 || DEP == 1 || DEP == 2 ? 2 : 1;
template <int NV, int DEP> constexpr int kUnrollB = kUnrollA<NV, DEP>;
// Of those, how many are computed on together: two particles of three components by stages would
// need more than the 128 registers (the same two 155 and 145 us).
template <int NV, int U> constexpr int kGroup = NV == 1 ? U : 1;
// Minimum wavefronts per SIMD the particle passes are compiled for: one 1024-thread
// workgroup per CU is 4 per SIMD (at most 128 VGPRs); 1D-3V keeps its registers.
template <int NV> constexpr int kWavesPerEU = NV == 1 ? 4 : 1;
// Largest workgroup of the particle passes.
template <int NV> constexpr int kMaxThreads = 1024;

// Run::scheme of the electromagnetic schemes, EMEC(LI), EMEC(PSATD) and EMEC(LF).
__host__ __device__ constexpr bool em_scheme(int s) { return s == 2 || s == kPsatd || s == kLeapfrog; }

// Threads of the (1-D) workgroup: the group-size field of the implicit kernel arguments
// (a 16-bit field at byte 12), read with a scalar load of the dword that holds it.
// blockDim.x also allows for a partial last workgroup, which these launches never have,
// and is read with a vector load; vector loads complete in order, so waiting for it
// would also wait for every particle load issued before it.  (The dispatch packet holds
// the same number but may sit in host memory.)
__device__ __forceinline__ unsigned nthreads()
{
    typedef const __attribute__((address_space(4))) unsigned int *kernarg_ptr;
    return ((kernarg_ptr)__builtin_amdgcn_implicitarg_ptr())[3] & 0xffffu;
}

// A run's scalars in constant memory: the first kernel argument of the plain passes, an entry
// of the run table in the batched ones.
typedef const __attribute__((address_space(4))) Run *RunPtr;

__device__ __forceinline__ RunPtr kernarg_run()
{
    return (RunPtr)__builtin_amdgcn_kernarg_segment_ptr();
}

// A value that is the same in every lane, in a scalar register pair of its own.
__device__ __forceinline__ double scalar_pair(double v)
{
    unsigned lo = __double2loint(v), hi = __double2hiint(v);
    asm("" : "+s"(lo), "+s"(hi));
    return __hiloint2double((int)hi, (int)lo);
}

// The run's scalars read (again) at this point, with scalar loads.  The passes read them once
// for their prologue and once for the particle loop: values held from one to the other would
// not fit the scalar registers beside the prologue's addresses, and the loop would fetch its
// constants from spill lanes (150 of 670 vector instructions of a pass-B iteration).
__device__ __forceinline__ Run reload(RunPtr p)
{
    asm volatile("" : "+s"(p));
    struct Words {
        int w[sizeof(Run) / 4];
    };
    typedef const __attribute__((address_space(4))) Words *words;
    Run r = __builtin_bit_cast(Run, *(words)p);
    // one register pair each: as parts of the wide loads they would be spilled eight at a time
    double *c[] = {&r.dt, &r.hdt, &r.L, &r.inv_L, &r.inv_h, &r.hinv_h, &r.qs, &r.wu, &r.xshift};
#pragma unroll
    for (double *d : c)
        *d = scalar_pair(*d);
    return r;
}

// Likewise a pointer that the particle loop uses.
template <typename P> __device__ __forceinline__ void settle_pointer(P &p)
{
    typedef __attribute__((address_space(1))) double *global_ptr;   // (stays a global address)
    p = (P)(global_ptr)__builtin_bit_cast(unsigned long long,
                                          scalar_pair(__builtin_bit_cast(double, (unsigned long long)p)));
}

// Written by k_group_size_probe: nthreads() as read in one-workgroup launches of 64 and
// 256 threads (the library checks them once per device before its first launch).
__device__ int g_group_size_probe[2];

__global__ void k_group_size_probe(int slot)
{
    if (threadIdx.x == 0)
        g_group_size_probe[slot] = (int)nthreads();
}

// A thread's batch of U particles (lane l of a wavefront takes b + l + 64 u, u < U; see
// BatchAddr), loaded together.  The particle loops keep the next batch's loads in flight
// while they compute on the current one (and the first batch's loads in flight during the
// field prologue), so HBM latency overlaps LDS and ALU work.
template <int U, int NV> struct PBatch {
    double x[U], v[U][NV], w[U];
};

// Particles u0 .. u0 + G - 1 of a lane's batch.
template <int G, int U, int NV>
__device__ __forceinline__ PBatch<G, NV> batch_group(const PBatch<U, NV> &b, int u0)
{
    PBatch<G, NV> o;
#pragma unroll
    for (int u = 0; u < G; ++u) {
        o.x[u] = b.x[u0 + u];
        o.w[u] = b.w[u0 + u];
#pragma unroll
        for (int c = 0; c < NV; ++c)
            o.v[u][c] = b.v[u0 + u][c];
    }
    return o;
}

// Addressing of a wavefront's batch of 64 U consecutive particles starting at `start` (the
// same in every lane): lane l takes start + l + 64 u.  Entries past p1 are clamped to
// particle p1 - 1 (every range holds at least one particle), so loads are issued without a
// per-lane branch.  The base is wavefront-uniform and the per-lane offset 32-bit, which
// lets the loads use a scalar base register instead of 64-bit vector address arithmetic.
struct BatchAddr {
    int64_t b0;        // first particle of the batch, clamped to p1 - 1
    unsigned lim;      // largest offset inside [b0, p1)
    __device__ __forceinline__ BatchAddr(int64_t start, int64_t p1, unsigned span)
    {
        b0 = (int64_t)min((uint64_t)start, (uint64_t)(p1 - 1));      // (as batch_begins compares)
        lim = (unsigned)min(p1 - 1 - b0, (int64_t)(span - 1));
    }
    __device__ __forceinline__ unsigned off(unsigned lane, int u) const
    {
        return min(lane + 64u * (unsigned)u, lim);
    }
};

// Loads the batch at `start` (U particles per lane, with their weights W[p], or wu when W is
// null).  The weights come with the batch: loaded when the batch is processed, they would be
// waited for in the middle of it, and with them, in order, the next batch's loads.  Callers
// mask the entries past p1 with their own bounds test.
template <int U, int NV>
__device__ __forceinline__ void load_batch(PBatch<U, NV> &b, const double *__restrict__ X,
                                           const double *__restrict__ V, int64_t vstride,
                                           const double *__restrict__ W, double wu,
                                           int64_t start, int64_t p1)
{
    const BatchAddr a(start, p1, 64u * U);
    const unsigned lane = threadIdx.x & 63;
    const double *Xb = X + a.b0;
#pragma unroll
    for (int u = 0; u < U; ++u) {
        const unsigned o = a.off(lane, u);
        b.x[u] = Xb[o];
#pragma unroll
        for (int c = 0; c < NV; ++c)
            b.v[u][c] = (V + c * vstride + a.b0)[o];
        b.w[u] = wu;
    }
    if (W) {
#pragma unroll
        for (int u = 0; u < U; ++u)
            b.w[u] = (W + a.b0)[a.off(lane, u)];
    }
}

// A workgroup's particles go to its wavefronts in batches of 64 U consecutive particles
// (lane l takes b + l + 64 u): wavefront w starts with the workgroup's batch w, and each
// then claims the next unclaimed batch from a counter in LDS.  The hardware issues older
// wavefronts first, so a fixed split leaves the youngest ones finishing alone at the end
// of the pass; claiming batches as they go, the wavefronts of a workgroup finish within
// about one batch of each other.  The counter is set by reset() before a barrier that
// precedes the first claim.
//
// Batch k of a workgroup starts at origin + k step (batch_order).  Chunks (the default): the
// workgroup's particles are [p0, p1), origin = p0 and step = one batch.  Interleaved:
// batches are dealt to the workgroups round-robin, origin = b batches for workgroup b
// and step = nblocks batches, so that at any moment the grid reads one region of the
// state rather than nblocks separate ones; with the state streaming from HBM this reads
// faster, with it in the Infinity Cache the chunks do (callers pass p1 = N_p).
//
// Static (the deterministic mode): wavefront w takes batches w, w + W, w + 2W, ... of
// its workgroup's W wavefronts, so every thread always sees the same particles in the
// same order and its running sums (kinetic energy) are reproducible bit for bit.
template <int U> struct WaveBatches {
    BatchOrder o;
    int *ctr;
    int fixed;             // 1: static assignment
    int k;                 // static: index of the wavefront's current batch
    int nw;
    // Interleaved runs (the state larger than the 256 MB Infinity Cache) can walk the state
    // from its end (a reversed order): a pass that starts where the previous pass ended finds
    // up to 256 MB of the state still in the cache.  The set of batches is the same either way.
    __device__ __forceinline__ WaveBatches(const BatchOrder &order, int *counter, unsigned nt, int static_order = 0)
        : o(order), ctr(counter), fixed(static_order), nw((int)(nt >> 6))
    {
        k = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    }
    __device__ __forceinline__ void reset() const
    {
        if (threadIdx.x == 0)
            *ctr = nw;
    }
    // first particle of this wavefront's first batch (the same in every lane)
    __device__ __forceinline__ int64_t first() const
    {
        return o.origin + __builtin_amdgcn_readfirstlane(threadIdx.x >> 6) * o.step;
    }
    // claim the next batch (every lane of the wavefront active)
    __device__ __forceinline__ int64_t claim()
    {
        if (fixed) {
            k += nw;
            return batch_start(o, k);
        }
        // (an address the compiler takes to differ by lane keeps it from wrapping the one
        // lane's atomic in a wavefront-wide sum)
        int kc = 0;
        unsigned zero = 0;
        asm("" : "+v"(zero));
        if ((threadIdx.x & 63) == 0)
            kc = atomicAdd(ctr + zero, 1);
        return batch_start(o, __builtin_amdgcn_readlane(kc, 0));
    }
};

// ------------------------------------------------------------------ shape functions
// Cardinal B-spline weights of degree ORDER for a particle at xi = x / h - shift
// (section 2.2).  first = index of the leftmost node of the ORDER + 1 node stencil.
template <int ORDER> struct Stencil {
    int first;
    double w[ORDER + 1];
};

__device__ __forceinline__ Stencil<1> stencil1(double xi)
{
    double f = floor(xi);
    double d = xi - f;
    Stencil<1> s;
    s.first = (int)f;
    s.w[0] = 1.0 - d;
    s.w[1] = d;
    return s;
}

// Quadratic weights (1/2 - d)^2 / 2, 3/4 - d^2, (1/2 + d)^2 / 2, expanded as
// t -+ d/2 with t = 1/8 + d^2/2 (five operations; gather and deposit share them).
__device__ __forceinline__ Stencil<2> stencil2(double xi)
{
    double f = floor(xi + 0.5);
    double d = xi - f;                       // in [-1/2, 1/2)
    double hd = 0.5 * d;
    double t = fma(hd, d, 0.125);
    Stencil<2> s;
    s.first = (int)f - 1;
    s.w[0] = t - hd;
    s.w[1] = fma(-d, d, 0.75);
    s.w[2] = t + hd;
    return s;
}

template <int ORDER> __device__ __forceinline__ Stencil<ORDER> stencil(double xi);
template <> __device__ __forceinline__ Stencil<1> stencil<1>(double xi) { return stencil1(xi); }
template <> __device__ __forceinline__ Stencil<2> stencil<2>(double xi) { return stencil2(xi); }

// Periodic node index.  Positions handed to the passes are within a few cells of
// [0, L), so the first two tests decide; the modulo keeps any input (even NaN, which
// converts to an arbitrary int) inside the tile.
__device__ __forceinline__ int wrap_node(int i, int ng)
{
    if ((unsigned)i < (unsigned)ng)
        return i;
    if (i < 0 && i >= -ng)
        return i + ng;
    if (i >= ng && i < 2 * ng)
        return i - ng;
    int r = i % ng;
    return r < 0 ? r + ng : r;
}

// The node of a tile slot (an index within kGhost of [0, ng), ng >= 3): two conditional steps
// either way, without the set-up of a modulo.
static_assert(kGhost <= 6, "two periods of the smallest grid cover the ghosts");
__device__ __forceinline__ int wrap_ghost(int i, int ng)
{
    i += i < 0 ? ng : 0;
    i += i < 0 ? ng : 0;
    i -= i >= ng ? ng : 0;
    i -= i >= ng ? ng : 0;
    return i;
}

// LDS tiles hold N_g nodes plus kGhost periodic copies on each side: node i of
// component c sits at slot c * tw + kGhost + i (tw = N_g + 2 kGhost).  The ORDER + 1
// slots of a stencil are always consecutive: a stencil whose nodes fall inside the padded
// range indexes the tile directly, and one beyond the ghost band has its first node
// wrapped into [0, N_g), which keeps the rest inside the right ghost band (ORDER <=
// kGhost).  So the LDS accesses of one stencil share a base address.
static_assert(kGhost >= 2, "a wrapped quadratic stencil must fit the right ghost band");
template <int ORDER> struct Slots {
    int n[ORDER + 1];
};

template <int ORDER>
__device__ __forceinline__ Slots<ORDER> slots_of(const Stencil<ORDER> &s, int ng)
{
    int b = s.first + kGhost;
    if ((unsigned)b > (unsigned)(ng + 2 * kGhost - ORDER - 1))
        b = wrap_node(s.first, ng) + kGhost;
    Slots<ORDER> o;
#pragma unroll
    for (int k = 0; k <= ORDER; ++k)
        o.n[k] = b + k;
    return o;
}

__device__ __forceinline__ int slot_of_node(int i, int ng)
{
    return (unsigned)(i + kGhost) < (unsigned)(ng + 2 * kGhost) ? i + kGhost
                                                                 : wrap_node(i, ng) + kGhost;
}

template <int ORDER>
__device__ __forceinline__ double gather1(const double *tile, const Stencil<ORDER> &s,
                                          const Slots<ORDER> &n)
{
    double acc = 0.0;
#pragma unroll
    for (int k = 0; k <= ORDER; ++k)
        acc = fma(tile[n.n[k]], s.w[k], acc);
    return acc;
}

// Gathers that deposit nothing at the same position use the field as a polynomial in the
// particle's offset d inside its cell (d as in stencil<ORDER>): sum_k E_k w_k(d) expanded
// once per cell in the prologue, so a gather costs ORDER FMAs instead of the weights and
// ORDER + 1 FMAs.  Coefficient tile: slot s holds the ORDER + 1 coefficients of the cell
// whose stencil starts at slot s.
template <int ORDER> struct Cell {
    int base;            // slot of the stencil's first node
    double d;
};

// The particle loops treat the U particles of a lane together, stage by stage, so that their
// dependent chains overlap (a pass on few particles has one wavefront per SIMD and nothing
// else to issue) and the rare cases (a stencil beyond the ghost band, a wrap, a large
// correction) cost one test per stage: a branch the whole wavefront takes or not.

// Where a particle sits on the grid: its node (the nearest one for the quadratic shape, the
// lower one for the tent) and the offset from it, both of the coordinate s scale - shift.
// Adding 1.5 2^52 rounds to the nearest integer and leaves it in the sum's low bits, so
// neither the coordinate itself nor a conversion is needed.  (A tie may round to either node;
// the spline's two pieces agree there.)  The sum less the constant, as 64-bit numbers, is the
// node of a coordinate up to 2^51.  Beyond, and for one that is not finite, it is some large
// number, and the quadratic shape's offset is no longer the distance from a whole number:
// slot_bases puts such a particle inside the tile and its offset into [-1/2, 1/2].  The tent's
// offset always lies in [0, 1), so the low 32 bits do there: beyond 2^31 they are some node.
constexpr double kRoundMagic = 6755399441055744.0;   // 1.5 * 2^52
struct Pos {
    long long n;
    double d;
};

template <int ORDER> __device__ __forceinline__ Pos locate(double s, double scale, double shift)
{
    Pos p;
    if constexpr (ORDER == 2) {
        const double t = fma(s, scale, kRoundMagic);   // (shift is 0: half-node grids use tents)
        p.n = __double_as_longlong(t) - __double_as_longlong(kRoundMagic);
        p.d = fma(s, scale, -(t - kRoundMagic));
    } else {
        const double xi = fma(s, scale, -shift), f = floor(xi);
        p.n = __double2loint(f + kRoundMagic);
        p.d = xi - f;
    }
    return p;
}

// The same particle on the half nodes (i + 1/2).
template <int ORDER> __device__ __forceinline__ Pos half_node(const Pos &p)
{
    Pos o;
    if constexpr (ORDER == 2) {
        // nearest half node: i or i - 1 by the sign of the offset
        o.d = p.d - __builtin_copysign(0.5, p.d);
        o.n = p.n + (__double2hiint(p.d) >> 31);
    } else {
        const bool low = p.d < 0.5;
        o.d = low ? p.d + 0.5 : p.d - 0.5;
        o.n = low ? p.n - 1 : p.n;
    }
    return o;
}

// The stencil of a particle (the weights of stencil<ORDER> from its offset).
template <int ORDER> __device__ __forceinline__ Stencil<ORDER> stencil_at(const Pos &p)
{
    Stencil<ORDER> s;
    if constexpr (ORDER == 2) {
        const double hd = 0.5 * p.d, t = fma(hd, p.d, 0.125);
        s.first = (int)(p.n - 1);
        s.w[0] = t - hd;
        s.w[1] = fma(-p.d, p.d, 0.75);
        s.w[2] = t + hd;
    } else {
        s.first = (int)p.n;
        s.w[0] = 1.0 - p.d;
        s.w[1] = p.d;
    }
    return s;
}

// A quadratic shape's offset out of [-1/2, 1/2] (see Pos) taken as the distance from the
// nearest whole number: its weights, which grow with it, stay those of some particle.
template <int ORDER> __device__ __forceinline__ void near_offset(Pos &p)
{
    if (ORDER == 2 && !(fabs(p.d) <= 0.5))
        p.d -= rint(p.d);
}

// The slot of the first node of a particle's stencil if the tile holds it there (see Slots),
// any larger number if not.  (Of the quadratic shape's 64 bits the comparison with the largest
// slot is the test for a far offset as well; as a test of its own that was 1-3 % of a step.)
template <int ORDER> __device__ __forceinline__ auto first_slot(const Pos &p)
{
    if constexpr (ORDER == 2)
        return (unsigned long long)p.n + (kGhost - 1);
    else
        return (unsigned)p.n + kGhost;
}

// A particle that is not in the tile there: its slot, its offset near.
template <int ORDER> __device__ __forceinline__ int far_slot(Pos &p, int ng)
{
    near_offset<ORDER>(p);
    return wrap_node((int)(p.n - (ORDER == 2 ? 1 : 0)), ng) + kGhost;
}

// Slots of the first nodes of the particles' stencils.
template <int ORDER, int U>
__device__ __forceinline__ void slot_bases(int (&b)[U], Pos (&p)[U], int ng)
{
    const unsigned lim = (unsigned)(ng + 2 * kGhost - ORDER - 1);
    bool out = false;
#pragma unroll
    for (int u = 0; u < U; ++u) {
        b[u] = (int)first_slot<ORDER>(p[u]);
        out |= first_slot<ORDER>(p[u]) > lim;
    }
    if (__any(out)) {
#pragma unroll
        for (int u = 0; u < U; ++u)
            if (first_slot<ORDER>(p[u]) > lim)
                b[u] = far_slot<ORDER>(p[u], ng);
    }
}

template <int ORDER, int U>
__device__ __forceinline__ void cells_at(Cell<ORDER> (&c)[U], Pos (&p)[U], int ng)
{
    int b[U];
    slot_bases<ORDER, U>(b, p, ng);
#pragma unroll
    for (int u = 0; u < U; ++u) {
        c[u].base = b[u];
        c[u].d = p[u].d;
    }
}

// Stencils of the particles and the slots of their first nodes.
template <int ORDER, int U>
__device__ __forceinline__ void stencils_at(Stencil<ORDER> (&st)[U], int (&b)[U], Pos (&p)[U], int ng)
{
    slot_bases<ORDER, U>(b, p, ng);
#pragma unroll
    for (int u = 0; u < U; ++u)
        st[u] = stencil_at<ORDER>(p[u]);
}

template <int ORDER>
__device__ __forceinline__ double gather_at(const double *tile, const Stencil<ORDER> &s, int base)
{
    double acc = 0.0;
#pragma unroll
    for (int k = 0; k <= ORDER; ++k)
        acc = fma(tile[base + k], s.w[k], acc);
    return acc;
}

template <int ORDER>
__device__ __forceinline__ double gather_poly(const double *ct, const Cell<ORDER> &c)
{
    // (base is a slot number: the 24-bit product runs at full rate, the 64-bit one does not)
    const double *k = ct + __umul24((unsigned)c.base, ORDER + 1);
    if constexpr (ORDER == 1)
        return fma(c.d, k[1], k[0]);
    else
        return fma(c.d, fma(c.d, k[2], k[1]), k[0]);
}

// Coefficients of every cell of a tile from its node values f(0..ng) (periodic).
//   tent:      E(d) = E_0 + d (E_1 - E_0)
//   quadratic: E(d) = (E_0 + E_2)/8 + 3 E_1/4 + d (E_2 - E_0)/2 + d^2 ((E_0 + E_2)/2 - E_1)
template <int ORDER>
__device__ __forceinline__ void coefs(double *c, const double (&e)[ORDER + 1])
{
    if constexpr (ORDER == 1) {
        c[0] = e[0];
        c[1] = e[1] - e[0];
    } else {
        c[0] = 0.125 * (e[0] + e[2]) + 0.75 * e[1];
        c[1] = 0.5 * (e[2] - e[0]);
        c[2] = 0.5 * (e[0] + e[2]) - e[1];
    }
}

template <int ORDER, typename F>
__device__ __forceinline__ void coef_fill(double *ct, F &&f, int ng, int tw, unsigned nt)
{
    for (int s = threadIdx.x; s < tw - ORDER; s += nt) {
        const int i0 = wrap_ghost(s - kGhost, ng), i1 = i0 + 1 == ng ? 0 : i0 + 1;
        double e[ORDER + 1] = {f(i0), f(i1)};
        if constexpr (ORDER == 2)
            e[2] = f(i1 + 1 == ng ? 0 : i1 + 1);
        coefs<ORDER>(ct + (ORDER + 1) * s, e);
    }
}

// Add a workgroup's ghost-padded LDS current tile (ncomp components) into the global
// current (hardware FP64 atomics); ghost slots go to their periodic nodes, zero entries
// (common when the particles are cell-sorted) are skipped.
__device__ __forceinline__ void tile_flush(const double *tile, double *J, int ncomp, int ng,
                                           int tw)
{
    for (int c = 0; c < ncomp; ++c)
        for (int j = threadIdx.x; j < tw; j += nthreads()) {
            const double val = tile[c * tw + j];
            if (val != 0.0)
                unsafeAtomicAdd(&J[c * ng + wrap_ghost(j - kGhost, ng)], val);
        }
}

__device__ __forceinline__ double read_lane(double v, int lane)
{
    return __hiloint2double(__builtin_amdgcn_readlane(__double2hiint(v), lane),
                            __builtin_amdgcn_readlane(__double2loint(v), lane));
}

// Deposit accumulator of one thread for NC current components (tile stride tw).
// DEP = 0: each particle adds its ORDER + 1 contributions with LDS atomics on a 64-bit
//          fixed-point tile (below).
// DEP = 1 (particles cell-sorted, so a thread's successive particles share a cell or
//          two): contributions are summed in registers over a window of ORDER + 3 nodes
//          anchored one node left of the stencil that opened it, and added to the tile
//          only when a particle's stencil leaves the window, and at the end.
// DEP = 2: a register window shared by the wavefront (below).
// DEP = 3: each particle adds its contributions with FP64 LDS atomics.
// Every kind has init(side, run), add(...), finish(tile, tw, ng); after the workgroup has
// synchronised, flush_tile(tile, J, ncomp, ng, tw) adds the tile into the global current.
template <int ORDER, int NC, int DEP> struct Depo;

// DEP = 0.  A contribution c is stored as round(c 2^S): one FMA against 1.5 2^52 rounds
// c 2^S to an integer exactly while |c 2^S| < 2^51, and the integer is added with
// ds_add_u64, which runs at about twice the rate of FP64 LDS atomics on random addresses.
// Sums inside a workgroup are then exact and independent of the order of the adds.  The
// scale 2^S is chosen at initialisation (k_fx_setup) so that twice the largest
// contribution of the initial particles, 2 max_p w_p |v_p| / h, stays below Run::fx_lim
// (<= 2^62 / chunk): each entry receives at most one contribution per particle of the
// workgroup, so no entry can overflow.  A contribution at or beyond the bound (a particle
// more than twice as fast as the fastest initial one, or a non-finite value) leaves the
// fixed-point path:
//   default            - it is added to an FP64 side tile with FP64 LDS atomics;
//   deterministic mode - it is rounded to a coarser fixed point, 2^(S - kFxCoarse), in the
//                        same side tile (as integers; exact and order-independent too),
//                        while |c| 2^(S - kFxCoarse) < fx_lim; beyond that (or not finite)
//                        it is dropped and `over` is set (the step is then reported as
//                        non-finite).
constexpr double kFxMagic = 6755399441055744.0;   // 1.5 * 2^52
constexpr int kFxCoarse = 12;

// The integer that v + kFxMagic (rounded) holds.
__device__ __forceinline__ long long fx_round_of(double sum)
{
    return __double_as_longlong(sum) - __double_as_longlong(kFxMagic);
}

__device__ __forceinline__ long long fx_round(double v) { return fx_round_of(v + kFxMagic); }

template <int ORDER, int NC> struct Depo<ORDER, NC, 0> {
    double *side;
    double scale, lim, inv;
    int det;
    int over;              // deterministic mode: a contribution was out of range
    __device__ __forceinline__ void init(double *side_tile, const Run &r, const DevState *st,
                                         int which = 0)
    {
        side = side_tile;
        // through vector loads (an index the compiler takes to differ by lane): a scalar
        // load would be waited for at once, before the loads and the clearing around it
        unsigned k = (unsigned)which;
        asm("" : "+v"(k));
        scale = st->fx_scale[k];
        inv = st->fx_inv[k];
        lim = r.fx_lim;
        det = r.det;
        over = 0;
    }
    // Before the first add: the scales (the same in every lane) into scalar registers.
    __device__ __forceinline__ void settle()
    {
        scale = read_lane(scale, 0);
        inv = read_lane(inv, 0);
    }
    __device__ __forceinline__ void add(double *jt, int tw, int ng, const Stencil<ORDER> &s,
                                        const double (&q)[NC], bool = true, bool = true)
    {
        add_at(jt, tw, slots_of<ORDER>(s, ng), s, q);
    }
    __device__ __forceinline__ void add_at(double *jt, int tw, const Slots<ORDER> &sl,
                                           const Stencil<ORDER> &s, const double (&q)[NC])
    {
        unsigned long long *ti = reinterpret_cast<unsigned long long *>(jt);
#pragma unroll
        for (int c = 0; c < NC; ++c) {
            const double qs = q[c] * scale;
            if (fabs(qs) < lim) {
#pragma unroll
                for (int k = 0; k <= ORDER; ++k) {
                    const double m = fma(qs, s.w[k], kFxMagic);
                    const long long iv = __double_as_longlong(m) - __double_as_longlong(kFxMagic);
                    atomicAdd(&ti[c * tw + sl.n[k]], (unsigned long long)iv);
                }
            } else if (!det) {
#pragma unroll
                for (int k = 0; k <= ORDER; ++k)
                    atomicAdd(&side[c * tw + sl.n[k]], q[c] * s.w[k]);
            } else {
                const double qc = qs * (1.0 / (double)(1 << kFxCoarse));
                if (fabs(qc) < lim) {
                    unsigned long long *si = reinterpret_cast<unsigned long long *>(side);
#pragma unroll
                    for (int k = 0; k <= ORDER; ++k)
                        atomicAdd(&si[c * tw + sl.n[k]], (unsigned long long)fx_round(qc * s.w[k]));
                } else {
                    over = 1;
                }
            }
        }
    }
    // The contributions of a lane's U particles: straight to the tile unless one of the
    // wavefront's is out of range.
    template <int U>
    __device__ __forceinline__ void add_all(double *jt, int tw, int ng, Pos (&p)[U],
                                            const double (&q)[U][NC], const bool (&valid)[U])
    {
        Stencil<ORDER> st[U];
        int b[U];
        stencils_at<ORDER, U>(st, b, p, ng);
        double qs[U][NC];
        bool out = false;
#pragma unroll
        for (int u = 0; u < U; ++u)
#pragma unroll
            for (int c = 0; c < NC; ++c) {
                qs[u][c] = q[u][c] * scale;
                out |= !(fabs(qs[u][c]) < lim);     // (lanes past the end carry no weight)
            }
        if (__any(out)) {
#pragma unroll
            for (int u = 0; u < U; ++u)
                if (valid[u])
                    add(jt, tw, ng, st[u], q[u]);
            return;
        }
        unsigned long long *ti = reinterpret_cast<unsigned long long *>(jt);
#pragma unroll
        for (int u = 0; u < U; ++u)
            if (valid[u])
#pragma unroll
                for (int c = 0; c < NC; ++c)
#pragma unroll
                    for (int k = 0; k <= ORDER; ++k)
                        atomicAdd(&ti[c * tw + b[u] + k],
                                  (unsigned long long)fx_round_of(fma(qs[u][c], st[u].w[k], kFxMagic)));
    }
    __device__ __forceinline__ void finish(double *, int, int) {}
    // Tile slot `idx` as a double: the integer sum times 2^-S plus the side tile.
    __device__ __forceinline__ double value(const double *jt, int idx) const
    {
        const double fine = (double)__double_as_longlong(jt[idx]) * inv;
        if (!det)
            return fine + side[idx];
        return fine + (double)__double_as_longlong(side[idx]) * (inv * (double)(1 << kFxCoarse));
    }
    // Default: each entry back to a double on its way into the global current (FP64
    // atomics).  Deterministic mode: J is this workgroup's row of the partial sums; node i
    // receives its interior slot and its periodic ghost images, added in slot order.
    __device__ __forceinline__ void flush_tile(const double *jt, double *J, int ncomp, int ng,
                                               int tw)
    {
        if (det) {
            for (int idx = threadIdx.x; idx < ncomp * ng; idx += nthreads()) {
                const int c = idx / ng, i = idx % ng;
                double acc = 0.0;
                for (int j = (i + kGhost) % ng; j < tw; j += ng)
                    acc += value(jt, c * tw + j);
                J[c * ng + i] = acc;
            }
            return;
        }
        for (int c = 0; c < ncomp; ++c)
            for (int j = threadIdx.x; j < tw; j += nthreads()) {
                const double val = value(jt, c * tw + j);
                if (val != 0.0)
                    unsafeAtomicAdd(&J[c * ng + wrap_ghost(j - kGhost, ng)], val);
            }
    }
};

template <int ORDER, int NC> struct Depo<ORDER, NC, 3> {
    int over = 0;
    __device__ __forceinline__ void init(double *, const Run &, const DevState *, int = 0) {}
    __device__ __forceinline__ void settle() {}
    __device__ __forceinline__ void add(double *jt, int tw, int ng, const Stencil<ORDER> &s,
                                        const double (&q)[NC], bool = true, bool = true)
    {
        add_at(jt, tw, slots_of<ORDER>(s, ng), s, q);
    }
    __device__ __forceinline__ void add_at(double *jt, int tw, const Slots<ORDER> &sl,
                                           const Stencil<ORDER> &s, const double (&q)[NC])
    {
#pragma unroll
        for (int c = 0; c < NC; ++c)
#pragma unroll
            for (int k = 0; k <= ORDER; ++k)
                atomicAdd(&jt[c * tw + sl.n[k]], q[c] * s.w[k]);
    }
    __device__ __forceinline__ void finish(double *, int, int) {}
    __device__ __forceinline__ void flush_tile(const double *jt, double *J, int ncomp, int ng,
                                               int tw)
    {
        tile_flush(jt, J, ncomp, ng, tw);
    }
};


template <int ORDER, int NC> struct Depo<ORDER, NC, 1> {
    static constexpr int W = ORDER + 3;
    int anchor;
    bool live;
    int over = 0;
    double acc[NC][W];
    __device__ __forceinline__ void settle() {}
    __device__ __forceinline__ void clear()
    {
#pragma unroll
        for (int c = 0; c < NC; ++c)
#pragma unroll
            for (int j = 0; j < W; ++j)
                acc[c][j] = 0.0;
    }
    __device__ __forceinline__ void init(double *, const Run &, const DevState *, int = 0)
    {
        live = false;
        anchor = 0;
        clear();
    }
    __device__ __forceinline__ void flush_tile(const double *jt, double *J, int ncomp, int ng,
                                               int tw)
    {
        tile_flush(jt, J, ncomp, ng, tw);
    }
    __device__ __forceinline__ void flush(double *jt, int tw, int ng)
    {
        if (!live)
            return;
#pragma unroll
        for (int j = 0; j < W; ++j) {
            const int slot = slot_of_node(anchor + j, ng);
#pragma unroll
            for (int c = 0; c < NC; ++c)
                if (acc[c][j] != 0.0)
                    atomicAdd(&jt[c * tw + slot], acc[c][j]);
        }
        clear();
    }
    __device__ __forceinline__ void add(double *jt, int tw, int ng, const Stencil<ORDER> &s,
                                        const double (&q)[NC], bool = true, bool = true)
    {
        int d = s.first - anchor;
        if (!live || d < 0 || d > W - ORDER - 1) {
            flush(jt, tw, ng);
            anchor = s.first - 1;
            live = true;
            d = 1;
        }
#pragma unroll
        for (int j = 0; j < W; ++j) {
            double a = 0.0;
#pragma unroll
            for (int k = 0; k <= ORDER; ++k)
                if (j - k >= 0 && j - k <= W - ORDER - 1)
                    a = (d == j - k) ? s.w[k] : a;
#pragma unroll
            for (int c = 0; c < NC; ++c)
                acc[c][j] = fma(q[c], a, acc[c][j]);
        }
    }
    __device__ __forceinline__ void finish(double *jt, int tw, int ng) { flush(jt, tw, ng); }
};

// Cross-lane move within rows of 16 lanes (DPP), for a double.
template <int CTRL> __device__ __forceinline__ double dpp_mov(double v)
{
    const int lo = __builtin_amdgcn_update_dpp(0, __double2loint(v), CTRL, 0xF, 0xF, false);
    const int hi = __builtin_amdgcn_update_dpp(0, __double2hiint(v), CTRL, 0xF, 0xF, false);
    return __hiloint2double(hi, lo);
}

// Sum over the 64 lanes of a wavefront (all lanes active): butterflies within rows of 16
// with DPP (quad permutations, half-row and row mirrors), then across rows.
__device__ __forceinline__ double wave_sum_dpp(double v)
{
    v += dpp_mov<0xB1>(v);     // quad_perm [1, 0, 3, 2]
    v += dpp_mov<0x4E>(v);     // quad_perm [2, 3, 0, 1]
    v += dpp_mov<0x141>(v);    // row_half_mirror
    v += dpp_mov<0x140>(v);    // row_mirror
    v += __shfl_xor(v, 16, 64);
    v += __shfl_xor(v, 32, 64);
    return v;
}

// DEP = 2 (particles cell-sorted; every lane of the wavefront calls add, with `valid`
// false past the end of the range): each lane sums its contributions in registers over a
// window of ORDER + 3 nodes shared by the whole wavefront.  The window is placed one node
// left of the stencil of the wavefront's first particle and stays put while that stencil
// remains inside it (sub-cell wobble does not move it); when it leaves, the window is
// summed across the wavefront (DPP) and one lane adds it to the LDS tile.  A run of
// sorted particles thus costs a few LDS atomics per wavefront instead of ORDER + 1 per
// particle.  A lane whose stencil is outside the window adds it with LDS atomics.  The
// window may move only at calls with `may_move` (the first particle of each batch), so
// the reduction code appears once in the unrolled particle loop.
template <int ORDER, int NC> struct Depo<ORDER, NC, 2> {
    static constexpr int W = ORDER + 3;
    int anchor;            // the same in every lane of the wavefront
    bool live;
    int over = 0;
    double acc[NC][W];
    __device__ __forceinline__ void settle() {}
    __device__ __forceinline__ void clear()
    {
#pragma unroll
        for (int c = 0; c < NC; ++c)
#pragma unroll
            for (int j = 0; j < W; ++j)
                acc[c][j] = 0.0;
    }
    __device__ __forceinline__ void init(double *, const Run &, const DevState *, int = 0)
    {
        live = false;
        anchor = 0;
        clear();
    }
    __device__ __forceinline__ void flush_tile(const double *jt, double *J, int ncomp, int ng,
                                               int tw)
    {
        tile_flush(jt, J, ncomp, ng, tw);
    }
    // all lanes of the wavefront active
    __device__ __forceinline__ void flush(double *jt, int tw, int ng)
    {
        if (!live)
            return;
        const bool lead = (threadIdx.x & 63) == 0;
#pragma unroll
        for (int j = 0; j < W; ++j) {
            const int slot = slot_of_node(anchor + j, ng);
#pragma unroll
            for (int c = 0; c < NC; ++c) {
                const double t = wave_sum_dpp(acc[c][j]);
                if (lead && t != 0.0)
                    atomicAdd(&jt[c * tw + slot], t);
            }
        }
        clear();
    }
    __device__ __forceinline__ void add(double *jt, int tw, int ng, const Stencil<ORDER> &s,
                                        const double (&q)[NC], bool valid, bool may_move)
    {
        if (may_move) {
            // lane 0 holds the wavefront's lowest particle index; invalid lanes are the
            // highest ones, so an invalid lane 0 means the whole wavefront is past the end
            const int f0 = __builtin_amdgcn_readfirstlane(s.first);
            const int v0 = __builtin_amdgcn_readfirstlane((int)valid);
            const int d0 = f0 - anchor;
            if (v0 && (!live || d0 < 0 || d0 > W - ORDER - 1)) {
                flush(jt, tw, ng);
                anchor = f0 - 1;
                live = true;
            }
        }
        if (!valid)
            return;
        if (!live) {
            // (only before the first window is placed) add directly
            const Slots<ORDER> sl = slots_of<ORDER>(s, ng);
#pragma unroll
            for (int c = 0; c < NC; ++c)
#pragma unroll
                for (int k = 0; k <= ORDER; ++k)
                    atomicAdd(&jt[c * tw + sl.n[k]], q[c] * s.w[k]);
            return;
        }
        const int d = s.first - anchor;
        if (d >= 0 && d <= W - ORDER - 1) {
#pragma unroll
            for (int j = 0; j < W; ++j) {
                double a = 0.0;
#pragma unroll
                for (int k = 0; k <= ORDER; ++k)
                    if (j - k >= 0 && j - k <= W - ORDER - 1)
                        a = (d == j - k) ? s.w[k] : a;
#pragma unroll
                for (int c = 0; c < NC; ++c)
                    acc[c][j] = fma(q[c], a, acc[c][j]);
            }
        } else {
            const Slots<ORDER> sl = slots_of<ORDER>(s, ng);
#pragma unroll
            for (int c = 0; c < NC; ++c)
#pragma unroll
                for (int k = 0; k <= ORDER; ++k)
                    atomicAdd(&jt[c * tw + sl.n[k]], q[c] * s.w[k]);
        }
    }
    __device__ __forceinline__ void finish(double *jt, int tw, int ng) { flush(jt, tw, ng); }
};

// A lane's U particles into any kind of accumulator (Depo<., ., 2> wants every lane).
template <int ORDER, int NC, int DEP, int U>
__device__ __forceinline__ void deposit_all(Depo<ORDER, NC, DEP> &dep, double *jt, int tw, int ng,
                                            Pos (&p)[U], const double (&q)[U][NC],
                                            const bool (&valid)[U], bool first = true)
{
    if constexpr (DEP == 0) {
        dep.template add_all<U>(jt, tw, ng, p, q, valid);
    } else {
#pragma unroll
        for (int u = 0; u < U; ++u) {
            near_offset<ORDER>(p[u]);
            if (DEP == 2 || valid[u])
                dep.add(jt, tw, ng, stencil_at<ORDER>(p[u]), q[u], valid[u], first && u == 0);
        }
    }
}

// Periodic position in [0, L).  A particle moves less than a period per step, so one
// conditional add or subtract almost always suffices; otherwise x - L floor(x / L),
// with rounding that lands on L mapped to 0.
__device__ __forceinline__ double wrap_pos(double x, double L)
{
    if (x < 0.0)
        x += L;
    else if (x >= L)
        x -= L;
    if (x < 0.0 || x >= L || !(x == x)) {
        x = x - L * floor(x / L);
        if (x < 0.0)
            x += L;
        if (x >= L)
            x = 0.0;
    }
    return x;
}

// The passes' periodic positions: x1 - L floor(x1 / L) in one rounding, which is x1, x1 + L
// or x1 - L for a particle that moved less than a period; what lands outside [0, L) by the
// rounding of x1 / L (or is not finite) goes through wrap_pos.
template <int U>
__device__ __forceinline__ void wrap_all(double (&xw)[U], const double (&x1)[U], const Run &r)
{
    bool out = false;
#pragma unroll
    for (int u = 0; u < U; ++u) {
        xw[u] = fma(-r.L, floor(x1[u] * r.inv_L), x1[u]);
        out |= !(xw[u] >= 0.0 && xw[u] < r.L);
    }
    if (__any(out)) {
#pragma unroll
        for (int u = 0; u < U; ++u)
            if (!(xw[u] >= 0.0 && xw[u] < r.L))
                xw[u] = wrap_pos(x1[u], r.L);
    }
}

__device__ __forceinline__ double wrap_one(double x1, const Run &r)
{
    const double in[1] = {x1};
    double xw[1];
    wrap_all<1>(xw, in, r);
    return xw[0];
}

// Exact charge conservation (section 3.5; Run::cc; tent shapes): the centred current and
// v-dagger's field go through the pieces of the particle's path x0 -> x1 (x0 wrapped, as
// stored; x1 unwrapped) between the half nodes, where the tent has its kinks.  In
// u = x / h - 1/2 the half nodes are the integers; a piece [s, e] is visited at its
// midpoint with the fraction (e - s) / |u1 - u0| of the path (on a piece the tent is
// linear, so its value at the midpoint is its time average there, and eq. (detbal) holds
// piece by piece).  Coordinates are taken relative to the whole cell `base` = floor(u0),
// and the end point as its wrapped image's u plus the whole periods in between: that is
// the number the next step starts from, whereas x / h itself is not exactly periodic in
// floating point (over many boundary crossings the difference would drift Gauss' law).
// The pieces of a path lie in consecutive cells, so the cell and its slot are counted up from
// the first one instead of being found again from each midpoint; visit(slot, d, frac) gets the
// slot of the cell's lower half node and the midpoint's offset in the cell.  A path with no
// length, or one longer than 2^30 cells (only a non-finite or absurd state), is one piece.
template <typename F>
__device__ __forceinline__ void cc_pieces(const Run &r, double x0, double x1, F &&visit)
{
    const double ua = x0 * r.inv_h - 0.5;
    const double base = floor(ua);
    const double xw = wrap_one(x1, r);
    // whole periods between x1 and xw (x1 - xw is a multiple of L up to rounding)
    const double m = rint((x1 - xw) * r.inv_L);
    const double ta = ua - base;
    const double tb = (xw * r.inv_h - 0.5) + (m * (double)r.ng - base);
    const double lo = fmin(ta, tb), hi = fmax(ta, tb), len = hi - lo;
    const bool one = !(len > 0.0) || !(len < 1073741824.0);
    double t = one ? 0.5 * (ta + tb) : lo;
    double f = floor(t);
    int node = (int)(base + f);
    const unsigned lim = (unsigned)(r.ng + 2 * kGhost - 2);
    auto slot = [&](int n) {
        const unsigned b = (unsigned)n + kGhost;
        return b <= lim ? (int)b : wrap_node(n, r.ng) + kGhost;
    };
    if (one) {
        visit(slot(node), t - f, 1.0);
        return;
    }
    double il = __builtin_amdgcn_rcp(len);          // one reciprocal per path
    il = fma(il, fma(-len, il, 1.0), il);
    il = fma(il, fma(-len, il, 1.0), il);
    for (;;) {
        const double e = fmin(f + 1.0, hi);
        visit(slot(node), 0.5 * (t + e) - f, (e - t) * il);
        if (e >= hi)
            break;
        t = e;
        f += 1.0;
        node = (int)((unsigned)node + 1u);
    }
}

// The tent stencil of a piece and its slots.
__device__ __forceinline__ Stencil<1> cc_stencil(double d)
{
    Stencil<1> s;
    s.first = 0;            // (the slot is known)
    s.w[0] = 1.0 - d;
    s.w[1] = d;
    return s;
}

__device__ __forceinline__ Slots<1> cc_slots(int slot)
{
    Slots<1> o;
    o.n[0] = slot;
    o.n[1] = slot + 1;
    return o;
}

// v-dagger's field through the pieces of the path x0 -> x1 (tent coefficient tile ct).
__device__ __forceinline__ double cc_gather(const Run &r, const double *ct, double x0, double x1)
{
    double acc = 0.0;
    cc_pieces(r, x0, x1, [&](int slot, double d, double f) {
        Cell<1> c;
        c.base = slot;
        c.d = d;
        acc = fma(f, gather_poly<1>(ct, c), acc);
    });
    return acc;
}


// --------------------------------------------------------------- block reductions
// Workgroup barrier that orders LDS only.  __syncthreads also waits for every global load
// and store the wavefront has in flight (particle writes, the last prefetch), which costs
// microseconds at the end of a pass; exchanges through LDS need only the LDS operations
// complete.  Global memory written before it is not made visible to the workgroup.
__device__ __forceinline__ void lds_barrier()
{
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup", "local");
    __builtin_amdgcn_s_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup", "local");
}

// Sum (max) over the 64 lanes of a wavefront, all lanes active; every lane gets the same
// value.  Within each row of 16 lanes, DPP butterflies (quad permutations, half-row and row
// mirrors) leave the row's sum in all of its lanes (each addition pairs the same two
// values in both lanes, so the lanes agree bit for bit); the four row sums are then read
// from lanes 0, 16, 32, 48 and combined in that order.  No LDS round trips.
__device__ __forceinline__ double wave_sum(double v)
{
    v += dpp_mov<0xB1>(v);     // quad_perm [1, 0, 3, 2]
    v += dpp_mov<0x4E>(v);     // quad_perm [2, 3, 0, 1]
    v += dpp_mov<0x141>(v);    // row_half_mirror
    v += dpp_mov<0x140>(v);    // row_mirror
    return ((read_lane(v, 0) + read_lane(v, 16)) + read_lane(v, 32)) + read_lane(v, 48);
}

__device__ __forceinline__ double wave_max(double v)
{
    v = fmax(v, dpp_mov<0xB1>(v));
    v = fmax(v, dpp_mov<0x4E>(v));
    v = fmax(v, dpp_mov<0x141>(v));
    v = fmax(v, dpp_mov<0x140>(v));
    return fmax(fmax(fmax(read_lane(v, 0), read_lane(v, 16)), read_lane(v, 32)), read_lane(v, 48));
}

// LDS for the block reductions: up to 4 values per wavefront of a 1024-thread workgroup.
constexpr int kRedSize = 64;
// Ordered sums over many rows (k_reduce_partials): a workgroup of 256 threads
// takes kRedEntries consecutive entries, kRedSegments threads per entry.
constexpr int kRedEntries = 32, kRedSegments = 8;

// Deterministic reduction of N values over the workgroup in one round of LDS: value k is
// summed, or maximised where bit k of MAXMASK is set, always in the same fixed order for a
// given blockDim (so a value gives the same result whatever is reduced beside it); every
// thread gets the results.  red: kRedSize doubles of LDS.  The barriers order LDS only.
template <unsigned MAXMASK, int N>
__device__ __forceinline__ void block_reduce(double (&v)[N], double *red)
{
    static_assert(N >= 1 && N * 16 <= kRedSize, "reduction too wide");
    const int lane = threadIdx.x & 63, wid = threadIdx.x >> 6, nw = (nthreads() + 63) >> 6;
#pragma unroll
    for (int k = 0; k < N; ++k)
        v[k] = (MAXMASK >> k) & 1u ? wave_max(v[k]) : wave_sum(v[k]);
    lds_barrier();
    if (lane == 0) {
#pragma unroll
        for (int k = 0; k < N; ++k)
            red[k * 16 + wid] = v[k];
    }
    lds_barrier();
#pragma unroll
    for (int k = 0; k < N; ++k) {
        const double *rk = red + k * 16;
        double t;
        if ((MAXMASK >> k) & 1u) {
            t = rk[0];
            for (int i = 1; i < nw; ++i)
                t = fmax(t, rk[i]);
        } else {
            t = 0.0;
            for (int i = 0; i < nw; ++i)
                t += rk[i];
        }
        v[k] = t;
    }
    lds_barrier();
}

// A block reduction in two halves around a barrier that the caller has anyway:
// wave_partials leaves each wavefront's value k in red; after the barrier wave_total(red, k,
// nw) combines the nw wavefronts' values, in every lane of any wavefront that asks (all
// lanes active).  The lanes read the values side by side and combine them within rows of 16
// (DPP), a fixed order; reading them one after the other, as block_reduce does, is a chain of
// nw LDS round trips.
template <unsigned MAXMASK, int N>
__device__ __forceinline__ void wave_partials(const double (&v)[N], double *red)
{
    static_assert(N >= 1 && N * 16 <= kRedSize, "reduction too wide");
    const int wid = threadIdx.x >> 6;
#pragma unroll
    for (int k = 0; k < N; ++k) {
        const double t = (MAXMASK >> k) & 1u ? wave_max(v[k]) : wave_sum(v[k]);
        if ((threadIdx.x & 63) == 0)
            red[k * 16 + wid] = t;
    }
}

template <bool MAX = false>
__device__ __forceinline__ double wave_total(const double *red, int k, unsigned nw)
{
    const unsigned i = threadIdx.x & 15;
    double v = red[k * 16 + (i < nw ? i : 0)];
    if (!MAX && i >= nw)
        v = 0.0;
    if constexpr (MAX) {
        v = fmax(v, dpp_mov<0xB1>(v));
        v = fmax(v, dpp_mov<0x4E>(v));
        v = fmax(v, dpp_mov<0x141>(v));
        v = fmax(v, dpp_mov<0x140>(v));
    } else {
        v += dpp_mov<0xB1>(v);
        v += dpp_mov<0x4E>(v);
        v += dpp_mov<0x141>(v);
        v += dpp_mov<0x140>(v);
    }
    return v;
}

__device__ __forceinline__ double block_sum(double v, double *red)
{
    double a[1] = {v};
    block_reduce<0u>(a, red);
    return a[0];
}

// Mean of n values (LDS or global), identical in every workgroup of a launch.
__device__ __forceinline__ double block_mean(const double *a, int n, double *red)
{
    double s = 0.0;
    for (int i = threadIdx.x; i < n; i += nthreads())
        s += a[i];
    return block_sum(s, red) / n;
}


// Component value J[i] summed over nrep <= kMaxRep replicas of stride rs, in replica
// order; the loads are issued together, without a branch (those past nrep repeat the last
// replica and count as zero).
__device__ __forceinline__ double rep_sum(const double *J, int i, int nrep, int rs)
{
    double a[kMaxRep];
#pragma unroll
    for (int k = 0; k < kMaxRep; ++k)
        a[k] = (J + (size_t)((unsigned)min(k, nrep - 1) * (unsigned)rs))[i];
    double s = a[0];
#pragma unroll
    for (int k = 1; k < kMaxRep; ++k)
        s += k < nrep ? a[k] : 0.0;
    return s;
}

// Sum of the replicas of the first n values of J into dst (LDS or global).
__device__ __forceinline__ void rep_gather(double *dst, const double *J, int n, int nrep, int rs)
{
    for (int i = threadIdx.x; i < n; i += nthreads())
        dst[i] = rep_sum(J, i, nrep, rs);
}

// Zero every replica of the first n values of J.
__device__ __forceinline__ void rep_zero(double *J, int n, int nrep, int rs)
{
    for (int k = 0; k < nrep; ++k)
        for (int i = threadIdx.x; i < n; i += nthreads())
            J[(size_t)k * rs + i] = 0.0;
}

// Zero share `part` of `nparts` >= nrep of every replica of the first n values of J (the
// shares together cover them once), so that all workgroups of a launch share the clearing:
// share p takes a slice of replica p mod nrep.
__device__ __forceinline__ void rep_zero_part(double *J, int n, int nrep, int rs, int part,
                                              int nparts, unsigned nt)
{
    const unsigned k = (unsigned)part % (unsigned)nrep, j = (unsigned)part / (unsigned)nrep;
    const unsigned slices = ((unsigned)nparts - k + nrep - 1) / (unsigned)nrep;
    const unsigned per = ((unsigned)n + slices - 1) / slices;
    const unsigned e1 = min((unsigned)n, (j + 1) * per);
    double *Jk = J + (size_t)k * rs;
    for (unsigned e = j * per + threadIdx.x; e < e1; e += nt)
        Jk[e] = 0.0;
}

// The replica a workgroup adds into.
__device__ __forceinline__ double *rep_slot(double *J, int nrep, int ng)
{
    return J + (size_t)(blockIdx.x % nrep) * 3 * ng;
}

// Where a workgroup's deposit tile goes: its replica of the current J, or in the
// deterministic mode its own row of the partial sums (k_reduce_partials then writes J).
// Called in the prologue, under the loads (its modulo is a chain of 20 instructions).
__device__ __forceinline__ double *dep_target(const Run &r, const Work &wk, double *J)
{
    double *t = r.det ? wk.part + (size_t)blockIdx.x * 3 * r.ng : rep_slot(J, r.nrep, r.ng);
    settle_pointer(t);
    return t;
}

// A deterministic-mode deposit met a value it cannot hold: report it with the next record.
template <typename D> __device__ __forceinline__ void flag_over(const D &dep, const Work &wk)
{
    if (dep.over)
        atomicOr(&wk.st->flag_a, 1);
}

__device__ __forceinline__ void tile_load(double *dst, const double *src, int n,
                                          unsigned nt = nthreads())
{
    for (int i = threadIdx.x; i < n; i += nt)
        dst[i] = src[i];
}

__device__ __forceinline__ void tile_zero(double *dst, int n,
                                          unsigned nt = nthreads())
{
    for (int i = threadIdx.x; i < n; i += nt)
        dst[i] = 0.0;
}

// Fill the ghost slots of ncomp tile components from their periodic images (the
// interior must be written and visible).
__device__ __forceinline__ void ghost_fill(double *tile, int ncomp, int ng, int tw,
                                          unsigned nt = nthreads())
{
    for (int idx = threadIdx.x; idx < ncomp * 2 * kGhost; idx += nt) {
        const int c = idx / (2 * kGhost), j = idx % (2 * kGhost);
        const int slot = j < kGhost ? j : ng + j;
        tile[c * tw + slot] = tile[c * tw + wrap_ghost(slot - kGhost, ng) + kGhost];
    }
}

// Interiors of the ghost-padded E [3][tw] and B [2][tw] tiles from a field block
// E [3][ng] | B [2][ng] (Work::ps or Work::pf); the caller fills the ghosts.
__device__ __forceinline__ void psatd_tiles(const Run &r, const double *src, double *et, double *bt,
                                            unsigned nt)
{
    const int ng = r.ng, tw = r.tw, n = 5 * ng;
    auto put = [&](int idx, double v) {
        const int c = (idx >= ng) + (idx >= 2 * ng) + (idx >= 3 * ng) + (idx >= 4 * ng);
        if (idx < n)
            (c < 3 ? et + c * tw : bt + (c - 3) * tw)[kGhost + idx - c * ng] = v;
    };
    for (int idx = threadIdx.x; idx < n; idx += 2 * (int)nt) {
        const double v0 = src[idx], v1 = src[min(idx + (int)nt, n - 1)];
        put(idx, v0);
        put(idx + (int)nt, v1);
    }
}

// ------------------------------------------------------------------ grid operations
// Staggered differences: nodes f[i] at i h, half nodes g[i] at (i + 1/2) h.
__device__ __forceinline__ double dplus(const double *f, int i, int ng, double inv_h)
{
    return (f[i + 1 == ng ? 0 : i + 1] - f[i]) * inv_h;
}
__device__ __forceinline__ double dminus(const double *g, int i, int ng, double inv_h)
{
    return (g[i] - g[i == 0 ? ng - 1 : i - 1]) * inv_h;
}

// EMEC(LF) magnetic half step at half node i, component c (0: B_y, 1: B_z):
// B^{n+1/2} = B^{n-1/2} - dt curl E^n, (curl E)_y = -D+E_z, (curl E)_z = D+E_y
// (eq. (EMleapfrog), second line).  E [3][ng], B [2][ng] in global memory.
__device__ __forceinline__ double lf_bhalf(const Run &r, const double *E, const double *B, int c,
                                           int i)
{
    const int ng = r.ng, ip = i + 1 == ng ? 0 : i + 1;
    if (c == 0)
        return B[i] + r.dt * ((E[2 * ng + ip] - E[2 * ng + i]) * r.inv_h);
    return B[ng + i] - r.dt * ((E[ng + ip] - E[ng + i]) * r.inv_h);
}

// EMEC(LF)'s magnetic energy of the state (E^n, B^{n-1/2}) (section 4.1):
// W_B^n = c^2/2 h sum B^{n+1/2} . B^{n-1/2}.  Computed by one wavefront (all lanes active)
// in an order fixed by N_g alone, so that every writer of a record (a pass's lead, the
// end-of-call launch, initialisation) gets the same bits.
__device__ __forceinline__ double lf_magnetic_energy(const Run &r, const double *E, const double *B)
{
    const int ng = r.ng;
    double s = 0.0;
    for (int idx = threadIdx.x & 63; idx < 2 * ng; idx += 64) {
        const int c = idx >= ng ? 1 : 0, i = idx - c * ng;
        s = fma(lf_bhalf(r, E, B, c, i), B[idx], s);
    }
    return 0.5 * r.c2 * r.h * wave_sum(s);
}

// Electromagnetic predictor fields into the interiors of the LDS tiles es [3][tw], bs [2][tw]
// from E^n, B^n and j^{n,*} (the caller fills the ghosts; the electrostatic passes build
// theirs from NodeLoad):
//   EM   : E* = E + dt/2 (c^2 curl B - j), B* = B - dt/2 curl E   (eq. (EMbasic))
//   EMEC(LF): B^{n+1/2} = B - dt curl E into bs, E* = E + dt/2 (c^2 curl B^{n+1/2} - j)
//          (eq. (EMleapfrog); the workgroup synchronises between the two)
// In 1D: (curl B)_y = -D-B_z, (curl B)_z = D-B_y, (curl E)_y = -D+E_z, (curl E)_z = D+E_y.
__device__ __forceinline__ void predictor_fields(const Run &r, const double *E, const double *B,
                                 const double *J, double *es, double *bs, int nrep)
{
    const int ng = r.ng, tw = r.tw, rs = 3 * ng;
    double *e0 = es + kGhost, *b0 = bs + kGhost;
    const double *Ex = E, *Ey = E + ng, *Ez = E + 2 * ng;
    const double *By = B, *Bz = B + ng;
    if (r.scheme == kLeapfrog) {
        // B^{n+1/2} into bs first (E* takes its curl), then E* (eq. (EMleapfrog))
        for (int i = threadIdx.x; i < ng; i += nthreads()) {
            b0[i] = lf_bhalf(r, E, B, 0, i);
            b0[tw + i] = lf_bhalf(r, E, B, 1, i);
        }
        lds_barrier();
        for (int i = threadIdx.x; i < ng; i += nthreads()) {
            const int im = i == 0 ? ng - 1 : i - 1;
            e0[i] = Ex[i] - r.hdt * rep_sum(J, i, nrep, rs);
            e0[tw + i] = Ey[i] + r.hdt * (-r.c2 * ((b0[tw + i] - b0[tw + im]) * r.inv_h)
                                          - rep_sum(J, ng + i, nrep, rs));
            e0[2 * tw + i] = Ez[i] + r.hdt * (r.c2 * ((b0[i] - b0[im]) * r.inv_h)
                                              - rep_sum(J, 2 * ng + i, nrep, rs));
        }
        return;
    }
    for (int i = threadIdx.x; i < ng; i += nthreads()) {
        e0[i] = Ex[i] - r.hdt * rep_sum(J, i, nrep, rs);
        e0[tw + i] = Ey[i] + r.hdt * (-r.c2 * dminus(Bz, i, ng, r.inv_h) - rep_sum(J, ng + i, nrep, rs));
        e0[2 * tw + i] = Ez[i] + r.hdt * (r.c2 * dminus(By, i, ng, r.inv_h) - rep_sum(J, 2 * ng + i, nrep, rs));
        b0[i] = By[i] + r.hdt * dplus(Ez, i, ng, r.inv_h);
        b0[tw + i] = Bz[i] - r.hdt * dplus(Ey, i, ng, r.inv_h);
    }
}

// Electromagnetic field update (EMEC(LI)) from the centred current J (global): new fields
// into e1 [3][ng] and b1 [2][ng] (LDS), averaged fields into the interiors of the tiles eb
// [3][tw], bb [2][tw] (the caller fills the ghosts).  Single runs take these from the field
// launch (k_em_fields) instead; the batched form solves them here.
//   a = dt/2, s = a^2 c^2, L_h = D-D+, eq. (EMbasic) with Crank-Nicolson:
//     (I - s L_h) E_y' = (I + s L_h) E_y - dt c^2 D-B_z - dt j_y,  B_z' = B_z - a D+(E_y + E_y')
//     (I - s L_h) E_z' = (I + s L_h) E_z + dt c^2 D-B_y - dt j_z,  B_y' = B_y + a D+(E_z + E_z')
//     E_x' = E_x - dt j_x
//   The circulant system is solved with the first row g of its inverse.
// scratch: 7 N_g doubles of LDS (E^n, B^n, right-hand sides).
__device__ __forceinline__ void field_update(const Run &r, const Work &wk, const double *E, const double *B,
                             const double *J, double *e1, double *b1, double *eb, double *bb,
                             double *scratch, int nrep)
{
    const int ng = r.ng, tw = r.tw, rs = 3 * ng;
    double *E0 = scratch;            // [3][ng]
    double *B0 = E0 + 3 * ng;        // [2][ng]
    double *R = B0 + 2 * ng;         // [2][ng]
    double *g2 = b1;                 // [2][ng]: g twice (b1 is written after their last use)
    tile_load(E0, E, 3 * ng);
    tile_load(B0, B, 2 * ng);
    for (int i = threadIdx.x; i < ng; i += nthreads())
        g2[i] = g2[ng + i] = wk.cninv[i];
    __syncthreads();
    const double a = r.hdt, s = a * a * r.c2, ih2 = r.inv_h * r.inv_h;
    const double *Ey = E0 + ng, *Ez = E0 + 2 * ng, *By = B0, *Bz = B0 + ng;
    for (int i = threadIdx.x; i < ng; i += nthreads()) {
        const int ip = i + 1 == ng ? 0 : i + 1, im = i == 0 ? ng - 1 : i - 1;
        e1[i] = E0[i] - r.dt * rep_sum(J, i, nrep, rs);
        R[i] = Ey[i] + s * (Ey[ip] - 2.0 * Ey[i] + Ey[im]) * ih2
               - r.dt * r.c2 * dminus(Bz, i, ng, r.inv_h) - r.dt * rep_sum(J, ng + i, nrep, rs);
        R[ng + i] = Ez[i] + s * (Ez[ip] - 2.0 * Ez[i] + Ez[im]) * ih2
                    + r.dt * r.c2 * dminus(By, i, ng, r.inv_h) - r.dt * rep_sum(J, 2 * ng + i, nrep, rs);
    }
    __syncthreads();
    // (The row twice over, so that no index wraps: with a selection on each one it was left to
    // the registers of the surrounding pass whether the reads overlap, and the solve took what
    // they gave: batches of 16 runs of 1e5 particles x 512 cells 225 to 290 us a step, now 155.)
    for (int i = threadIdx.x; i < ng; i += nthreads()) {
        const double *gi = g2 + ng + i;
        double ay = 0.0, az = 0.0;
#pragma unroll 4
        for (int j = 0; j < ng; ++j) {
            ay += gi[-j] * R[j];
            az += gi[-j] * R[ng + j];
        }
        e1[ng + i] = ay;
        e1[2 * ng + i] = az;
    }
    __syncthreads();
    for (int i = threadIdx.x; i < ng; i += nthreads()) {
        const int ip = i + 1 == ng ? 0 : i + 1;
        b1[ng + i] = Bz[i] - a * ((Ey[ip] + e1[ng + ip]) - (Ey[i] + e1[ng + i])) * r.inv_h;
        b1[i] = By[i] + a * ((Ez[ip] + e1[2 * ng + ip]) - (Ez[i] + e1[2 * ng + i])) * r.inv_h;
    }
    __syncthreads();
    for (int i = threadIdx.x; i < 3 * ng; i += nthreads())
        eb[(i / ng) * tw + kGhost + i % ng] = 0.5 * (E0[i] + e1[i]);
    for (int i = threadIdx.x; i < 2 * ng; i += nthreads())
        bb[(i / ng) * tw + kGhost + i % ng] = 0.5 * (B0[i] + b1[i]);
}

// EMEC(LF)'s full step in pass B (eq. (EMleapfrog)), after predictor_fields has put
// B^{n+1/2} into the interior of bs: E^{n+1} = E^n + dt (c^2 curl B^{n+1/2} - j^{*,n+1/2})
// into e1 [3][ng], B^{n+1/2} (the next state's B) into b1 [2][ng], and what v-dagger
// gathers into the interiors of eb ((E^n + E^{n+1})/2) and bb (B^{n+1/2}).
__device__ __forceinline__ void lf_full_fields(const Run &r, const double *E, const double *J,
                                               const double *bs, double *e1, double *b1,
                                               double *eb, double *bb, int nrep)
{
    const int ng = r.ng, tw = r.tw, rs = 3 * ng;
    const double *by = bs + kGhost, *bz = bs + tw + kGhost;
    for (int i = threadIdx.x; i < ng; i += nthreads()) {
        const int im = i == 0 ? ng - 1 : i - 1;
        const double ex = E[i], ey = E[ng + i], ez = E[2 * ng + i];
        const double nx = ex - r.dt * rep_sum(J, i, nrep, rs);
        const double ny = ey + r.dt * (-r.c2 * ((bz[i] - bz[im]) * r.inv_h) - rep_sum(J, ng + i, nrep, rs));
        const double nz = ez + r.dt * (r.c2 * ((by[i] - by[im]) * r.inv_h) - rep_sum(J, 2 * ng + i, nrep, rs));
        e1[i] = nx;
        e1[ng + i] = ny;
        e1[2 * ng + i] = nz;
        eb[kGhost + i] = 0.5 * (ex + nx);
        eb[tw + kGhost + i] = 0.5 * (ey + ny);
        eb[2 * tw + kGhost + i] = 0.5 * (ez + nz);
        b1[i] = by[i];
        b1[ng + i] = bz[i];
        bb[kGhost + i] = by[i];
        bb[tw + kGhost + i] = bz[i];
    }
}

// What an electrostatic pass builds its fields from, one node per thread and round: E^n and
// the replicas of the predictor current (J1) and, in pass B, of the centred current (J2);
// null: none (ESEC1 has no predictor current).  issue() starts the loads, commit() sums
// the replicas in order and leaves the three values of the node in LDS.  The passes issue the
// first round, then their first particle loads (completions are counted in order, so loads
// issued before these would be waited for too) and the clearing of their tiles, and commit
// after that, so the clearing is done while the loads are under way.
// (All kMaxRep replicas are read without a branch; those past nrep repeat the last one and
// count as zero.)
template <bool TWO> struct NodeLoad {
    double e, a[kMaxRep], b[TWO ? kMaxRep : 1];
    __device__ __forceinline__ void issue(const Run &r, const double *E, const double *J1,
                                          const double *J2, int node)
    {
        live = J1 ? r.nrep : 0;
        // (wavefronts without a node load nothing: the loads of a 1024-thread workgroup on
        // 256 cells would otherwise keep the CU's memory pipe busy for about a microsecond)
        if (__builtin_amdgcn_readfirstlane(node) >= r.ng)
            return;
        const unsigned i = (unsigned)min(node, r.ng - 1);
        const unsigned rs = 3u * (unsigned)r.ng;
        const double *A = J1 ? J1 : E;
        const int na = J1 ? r.nrep : 1;
        e = E[i];
#pragma unroll
        for (int k = 0; k < kMaxRep; ++k) {
            a[k] = (A + (size_t)((unsigned)min(k, na - 1) * rs))[i];
            if constexpr (TWO)
                b[k] = (J2 + (size_t)((unsigned)min(k, r.nrep - 1) * rs))[i];
        }
    }
    int live;             // replicas of J1 that count
    __device__ __forceinline__ void commit(const Run &r, int i, double *re, double *ra, double *rb,
                                           double &sa, double &sb, double *save) const
    {
        if (i >= r.ng)
            return;
        double ja = live > 0 ? a[0] : 0.0;
#pragma unroll
        for (int k = 1; k < kMaxRep; ++k)
            ja += k < live ? a[k] : 0.0;
        re[i] = e;
        ra[i] = ja;
        sa += ja;
        if constexpr (TWO) {
            double jb = b[0];
#pragma unroll
            for (int k = 1; k < kMaxRep; ++k)
                jb += k < r.nrep ? b[k] : 0.0;
            rb[i] = jb;
            sb += jb;
            if (save) {
                save[i] = e;
                save[r.ng + i] = ja;
                save[2 * r.ng + i] = jb;
            }
        }
    }
};

// The rounds after the first (grids with more nodes than the workgroup has threads), two
// nodes in flight per thread.
template <bool TWO>
__device__ __forceinline__ void node_rounds(const Run &r, const double *E, const double *J1,
                                            const double *J2, double *re, double *ra, double *rb,
                                            double &sa, double &sb, double *save, int nt)
{
    for (int i = threadIdx.x + nt; i < r.ng; i += 2 * nt) {
        NodeLoad<TWO> p, q;
        p.issue(r, E, J1, J2, i);
        q.issue(r, E, J1, J2, i + nt);
        p.commit(r, i, re, ra, rb, sa, sb, save);
        q.commit(r, i + nt, re, ra, rb, sa, sb, save);
    }
}

// W_E = h/2 sum |E|^2 and W_B = c^2 h/2 sum |B|^2 (section 5.1) of LDS/global fields;
// every thread gets the result.
__device__ __forceinline__ void field_energies(const Run &r, const double *E, const double *B, double *we,
                               double *wb, double *red)
{
    const bool em = em_scheme(r.scheme);
    const int ng = r.ng, ne = em ? 3 : 1;
    double se = 0.0, sb = 0.0;
    for (int i = threadIdx.x; i < ne * ng; i += nthreads())
        se += E[i] * E[i];
    if (em)
        for (int i = threadIdx.x; i < 2 * ng; i += nthreads())
            sb += B[i] * B[i];
    *we = 0.5 * r.h * block_sum(se, red);
    *wb = em ? 0.5 * r.c2 * r.h * block_sum(sb, red) : 0.0;
}

// Write the record of `step` from the pass-B scalars of every workgroup and the field
// energies in st.  One wavefront (all lanes active) writes it, without a barrier, so in a
// pass the lead workgroup's other wavefronts go on with its particles meanwhile: the record
// is a chain of three memory round trips (2.5 us at 256 workgroups), which used to sit in
// front of the lead's particles (pass A of Landau 1e5 x 64: 7.2 us on the lead, 5.9 on the
// others).  Lane l takes workgroups l, l + 64, ... in turn and the lanes are summed in a fixed
// order, so every writer of a record gets the same bits.
// The standard scheme (Run::scheme == kStandard) has its fields at half steps: its record
// of step n >= 1 is TE at (n - 1/2) dt, the mean of the kinetic energies of steps n - 1
// (slot 4, written by the same pass) and n plus the field energy of E^{n-1/2}.
__device__ __forceinline__ void write_record(const Run &r, const Work &wk, int64_t step)
{
    const bool half = r.scheme == kStandard && step > 0;
    const int lane = threadIdx.x & 63;
    DevState *st = wk.st;
    const double we = st->we, wb = st->wb, te_start = st->te0;
    const int64_t fb_before = step == 0 ? 0 : st->fb_total;
    const int32_t sticky = step == 0 ? 0 : st->nonfinite_sticky;
    double ke = 0.0, fb = 0.0, gd = 0.0, nf = 0.0;
#pragma unroll 4
    for (int b = lane; b < r.nblocks; b += 64) {
        const double *sp = wk.spart + (size_t)b * kNS;
        ke += half ? 0.5 * (sp[0] + sp[4]) : sp[0];
        fb += sp[1];
        gd = fmax(gd, sp[2]);
        nf = fmax(nf, sp[3]);
    }
    ke = wave_sum(ke);
    fb = wave_sum(fb);
    gd = wave_max(gd);
    nf = wave_max(nf);
    if (lane == 0) {
        // (exchanged: workgroups of this pass may set it for the next record meanwhile; only
        // the deterministic mode sets it, and the round trip is on the record's chain: Landau
        // runs 265 -> 261 us per 20 steps at 1e4 particles without it)
        if (r.det && atomicExch(&st->flag_a, 0))
            nf = 1.0;
        const double te = ke + we + wb, te0 = step == 0 ? te : te_start;
        const int64_t fb_total = fb_before + (int64_t)fb;
        st->te0 = te0;
        st->fb_total = fb_total;
        st->nonfinite_sticky = sticky | (nf != 0.0);
        DevRecord rec;
        rec.step = step;
        rec.time = ((double)step - (half ? 0.5 : 0.0)) * r.dt;
        rec.kinetic = ke;
        rec.field_e = we;
        rec.field_b = wb;
        rec.total = te;
        rec.rel_energy_err = fabs(te - te0) / te0;
        rec.max_gamma_dev = gd;
        rec.fallbacks = (int64_t)fb;
        rec.fallbacks_total = fb_total;
        rec.nonfinite = nf != 0.0;
        rec.pad = 0;
        wk.rec[step < ((int64_t)1 << 31) ? (int64_t)((uint32_t)step % (uint32_t)r.rec_cap) : step % r.rec_cap] = rec;
        st->recorded = step;
    }
}

// The wavefront of a workgroup that writes records and energies: its last one.
__device__ __forceinline__ bool record_wave(unsigned nt = nthreads())
{
    return (unsigned)__builtin_amdgcn_readfirstlane(threadIdx.x >> 6) == (nt >> 6) - 1;
}

// h/2 sum_i f(i) over n values, by one wavefront (all lanes active).
template <typename F> __device__ __forceinline__ double wave_energy(double half_h, int n, F &&f)
{
    double s = 0.0;
    for (int i = threadIdx.x & 63; i < n; i += 64)
        s += f(i);
    return half_h * wave_sum(s);
}

// --------------------------------------------------------------- particle kernels
// The double buffers of a run with those of parity par at index 0 (see pass_a_body): the
// passes then index them with constants, which also keeps a batched run's descriptor in
// registers rather than in scratch memory.
__host__ __device__ inline Work by_parity(Work w, int par)
{
    if (par) {
        const double *t[4] = {w.Ef[0], w.Bf[0], w.J1[0], w.J2[0]};
        w.Ef[0] = w.Ef[1];
        w.Bf[0] = w.Bf[1];
        w.J1[0] = w.J1[1];
        w.J2[0] = w.J2[1];
        w.Ef[1] = const_cast<double *>(t[0]);
        w.Bf[1] = const_cast<double *>(t[1]);
        w.J1[1] = const_cast<double *>(t[2]);
        w.J2[1] = const_cast<double *>(t[3]);
    }
    return w;
}

template <int NV, bool EM> struct TileSizes {
    static constexpr int ne = EM ? 3 : 1;      // E components gathered
    static constexpr int nb = EM ? 2 : 0;      // B components gathered
    static constexpr int ncur = EM ? 3 : 1;    // current components deposited
};

// Gamma = sqrt(r), r = 1 + rho, rho = num2 / den with num2 = 2 num (eq. (opt_solution));
// r < 0 or a non-finite r (e.g. den = 0) takes the fallback Gamma = 1 and is counted.
// Gamma - 1 is tiny for almost every particle (O(dt^4) for ESEC2): |rho| < 1e-4 evaluates
// rho with the hardware reciprocal refined by one Newton step (relative error about 2^-46,
// so below 1e-18 in Gamma) and sqrt(1 + rho) by its Taylor series through rho^4 (truncation
// below 3e-22).  A wavefront that holds any other rho (slow particles: half of the
// wavefronts of a thermal plasma) takes the square root of r = 1 + num2 / den as well, with
// the quotient and the root corrected to their last bit by one more Newton step each
// (methods of Goldschmidt and Markstein); a den below the range of the reciprocal's steps
// divides instead.
template <int NV, int U>
__device__ __forceinline__ void gamma_all(double (&g)[U], const double (&vs)[U][NV],
                                          const double (&vd)[U][NV], const double (&v)[U][NV],
                                          const bool (&valid)[U], int &fallbacks)
{
    // num2 = 2 num = sum (2 v* - (v-dagger + v)) . (v-dagger - v)
    double num2[U], den[U], rc[U], rho[U];
    bool large[U];
    double c3 = 0.0625;
    asm("" : "+v"(c3));        // (kept in registers: an FMA takes one constant that is not)
#pragma unroll
    for (int u = 0; u < U; ++u) {
        num2[u] = 0.0;
        den[u] = 0.0;
#pragma unroll
        for (int c = 0; c < NV; ++c) {
            const double a2 = fma(2.0, vs[u][c], -(vd[u][c] + v[u][c]));
            num2[u] = fma(a2, vd[u][c] - v[u][c], num2[u]);
            den[u] = fma(vd[u][c], vd[u][c], den[u]);
        }
        const double y = __builtin_amdgcn_rcp(den[u]);
        rc[u] = fma(y, fma(-den[u], y, 1.0), y);
        rho[u] = num2[u] * rc[u];
        large[u] = !(fabs(rho[u]) < 1e-4);
        g[u] = fma(rho[u], fma(rho[u], fma(rho[u], fma(rho[u], -0.0390625, c3), -0.125), 0.5), 1.0);
    }
#pragma unroll
    for (int u = 0; u < U; ++u)
        if (__any(large[u])) {
            const double y = fma(rc[u], fma(-den[u], rc[u], 1.0), rc[u]);
            double quo = num2[u] * y;
            quo = fma(fma(-quo, den[u], num2[u]), y, quo);
            if (__any(large[u] && den[u] < 1e-280)) {
                asm volatile("");      // (not to be computed beside the usual quotient)
                quo = den[u] < 1e-280 ? num2[u] / den[u] : quo;
            }
            const double rr = 1.0 + quo;
            const double s = __builtin_amdgcn_rsq(rr);
            double root = rr * s, half = 0.5 * s;
            const double e = fma(-half, root, 0.5);
            root = fma(root, e, root);
            half = fma(half, e, half);
            root = fma(fma(-root, root, rr), half, root);
            root = rr > 0.0 ? root : 0.0;
            const bool ok = rr >= 0.0 && isfinite(rr);
            if (large[u]) {
                g[u] = ok ? root : 1.0;
                fallbacks += (!ok && valid[u]) ? 1 : 0;
            }
        }
}

// v* solves v* = u + v* x t with u = v^n + dt/2 E**, t = dt/2 B** (eq. (good_translation)
// second line, eq. (EMbasic) fourth line): v* = (u + u x t + (u.t) t) / (1 + |t|^2).
__device__ __forceinline__ void rotate_half(const double u[3], const double t[3], double o[3])
{
    double ut = u[0] * t[0] + u[1] * t[1] + u[2] * t[2];
    double tt = t[0] * t[0] + t[1] * t[1] + t[2] * t[2];
    double inv = 1.0 / (1.0 + tt);
    o[0] = (u[0] + (u[1] * t[2] - u[2] * t[1]) + ut * t[0]) * inv;
    o[1] = (u[1] + (u[2] * t[0] - u[0] * t[2]) + ut * t[1]) * inv;
    o[2] = (u[2] + (u[0] * t[1] - u[1] * t[0]) + ut * t[2]) * inv;
}

// v* and x^{n+1} (unwrapped) of a lane's particles, computed identically in both passes.
// tiles: EM: es[3][tw] predictor E, bs[2][tw] predictor B, ghost-padded; ES: es is the
// coefficient tile of E_x (coef_fill)
template <int ORDER, int NV, bool EM, int U>
__device__ __forceinline__ void half_steps(const Run &r, const double (&x)[U], const double (&v)[U][NV],
                                           const double *es, const double *bs, double (&vs)[U][NV],
                                           double (&x1)[U])
{
    Pos p[U];
#pragma unroll
    for (int u = 0; u < U; ++u)
        p[u] = locate<ORDER>(fma(r.hdt, v[u][0], x[u]), r.inv_h, r.xshift);     // x*
    if constexpr (EM) {
        Stencil<ORDER> s[U], sh[U];
        int n[U], nh[U];
        stencils_at<ORDER, U>(s, n, p, r.ng);
#pragma unroll
        for (int u = 0; u < U; ++u)
            p[u] = half_node<ORDER>(p[u]);
        stencils_at<ORDER, U>(sh, nh, p, r.ng);
#pragma unroll
        for (int u = 0; u < U; ++u) {
            double a[3], t[3];
#pragma unroll
            for (int c = 0; c < 3; ++c)
                a[c] = fma(r.hdt, gather_at<ORDER>(es + c * r.tw, s[u], n[u]), v[u][c]);
            t[0] = r.hdt * r.bext[0];
            t[1] = r.hdt * (r.bext[1] + gather_at<ORDER>(bs, sh[u], nh[u]));
            t[2] = r.hdt * (r.bext[2] + gather_at<ORDER>(bs + r.tw, sh[u], nh[u]));
            rotate_half(a, t, vs[u]);
        }
    } else {
        Cell<ORDER> c[U];
        cells_at<ORDER, U>(c, p, r.ng);
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const double a0 = fma(r.hdt, gather_poly<ORDER>(es, c[u]), v[u][0]);
            if constexpr (NV == 1) {
                vs[u][0] = a0;
            } else {
                const double a[3] = {a0, v[u][1], v[u][2]};
                const double t[3] = {r.hdt * r.bext[0], r.hdt * r.bext[1], r.hdt * r.bext[2]};
                rotate_half(a, t, vs[u]);
            }
        }
    }
#pragma unroll
    for (int u = 0; u < U; ++u)
        x1[u] = fma(r.dt, vs[u][0], x[u]);
}

// x^{n+1/2} = (x^n + x^{n+1}) / 2 on the nodes (hinv_h = 1 / 2h).
template <int ORDER, int U>
__device__ __forceinline__ void mid_points(Pos (&p)[U], const double (&x)[U], const double (&x1)[U],
                                           const Run &r)
{
#pragma unroll
    for (int u = 0; u < U; ++u)
        p[u] = locate<ORDER>(x[u] + x1[u], r.hinv_h, 0.0);
}

// v-dagger of an electrostatic particle from E-bar at x^{n+1/2} (eq. (good_translation)).
template <int NV>
__device__ __forceinline__ void dagger_es(double (&vd)[NV], const double (&v)[NV], const double (&vs)[NV],
                                          double e, const Run &r)
{
    if constexpr (NV == 1) {
        vd[0] = fma(r.dt, e, v[0]);
    } else {
        const double *b = r.bext;
        vd[0] = v[0] + r.dt * (e + (vs[1] * b[2] - vs[2] * b[1]));
        vd[1] = v[1] + r.dt * (vs[2] * b[0] - vs[0] * b[2]);
        vd[2] = v[2] + r.dt * (vs[0] * b[1] - vs[1] * b[0]);
    }
}

// A lane's new state of a pass that starts at particle b0 of its batch, and its scalars.
// The state is written through to memory (system-scope relaxed stores): nothing in the
// pass reads it back, and lines left dirty in the L2 of each XCD would be written back at
// the end of the kernel.  A non-finite state makes the kinetic energy non-finite, which is
// where the passes look for one.
template <int NV, int U>
__device__ __forceinline__ void store_all(const double (&xw)[U], const double (&vn)[U][NV],
                                          const bool (&valid)[U], double *Xo, double *Vo, int64_t b0,
                                          int64_t vstride)
{
    const unsigned lane = threadIdx.x & 63;
#pragma unroll
    for (int u = 0; u < U; ++u)
        if (valid[u]) {
            const unsigned o = lane + 64u * u;
#pragma unroll
            for (int c = 0; c < NV; ++c)
                __hip_atomic_store(&(Vo + c * vstride + b0)[o], vn[u][c], __ATOMIC_RELAXED,
                                   __HIP_MEMORY_SCOPE_SYSTEM);
            __hip_atomic_store(&(Xo + b0)[o], xw[u], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
        }
}

// Pass A of step n.  The passes take the run's arrays with those of the step's parity at
// index 0 (Work's double buffers turned by the caller, by_parity), so their addresses come with the
// kernel arguments instead of from a second, dependent read of them.
// LDS: EM: jt[ncur][tw] | es[ne][tw] | bs[nb][tw] | side[ncur][tw]; ES: jt[tw] | es[tw]
//      (j^{n,*}) | side[tw] | eraw[tw] (E^n) | coefficients of E*
// pass_a_body processes particles [p0, p1) of one run, its workgroup `slot`; `lead` marks
// the one workgroup (per run and launch) that also writes the record.
template <int ORDER, int NV, bool EM, int DEP, int U = kUnrollA<NV, DEP>, int G = kGroup<NV, U>>
__device__ __forceinline__ void pass_a_body(const Run &r0, RunPtr rp, const Work &wk, int64_t step,
                                            const double *__restrict__ X,
                                            const double *__restrict__ V, int64_t p0,
                                            int64_t p1, bool lead, int slot, double *smem,
                                            double *red, int *wctr)
{
    const Run &r = r0;
    using T = TileSizes<NV, EM>;
    const int ng = r.ng, tw = r.tw;
    const unsigned lane = threadIdx.x & 63, nt = nthreads();
    double *jt = smem;
    double *es = jt + T::ncur * tw;
    double *bs = es + T::ne * tw;
    double *side = bs + T::nb * tw;       // [ncur][tw] FP64 side tile of the deposit
    double *eraw = side + T::ncur * tw;   // ES: E^n (es: j^{n,*})
    double *ct = smem + coef_offset((2 * T::ncur + T::ne + T::nb + 1) * tw);   // ES: coefficients
    Depo<ORDER, T::ncur, DEP> dep;
    // pass A walks the state from its end, pass B from its start (see WaveBatches)
    WaveBatches<U> wb(batch_order(p0, 64 * U, r.interleave != 0, blockIdx.x, r.nblocks, r.np, true), wctr, nt, r.det);
    PBatch<U, NV> cur, nxt;
    int64_t bcur = wb.first();
    wb.reset();
    NodeLoad<false> nodes;
    // ESEC1 gathers E^n itself: no predictor current
    const double *j1 = EM || r.scheme != 0 ? nullptr : wk.J1[0];
    if constexpr (!EM) {
        nodes.issue(r, wk.Ef[0], j1, nullptr, threadIdx.x);
        dep.init(side, r, wk.st);
        __builtin_amdgcn_sched_barrier(0);
        load_batch(cur, X, V, r.vstride, r.w, r.wu, bcur, p1);
    } else {
        dep.init(side, r, wk.st);
    }
    tile_zero(jt, T::ncur * tw, nt);
    tile_zero(side, T::ncur * tw, nt);
    double *target = dep_target(r, wk, wk.J2[0]);
    // the currents of the next step accumulate into the other buffers (nothing reads them
    // in this pass): every workgroup clears its share
    if (r.scheme != 1)
        rep_zero_part(wk.J1[1], T::ncur * ng, r.nrep, 3 * ng, slot, r.nblocks, nt);
    rep_zero_part(wk.J2[1], T::ncur * ng, r.nrep, 3 * ng, slot, r.nblocks, nt);
    if constexpr (EM) {
        if (r.scheme == kPsatd)
            psatd_tiles(r, wk.ps, es, bs, nt);    // E*, B* come from the field launch before
        else
            predictor_fields(r, wk.Ef[0], wk.Bf[0], wk.J1[0], es, bs, r.nrep);
        load_batch(cur, X, V, r.vstride, r.w, r.wu, bcur, p1);
        lds_barrier();
        ghost_fill(es, T::ne, ng, tw, nt);
        ghost_fill(bs, T::nb, ng, tw, nt);
    } else {
        double m[1] = {0.0}, unused = 0.0;
        nodes.commit(r, threadIdx.x, eraw, es, nullptr, m[0], unused, nullptr);
        node_rounds<false>(r, wk.Ef[0], j1, nullptr, eraw, es, nullptr, m[0], unused, nullptr, nt);
        wave_partials<0u>(m, red);
        lds_barrier();
        const double mean = wave_total(red, 0, nt >> 6) * r.inv_ng;
        coef_fill<ORDER>(ct, [&](int i) { return eraw[i] - r.hdt * (es[i] - mean); }, ng, tw, nt);
    }
    lds_barrier();
    // the record of the state this step starts from, if not written yet
    if (lead && record_wave(nt) && step > wk.st->recorded) {
        if (EM && r.scheme == kLeapfrog) {
            const double wbl = lf_magnetic_energy(r, wk.Ef[0], wk.Bf[0]);
            if (lane == 0)
                wk.st->wb = wbl;
        }
        write_record(r, wk, step);
    }
    const double *eg = EM ? es : ct;     // what half_steps gathers E from

    const Run q = reload(rp);
    settle_pointer(X);
    settle_pointer(V);
    dep.settle();
    // whole wavefronts run the loop (DEP = 2 needs them in its deposit); particles past the
    // end are masked with `valid`
    while (batch_begins(bcur, p1)) {
        const int64_t bnxt = wb.claim();
        const unsigned nval = (unsigned)min(p1 - bcur, (int64_t)(64 * U));
        load_batch(nxt, X, V, q.vstride, q.w, q.wu, bnxt, p1);   // the last one is discarded
        bool in[U];
#pragma unroll
        for (int u = 0; u < U; ++u)
            in[u] = lane + 64u * u < nval;
        if (nval < 64u * U)       // lanes past the end repeat the last particle, without weight
#pragma unroll
            for (int u = 0; u < U; ++u)
                cur.w[u] = in[u] ? cur.w[u] : 0.0;
        auto process = [&](const PBatch<G, NV> &p, const bool (&valid)[G], int u0) __attribute__((always_inline)) {
            double vs[G][NV], x1[G];
            half_steps<ORDER, NV, EM, G>(q, p.x, p.v, eg, bs, vs, x1);
            double qv[G][T::ncur];
#pragma unroll
            for (int u = 0; u < G; ++u) {
                const double qw = p.w[u] * q.qs;
#pragma unroll
                for (int c = 0; c < T::ncur; ++c)
                    qv[u][c] = qw * vs[u][c];
            }
            bool done = false;
            if constexpr (!EM && ORDER == 1 && (DEP == 0 || DEP == 3)) {
                if (q.cc) {
                    // exact charge conservation: through the pieces of the path x^n -> x^{n+1}
#pragma unroll
                    for (int u = 0; u < G; ++u)
                        if (valid[u])
                            cc_pieces(q, p.x[u], x1[u], [&](int slot, double d, double f) {
                                double qf[T::ncur];
#pragma unroll
                                for (int c = 0; c < T::ncur; ++c)
                                    qf[c] = qv[u][c] * f;
                                dep.add_at(jt, tw, cc_slots(slot), cc_stencil(d), qf);
                            });
                    done = true;
                }
            }
            if (!done) {
                Pos pos[G];
                mid_points<ORDER, G>(pos, p.x, x1, q);
                deposit_all<ORDER, T::ncur, DEP, G>(dep, jt, tw, ng, pos, qv, valid, u0 == 0);
            }
        };
        if constexpr (G == U) {
            process(cur, in, 0);
        } else {
#pragma unroll
            for (int u0 = 0; u0 < U; u0 += G) {
                bool valid[G];
#pragma unroll
                for (int u = 0; u < G; ++u)
                    valid[u] = in[u0 + u];
                process(batch_group<G>(cur, u0), valid, u0);
            }
        }
        cur = nxt;
        bcur = bnxt;
    }
    dep.finish(jt, tw, ng);
    flag_over(dep, wk);
    lds_barrier();
    dep.flush_tile(jt, target, T::ncur, ng, tw);
}

template <int ORDER, int NV, bool EM, int DEP>
__global__ __launch_bounds__(kMaxThreads<NV>) __attribute__((amdgpu_waves_per_eu(kWavesPerEU<NV>)))
void k_pass_a(Run r, Work wk, int64_t step,
                                                 const double *__restrict__ X,
                                                 const double *__restrict__ V)
{
    extern __shared__ double smem[];
    __shared__ double red[kRedSize];
    __shared__ int wctr;
    const int64_t p0 = (int64_t)blockIdx.x * r.chunk;
    // the lead (one of whose wavefronts also writes the record) is the last workgroup, whose
    // chunk is the smallest when N_p is not a multiple of it
    pass_a_body<ORDER, NV, EM, DEP>(r, kernarg_run(), wk, step, X, V, p0,
                                    r.interleave ? r.np : min(r.np, p0 + r.chunk),
                                    (int)blockIdx.x == r.nblocks - 1, blockIdx.x, smem, red,
                                    &wctr);
}

// A workgroup's scalars from the wavefronts' partials in red (after the barrier): kinetic
// energy (halved here) and fallbacks are sums, max |Gamma - 1| and the non-finite flag
// maxima.  Written by the record wavefront.
__device__ __forceinline__ void write_scalars(double *sp, const double *red, unsigned nt)
{
    if (record_wave(nt)) {
        const unsigned nw = nt >> 6;
        const double ke = 0.5 * wave_total(red, 0, nw), fb = wave_total(red, 1, nw);
        const double gd = wave_total<true>(red, 2, nw), nf = wave_total<true>(red, 3, nw);
        if ((threadIdx.x & 63) == 0) {
            sp[0] = ke;
            sp[1] = fb;
            sp[2] = gd;
            sp[3] = nf;
        }
    }
}

// Pass B of step n: new fields, second gather, Gamma, state write and
// (PRED) the next step's predictor deposit.
// LDS: jt[ncur][tw] | es[ne][tw] | bs[nb][tw] | eb[ne][tw] | bb[nb][tw] | e1[ne][ng] |
//      b1[nb][ng] | EM scratch[8 ng] | side[ncur][tw]; ES: es, eb, e1 hold j^{n,*}, E^n,
//      j^{*,n+1/2}, and the coefficients of E* and E-bar follow side
// pass_b_body processes particles [p0, p1) of one run and leaves its scalars in
// spart[slot]; `lead` marks the workgroup that publishes the new fields of the run.
template <int ORDER, int NV, bool EM, bool PRED, int DEP, int U = kUnrollB<NV, DEP>, int G = kGroup<NV, U>>
__device__ __forceinline__ void pass_b_body(const Run &r0, RunPtr rp, const Work &wk, const double *X,
                                            const double *V, double *Xo, double *Vo,
                                            int64_t p0, int64_t p1, bool lead, int slot,
                                            double *smem, double *red, int *wctr)
{
    const Run &r = r0;
    using T = TileSizes<NV, EM>;
    const int ng = r.ng, tw = r.tw;
    const unsigned lane = threadIdx.x & 63, nt = nthreads();
    WaveBatches<U> wb(batch_order(p0, 64 * U, r.interleave != 0, blockIdx.x, r.nblocks, r.np, false), wctr, nt, r.det);
    PBatch<U, NV> cur, nxt;
    int64_t bcur = wb.first();
    wb.reset();
    double *jt = smem;
    double *es = jt + T::ncur * tw;
    double *bs = es + T::ne * tw;
    double *eb = bs + T::nb * tw;
    double *bb = eb + T::ne * tw;
    double *e1 = bb + T::nb * tw;
    double *b1 = e1 + T::ne * ng;
    double *scratch = b1 + T::nb * ng;
    double *side = scratch + (EM ? 8 * ng : 0);   // [ncur][tw] FP64 side tile of the deposit
    // ES: coefficient tiles of E* and E-bar
    double *cts = smem + coef_offset((2 * T::ncur + 2 * T::ne + 2 * T::nb) * tw + (T::ne + T::nb + (EM ? 8 : 0)) * ng);
    double *ctb = cts + (ORDER + 1) * tw;
    const double *En = wk.Ef[0];
    const double *Bn = EM ? wk.Bf[0] : nullptr;
    Depo<ORDER, T::ncur, DEP> dep;
    NodeLoad<true> nodes;
    const double *j1 = EM || r.scheme != 0 ? nullptr : wk.J1[0];
    if constexpr (!EM) {
        nodes.issue(r, En, j1, wk.J2[0], threadIdx.x);
        dep.init(side, r, wk.st);
        __builtin_amdgcn_sched_barrier(0);
        load_batch(cur, X, V, r.vstride, r.w, r.wu, bcur, p1);
    } else {
        dep.init(side, r, wk.st);
    }
    if constexpr (PRED) {
        tile_zero(jt, T::ncur * tw, nt);
        tile_zero(side, T::ncur * tw, nt);
    }
    double *target = PRED ? dep_target(r, wk, wk.J1[1]) : nullptr;
    if constexpr (EM) {
        if (r.em_fields) {
            // the fields v-dagger gathers come from the field launch before this pass, which
            // has also published E^{n+1}, B^{n+1} (the lead reads those back for their
            // energies); E*, B* from the predictor launch (PSATD) or, for the local LI
            // predictor, as in pass A
            if (r.scheme == kPsatd)
                psatd_tiles(r, wk.ps, es, bs, nt);
            else
                predictor_fields(r, En, Bn, wk.J1[0], es, bs, r.nrep);
            psatd_tiles(r, wk.pf, eb, bb, nt);
            if (lead) {
                tile_load(e1, wk.Ef[1], 3 * ng, nt);
                tile_load(b1, wk.Bf[1], 2 * ng, nt);
            }
            load_batch(cur, X, V, r.vstride, r.w, r.wu, bcur, p1);
        } else if (r.scheme == kLeapfrog) {
            predictor_fields(r, En, Bn, wk.J1[0], es, bs, r.nrep);
            load_batch(cur, X, V, r.vstride, r.w, r.wu, bcur, p1);
            lf_full_fields(r, En, wk.J2[0], bs, e1, b1, eb, bb, r.nrep);
        } else {
            predictor_fields(r, En, Bn, wk.J1[0], es, bs, r.nrep);
            load_batch(cur, X, V, r.vstride, r.w, r.wu, bcur, p1);
            field_update(r, wk, En, Bn, wk.J2[0], e1, b1, eb, bb, scratch, r.nrep);
        }
        lds_barrier();
        ghost_fill(es, T::ne, ng, tw, nt);
        ghost_fill(eb, T::ne, ng, tw, nt);
        ghost_fill(bs, T::nb, ng, tw, nt);
        ghost_fill(bb, T::nb, ng, tw, nt);
        if (lead) {
            // publish E^{n+1}, B^{n+1} and their energies (pass A clears the next currents)
            if (!r.em_fields) {
                for (int i = threadIdx.x; i < T::ne * ng; i += nt)
                    wk.Ef[1][i] = e1[i];
                for (int i = threadIdx.x; i < 2 * ng; i += nt)
                    wk.Bf[1][i] = b1[i];
            }
            if (record_wave(nt)) {
                const double we = wave_energy(0.5 * r.h, 3 * ng, [&](int i) { return e1[i] * e1[i]; });
                const double wb = wave_energy(0.5 * r.c2 * r.h, 2 * ng, [&](int i) { return b1[i] * b1[i]; });
                if (lane == 0) {
                    wk.st->we = we;
                    // EMEC(LF)'s W_B needs B^{n+3/2}: the writer of the next record computes it
                    if (r.scheme != kLeapfrog)
                        wk.st->wb = wb;
                }
            }
        }
    } else {
        // E* = E^n - dt/2 (j^{n,*} - mean) (eq. (good_translation); ESEC1: E^n) and
        // E^{n+1} = E^n - dt (j^{*,n+1/2} - mean) (eq. (ampere) in 1D), from the node values
        double *save = lead ? wk.grid_save : nullptr;
        double m[2] = {0.0, 0.0};
        nodes.commit(r, threadIdx.x, eb, es, e1, m[0], m[1], save);
        node_rounds<true>(r, En, j1, wk.J2[0], eb, es, e1, m[0], m[1], save, nt);
        wave_partials<0u>(m, red);
        lds_barrier();
        const double mean1 = wave_total(red, 0, nt >> 6) * r.inv_ng, mean2 = wave_total(red, 1, nt >> 6) * r.inv_ng;
        auto star = [&](int i) { return eb[i] - r.hdt * (es[i] - mean1); };
        auto next = [&](int i) { return eb[i] - r.dt * (e1[i] - mean2); };
        auto bar = [&](int i) { return 0.5 * (eb[i] + next(i)); };
        coef_fill<ORDER>(cts, star, ng, tw, nt);
        coef_fill<ORDER>(ctb, bar, ng, tw, nt);
        if (lead) {
            // publish E^{n+1} and its energy (pass A clears the next currents)
            for (int i = threadIdx.x; i < ng; i += nt)
                wk.Ef[1][i] = next(i);
            if (save)
                // the fields this step gathers, for the adjoint's reverse passes
                for (int i = threadIdx.x; i < ng; i += nt) {
                    save[3 * ng + i] = star(i);
                    save[4 * ng + i] = bar(i);
                    save[5 * ng + i] = next(i);
                }
            if (record_wave(nt)) {
                const double we = wave_energy(0.5 * r.h, ng, [&](int i) { return next(i) * next(i); });
                if (lane == 0) {
                    wk.st->we = we;
                    wk.st->wb = 0.0;
                }
            }
        }
    }
    const double *eg = EM ? es : cts;    // what half_steps gathers E* from
    lds_barrier();

    double ke = 0.0, gdev = 0.0;
    int fb = 0;
    const Run q = reload(rp);
    settle_pointer(X);
    settle_pointer(V);
    settle_pointer(Xo);
    settle_pointer(Vo);
    dep.settle();
    while (batch_begins(bcur, p1)) {
        const int64_t bnxt = wb.claim();
        const unsigned nval = (unsigned)min(p1 - bcur, (int64_t)(64 * U));
        load_batch(nxt, X, V, q.vstride, q.w, q.wu, bnxt, p1);   // the last one is discarded
        bool in[U];
#pragma unroll
        for (int u = 0; u < U; ++u)
            in[u] = lane + 64u * u < nval;
        if (nval < 64u * U)       // lanes past the end repeat the last particle, without weight
#pragma unroll
            for (int u = 0; u < U; ++u)
                cur.w[u] = in[u] ? cur.w[u] : 0.0;
        auto process = [&](const PBatch<G, NV> &p, const bool (&valid)[G], int u0) __attribute__((always_inline)) {
            double vs[G][NV], x1[G], vd[G][NV];
            Pos pos[G];
            half_steps<ORDER, NV, EM, G>(q, p.x, p.v, eg, bs, vs, x1);
            mid_points<ORDER, G>(pos, p.x, x1, q);
            if constexpr (EM) {
                Stencil<ORDER> s[G], sh[G];
                int n[G], nh[G];
                stencils_at<ORDER, G>(s, n, pos, ng);
#pragma unroll
                for (int u = 0; u < G; ++u)
                    pos[u] = half_node<ORDER>(pos[u]);
                stencils_at<ORDER, G>(sh, nh, pos, ng);
#pragma unroll
                for (int u = 0; u < G; ++u) {
                    // v-dagger = v^n + dt (E-bar + v* x B-bar)   (eq. (good_translation), (EMbasic))
                    const double e[3] = {gather_at<ORDER>(eb, s[u], n[u]), gather_at<ORDER>(eb + tw, s[u], n[u]),
                                         gather_at<ORDER>(eb + 2 * tw, s[u], n[u])};
                    const double b[3] = {q.bext[0], q.bext[1] + gather_at<ORDER>(bb, sh[u], nh[u]),
                                         q.bext[2] + gather_at<ORDER>(bb + tw, sh[u], nh[u])};
                    const double *v = p.v[u], *a = vs[u];
                    vd[u][0] = v[0] + q.dt * (e[0] + (a[1] * b[2] - a[2] * b[1]));
                    vd[u][1] = v[1] + q.dt * (e[1] + (a[2] * b[0] - a[0] * b[2]));
                    vd[u][2] = v[2] + q.dt * (e[2] + (a[0] * b[1] - a[1] * b[0]));
                }
            } else {
                double e[G];
                bool done = false;
                if constexpr (ORDER == 1) {
                    if (q.cc) {
#pragma unroll
                        for (int u = 0; u < G; ++u)
                            e[u] = cc_gather(q, ctb, p.x[u], x1[u]);
                        done = true;
                    }
                }
                if (!done) {
                    Cell<ORDER> c[G];
                    cells_at<ORDER, G>(c, pos, ng);
#pragma unroll
                    for (int u = 0; u < G; ++u)
                        e[u] = gather_poly<ORDER>(ctb, c[u]);
                }
#pragma unroll
                for (int u = 0; u < G; ++u)
                    dagger_es<NV>(vd[u], p.v[u], vs[u], e[u], q);
            }
            // Gamma (eq. (opt_solution)); an imaginary or undefined root falls back to 1
            double g[G], vn[G][NV], xw[G], v2[G];
            gamma_all<NV, G>(g, vs, vd, p.v, valid, fb);
#pragma unroll
            for (int u = 0; u < G; ++u) {
                v2[u] = 0.0;
#pragma unroll
                for (int c = 0; c < NV; ++c) {
                    vn[u][c] = g[u] * vd[u][c];
                    v2[u] = fma(vn[u][c], vn[u][c], v2[u]);
                }
            }
            wrap_all<G>(xw, x1, q);
            store_all<NV, G>(xw, vn, valid, Xo, Vo, bcur + 64 * u0, q.vstride);
#pragma unroll
            for (int u = 0; u < G; ++u) {
                gdev = fmax(gdev, fabs(g[u] - 1.0));
                ke = fma(p.w[u], v2[u], ke);
            }
            if constexpr (PRED) {
                double qv[G][T::ncur];
#pragma unroll
                for (int u = 0; u < G; ++u) {
                    const double qw = p.w[u] * q.qs;
#pragma unroll
                    for (int c = 0; c < T::ncur; ++c)
                        qv[u][c] = qw * vn[u][c];
                    pos[u] = locate<ORDER>(fma(q.hdt, vn[u][0], xw[u]), q.inv_h, q.xshift);
                }
                deposit_all<ORDER, T::ncur, DEP, G>(dep, jt, tw, ng, pos, qv, valid, u0 == 0);
            }
        };
        if constexpr (G == U) {
            process(cur, in, 0);
        } else {
#pragma unroll
            for (int u0 = 0; u0 < U; u0 += G) {
                bool valid[G];
#pragma unroll
                for (int u = 0; u < G; ++u)
                    valid[u] = in[u0 + u];
                process(batch_group<G>(cur, u0), valid, u0);
            }
        }
        cur = nxt;
        bcur = bnxt;
    }
    int nonfinite = isfinite(ke) ? 0 : 1;
    if constexpr (PRED) {
        dep.finish(jt, tw, ng);
        nonfinite |= dep.over;
    }
    // kinetic energy and fallbacks (sums), max |Gamma - 1| and the non-finite flag (maxima)
    const double sc[4] = {ke, (double)fb, gdev, (double)nonfinite};
    wave_partials<0xcu>(sc, red);
    lds_barrier();
    if constexpr (PRED)
        dep.flush_tile(jt, target, T::ncur, ng, tw);
    write_scalars(wk.spart + (size_t)slot * kNS, red, nt);
}

template <int ORDER, int NV, bool EM, bool PRED, int DEP>
__global__ __launch_bounds__(kMaxThreads<NV>) __attribute__((amdgpu_waves_per_eu(kWavesPerEU<NV>)))
void k_pass_b(Run r, Work wk, const double *X,
                                                 const double *V, double *Xo, double *Vo)
{
    extern __shared__ double smem[];
    __shared__ double red[kRedSize];
    __shared__ int wctr;
    const int64_t p0 = (int64_t)blockIdx.x * r.chunk;
    pass_b_body<ORDER, NV, EM, PRED, DEP>(r, kernarg_run(), wk, X, V, Xo, Vo, p0,
                                          r.interleave ? r.np : min(r.np, p0 + r.chunk),
                                          (int)blockIdx.x == r.nblocks - 1, blockIdx.x, smem,
                                          red, &wctr);
}

// ------------------------------------------------------------ ESEC1 in one pass
// ESEC1 (eq. (naivetranslation) with eq. (PICmodification)) has a single grid-wide
// dependency per step: v* uses E^n, which is known before the step, so only the centred
// current j^{n+1/2} -> E^{n+1} needs every particle.  One launch per step therefore
// suffices: it finishes step n (E^{n+1} from j^{n+1/2}, v-dagger, Gamma, the state
// write) and, with x^{n+1}, v^{n+1} still in registers, already computes step n+1's v*
// (gathering the E^{n+1} it has just built) and deposits j^{n+3/2}.  The state is read
// once and written once per step (32 B per particle in 1D-1V).  Step n + 1 recomputes that
// v* from the stored x^{n+1}, v^{n+1} and the stored E^{n+1} with the same instructions,
// so the deposit and the later gather see a bit-identical x^{n+3/2}.  The first step's
// current j^{1/2} is deposited at initialisation by a pass A.
// Currents rotate through three buffers: the pass reads j^{n+1/2} (Jr), deposits
// j^{n+3/2} (Jd) and clears the buffer that held j^{n-1/2} (Jc), which step n + 1 deposits
// into.  The per-workgroup scalars alternate between two arrays as well: this pass's lead
// writes the record of step n from the scalars of the previous pass (wk.spart) while
// the other workgroups write theirs for step n + 1 (spw).
// LDS: jt[tw] | es[tw] (E^n) | e1[ng] (j^{n+1/2}) | side[tw] | three coefficient tiles (E^n,
//      E-bar, E^{n+1}).
template <int ORDER, int NV, int DEP, int U = kUnrollB<NV, 0>>
__device__ __forceinline__ void esec1_body(const Run &r0, RunPtr rp, const Work &wk, int64_t step,
                                           const double *X, const double *V, double *Xo,
                                           double *Vo, const double *Jr, double *Jd, double *Jc,
                                           double *spw, int64_t p0, int64_t p1, bool lead,
                                           int slot, double *smem, double *red, int *wctr)
{
    const Run &r = r0;
    const int ng = r.ng, tw = r.tw;
    const unsigned lane = threadIdx.x & 63, nt = nthreads();
    // one pass per step: alternate directions (see WaveBatches)
    WaveBatches<U> wb(batch_order<true>(p0, 64 * U, r.interleave != 0, blockIdx.x, r.nblocks, r.np, (step & 1) != 0),
                      wctr, nt, r.det);
    PBatch<U, NV> cur, nxt;
    int64_t bcur = wb.first();
    wb.reset();
    double *jt = smem;
    double *es = jt + tw;
    double *e1 = es + tw;
    double *side = e1 + ng;
    double *ctn = smem + coef_offset(3 * tw + ng);     // E^n
    double *ctb = ctn + (ORDER + 1) * tw;               // E-bar
    double *ct1 = ctb + (ORDER + 1) * tw;               // E^{n+1}
    const double *En = wk.Ef[0];
    Depo<ORDER, 1, DEP> dep;
    // node values: E^n into es, j^{n+1/2} into e1 (see pass_b_body)
    NodeLoad<false> nodes;
    nodes.issue(r, En, Jr, nullptr, threadIdx.x);
    dep.init(side, r, wk.st);
    __builtin_amdgcn_sched_barrier(0);
    load_batch(cur, X, V, r.vstride, r.w, r.wu, bcur, p1);
    tile_zero(jt, tw, nt);
    tile_zero(side, tw, nt);
    double *target = dep_target(r, wk, Jd);
    rep_zero_part(Jc, ng, r.nrep, 3 * ng, slot, r.nblocks, nt);
    double m[1] = {0.0}, unused = 0.0;
    nodes.commit(r, threadIdx.x, es, e1, nullptr, m[0], unused, nullptr);
    node_rounds<false>(r, En, Jr, nullptr, es, e1, nullptr, m[0], unused, nullptr, nt);
    wave_partials<0u>(m, red);
    lds_barrier();
    const double mean = wave_total(red, 0, nt >> 6) * r.inv_ng;
    auto next = [&](int i) { return es[i] - r.dt * (e1[i] - mean); };     // E^{n+1}
    coef_fill<ORDER>(ctn, [&](int i) { return es[i]; }, ng, tw, nt);
    coef_fill<ORDER>(ctb, [&](int i) { return 0.5 * (es[i] + next(i)); }, ng, tw, nt);
    coef_fill<ORDER>(ct1, next, ng, tw, nt);
    if (lead)
        for (int i = threadIdx.x; i < ng; i += nt)
            wk.Ef[1][i] = next(i);
    lds_barrier();
    if (lead && record_wave(nt)) {
        // the record of step n (its kinetic energy from the previous pass's scalars, its
        // field energy from st->we), then the energy of E^{n+1} for step n + 1
        if (step > wk.st->recorded)
            write_record(r, wk, step);
        const double we = wave_energy(0.5 * r.h, ng, [&](int i) { return next(i) * next(i); });
        if (lane == 0) {
            wk.st->we = we;
            wk.st->wb = 0.0;
        }
    }

    double ke = 0.0, gdev = 0.0;
    int fb = 0;
    const Run q = reload(rp);
    settle_pointer(X);
    settle_pointer(V);
    settle_pointer(Xo);
    settle_pointer(Vo);
    dep.settle();
    while (batch_begins(bcur, p1)) {
        const int64_t bnxt = wb.claim();
        const unsigned nval = (unsigned)min(p1 - bcur, (int64_t)(64 * U));
        load_batch(nxt, X, V, q.vstride, q.w, q.wu, bnxt, p1);   // the last one is discarded
        bool valid[U];
#pragma unroll
        for (int u = 0; u < U; ++u)
            valid[u] = lane + 64u * u < nval;
        if (nval < 64u * U)       // lanes past the end repeat the last particle, without weight
#pragma unroll
            for (int u = 0; u < U; ++u)
                cur.w[u] = valid[u] ? cur.w[u] : 0.0;
        double vs[U][NV], x1[U], vd[U][NV];
        Pos pos[U];
        half_steps<ORDER, NV, false, U>(q, cur.x, cur.v, ctn, nullptr, vs, x1);
        mid_points<ORDER, U>(pos, cur.x, x1, q);
        Cell<ORDER> c[U];
        cells_at<ORDER, U>(c, pos, ng);
#pragma unroll
        for (int u = 0; u < U; ++u)
            dagger_es<NV>(vd[u], cur.v[u], vs[u], gather_poly<ORDER>(ctb, c[u]), q);
        double g[U], vn[U][NV], xw[U], v2[U];
        gamma_all<NV, U>(g, vs, vd, cur.v, valid, fb);
#pragma unroll
        for (int u = 0; u < U; ++u) {
            v2[u] = 0.0;
#pragma unroll
            for (int c = 0; c < NV; ++c) {
                vn[u][c] = g[u] * vd[u][c];
                v2[u] = fma(vn[u][c], vn[u][c], v2[u]);
            }
        }
        wrap_all<U>(xw, x1, q);
        store_all<NV, U>(xw, vn, valid, Xo, Vo, bcur, q.vstride);
#pragma unroll
        for (int u = 0; u < U; ++u) {
            gdev = fmax(gdev, fabs(g[u] - 1.0));
            ke = fma(cur.w[u], v2[u], ke);
        }
        // step n + 1: v* from E^{n+1} at x*_{n+1}, and the centred deposit j^{n+3/2}
        double va[U][NV], xa[U], qv[U][1];
        half_steps<ORDER, NV, false, U>(q, xw, vn, ct1, nullptr, va, xa);
        mid_points<ORDER, U>(pos, xw, xa, q);
#pragma unroll
        for (int u = 0; u < U; ++u)
            qv[u][0] = (cur.w[u] * q.qs) * va[u][0];
        deposit_all<ORDER, 1, DEP, U>(dep, jt, tw, ng, pos, qv, valid);
        cur = nxt;
        bcur = bnxt;
    }
    dep.finish(jt, tw, ng);
    const int nonfinite = isfinite(ke) ? dep.over : 1;
    const double sc[4] = {ke, (double)fb, gdev, (double)nonfinite};
    wave_partials<0xcu>(sc, red);
    lds_barrier();
    dep.flush_tile(jt, target, 1, ng, tw);
    write_scalars(spw + (size_t)slot * kNS, red, nt);
}

template <int ORDER, int NV, int DEP>
__global__ __launch_bounds__(kMaxThreads<NV>) __attribute__((amdgpu_waves_per_eu(kWavesPerEU<NV>)))
void k_esec1(Run r, Work wk, int64_t step, const double *X, const double *V, double *Xo,
             double *Vo, const double *Jr, double *Jd, double *Jc, double *spw)
{
    extern __shared__ double smem[];
    __shared__ double red[kRedSize];
    __shared__ int wctr;
    const int64_t p0 = (int64_t)blockIdx.x * r.chunk;
    esec1_body<ORDER, NV, DEP>(r, kernarg_run(), wk, step, X, V, Xo, Vo, Jr, Jd, Jc, spw, p0,
                               r.interleave ? r.np : min(r.np, p0 + r.chunk),
                               (int)blockIdx.x == r.nblocks - 1, blockIdx.x, smem, red, &wctr);
}

// ------------------------------------------------ standard explicit PIC (comparison)
// The scheme section 5 compares against: Vlasov-Poisson with the leapfrog/Boris push in
// its symmetric form, eq. (symm_Boris): x* = x^n + dt/2 v^n; v^{n+1} = v^n + dt (E^{n+1/2}(x*)
// + v^{n+1/2} x B); x^{n+1} = x* + dt/2 v^{n+1}; E^{n+1/2} is the Gauss field of the charge
// density at the positions x*.  Each step is a field launch (k_std_field: density ->
// E^{n+1/2}) and one particle pass (k_std_pass), which ends by depositing the density at
// x*_{n+1} = x^{n+1} + dt/2 v^{n+1} for the next field launch; the next pass recomputes
// that x* from the stored state with the same instruction.  32 B per particle-step.

// Row of the spectral Gauss solve as a convolution, E_i = sum_j G_{(i - j) mod N} rho_j:
// G_d = (2/N) sum_{m=1}^{M} sin(2 pi m d / N) / k_m, k_m = 2 pi m / L, with M the largest
// mode below the Nyquist mode (the mean and Nyquist modes of E are zero, as in gauss_body).
__device__ void std_green_body(const Run &r, const Work &wk)
{
    const int ng = r.ng;
    for (int d = threadIdx.x; d < ng; d += nthreads()) {
        double acc = 0.0;
        for (int m = 1; 2 * m < ng; ++m) {
            const long long md = ((long long)m * d) % ng;
            const double k = 2.0 * M_PI * m / r.L;
            acc += sinpi(2.0 * (double)md / ng) / k;
        }
        wk.cninv[d] = 2.0 * acc / ng;
    }
}

__global__ __launch_bounds__(1024) void k_std_green(Run r, Work wk) { std_green_body(r, wk); }

// sum_j K[(i - j) mod ng] f[j] by one wavefront: lane l takes j = l, l + 64, ... (both rows
// are then read without bank conflicts) and the lanes are summed in a fixed order, so the
// result does not depend on the launch.  Every lane gets it.
template <int N>
__device__ __forceinline__ double wave_convolve(const double *const (&K)[N], const double *const (&f)[N],
                                                int i, int ng)
{
    double acc = 0.0;
    for (int j = threadIdx.x & 63; j < ng; j += 64) {
        int k = i - j;
        k += k < 0 ? ng : 0;
#pragma unroll
        for (int n = 0; n < N; ++n)
            acc = fma(K[n][k], f[n][j], acc);
    }
    return wave_sum(acc);
}

// E^{n+1/2} from the density replicas in rho (optionally binomial-filtered once, (1/4,
// 1/2, 1/4)) into E.  A workgroup of kFieldNodes wavefronts computes as many consecutive
// nodes, one per wavefront.  The launch is a round of loads, a barrier and a few iterations:
// with 64 lanes to a node the convolution is N_g / 64 iterations long (eight lanes to a node,
// 32 iterations at 256 cells: 4.7 us, the shortest 3.9; now 4.4 and 2.4).
// LDS: rho[ng] | g[ng] | filtered rho[ng].
constexpr int kFieldNodes = 8;

__global__ __launch_bounds__(64 * kFieldNodes) void k_std_field(Run r, Work wk, const double *rho_rep,
                                                                double *E, int filter)
{
    extern __shared__ double smem[];
    const int ng = r.ng;
    const unsigned nt = nthreads();
    double *rho = smem, *g = smem + ng, *rf = smem + 2 * ng;
    for (int i = threadIdx.x; i < ng; i += nt) {
        g[i] = wk.cninv[i];
        rho[i] = rep_sum(rho_rep, i, r.nrep, 3 * ng);
    }
    __syncthreads();
    if (filter) {
        for (int i = threadIdx.x; i < ng; i += nt)
            rf[i] = 0.25 * rho[i == 0 ? ng - 1 : i - 1] + 0.5 * rho[i] + 0.25 * rho[i + 1 == ng ? 0 : i + 1];
        __syncthreads();
        rho = rf;
    }
    const int i = blockIdx.x * kFieldNodes + (threadIdx.x >> 6);
    if (i >= ng)
        return;
    const double *const K[1] = {g}, *const f[1] = {rho};
    const double e = wave_convolve<1>(K, f, i, ng);
    if ((threadIdx.x & 63) == 0)
        E[i] = e;
}

// Charge density at x*_0 = x^0 + dt/2 v^0 into J (the first field launch's input).
template <int ORDER>
__device__ __forceinline__ void std_prime_body(const Run &r, const Work &wk,
                                               const double *__restrict__ X,
                                               const double *__restrict__ V, double *J,
                                               int64_t p0, int64_t p1, double *smem)
{
    double *jt = smem;
    double *side = jt + r.tw;
    tile_zero(jt, 2 * r.tw);
    __syncthreads();
    Depo<ORDER, 1, 0> dep;
    dep.init(side, r, wk.st, 1);
    for (int64_t p = p0 + threadIdx.x; p < p1; p += nthreads()) {
        const double q[1] = {(r.w ? r.w[p] : r.wu) * r.qs};
        dep.add(jt, r.tw, r.ng, stencil<ORDER>(fma(r.hdt, V[p], X[p]) * r.inv_h), q);
    }
    flag_over(dep, wk);
    __syncthreads();
    dep.flush_tile(jt, dep_target(r, wk, J), 1, r.ng, r.tw);
}

template <int ORDER>
__global__ __launch_bounds__(1024) void k_std_prime(Run r, Work wk, const double *__restrict__ X,
                                                    const double *__restrict__ V, double *J)
{
    extern __shared__ double smem[];
    const int64_t p0 = (int64_t)blockIdx.x * r.chunk;
    std_prime_body<ORDER>(r, wk, X, V, J, p0, min(r.np, p0 + r.chunk), smem);
}

// One particle pass of step n: gather E^{n+1/2} at x*, the Boris velocity update, the new
// state, the kinetic energies before and after, and the density at x*_{n+1}.
// LDS: jt[tw] | es[tw] | side[tw] | coefficient tile of E^{n+1/2}.
template <int ORDER, int NV, int DEP, int U = kUnrollB<NV, 0>>
__device__ __forceinline__ void std_pass_body(const Run &r0, RunPtr rp, const Work &wk, int64_t step,
                                              const double *X, const double *V, double *Xo,
                                              double *Vo, double *Jd, double *Jc, double *spw,
                                              int64_t p0, int64_t p1, bool lead, int slot,
                                              double *smem, double *red, double *red0, int *wctr)
{
    const Run &r = r0;
    const int ng = r.ng, tw = r.tw;
    const unsigned lane = threadIdx.x & 63, nt = nthreads();
    // one pass per step: alternate directions (see WaveBatches)
    WaveBatches<U> wb(batch_order<true>(p0, 64 * U, r.interleave != 0, blockIdx.x, r.nblocks, r.np, (step & 1) != 0),
                      wctr, nt, r.det);
    PBatch<U, NV> cur, nxt;
    int64_t bcur = wb.first();
    wb.reset();
    double *jt = smem;
    double *es = jt + tw;
    double *side = es + tw;
    double *ct = smem + coef_offset(3 * tw);
    const double *Eh = wk.Ef[0];
    Depo<ORDER, 1, DEP> dep;
    const double eh0 = Eh[min((int)threadIdx.x, ng - 1)];
    dep.init(side, r, wk.st, 1);
    __builtin_amdgcn_sched_barrier(0);
    load_batch(cur, X, V, r.vstride, r.w, r.wu, bcur, p1);
    tile_zero(jt, tw, nt);
    tile_zero(side, tw, nt);
    double *target = dep_target(r, wk, Jd);
    rep_zero_part(Jc, ng, r.nrep, 3 * ng, slot, r.nblocks, nt);
    if ((int)threadIdx.x < ng)
        es[threadIdx.x] = eh0;
    for (int i = threadIdx.x + nt; i < ng; i += nt)
        es[i] = Eh[i];
    lds_barrier();
    coef_fill<ORDER>(ct, [&](int i) { return es[i]; }, ng, tw, nt);
    lds_barrier();
    if (lead && record_wave(nt)) {
        if (step > wk.st->recorded)
            write_record(r, wk, step);
        const double we = wave_energy(0.5 * r.h, ng, [&](int i) { return es[i] * es[i]; });
        if (lane == 0) {
            wk.st->we = we;
            wk.st->wb = 0.0;
        }
    }

    double ke1 = 0.0, ke0 = 0.0;
    const Run q = reload(rp);
    settle_pointer(X);
    settle_pointer(V);
    settle_pointer(Xo);
    settle_pointer(Vo);
    dep.settle();
    while (batch_begins(bcur, p1)) {
        const int64_t bnxt = wb.claim();
        const unsigned nval = (unsigned)min(p1 - bcur, (int64_t)(64 * U));
        load_batch(nxt, X, V, q.vstride, q.w, q.wu, bnxt, p1);   // the last one is discarded
        bool valid[U];
#pragma unroll
        for (int u = 0; u < U; ++u)
            valid[u] = lane + 64u * u < nval;
        if (nval < 64u * U)       // lanes past the end repeat the last particle, without weight
#pragma unroll
            for (int u = 0; u < U; ++u)
                cur.w[u] = valid[u] ? cur.w[u] : 0.0;
        double xs[U], vn[U][NV], x1[U], xw[U];
        Pos pos[U];
#pragma unroll
        for (int u = 0; u < U; ++u) {
            xs[u] = fma(q.hdt, cur.v[u][0], cur.x[u]);
            pos[u] = locate<ORDER>(xs[u], q.inv_h, 0.0);
        }
        Cell<ORDER> c[U];
        cells_at<ORDER, U>(c, pos, ng);
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const double ep = gather_poly<ORDER>(ct, c[u]);
            const double *v = cur.v[u];
            if constexpr (NV == 1) {
                vn[u][0] = fma(q.dt, ep, v[0]);
            } else {
                // v^{n+1/2} = a + v^{n+1/2} x t, a = v^n + dt/2 E, t = dt/2 B; v^{n+1} = 2 v^{n+1/2} - v^n
                const double a[3] = {fma(q.hdt, ep, v[0]), v[1], v[2]};
                const double t[3] = {q.hdt * q.bext[0], q.hdt * q.bext[1], q.hdt * q.bext[2]};
                double vh[3];
                rotate_half(a, t, vh);
#pragma unroll
                for (int k = 0; k < 3; ++k)
                    vn[u][k] = fma(2.0, vh[k], -v[k]);
            }
            x1[u] = fma(q.hdt, vn[u][0], xs[u]);
        }
        wrap_all<U>(xw, x1, q);
        store_all<NV, U>(xw, vn, valid, Xo, Vo, bcur, q.vstride);
        // the density of step n + 1 at x*_{n+1}
        double qv[U][1];
#pragma unroll
        for (int u = 0; u < U; ++u) {
            double v2 = 0.0, v20 = 0.0;
#pragma unroll
            for (int k = 0; k < NV; ++k) {
                v2 = fma(vn[u][k], vn[u][k], v2);
                v20 = fma(cur.v[u][k], cur.v[u][k], v20);
            }
            ke1 = fma(cur.w[u], v2, ke1);
            ke0 = fma(cur.w[u], v20, ke0);
            qv[u][0] = cur.w[u] * q.qs;
            pos[u] = locate<ORDER>(fma(q.hdt, vn[u][0], xw[u]), q.inv_h, 0.0);
        }
        deposit_all<ORDER, 1, DEP, U>(dep, jt, tw, ng, pos, qv, valid);
        cur = nxt;
        bcur = bnxt;
    }
    dep.finish(jt, tw, ng);
    const int nonfinite = isfinite(ke1) ? dep.over : 1;
    // slots: kinetic energy after, no fallbacks, no Gamma, non-finite; kinetic energy before
    const double sc[4] = {ke1, 0.0, 0.0, (double)nonfinite};
    wave_partials<0xcu>(sc, red);
    const double ke0w = wave_sum(ke0);
    if (lane == 0)
        red0[threadIdx.x >> 6] = ke0w;
    lds_barrier();
    dep.flush_tile(jt, target, 1, ng, tw);
    write_scalars(spw + (size_t)slot * kNS, red, nt);
    if (record_wave(nt)) {
        const double k0 = 0.5 * wave_total(red0, 0, nt >> 6);
        if (lane == 0)
            spw[(size_t)slot * kNS + 4] = k0;
    }
}

template <int ORDER, int NV, int DEP>
__global__ __launch_bounds__(kMaxThreads<NV>) __attribute__((amdgpu_waves_per_eu(kWavesPerEU<NV>)))
void k_std_pass(Run r, Work wk, int64_t step, const double *X, const double *V, double *Xo,
                double *Vo, double *Jd, double *Jc, double *spw)
{
    extern __shared__ double smem[];
    __shared__ double red[kRedSize], red0[16];
    __shared__ int wctr;
    const int64_t p0 = (int64_t)blockIdx.x * r.chunk;
    std_pass_body<ORDER, NV, DEP>(r, kernarg_run(), wk, step, X, V, Xo, Vo, Jd, Jc, spw, p0,
                                  r.interleave ? r.np : min(r.np, p0 + r.chunk),
                                  (int)blockIdx.x == r.nblocks - 1, blockIdx.x, smem, red, red0,
                                  &wctr);
}

// End of a pic_step call (one workgroup): the record of the newest state and a copy of
// the newest fields into the caller's arrays.
__device__ void finish_body(const Run &r, const Work &wk, int par, int64_t step)
{
    if (record_wave() && step > wk.st->recorded) {
        if (r.scheme == kLeapfrog) {
            const double wbl = lf_magnetic_energy(r, wk.Ef[par], wk.Bf[par]);
            if ((threadIdx.x & 63) == 0)
                wk.st->wb = wbl;
        }
        write_record(r, wk, step);
    }
    for (int i = threadIdx.x; i < 3 * r.ng; i += nthreads())
        wk.E[i] = wk.Ef[par][i];
    if (em_scheme(r.scheme))
        for (int i = threadIdx.x; i < 2 * r.ng; i += nthreads())
            wk.B[i] = wk.Bf[par][i];
}

__global__ __launch_bounds__(1024) void k_finish(Run r, Work wk, int par, int64_t step)
{
    finish_body(r, wk, par, step);
}

// Copy of the newest record into a caller's device pic_diag (one thread).
__global__ void k_copy_record(Work wk, int rec_cap, DevRecord *dst)
{
    if (blockIdx.x == 0 && threadIdx.x == 0)
        *dst = wk.rec[wk.st->recorded % rec_cap];
}

// ------------------------------------------------------------------- initialisation
// Predictor deposit of the initial state, w v^0 at x*_0 = x^0 + dt/2 v^0, into J1[0].
template <int ORDER, int NV, bool EM>
__device__ __forceinline__ void predeposit_body(const Run &r, const Work &wk,
                                                const double *__restrict__ X,
                                                const double *__restrict__ V, int64_t p0,
                                                int64_t p1, double *smem)
{
    using T = TileSizes<NV, EM>;
    double *jt = smem;
    double *side = jt + T::ncur * r.tw;
    tile_zero(jt, 2 * T::ncur * r.tw);
    __syncthreads();
    Depo<ORDER, T::ncur, 0> dep;
    dep.init(side, r, wk.st);
    for (int64_t p = p0 + threadIdx.x; p < p1; p += nthreads()) {
        const double q = (r.w ? r.w[p] : r.wu) * r.qs;
        double qv[T::ncur];
#pragma unroll
        for (int c = 0; c < T::ncur; ++c)
            qv[c] = q * V[c * r.vstride + p];
        dep.add(jt, r.tw, r.ng, stencil<ORDER>(fma(r.hdt, V[p], X[p]) * r.inv_h - r.xshift), qv);
    }
    flag_over(dep, wk);
    __syncthreads();
    dep.flush_tile(jt, dep_target(r, wk, wk.J1[0]), T::ncur, r.ng, r.tw);
}

template <int ORDER, int NV, bool EM>
__global__ __launch_bounds__(1024) void k_predeposit(Run r, Work wk, const double *__restrict__ X,
                                                     const double *__restrict__ V)
{
    extern __shared__ double smem[];
    const int64_t p0 = (int64_t)blockIdx.x * r.chunk;
    predeposit_body<ORDER, NV, EM>(r, wk, X, V, p0, min(r.np, p0 + r.chunk), smem);
}

// Charge deposit rho_i = (1/h) sum_p w_p S(x_i - x_p) into J2[0] (scratch for Gauss).
template <int ORDER>
__device__ __forceinline__ void deposit_rho_body(const Run &r, const Work &wk,
                                                 const double *__restrict__ X, int64_t p0,
                                                 int64_t p1, double *smem)
{
    double *jt = smem;
    double *side = jt + r.tw;
    tile_zero(jt, 2 * r.tw);
    __syncthreads();
    Depo<ORDER, 1, 0> dep;
    dep.init(side, r, wk.st, 1);
    for (int64_t p = p0 + threadIdx.x; p < p1; p += nthreads()) {
        const double q[1] = {(r.w ? r.w[p] : r.wu) * r.qs};
        dep.add(jt, r.tw, r.ng, stencil<ORDER>(X[p] * r.inv_h), q);
    }
    flag_over(dep, wk);
    __syncthreads();
    dep.flush_tile(jt, dep_target(r, wk, wk.J2[0]), 1, r.ng, r.tw);
}

template <int ORDER>
__global__ __launch_bounds__(1024) void k_deposit_rho(Run r, Work wk, const double *__restrict__ X)
{
    extern __shared__ double smem[];
    const int64_t p0 = (int64_t)blockIdx.x * r.chunk;
    deposit_rho_body<ORDER>(r, wk, X, p0, min(r.np, p0 + r.chunk), smem);
}

// Both deposits of an ESEC2 start with the Gauss solve in one launch: the charge density into
// J2[0] and the predictor current into J1[0] (electrostatic; not in the deterministic mode,
// whose partial sums hold one deposit at a time).  LDS: two tiles with their side tiles.
template <int ORDER>
__global__ __launch_bounds__(1024) void k_init_deposits(Run r, Work wk, const double *__restrict__ X,
                                                        const double *__restrict__ V)
{
    extern __shared__ double smem[];
    const int tw = r.tw, ng = r.ng;
    const unsigned nt = nthreads();
    double *jr = smem, *sr = jr + tw, *jj = sr + tw, *sj = jj + tw;
    tile_zero(smem, 4 * tw, nt);
    Depo<ORDER, 1, 0> dr, dj;
    dr.init(sr, r, wk.st, 1);
    dj.init(sj, r, wk.st);
    __syncthreads();
    const int64_t p0 = (int64_t)blockIdx.x * r.chunk, p1 = min(r.np, p0 + r.chunk);
    for (int64_t p = p0 + threadIdx.x; p < p1; p += nt) {
        const double x = X[p], v = V[p], q = (r.w ? r.w[p] : r.wu) * r.qs;
        const double qr[1] = {q}, qj[1] = {q * v};
        dr.add(jr, tw, ng, stencil<ORDER>(x * r.inv_h), qr);
        dj.add(jj, tw, ng, stencil<ORDER>(fma(r.hdt, v, x) * r.inv_h - r.xshift), qj);
    }
    __syncthreads();
    dr.flush_tile(jr, rep_slot(wk.J2[0], r.nrep, ng), 1, ng, tw);
    dj.flush_tile(jj, rep_slot(wk.J1[0], r.nrep, ng), 1, ng, tw);
}

// ------------------------------------------------------------- counting-sort rebin
// Particles are reordered by key = kVBins * cell + (v_x >= 0): particles of one cell and
// one direction of motion become contiguous, so a wavefront's particles share a cell or
// two for many steps (gathers become LDS broadcasts, deposits can be summed in registers
// and the global tile flush touches few nodes).  Counting sort: per-workgroup histograms
// (LDS), an exclusive scan of the [key][workgroup] counts, and a scatter in which each
// workgroup places its particles at its own offsets (order inside a key and workgroup is
// unspecified).
__device__ __forceinline__ int sort_key(const Run &r, double x, double vx)
{
    const double cf = floor(x * r.inv_h);
    const int c = (cf >= 0.0 && cf < (double)r.ng) ? (int)cf : (cf >= (double)r.ng ? r.ng - 1 : 0);
    return kVBins * c + (vx >= 0.0 ? 1 : 0);
}

// hist[key * nblocks + b] = number of particles of workgroup b with that key.
__global__ __launch_bounds__(1024) void k_rebin_count(Run r, Work wk, const double *__restrict__ X,
                                                      const double *__restrict__ V)
{
    extern __shared__ int ihist[];
    const int nbins = kVBins * r.ng;
    for (int i = threadIdx.x; i < nbins; i += nthreads())
        ihist[i] = 0;
    __syncthreads();
    const int64_t p0 = (int64_t)blockIdx.x * r.chunk;
    const int64_t p1 = min(r.np, p0 + r.chunk);
    for (int64_t p = p0 + threadIdx.x; p < p1; p += nthreads())
        atomicAdd(&ihist[sort_key(r, X[p], V[p])], 1);
    __syncthreads();
    for (int i = threadIdx.x; i < nbins; i += nthreads())
        wk.hist[(int64_t)i * r.nblocks + blockIdx.x] = ihist[i];
}

// Exclusive scan of hist (length n) in three launches: per-segment sums, a scan of the
// segment sums (one workgroup), and the per-segment rescans.
__global__ __launch_bounds__(1024) void k_scan_sums(const int64_t *a, int64_t n, int64_t seg,
                                                    int64_t *segsum)
{
    __shared__ double red[kRedSize];
    const int64_t s0 = (int64_t)blockIdx.x * seg, s1 = min(n, s0 + seg);
    double acc = 0.0;     // counts are exact in double below 2^53
    for (int64_t i = s0 + threadIdx.x; i < s1; i += nthreads())
        acc += (double)a[i];
    acc = block_sum(acc, red);
    if (threadIdx.x == 0)
        segsum[blockIdx.x] = (int64_t)acc;
}

__global__ __launch_bounds__(1024) void k_scan_top(int64_t *segsum, int nseg)
{
    // nseg <= blockDim: one value per thread, Hillis-Steele in LDS
    __shared__ int64_t buf[1024];
    const int t = threadIdx.x;
    const int64_t mine = t < nseg ? segsum[t] : 0;
    buf[t] = mine;
    __syncthreads();
    for (int off = 1; off < (int)nthreads(); off <<= 1) {
        const int64_t add = t >= off ? buf[t - off] : 0;
        __syncthreads();
        buf[t] += add;
        __syncthreads();
    }
    if (t < nseg)
        segsum[t] = buf[t] - mine;     // exclusive
}

__global__ __launch_bounds__(1024) void k_scan_apply(int64_t *a, int64_t n, int64_t seg,
                                                     const int64_t *segsum)
{
    // in-place exclusive scan of one segment, processed in chunks of blockDim elements
    __shared__ int64_t buf[1024];
    const int t = threadIdx.x;
    const int64_t s0 = (int64_t)blockIdx.x * seg, s1 = min(n, s0 + seg);
    int64_t carry = segsum[blockIdx.x];
    for (int64_t c0 = s0; c0 < s1; c0 += nthreads()) {
        const int64_t i = c0 + t;
        const int64_t mine = i < s1 ? a[i] : 0;
        buf[t] = mine;
        __syncthreads();
        for (int off = 1; off < (int)nthreads(); off <<= 1) {
            const int64_t add = t >= off ? buf[t - off] : 0;
            __syncthreads();
            buf[t] += add;
            __syncthreads();
        }
        if (i < s1)
            a[i] = carry + buf[t] - mine;
        const int64_t total = buf[nthreads() - 1];
        __syncthreads();
        carry += total;
    }
}

// Scatter the state (and ids, weights) of each workgroup's particles to their sorted
// positions in the second buffers.
template <int NV>
__global__ __launch_bounds__(1024) void k_rebin_scatter(Run r, Work wk, const double *__restrict__ X,
                                                        const double *__restrict__ V,
                                                        const int64_t *__restrict__ ID)
{
    extern __shared__ int64_t cursor[];
    const int nbins = kVBins * r.ng;
    for (int i = threadIdx.x; i < nbins; i += nthreads())
        cursor[i] = wk.hist[(int64_t)i * r.nblocks + blockIdx.x];
    __syncthreads();
    const int64_t p0 = (int64_t)blockIdx.x * r.chunk;
    const int64_t p1 = min(r.np, p0 + r.chunk);
    for (int64_t p = p0 + threadIdx.x; p < p1; p += nthreads()) {
        const double x = X[p];
        const int key = sort_key(r, x, V[p]);
        const int64_t d = (int64_t)atomicAdd((unsigned long long *)&cursor[key], 1ull);
        wk.x2[d] = x;
#pragma unroll
        for (int c = 0; c < NV; ++c)
            wk.v2[c * r.np + d] = V[c * r.vstride + p];
        if (ID)
            wk.id2[d] = ID[p];
        if (wk.wcur)
            wk.w2[d] = wk.wcur[p];
    }
}

__global__ void k_copy_i64(int64_t *dst, const int64_t *src, int64_t n)
{
    for (int64_t i = (int64_t)blockIdx.x * nthreads() + threadIdx.x; i < n;
         i += (int64_t)gridDim.x * nthreads())
        dst[i] = src[i];
}

__global__ void k_copy_f64(double *dst, const double *src, int64_t n)
{
    for (int64_t i = (int64_t)blockIdx.x * nthreads() + threadIdx.x; i < n;
         i += (int64_t)gridDim.x * nthreads())
        dst[i] = src[i];
}

// Wrap positions into [0, L); the initial kinetic energy and non-finite flag go to
// spart[slot] like the scalars of a pass B.
template <int NV>
__device__ __forceinline__ void init_particles_body(const Run &r, const Work &wk,
                                                    double *__restrict__ X,
                                                    const double *__restrict__ V, int64_t p0,
                                                    int64_t p1, int slot, double *red)
{
    double ke = 0.0, ws = 0.0, wmax = 0.0, wvmax = 0.0;
    int nonfinite = 0;
    for (int64_t p = p0 + threadIdx.x; p < p1; p += nthreads()) {
        double v2 = 0.0, vm = 0.0;
#pragma unroll
        for (int c = 0; c < NV; ++c) {
            const double vc = V[c * r.vstride + p];
            v2 += vc * vc;
            vm = fmax(vm, fabs(vc));
        }
        const double x = X[p];
        if (!isfinite(x) || !isfinite(v2))
            nonfinite = 1;
        X[p] = wrap_pos(x, r.L);
        const double wp = r.w ? r.w[p] : r.wu;
        ke += wp * v2;
        ws += wp;
        wmax = fmax(wmax, fabs(wp));
        wvmax = fmax(wvmax, fabs(wp) * vm);
    }
    double sums[2] = {ke, ws}, maxes[3] = {(double)nonfinite, wmax, wvmax};
    block_reduce<0u>(sums, red);
    block_reduce<7u>(maxes, red);
    if (threadIdx.x == 0) {
        wk.spart[slot * kNS + 0] = 0.5 * sums[0];
        wk.spart[slot * kNS + 1] = 0.0;
        wk.spart[slot * kNS + 2] = 0.0;
        wk.spart[slot * kNS + 3] = maxes[0];
        wk.spart[slot * kNS + 4] = sums[1];
        wk.spart[slot * kNS + 5] = maxes[1];
        wk.spart[slot * kNS + 6] = maxes[2];
    }
}

template <int NV>
__global__ __launch_bounds__(1024) void k_init_particles(Run r, Work wk, double *__restrict__ X,
                                                         const double *__restrict__ V)
{
    __shared__ double red[kRedSize];
    const int64_t p0 = (int64_t)blockIdx.x * r.chunk;
    init_particles_body<NV>(r, wk, X, V, p0, min(r.np, p0 + r.chunk), blockIdx.x, red);
}

// Fixed-point scales of the deposit tiles (one workgroup per run), from the initial
// particles' slots 4-6: the charge density's from the largest weight (a charge
// contribution is at most w / h), the currents' from twice the largest w |v| (or w, if
// that is larger: speeds are in thermal units).  2^S is the largest power of two with
// q 2^S <= Run::fx_lim for that reference contribution q.
__device__ void fx_setup_body(const Run &r, const Work &wk, double *red)
{
    double wmax = 0.0, wvmax = 0.0;
    for (int b = threadIdx.x; b < r.nblocks; b += nthreads()) {
        wmax = fmax(wmax, wk.spart[b * kNS + 5]);
        wvmax = fmax(wvmax, wk.spart[b * kNS + 6]);
    }
    double m[2] = {wmax, wvmax};
    block_reduce<3u>(m, red);
    if (threadIdx.x == 0) {
        const double qref[2] = {2.0 * fmax(m[1], m[0]) * r.inv_h, m[0] * r.inv_h};
        for (int k = 0; k < 2; ++k) {
            int S = 0;
            if (qref[k] > 0.0 && isfinite(qref[k]))
                S = (int)floor(log2(r.fx_lim / qref[k]));
            S = max(-1000, min(1000, S));
            wk.st->fx_scale[k] = ldexp(1.0, S);
            wk.st->fx_inv[k] = ldexp(1.0, -S);
        }
        wk.st->flag_a = 0;
    }
}

__global__ __launch_bounds__(1024) void k_fx_setup(Run r, Work wk)
{
    __shared__ double red[kRedSize];
    fx_setup_body(r, wk, red);
}

// Deterministic mode: J[c][i] = the sum over the workgroups b of part[b][c][i] (replica 0
// of a current; the deterministic mode keeps one replica), always in the same order: a
// workgroup of 256 threads takes 32 consecutive entries; for each entry, 8 threads sum
// consecutive eighths of the rows in row order, and the 8 sums are then added in order.

__global__ __launch_bounds__(256) void k_reduce_partials(const double *__restrict__ part,
                                                         double *__restrict__ J, int nblocks,
                                                         int n, int rowlen)
{
    __shared__ double seg[kRedSegments][kRedEntries];
    const int t = threadIdx.x, e = t % kRedEntries, sg = t / kRedEntries;
    const int idx = blockIdx.x * kRedEntries + e;
    const int per = (nblocks + kRedSegments - 1) / kRedSegments;
    const int b0 = min(nblocks, sg * per), b1 = min(nblocks, b0 + per);
    double acc = 0.0;
    if (idx < n) {
        int b = b0;
        for (; b + 8 <= b1; b += 8) {
            double v[8];
#pragma unroll
            for (int k = 0; k < 8; ++k)
                v[k] = part[(size_t)(b + k) * rowlen + idx];
#pragma unroll
            for (int k = 0; k < 8; ++k)
                acc += v[k];
        }
        for (; b < b1; ++b)
            acc += part[(size_t)b * rowlen + idx];
    }
    seg[sg][e] = acc;
    __syncthreads();
    if (sg == 0 && idx < n) {
        double s = seg[0][e];
#pragma unroll
        for (int k = 1; k < kRedSegments; ++k)
            s += seg[k][e];
        J[idx] = s;
    }
}

// Initial Gauss solve: dE/dx = rho - 1 with rho in J2[0], into the caller's E_x.
// Spectrally on the nodes: E_m = rho_m / (i k_m), k_m = 2 pi m / L for 0 < |m| < N/2, mean
// and Nyquist modes zero (the Poisson form, eq. (poisson), in 1D), as the convolution of rho
// with the row G_d = (2 / N_g) sum_m sin(2 pi m d / N_g) / k_m (0 < m < N_g / 2), which is odd
// in d.  The constant part of rho convolves to zero: rho_0 is taken off first, so it doesn't
// round into the sum.
// One workgroup, so the LDS bounds it: the row takes N_g^2 / 4 reads of the table of sines (m d
// mod N_g: bank conflicts) and the convolution N_g^2 of consecutive addresses, where the two
// transforms of the spectral form took 4 N_g^2 of the first kind (with the launch's other work,
// 512 cells 71.7 -> 26.7 us, 256 cells 24.1 -> 13.6, 64 cells 7.9 -> 6.7).  On grids of at
// most 512 cells S threads share an element of either sum, each taking a consecutive S-th of
// its terms, and the S parts are added in order.
// LDS: rho | sines of 2 pi j / N_g | 1 / k_m [N_g / 2] | G twice over [2 N_g] | partial sums
//      (for the largest of several grids: room for any of them)
__host__ __device__ constexpr size_t gauss_lds_doubles(int ng)
{
    return ng <= 512 ? 5 * (size_t)ng + 1024 : (ng <= 716 ? 3584 : 5 * (size_t)ng);
}

__device__ void gauss_body(const Run &r, const Work &wk, double *smem)
{
    const int ng = r.ng, nt = (int)nthreads(), M = (ng - 1) / 2;
    double *rho = smem, *ts = smem + ng, *ik = smem + 2 * ng, *G = ik + ng / 2 + 1, *part = smem + 5 * ng;
    auto split = [&](int n) { return ng <= 512 ? max(1, min(16, nt / n)) : 1; };
    rep_gather(rho, wk.J2[0], ng, r.nrep, 3 * ng);
    for (int j = threadIdx.x; j < ng; j += nt)
        ts[j] = sinpi(2.0 * (double)j / ng);
    for (int m = threadIdx.x; m <= M; m += nt)
        ik[m] = r.L / (M_PI * m * ng);         // (2 / N_g) / k_m
    __syncthreads();
    if (r.filter_rho) {
        // the standard scheme's filtered density (as in k_std_field), through G
        for (int i = threadIdx.x; i < ng; i += nt)
            G[i] = 0.25 * rho[i == 0 ? ng - 1 : i - 1] + 0.5 * rho[i] + 0.25 * rho[i + 1 == ng ? 0 : i + 1];
        __syncthreads();
        for (int i = threadIdx.x; i < ng; i += nt)
            rho[i] = G[i];
        __syncthreads();
    }
    // G_d, 0 < d < N_g / 2
    const int S1 = split(M), len1 = (M + S1 - 1) / S1;
    for (int it = threadIdx.x; it < S1 * M; it += nt) {
        const int sg = it / M, d = it - sg * M + 1, m0 = sg * len1 + 1, m1 = min(M, m0 + len1 - 1);
        double acc = 0.0;
        int md = (int)(((long long)m0 * d) % ng);      // m d mod N_g
#pragma unroll 4
        for (int m = m0; m <= m1; ++m) {
            acc = fma(ts[md], ik[m], acc);
            md += d;
            md -= md >= ng ? ng : 0;
        }
        if (S1 == 1)
            G[d] = acc;
        else
            part[it] = acc;
    }
    __syncthreads();
    // both periods of the row: G[N_g + d] and G[d] hold G_d, 0 <= d < N_g
    const double r0 = rho[0];
    __syncthreads();
    for (int i = threadIdx.x; i < ng; i += nt) {
        rho[i] -= r0;
        const int d = 2 * i < ng ? i : ng - i;
        double g = 0.0;
        if (i != 0 && 2 * i != ng) {
            if (S1 == 1)
                g = G[d];
            else
                for (int sg = 0; sg < S1; ++sg)
                    g += part[sg * M + d - 1];
            g = i == d ? g : -g;
        }
        G[ng + i] = g;
    }
    __syncthreads();
    for (int i = threadIdx.x; i < ng; i += nt)
        G[i] = G[ng + i];
    __syncthreads();
    // E_i = sum_j G_{i - j} rho_j
    const int S2 = split(ng), len2 = (ng + S2 - 1) / S2;
    for (int it = threadIdx.x; it < S2 * ng; it += nt) {
        const int sg = it / ng, i = it - sg * ng, j0 = sg * len2, j1 = min(ng, j0 + len2);
        const double *g = G + ng + i;
        double acc = 0.0;
#pragma unroll 8
        for (int j = j0; j < j1; ++j)
            acc = fma(g[-j], rho[j], acc);
        if (S2 == 1)
            wk.E[i] = acc;
        else
            part[it] = acc;
    }
    if (S2 == 1)
        return;
    __syncthreads();
    for (int i = threadIdx.x; i < ng; i += nt) {
        double acc = part[i];
        for (int sg = 1; sg < S2; ++sg)
            acc += part[sg * ng + i];
        wk.E[i] = acc;
    }
}

__global__ __launch_bounds__(1024) void k_gauss(Run r, Work wk)
{
    extern __shared__ double smem[];
    gauss_body(r, wk, smem);
}

// The Gauss solve and, the fields then being known, the rest of the initialisation
// (k_init_finish) in one launch.
__device__ void init_finish_body(const Run &r, const Work &wk, double *red);

__global__ __launch_bounds__(1024) void k_gauss_finish(Run r, Work wk)
{
    extern __shared__ double smem[];
    __shared__ double red[kRedSize];
    gauss_body(r, wk, smem);
    __syncthreads();
    init_finish_body(r, wk, red);
}

// Initial field of a charge-conserving run (Run::cc): Gauss' law on the half-node E,
// (E_{i+1/2} - E_{i-1/2}) / h = rho_i - mean(rho), by a running sum from the density in
// J2[0] (quadratic B-spline on the nodes), then the mean of E removed (E = -d(phi)/dx).
// One workgroup; the running sum is serial (N_g additions).
__global__ __launch_bounds__(1024) void k_gauss_cc(Run r, Work wk)
{
    extern __shared__ double smem[];
    __shared__ double red[kRedSize];
    const int ng = r.ng;
    double *rho = smem;
    rep_gather(rho, wk.J2[0], ng, r.nrep, 3 * ng);
    __syncthreads();
    const double m = block_mean(rho, ng, red);
    if (threadIdx.x == 0) {
        double e = 0.0;
        rho[0] = 0.0;               // rho[i] now holds E_{i+1/2}
        for (int i = 1; i < ng; ++i) {
            e += r.h * (rho[i] - m);
            rho[i] = e;
        }
    }
    __syncthreads();
    const double me = block_mean(rho, ng, red);
    for (int i = threadIdx.x; i < ng; i += nthreads())
        wk.E[i] = rho[i] - me;
}

// First row of (I - s L_h)^{-1} for the periodic 3-point Laplacian: circulant, so
// g_k = (1/N) sum_m cos(2 pi m k / N) / (1 + s (4/h^2) sin^2(pi m / N)).  Used by the
// batched form, whose pass B solves Crank-Nicolson in its prologue (field_update).
__device__ void cn_init_body(const Run &r, const Work &wk)
{
    const int ng = r.ng;
    const double s = r.hdt * r.hdt * r.c2;
    for (int k = threadIdx.x; k < ng; k += nthreads()) {
        double acc = 0.0;
        for (int m = 0; m < ng; ++m) {
            const double sn = sinpi((double)m / ng);
            const double lam = 1.0 + s * 4.0 * r.inv_h * r.inv_h * sn * sn;
            const long long mk = ((long long)m * k) % ng;
            acc += cospi(2.0 * (double)mk / ng) / lam;
        }
        wk.cninv[k] = acc / ng;
    }
}


// ------------------------------------------------------------------- EMEC(PSATD)
// Field updates of the electromagnetic schemes as real-space convolutions.
// EMEC(PSATD) (section 4.2): the semi-discrete Maxwell system with the
// current held fixed, dE/dt = c^2 curl B - j, dB/dt = -curl E, integrated exactly over a
// time tau for each Fourier mode (eq. (PSATDformula)), and the time average of E over the
// step (its time integral).  In 1D the transverse pairs (E_y, B_z) and (E_z, -B_y) both
// obey dE/dt = -c^2 D- B - j, dB/dt = -D+ E with E, j on the nodes and B on the half
// nodes; the curls are spectral on this staggered grid: D+ (nodes to half nodes)
// multiplies mode k by a = i k e^{i k h/2}, D- (half nodes to nodes) by
// b = i k e^{-i k h/2}, so that a b = -k^2.  With w = c |k|, C = cos(w tau),
// S = sin(w tau) and 1 - C = 2 sin^2(w tau / 2):
//   E(tau) = C E - c^2 b S/w B - S/w j,   B(tau) = C B - a S/w E + a (1 - C)/w^2 j,
//   <E>    = S/(w tau) E - c^2 b (1 - C)/(w^2 tau) B - (1 - C)/(w^2 tau) j,
// and mode 0: E - tau j, B, E - tau/2 j.  Each map is a circulant convolution in real
// space, out_i = sum_j K[(i - j) mod N] in_j, whose row K[d] = (1/N) Re sum_m K(m)
// e^{2 pi i m d / N} (m signed, |m| <= N/2; every symbol is real at the Nyquist mode)
// is computed once here: grid (ceil(N / blockDim), kPsatdRows).
__device__ __forceinline__ void psatd_symbol(const Run &r, int row, int ms, double &sr, double &si)
{
    const bool full = row >= kRowC2;
    const double tau = full ? r.dt : r.hdt;
    if (ms == 0) {
        sr = (row == kRowC1 || row == kRowC2 || row == kRowAE) ? 1.0
             : (row == kRowEJ1 || row == kRowEJ2) ? -tau
             : row == kRowAJ ? -0.5 * tau : 0.0;
        si = 0.0;
        return;
    }
    const double k = 2.0 * M_PI * (double)ms / r.L;
    const double w = sqrt(r.c2) * fabs(k);
    double sh, ch;                       // e^{i k h/2} = ch + i sh, k h/2 = pi ms / N
    sincospi((double)ms / r.ng, &sh, &ch);
    double S, C;
    sincos(w * tau, &S, &C);
    const double sh2 = sin(0.5 * w * tau);
    const double omc = 2.0 * sh2 * sh2;  // 1 - C
    // a = i k e^{i k h/2} = k (-sh + i ch),  b = i k e^{-i k h/2} = k (sh + i ch)
    switch (row) {
    case kRowC1: case kRowC2: sr = C; si = 0.0; break;
    case kRowEB1: case kRowEB2: sr = -r.c2 * S / w * k * sh; si = -r.c2 * S / w * k * ch; break;
    case kRowEJ1: case kRowEJ2: sr = -S / w; si = 0.0; break;
    case kRowBE1: case kRowBE2: sr = S / w * k * sh; si = -S / w * k * ch; break;
    case kRowBJ1: case kRowBJ2: sr = -omc / (w * w) * k * sh; si = omc / (w * w) * k * ch; break;
    case kRowAE: sr = S / (w * tau); si = 0.0; break;
    case kRowAB: sr = -r.c2 * omc / (w * w * tau) * k * sh; si = -r.c2 * omc / (w * w * tau) * k * ch; break;
    default: sr = -omc / (w * w * tau); si = 0.0; break;   // kRowAJ
    }
}

// The same rows for EMEC(LI) (eq. (EMbasic) with Crank-Nicolson), from the symbols of the
// staggered differences, D+ -> a = (e^{i k h} - 1)/h and D- -> b = (1 - e^{-i k h})/h, with
// lambda = s a b = -4 s sin^2(k h/2)/h^2 (s = (dt/2)^2 c^2) and d = 1 - lambda:
//   predictor (explicit half step): E* = E - dt/2 c^2 b B - dt/2 j, B* = B - dt/2 a E;
//   full step: E' = (1 + lambda)/d E - dt c^2 b/d B - dt/d j,
//              B' = B - dt/2 a (E + E') = (1 + lambda)/d B - dt a/d E + dt^2 a/(2 d) j;
//   average (E + E')/2 = E/d - dt c^2 b/(2 d) B - dt/(2 d) j.
__device__ __forceinline__ void cn_symbol(const Run &r, int row, int ms, double &sr, double &si)
{
    double st, ct, sh;                   // sin, cos of k h = 2 pi ms / N; sin(k h/2)
    sincospi(2.0 * (double)ms / r.ng, &st, &ct);
    sh = sinpi((double)ms / r.ng);
    const double omc = 2.0 * sh * sh;    // 1 - cos(k h)
    // a = (-omc + i st)/h,  b = (omc + i st)/h
    const double ar = -omc * r.inv_h, ai = st * r.inv_h, br = omc * r.inv_h, bi = st * r.inv_h;
    const double s = r.hdt * r.hdt * r.c2;
    const double lam = -4.0 * s * sh * sh * r.inv_h * r.inv_h, d = 1.0 - lam;
    const double dt = r.dt;
    switch (row) {
    case kRowC1: sr = 1.0; si = 0.0; break;
    case kRowEB1: sr = -r.hdt * r.c2 * br; si = -r.hdt * r.c2 * bi; break;
    case kRowEJ1: sr = -r.hdt; si = 0.0; break;
    case kRowBE1: sr = -r.hdt * ar; si = -r.hdt * ai; break;
    case kRowBJ1: sr = 0.0; si = 0.0; break;
    case kRowC2: sr = (1.0 + lam) / d; si = 0.0; break;
    case kRowEB2: sr = -dt * r.c2 * br / d; si = -dt * r.c2 * bi / d; break;
    case kRowEJ2: sr = -dt / d; si = 0.0; break;
    case kRowBE2: sr = -dt * ar / d; si = -dt * ai / d; break;
    case kRowBJ2: sr = dt * dt * ar / (2.0 * d); si = dt * dt * ai / (2.0 * d); break;
    case kRowAE: sr = 1.0 / d; si = 0.0; break;
    case kRowAB: sr = -dt * r.c2 * br / (2.0 * d); si = -dt * r.c2 * bi / (2.0 * d); break;
    default: sr = -dt / (2.0 * d); si = 0.0; break;   // kRowAJ
    }
}

// Rows of the electromagnetic field updates (EMEC(PSATD) or EMEC(LI) by Run::scheme):
// grid (ceil(N / blockDim), kPsatdRows).
__global__ __launch_bounds__(256) void k_em_rows(Run r, Work wk)
{
    extern __shared__ double sym[];      // [2][ng]: the row's symbol, real and imaginary
    const int ng = r.ng, row = blockIdx.y;
    for (int m = threadIdx.x; m < ng; m += nthreads()) {
        const int ms = 2 * m <= ng ? m : m - ng;
        if (r.scheme == kPsatd)
            psatd_symbol(r, row, ms, sym[m], sym[ng + m]);
        else
            cn_symbol(r, row, ms, sym[m], sym[ng + m]);
    }
    __syncthreads();
    const int d = blockIdx.x * nthreads() + threadIdx.x;
    if (d >= ng)
        return;
    double acc = 0.0;
    for (int m = 0; m < ng; ++m) {
        double sn, cs;
        const long long q = ((long long)m * d) % ng;
        sincospi(2.0 * (double)q / ng, &sn, &cs);
        acc += sym[m] * cs - sym[ng + m] * sn;
    }
    wk.prow[(size_t)row * ng + d] = acc / ng;
}

// One electromagnetic field update by the rows of k_em_rows.  full = 0: the predictor
// fields (E*, B*) into ps (EMEC(PSATD): PSATD(E^n, B^n, j^{n,*}, dt/2), eq. (EM_PSATD)
// second line); full = 1: (E^{n+1}, B^{n+1}) from E^n, B^n and j^{*,n+1/2} into
// Ef[par ^ 1], Bf[par ^ 1], and into pf the E that v-dagger gathers (PSATD: the time
// average <E> over the step; LI: (E^n + E^{n+1})/2) and B^{n+1/2} = (B^n + B^{n+1})/2.
// Grid (ceil(N / kFieldNodes), nq), one wavefront per node: blockIdx.y picks the pair p and the
// output o (predictor: q = 2 p + o, o = E, B; full: q = 3 p + o, o = E, B, <E>); each node is
// one wave_convolve, so the update is reproducible.  E_x has no curl term: E_x - tau j_x
// (average E_x - tau/2 j_x), written by q = 0.  (As k_std_field: the launch is round trips, and
// 64 lanes to a node instead of eight make it 6.3 -> 4.8 us at 251 cells, the shortest 5.9 ->
// 3.8.)
// LDS: e | B (signed) | j | the three rows [6][N].
__global__ __launch_bounds__(64 * kFieldNodes) void k_em_fields(Run r, Work wk, int full)
{
    extern __shared__ double sm[];
    const int ng = r.ng, rs = 3 * ng, q = blockIdx.y;
    const unsigned nt = nthreads();
    const int p = full ? q / 3 : q >> 1, o = full ? q % 3 : q & 1;
    const double *E = wk.Ef[0], *B = wk.Bf[0], *J = full ? wk.J2[0] : wk.J1[0];
    const int bc = p == 0 ? 1 : 0;       // pair 0: B_z, pair 1: B_y (taken as -B_y)
    const double sg = p == 0 ? 1.0 : -1.0;
    double *e = sm, *b = sm + ng, *jj = sm + 2 * ng, *k0 = sm + 3 * ng, *k1 = sm + 4 * ng,
           *k2 = sm + 5 * ng;
    int r0, r1, r2;
    if (o == 0) {
        r0 = full ? kRowC2 : kRowC1; r1 = full ? kRowEB2 : kRowEB1; r2 = full ? kRowEJ2 : kRowEJ1;
    } else if (o == 1) {
        r0 = full ? kRowBE2 : kRowBE1; r1 = full ? kRowC2 : kRowC1; r2 = full ? kRowBJ2 : kRowBJ1;
    } else {
        r0 = kRowAE; r1 = kRowAB; r2 = kRowAJ;
    }
    const int i = blockIdx.x * kFieldNodes + (threadIdx.x >> 6), ic = min(i, ng - 1);
    // what the node's own lane needs besides the sums, in the same round of loads
    const double bi = B[bc * ng + ic], exi = E[ic], jxi = q == 0 ? rep_sum(J, ic, r.nrep, rs) : 0.0;
    for (int n = threadIdx.x; n < ng; n += nt) {
        const double en = E[(1 + p) * ng + n], bn = B[bc * ng + n];
        const double a0 = wk.prow[(size_t)r0 * ng + n], a1 = wk.prow[(size_t)r1 * ng + n],
                     a2 = wk.prow[(size_t)r2 * ng + n];
        jj[n] = rep_sum(J, (1 + p) * ng + n, r.nrep, rs);
        e[n] = en;
        b[n] = sg * bn;
        k0[n] = a0;
        k1[n] = a1;
        k2[n] = a2;
    }
    __syncthreads();
    if (i >= ng)
        return;
    const double *const K[3] = {k0, k1, k2}, *const f[3] = {e, b, jj};
    const double acc = wave_convolve<3>(K, f, i, ng);
    if ((threadIdx.x & 63) != 0)
        return;
    if (!full) {
        if (o == 0)
            wk.ps[(1 + p) * ng + i] = acc;
        else
            wk.ps[(3 + bc) * ng + i] = sg * acc;
    } else if (o == 0) {
        wk.Ef[1][(1 + p) * ng + i] = acc;
    } else if (o == 1) {
        const double bn = sg * acc;
        wk.Bf[1][bc * ng + i] = bn;
        wk.pf[(3 + bc) * ng + i] = 0.5 * (bi + bn);
    } else {
        wk.pf[(1 + p) * ng + i] = acc;
    }
    if (q == 0) {
        if (full) {
            wk.Ef[1][i] = exi - r.dt * jxi;
            wk.pf[i] = exi - r.hdt * jxi;
        } else {
            wk.ps[i] = exi - r.hdt * jxi;
        }
    }
}


// Initial fields into the parity-0 buffers and the record of step 0 (one workgroup).
__device__ void init_finish_body(const Run &r, const Work &wk, double *red)
{
    const int ng = r.ng;
    for (int i = threadIdx.x; i < 3 * ng; i += nthreads())
        wk.Ef[0][i] = wk.E[i];
    if (em_scheme(r.scheme))
        for (int i = threadIdx.x; i < 2 * ng; i += nthreads())
            wk.Bf[0][i] = wk.B[i];
    double we, wb;
    field_energies(r, wk.E, wk.B, &we, &wb, red);
    if (r.scheme == kLeapfrog && threadIdx.x < 64)
        wb = lf_magnetic_energy(r, wk.E, wk.B);
    if (threadIdx.x == 0) {
        wk.st->we = we;
        wk.st->wb = wb;
        wk.st->recorded = -1;
    }
    // the charge scratch must be zero before the first centred deposit
    rep_zero(wk.J2[0], 3 * ng, r.nrep, 3 * ng);
    __syncthreads();
    if (threadIdx.x < 64)
        write_record(r, wk, 0);
}

__global__ __launch_bounds__(1024) void k_init_finish(Run r, Work wk)
{
    __shared__ double red[kRedSize];
    init_finish_body(r, wk, red);
}

__global__ void k_fill(double *p, int64_t n, double v)
{
    for (int64_t i = (int64_t)blockIdx.x * nthreads() + threadIdx.x; i < n;
         i += (int64_t)gridDim.x * nthreads())
        p[i] = v;
}

// Zero two ranges (the workspace's fields and currents, the caller's unused components of E).
__global__ void k_clear2(double *p, int64_t n, double *p2, int64_t n2)
{
    for (int64_t i = (int64_t)blockIdx.x * nthreads() + threadIdx.x; i < n + n2;
         i += (int64_t)gridDim.x * nthreads())
        *(i < n ? p + i : p2 + (i - n)) = 0.0;
}

// ----------------------------------------------------------------- batched ensemble
// Many independent runs (different N_p, N_g, L) advanced together.  Particles of all
// runs are packed in one structure of arrays; each run keeps its own fields, currents,
// state and records.  The work is a table of items, each a chunk of one run's
// particles (chunks of a run are consecutive; the first is the run's lead).  Every pass
// is ONE launch of a persistent grid whose workgroups stride over the table, so runs of
// very different sizes load-balance; the step number is read from a device counter so
// that a captured graph of several steps can be replayed unchanged.
struct BatchRun {
    Run r;                 // scalars; r.nblocks = items of this run, r.vstride = packed N
    Work wk;               // this run's arrays (spart points at its first item's slot)
    int64_t poff;          // first particle of the run in the packed arrays
};

struct BatchItem {
    int32_t run;
    int32_t slot;          // chunk index within the run (0 = lead)
    int64_t p0, p1;        // run-local particle range
};

// Copy of a structure that is the same for the whole workgroup (a run's scalars and
// arrays) into scalar registers, one 32-bit word at a time.
template <int N> struct Words {
    int w[N];
};

template <typename T> __device__ __forceinline__ T uniform_copy(const T &g)
{
    static_assert(sizeof(T) % 4 == 0, "32-bit words");
    constexpr int n = (int)(sizeof(T) / 4);
    Words<n> w = __builtin_bit_cast(Words<n>, g);
#pragma unroll
    for (int i = 0; i < n; ++i)
        w.w[i] = __builtin_amdgcn_readfirstlane(w.w[i]);
    return __builtin_bit_cast(T, w);
}

// A structure that no thread writes during the kernel and that the whole workgroup reads
// at one address, read with scalar loads (through the constant address space): the
// descriptors of the batched passes' work items, so that an item's prologue does not wait
// on a chain of vector loads.
template <typename T> __device__ __forceinline__ T uniform_load(const T *g)
{
    static_assert(sizeof(T) % 4 == 0, "32-bit words");
    typedef const __attribute__((address_space(4))) Words<sizeof(T) / 4> *const_ptr;
    return __builtin_bit_cast(T, *(const_ptr)g);
}

// Workgroups of the batched passes hold at most 512 threads: items are small, and two
// workgroups share a CU.
constexpr int kBatchMaxThreads = 512;
// Particles per lane in the batched passes, loaded and computed on together: two (96 Landau
// runs of 1e4 to 1e6 particles: four particles 183 us a step, three 181, two 180; 16 runs of
// 3e5 particles with three components: one particle 208, two 160).  The electrostatic pass B
// then needs a few registers more than its 128: 1 of them, with three components 3 to 10, are
// kept in scratch memory.
constexpr int kBatchUnroll = 2;
// Wavefronts per SIMD the batched passes are compiled for: two 512-thread workgroups per CU
// (at most 128 VGPRs), so that one's prologue and flush overlap the other's particles.  The
// electromagnetic pass B, 161 registers with two quadratic particles, is compiled for three:
// kept within 128 it took 414 us instead of 370 on 16 runs of 3e5 particles x 256 cells, 280
// instead of 225 on 16 of 1e5 x 512 (one particle per lane at four wavefronts 424 and 290).
template <bool EM> constexpr int kBatchWavesPerEU = EM ? 3 : 4;

struct Batch {
    const BatchRun *runs;
    const BatchItem *items;
    int32_t nitems, nruns;
    double *X, *V;         // packed particle arrays
    // Step counters on the device, so that a captured graph of steps can be replayed: pass A
    // of step n reads stepc[0] = n and leaves n + 1 in stepc[1], which pass B reads and
    // copies to stepc[0].  Neither writes the counter it reads, so no workgroup of a pass can
    // see it change, and no launch of its own is needed to advance it (4.8 us of a step).
    int64_t *stepc;
};

template <int ORDER, int NV, bool EM, int DEP>
__global__ __launch_bounds__(kBatchMaxThreads) __attribute__((amdgpu_waves_per_eu(kBatchWavesPerEU<false>))) void k_batch_pass_a(Batch b)
{
    extern __shared__ double smem[];
    __shared__ double red[kRedSize];
    __shared__ int wctr;
    const int64_t step = uniform_load(b.stepc);
    const int par = (int)(step & 1);
    if (blockIdx.x == 0 && threadIdx.x == 0)
        b.stepc[1] = step + 1;
    for (int it = blockIdx.x; it < b.nitems; it += gridDim.x) {
        const BatchItem item = uniform_load(b.items + it);
        const BatchRun br = uniform_load(b.runs + item.run);
        const Run &r = br.r;
        const Work wk = by_parity(br.wk, par);
        pass_a_body<ORDER, NV, EM, DEP, kBatchUnroll, kBatchUnroll>(
            r, (RunPtr)&b.runs[item.run].r, wk, step, b.X + br.poff, b.V + br.poff, item.p0, item.p1,
            item.slot == 0, item.slot, smem, red, &wctr);
        lds_barrier();
    }
}

template <int ORDER, int NV, bool EM, bool PRED, int DEP>
__global__ __launch_bounds__(kBatchMaxThreads) __attribute__((amdgpu_waves_per_eu(kBatchWavesPerEU<EM>))) void k_batch_pass_b(Batch b)
{
    extern __shared__ double smem[];
    __shared__ double red[kRedSize];
    __shared__ int wctr;
    const int64_t done = uniform_load(b.stepc + 1);     // this step's number + 1
    const int par = (int)((done - 1) & 1);
    if (blockIdx.x == 0 && threadIdx.x == 0)
        b.stepc[0] = done;
    for (int it = blockIdx.x; it < b.nitems; it += gridDim.x) {
        const BatchItem item = uniform_load(b.items + it);
        const BatchRun br = uniform_load(b.runs + item.run);
        const Run &r = br.r;
        const Work wk = by_parity(br.wk, par);
        pass_b_body<ORDER, NV, EM, PRED, DEP, kBatchUnroll, kBatchUnroll>(
            r, (RunPtr)&b.runs[item.run].r, wk, b.X + br.poff, b.V + br.poff, b.X + br.poff, b.V + br.poff, item.p0,
            item.p1, item.slot == 0, item.slot, smem, red, &wctr);
        lds_barrier();
    }
}

// One workgroup per run: newest record and fields into the caller's arrays.
__global__ __launch_bounds__(1024) void k_batch_finish(Batch b)
{
    const int64_t step = *b.stepc;
    const BatchRun &br = b.runs[blockIdx.x];
    const Run r = uniform_copy(br.r);
    const Work wk = uniform_copy(br.wk);
    finish_body(r, wk, (int)(step & 1), step);
}

template <int NV>
__global__ __launch_bounds__(1024) void k_batch_init_particles(Batch b)
{
    __shared__ double red[kRedSize];
    for (int it = blockIdx.x; it < b.nitems; it += gridDim.x) {
        const BatchItem item = b.items[it];
        const BatchRun &br = b.runs[item.run];
        const Run r = uniform_copy(br.r);
        const Work wk = uniform_copy(br.wk);
        init_particles_body<NV>(r, wk, b.X + br.poff, b.V + br.poff, item.p0, item.p1, item.slot,
                                red);
        __syncthreads();
    }
}

template <int ORDER>
__global__ __launch_bounds__(1024) void k_batch_deposit_rho(Batch b)
{
    extern __shared__ double smem[];
    for (int it = blockIdx.x; it < b.nitems; it += gridDim.x) {
        const BatchItem item = b.items[it];
        const BatchRun &br = b.runs[item.run];
        const Run r = uniform_copy(br.r);
        const Work wk = uniform_copy(br.wk);
        deposit_rho_body<ORDER>(r, wk, b.X + br.poff, item.p0, item.p1, smem);
        __syncthreads();
    }
}

template <int ORDER, int NV, bool EM>
__global__ __launch_bounds__(1024) void k_batch_predeposit(Batch b)
{
    extern __shared__ double smem[];
    for (int it = blockIdx.x; it < b.nitems; it += gridDim.x) {
        const BatchItem item = b.items[it];
        const BatchRun &br = b.runs[item.run];
        const Run r = uniform_copy(br.r);
        const Work wk = uniform_copy(br.wk);
        predeposit_body<ORDER, NV, EM>(r, wk, b.X + br.poff, b.V + br.poff, item.p0, item.p1, smem);
        __syncthreads();
    }
}

// One workgroup per run.
__global__ __launch_bounds__(1024) void k_batch_fx_setup(Batch b)
{
    __shared__ double red[kRedSize];
    const BatchRun &br = b.runs[blockIdx.x];
    const Run r = uniform_copy(br.r);
    const Work wk = uniform_copy(br.wk);
    fx_setup_body(r, wk, red);
}

__global__ __launch_bounds__(1024) void k_batch_gauss(Batch b)
{
    extern __shared__ double smem[];
    const BatchRun &br = b.runs[blockIdx.x];
    const Run r = uniform_copy(br.r);
    const Work wk = uniform_copy(br.wk);
    gauss_body(r, wk, smem);
}

__global__ __launch_bounds__(1024) void k_batch_cn_init(Batch b)
{
    const BatchRun &br = b.runs[blockIdx.x];
    const Run r = uniform_copy(br.r);
    const Work wk = uniform_copy(br.wk);
    cn_init_body(r, wk);
}

__global__ __launch_bounds__(1024) void k_batch_init_finish(Batch b)
{
    __shared__ double red[kRedSize];
    const BatchRun &br = b.runs[blockIdx.x];
    const Run r = uniform_copy(br.r);
    const Work wk = uniform_copy(br.wk);
    init_finish_body(r, wk, red);
    if (blockIdx.x == 0 && threadIdx.x == 0)
        *b.stepc = 0;
}

}  // namespace pic
