// stage.hip -- the fused finite-volume stage kernel of the Icarus hot path (gfx950, CDNA4).
//
// k_stage is the fused finite-volume stage (paper Sect. 2.1: TVDLF with a
// Woodward-type limiter, second order): a work-group marches along k (phi)
// through a leaf block (or through a part of it, down to one plane, for short
// work lists).
//
// For each k-plane the primitives of the plane and of its two-cell i/j halos
// sit in LDS.  The r- and theta-faces are done in passes of one wave each: rows
// (columns) of cells on adjacent lanes, every cell reconstructed once per
// direction, every face flux computed once, the face state of the cell below
// and the flux of the face above passed between lanes (DPP), and each cell's
// flux difference added to its place in LDS.  The phi-faces and the update
// belong to the thread of the column (i, j): flux differences with the
// finite-volume metric, hoop, Coriolis, centrifugal and gravity sources,
// floors, U_out = U_base + alpha dt L(U), in the second stage the CFL rate.
// Threads without a column turn the halo cells of the next plane into
// primitives.  Halo cells come from neighbouring blocks (same level), the
// block's own edge (outflow) or ghost slabs (inner boundary, coarse-fine
// faces).
//
// What bounds it: fp64 instructions and the latency between them.  Two
// work-groups share a CU (256 VGPRs a lane; 77 KB of LDS on 16 x 12 planes),
// two waves a SIMD; a fp64 operation issues every 4 cycles (at full load the
// clock takes that to 4.3 to 5.4 of 2.4 GHz) and its result is there after 8.
// Hence: few operations (limiters as minima and maxima, no reciprocal in the
// fast speed), the passes spread over the four waves so that no SIMD carries
// more than another (PassSplit), one barrier a plane (two planes of primitives
// and of differences in LDS), loads into registers a plane ahead, LDS rows
// pitched against bank conflicts, nothing spilled in the plane loop with eight
// variables (up to nine registers once per work item; with the tracer up to 24,
// and six scratch accesses a plane).
// Measured on 512 x 60 x 180 cells (2,400 blocks of 16 x 12 x 12): 403 us a
// launch (in XCD-contiguous order 390 to 410 on several cards), before 484 us;
// 4,096 blocks of 12^3: 543 to 559 us (13 G cells/s); 8 blocks of 12^3, one
// work-group each: 52 us, before 71 us (a wave without columns did nothing in the
// face phases of 12 x 12 planes).
#include "common.h"

// ---------------------------------------------------------------------------
// fused stage kernel
// ---------------------------------------------------------------------------

// Cell t of the 4 (BI + BJ) r/theta halo cells of plane k (two layers on each
// side, r-halo first, its two layers of one j adjacent): its (i, j).
template <int BI, int BJ>
DEV void halo_cell(int t, int &i, int &j)
{
    if (t < 4 * BJ) {                 // r-direction halo
        const int side = t / (2 * BJ), rem = t % (2 * BJ);
        const int l = rem % 2;
        j = rem / 2;
        i = side ? BI + l : l - 2;
    } else {                          // theta-direction halo
        const int q = t - 4 * BJ;
        const int side = q / (2 * BI), rem = q % (2 * BI);
        const int l = rem / BI;
        i = rem % BI;
        j = side ? BJ + l : l - 2;
    }
}

// Address spaces: what no launch of this kernel writes (work list, block
// descriptors, metric tables, dt) is read at uniform addresses through the
// constant space, as scalar loads; addresses that came through memory or an
// empty asm are named global, or their accesses would be flat ones.
#define AS_CONST __attribute__((address_space(4)))
#define AS_GLOBAL __attribute__((address_space(1)))
template <class T> DEV const AS_CONST T *in_const(const T *p) { return (const AS_CONST T *)(uintptr_t)p; }

// A k-plane of a block, or of its phi ghosts, for its columns: the value of
// variable v of column c = ci + BI cj is c + v sv doubles behind base.  The
// same for every lane: one address in scalar registers per plane (readfirstlane:
// or the compiler makes a copy of every load for each of the cases).
struct Plane {
    unsigned long long base;
    int sv;
};

// A value that every lane has, in scalar registers.
DEV unsigned long long uniform64(unsigned long long x)
{
    const unsigned lo = __builtin_amdgcn_readfirstlane((int)x), hi = __builtin_amdgcn_readfirstlane((int)(x >> 32));
    return (unsigned long long)hi << 32 | lo;
}

// The double at byte offset `off` behind a uniform base plus n doubles, and
// the other way round.
DEV double ld_at(unsigned long long base, int n, unsigned off)
{
    return *(const AS_GLOBAL double *)((const AS_GLOBAL char *)(base + 8ll * n) + off);
}
DEV void st_at(unsigned long long base, int n, unsigned off, double x)
{
    *(AS_GLOBAL double *)((AS_GLOBAL char *)(base + 8ll * n) + off) = x;
}

template <class S>
DEV Plane phi_plane(const KArgs &a, int slot, int n4, int n5, int k)
{
    constexpr int PL = S::B0 * S::B1;
    const bool in = k >= 0 && k < S::B2, up = k >= S::B2;
    const int code = in ? slot : up ? n5 : n4;
    const int l = up ? k - S::B2 : k + 2;                 // ghost layer, 0 nearest the low side
    const bool slab = code < 0 && code != NBR_OUTFLOW;
    const int blk = code < 0 ? slot : code;
    const int kk = in ? k : code < 0 ? (up ? S::B2 - 1 : 0) : (up ? l : S::B2 - 2 + l);
    const double *const pu = a.U + (size_t)blk * S::NV * S::NC + kk * PL;
    const double *const ps = a.slabs + (size_t)(slab ? nbr_slab(code) : 0) * a.slab_stride + l * PL;
    return Plane{uniform64((uintptr_t)(slab ? ps : pu)), __builtin_amdgcn_readfirstlane(slab ? 2 * PL : S::NC)};
}

// Halo cells behind one face of a block (direction d, face code as in
// BlockDesc::nbr): the cell of layer l (0 nearest the low side), in-face index
// a (j on an r-face, i on a theta-face, the column on a phi-face), plane k (not
// on a phi-face) and variable v is at base + l sl + a sa + k sk + v sv in the
// same-level neighbour, the block's own edge (outflow) or the ghost slab -- the
// cases of cell_addr, resolved once per face.
struct FaceMap {
    const double *base;
    int sl, sa, sk, sv;
};

template <class S>
DEV FaceMap face_map(const KArgs &a, int slot, int code, int d, int side)
{
    constexpr int PL = S::B0 * S::B1;
    const int Bd = S::dim(d), st = d == 0 ? 1 : d == 1 ? S::B0 : PL;        // cells and stride along d in a block
    FaceMap m;
    if (code >= 0 || code == NBR_OUTFLOW) {
        const int blk = code >= 0 ? code : slot;
        const int i0 = code >= 0 ? (side ? 0 : Bd - 2) : (side ? Bd - 1 : 0);   // layer 0 along d
        m.base = a.U + (size_t)blk * S::NV * S::NC + st * i0;
        m.sl = code >= 0 ? st : 0;
        m.sa = d == 0 ? S::B0 : 1;
        m.sk = PL;
        m.sv = S::NC;
    } else {
        const int FA = d == 0 ? S::B1 : S::B0, FB = d == 2 ? S::B1 : S::B2;     // slab layout of cell_addr
        m.base = a.slabs + (size_t)nbr_slab(code) * a.slab_stride;
        m.sl = FB * FA;
        m.sa = 1;
        m.sk = FA;
        m.sv = 2 * FB * FA;
    }
    return m;
}

// Metric records in LDS: the fields the kernel reads (im, ip scaled for the
// limiter, slope_scale).  The lanes of a row read the radial records of
// consecutive cells: 13 doubles apart the 32 lanes of a half-wave meet 32
// distinct bank pairs (16 doubles apart every second record falls on the same
// banks); the lanes of a column read the theta records likewise.
struct LdsR {
    double im, ip, ic, hm, hp, am, ap, rt, icfl, irc;
    double om2r, gg;                             // omega^2 r, G M / r^2
    double pad;
};
struct LdsT {
    double im, ip, ic, hm, hp, thm, thp, ctil, sinc, cosc, phf, icfl, isinc;
    double s2, c2;                               // 2 omega sin, 2 omega cos
};
struct LdsP {
    double im, ip, ic, hm, hp, iw;
};

// Work item of linear work index w when a.xcd_order is set: the work-groups
// of a launch go round-robin to the 8 XCDs (w % 8), so the items are split
// into 8 contiguous runs of the (Morton-ordered) work list, one per XCD, and
// neighbouring blocks -- which read each other's halos -- share an L2.
__device__ inline int xcd_item(int w, int n)
{
    const int q = n >> 3, rem = n & 7;
    const int x = w & 7, pos = w >> 3;
    return x * q + (x < rem ? x : rem) + pos;
}

// The value of the lane below (shr1) or above (shl1) in the wave.
template <int CTRL>
DEV double dpp64(double x)
{
    const long long b = __double_as_longlong(x);
    const int lo = (int)b, hi = (int)(b >> 32);
    const unsigned rl = __builtin_amdgcn_update_dpp(0, lo, CTRL, 0xf, 0xf, true);
    const unsigned rh = __builtin_amdgcn_update_dpp(0, hi, CTRL, 0xf, 0xf, true);
    return __longlong_as_double((long long)((unsigned long long)rh << 32 | rl));
}
// Pitch of rows of n doubles in LDS: the next number that is 2 modulo 4.
constexpr int tile_pitch(int n) { return n + (6 - n % 4) % 4; }

// Adds to a double in LDS (one lane and direction at a time reaches it).
DEV void lds_add(double *p, double x) { __hip_atomic_fetch_add(p, x, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP); }
DEV double shr1(double x) { return dpp64<0x138>(x); }
DEV double shl1(double x) { return dpp64<0x130>(x); }

// One cell's bookkeeping over a work item.
struct CellLog {
    int bad = -1;            // first non-physical stage input or second-stage result: its cell
    int nfr = 0, nfp = 0;    // cell updates the density / pressure floor acted on
    double rmax = 0.0;       // largest CFL rate
};

// Update of one cell: u (U_base in, U_out out) += adt (acc + sources), acc minus
// the flux differences and w the stage input's primitives (overwritten); then
// the floors and, in the second stage, the output check and the CFL rate,
// unless the cell lies on a refluxed face (they follow the reflux).
template <int NV>
DEV void update_cell(const KArgs &a, const Gas &gs, const LdsR &rr, const LdsT &tt, double iw, double adt, bool refluxed,
                     int cell, double *w, double *acc, double *u, CellLog &log)
{
    if (log.bad < 0 && unphysical<NV>(w)) log.bad = cell;
    if (!a.cart) {
        const double c = rr.om2r * tt.sinc;
        add_sources(w, rr.rt, tt.ctil, tt.s2, tt.c2, fma(c, tt.sinc, -rr.gg), c * tt.cosc, acc);
    }
#pragma unroll
    for (int v = 0; v < NV; ++v) u[v] = u[v] + adt * acc[v];
    if (refluxed) return;
    cons_to_prim<false, NV>(u, w, gs);
    if (u[0] < a.rho_floor || w[4] < a.p_floor) {                // rare
        const int f = apply_floors(u, gs, a.rho_floor, a.p_floor);
        log.nfr += f & 1;
        log.nfp += f >> 1;
        cons_to_prim<false, NV>(u, w, gs);
    }
    if (a.want_rate) {
        // the step's result: a non-finite value created in this stage would
        // otherwise drop out of the CFL maximum unnoticed
        if (log.bad < 0 && unphysical<NV>(w)) log.bad = cell;
        const double rate = cell_rate_of(w, rr.icfl, rr.irc * tt.icfl, rr.irc * tt.isinc * iw, gs);
        log.rmax = rate > log.rmax ? rate : log.rmax;
    }
}

// The end of a work item: a member's first bad cell, its floor counts, and the
// item's CFL maximum as part `part` of `parts` of the block (the last part
// clears the entries beyond).
template <int THREADS>
DEV void end_item(const KArgs &a, int slot, int mem, int part, int parts, const CellLog &log, double *sred)
{
    if (log.bad >= 0 && atomicCAS(&a.bad[2 * mem], 0, slot + 1) == 0) a.bad[2 * mem + 1] = log.bad;
    if (log.nfr | log.nfp) {
        atomicAdd(&a.floors[2 * mem], (unsigned long long)log.nfr);
        atomicAdd(&a.floors[2 * mem + 1], (unsigned long long)log.nfp);
    }
    if (a.want_rate) {
        const int tid = threadIdx.x;
        double m = wave_max(log.rmax);
        if ((tid & 63) == 0) sred[tid >> 6] = m;
        __syncthreads();
        if (tid < 64) {
            m = wave_max(tid < THREADS / 64 ? sred[tid] : 0.0);
            double *const r = a.rate + (size_t)slot * KSPLIT_MAX;
            if (tid == part) r[tid] = m;
            else if (part == parts - 1 && tid > part && tid < KSPLIT_MAX) r[tid] = 0.0;
        }
    }
}

// The metric tables of a block's cells (two ghosts a side) into LDS, phi cells
// kt .. kt + nk - 1 (counted with the ghosts); the threads t0 .. of three waves.
template <int BI, int BJ, int LIM>
DEV void load_tables(const KArgs &a, const AS_CONST LevelGeo *lg, int org0, int org1, int org2, int kt, int nk, int tid,
                     LdsR *sR, LdsT *sT, LdsP *sP)
{
    if (tid < BI + 4) {
        const AS_GLOBAL RecR *q = (const AS_GLOBAL RecR *)(uintptr_t)lg->r + org0 + tid;
        sR[tid] = LdsR{slope_scale<LIM>(q->idm), slope_scale<LIM>(q->idp), q->idc, q->hm, q->hp, q->am, q->ap,
                       q->rt, q->icfl, q->irc, a.omega * a.omega * q->rc, a.gm * IC_RCP(q->rc * q->rc), 0.0};
    } else if (tid >= 64 && tid < 64 + BJ + 4) {
        const AS_GLOBAL RecT *q = (const AS_GLOBAL RecT *)(uintptr_t)lg->t + org1 + tid - 64;
        sT[tid - 64] = LdsT{slope_scale<LIM>(q->idm), slope_scale<LIM>(q->idp), q->idc, q->hm, q->hp, q->thm, q->thp,
                            q->ctil, q->sinc, q->cosc, q->phf, q->icfl, q->isinc, 2.0 * a.omega * q->sinc,
                            2.0 * a.omega * q->cosc};
    } else if (tid >= 128 && tid < 128 + nk) {
        const AS_GLOBAL RecP *q = (const AS_GLOBAL RecP *)(uintptr_t)lg->p + org2 + kt + tid - 128;
        sP[tid - 128] = LdsP{slope_scale<LIM>(q->idm), slope_scale<LIM>(q->idp), q->idc, q->hm, q->hp, q->iw};
    }
}

// Which wave does which face passes of a plane.  A pass is one wave's worth of
// rows (r-faces) or columns (theta-faces); per plane a wave with columns has
// their phi-faces and updates besides (1.54 passes' worth of instructions), one
// without them only halo cells (about a quarter).  The passes go to the waves
// greedily, and the odd ones to another column wave from plane to plane (phase),
// so that the four SIMDs carry the same load: 3.5 passes' worth each on 16 x 12
// planes (2, 2, 1 and 3 passes) instead of 4, 4, 4 and 2, and on 12 x 12 planes
// (1, 1, 1 and 3) instead of 4, 4, 4 and 0.
struct PassSplit {
    unsigned begin[3];                           // first pass of wave w at bits 4 w of [phase]; wave 4: the end
};
constexpr PassSplit split_passes(int npass, int nwave, int ncolwave)
{
    PassSplit r{};
    for (int ph = 0; ph < 3; ++ph) {
        int load[4] = {0, 0, 0, 0}, cnt[4] = {0, 0, 0, 0};
        for (int w = 0; w < nwave; ++w) load[w] = w < ncolwave ? 154 : 25;
        for (int p = 0; p < npass; ++p) {
            int best = 0;
            for (int q = 0; q < nwave; ++q) {
                const int w = q < ncolwave ? (q + ph) % ncolwave : q;
                if (q == 0 || load[w] < load[best]) best = w;
            }
            load[best] += 100;
            cnt[best] += 1;
        }
        unsigned at = 0;
        for (int w = 0; w < nwave; ++w) {
            r.begin[ph] |= at << (4 * w);
            at += cnt[w];
        }
        r.begin[ph] |= at << (4 * nwave);
    }
    return r;
}

// NV: conserved variables (8, or 9 with the tracer); W: waves per SIMD the
// register allocation targets (a tuning choice); LIM: the limiter of the
// reconstruction (LIM_MC, the paper's, by default).
template <int BI, int BJ, int BK, int NV, int W, int LIM>
__global__ void __launch_bounds__(NT) __attribute__((amdgpu_waves_per_eu(W, W)))
k_stage(KArgs a)
{
    using S = Shape<BI, BJ, BK, NV>;
    // LDS rows are twice an odd number of doubles apart: the lanes of a theta
    // pass walk the rows of one column, on even bank pairs, those of the next
    // column on the odd ones (rows of 21 and differences of 16 doubles cost 38 %
    // of the LDS cycles in bank conflicts)
    constexpr int PI = BI + 4 + ((BI + 4) % 4 == 2 ? 0 : 2), PJ = BJ + 4;
    constexpr int DI = tile_pitch(BI);
    static_assert(PI % 4 == 2 && DI % 4 == 2, "LDS row pitch");
    constexpr int NCOL = BI * BJ;
    constexpr int NHALO = 4 * (BI + BJ);
    static_assert(NCOL + 64 <= NT, "plane too large for the work-group");
    constexpr int NHR = 4 * BJ;                  // r-halo cells (first; then the theta-halo)
    // the threads without a column take the halo cells, HIT (1 or 2) each
    constexpr int NSP = NT - NCOL, HIT = (NHALO + NSP - 1) / NSP;
    static_assert(HIT <= 2, "halo cells per thread without a column");

    // primitives of two consecutive planes: plane k in sW[k & 1], its r/theta
    // halos with it, and the column cells of plane k+1 in the other one (so that
    // no thread carries them in registers through the face phases)
    __shared__ double sW[2][NV][PJ][PI];
    // minus the r- and theta-flux differences of a plane's cells, plane k in
    // sD[k & 1]: zeroed, then added to by the lane of each direction (two
    // addends on zero give the same bits in either order)
    __shared__ double sD[2][NV][BJ][DI];
    __shared__ LdsR sR[BI + 4];
    __shared__ LdsT sT[BJ + 4];
    __shared__ LdsP sP[BK + 4];
    __shared__ double sred[NT / 64];

    const Gas gs = a.gas;
    const int nitems = *in_const(a.nitems);
    const int ks = a.ksplit;                     // parts of the march along k per block
    const int nwork = nitems * ks;
    for (int wi = blockIdx.x; wi < nwork; wi += gridDim.x) {
        // the thread index, opaque to the compiler once per work item: the
        // addresses and masks derived from it are formed per item instead of
        // being kept live (or spilled) across the whole kernel
        int tid = threadIdx.x;
        asm volatile("" : "+v"(tid));
        const bool col = tid < NCOL;
        const int ci = tid % BI, cj = tid / BI;      // column owned by this thread
        const unsigned tb = 8u * (unsigned)tid;      // its byte offset in a plane
        const int ww = a.xcd_order ? xcd_item(wi, nwork) : wi;
        const int it = ww / ks, part = ww % ks;
        const int k0 = part * BK / ks, k1 = (part + 1) * BK / ks;
        const int slot = in_const(a.items)[it];
        const AS_CONST BlockDesc *const bd = in_const(a.desc) + slot;
        const int mem = bd->member, mk = bd->reflux_mask;
        const int org0 = bd->org[0], org1 = bd->org[1], org2 = bd->org[2];
        const int fr0 = bd->freg[0], fr1 = bd->freg[1], fr2 = bd->freg[2], fr3 = bd->freg[3], fr4 = bd->freg[4],
                  fr5 = bd->freg[5];
        const Faces nb{bd->nbr[0], bd->nbr[1], bd->nbr[2], bd->nbr[3], bd->nbr[4], bd->nbr[5]};
        const double dt = in_const(a.dt)[mem];
        if (dt <= 0.0) continue;                 // member finished: state stays in place
        const double adt = a.alpha * dt;

        // --- prologue: the loads of the first planes go out first (they need
        // the descriptor only): column planes k0-2 .. k0+1 into P0 .. P3, or a
        // halo cell of plane k0 into P0 (and a second one into P1).  Every
        // thread loads all the way through (no branch: the compiler would give
        // each side registers of its own and spill); what it has no cell for
        // comes from its block's first column and is dropped.
        const unsigned tbc = col ? tb : 0u;
        const Plane q0 = phi_plane<S>(a, slot, nb.n4, nb.n5, k0 - 2), q1 = phi_plane<S>(a, slot, nb.n4, nb.n5, k0 - 1);
        const Plane q2 = phi_plane<S>(a, slot, nb.n4, nb.n5, k0), q3 = phi_plane<S>(a, slot, nb.n4, nb.n5, k0 + 1);
        // cell h of a thread without a column: at hp[h] + v hv[h] (bytes) in the
        // plane, hk[h] from plane to plane; hw: its place in sW, -1: none
        unsigned long long hp[2] = {q0.base, q1.base};
        int hv[2] = {8 * q0.sv, 8 * q1.sv}, hk[2] = {0, 0}, hw[2] = {-1, -1};
        {
            const FaceMap m0 = face_map<S>(a, slot, nb.n0, 0, 0), m1 = face_map<S>(a, slot, nb.n1, 0, 1);
            const FaceMap m2 = face_map<S>(a, slot, nb.n2, 1, 0), m3 = face_map<S>(a, slot, nb.n3, 1, 1);
#pragma unroll
            for (int h = 0; h < HIT; ++h) {
                const int t = tid - NCOL + h * NSP;
                int i, j;
                halo_cell<BI, BJ>(t, i, j);
                const bool rh = t < NHR;                  // r-halo, else theta-halo
                const int idx = rh ? i : j, bd_ = rh ? BI : BJ;
                const int side = idx >= bd_ ? 1 : 0, l = side ? idx - bd_ : idx + 2, q = rh ? j : i;
                const int f = (rh ? 0 : 2) + side;
                const double *fb = f == 0 ? m0.base : f == 1 ? m1.base : f == 2 ? m2.base : m3.base;
                const int fl = f == 0 ? m0.sl : f == 1 ? m1.sl : f == 2 ? m2.sl : m3.sl;
                const int fa = f == 0 ? m0.sa : f == 1 ? m1.sa : f == 2 ? m2.sa : m3.sa;
                const int fk = 8 * (f == 0 ? m0.sk : f == 1 ? m1.sk : f == 2 ? m2.sk : m3.sk);
                const int fv = 8 * (f == 0 ? m0.sv : f == 1 ? m1.sv : f == 2 ? m2.sv : m3.sv);
                const bool have = !col && t < NHALO;
                hw[h] = have ? (j + 2) * PI + i + 2 : -1;
                hk[h] = have ? fk : 0;
                hv[h] = have ? fv : hv[h];
                hp[h] = have ? (uintptr_t)(fb + l * fl + q * fa) + (long long)k0 * fk : hp[h] + tbc;
            }
            if (HIT < 2) hp[1] += tbc;
        }
        double P0[NV], P1[NV], P2[NV], P3[NV];
        {
            unsigned long long x = hp[0], y = hp[1];
#pragma unroll
            for (int v = 0; v < NV; ++v, x += hv[0]) P0[v] = *(const AS_GLOBAL double *)x;
#pragma unroll
            for (int v = 0; v < NV; ++v, y += hv[1]) P1[v] = *(const AS_GLOBAL double *)y;
        }
#pragma unroll
        for (int v = 0; v < NV; ++v) P2[v] = ld_at(q2.base, v * q2.sv, tbc);
#pragma unroll
        for (int v = 0; v < NV; ++v) P3[v] = ld_at(q3.base, v * q3.sv, tbc);
        const AS_CONST LevelGeo *const lg = in_const(a.geo) + bd->level;
        const AS_CONST RecP &pm1 = in_const(lg->p)[org2 + k0 + 1], &p0 = in_const(lg->p)[org2 + k0 + 2];
        __syncthreads();                         // the LDS of the item before is done with
        // the metric tables (read after the barrier that ends the prologue)
        load_tables<BI, BJ, LIM>(a, lg, org0, org1, org2, 0, BK + 4, tid, sR, sT, sP);
        // phi-face k0-1/2; registers carried along k: wL = face state of cell k
        // at k+1/2, Fm = flux at k-1/2; W(k) and W(k+1) of the own column sit in
        // LDS
        double wL[NV], Fm[NV];
        CellLog log;
        double *const W0 = &sW[0][0][0][0], *const D0 = &sD[0][0][0][0];
        constexpr int WV = PJ * PI, WB = NV * WV, DV = BJ * DI, DB = NV * DV;     // LDS strides per variable and plane
        int cw = (cj + 2) * PI + ci + 2, cd = cj * DI + ci;
        {
            double w0[NV], w1[NV], Wc[NV], Wn[NV];
            cons_to_prim<false, NV>(P0, w0, gs);
            cons_to_prim<false, NV>(P1, w1, gs);
            cons_to_prim<false, NV>(P2, Wc, gs);
            cons_to_prim<false, NV>(P3, Wn, gs);
            double *const Wk = W0 + (k0 & 1) * WB, *const Wk1 = W0 + (~k0 & 1) * WB;
            const int hw0 = col ? cw : hw[0];
            if (hw0 >= 0)
#pragma unroll
                for (int v = 0; v < NV; ++v) Wk[hw0 + v * WV] = col ? Wc[v] : w0[v];
            if (HIT > 1 && hw[1] >= 0)
#pragma unroll
                for (int v = 0; v < NV; ++v) Wk[hw[1] + v * WV] = w1[v];
            if (col)
#pragma unroll
                for (int v = 0; v < NV; ++v) Wk1[cw + v * WV] = Wn[v];
            double lo[NV], hi[NV], R0[NV];
            reconstruct<LIM, NV>(w0, w1, Wc, slope_scale<LIM>(pm1.idm), slope_scale<LIM>(pm1.idp), pm1.idc, pm1.hm,
                                 pm1.hp, lo, hi);
            reconstruct<LIM, NV>(w1, Wc, Wn, slope_scale<LIM>(p0.idm), slope_scale<LIM>(p0.idp), p0.idc, p0.hm, p0.hp,
                                 R0, wL);
            rusanov<2, NV>(hi, R0, Fm, gs);
            if (k0 == 0 && fr4 >= 0 && col)
                for (int v = 0; v < NV; ++v) st_at((uintptr_t)(a.freg + (size_t)fr4 * a.reg_stride), v * NCOL, tb, Fm[v]);
        }

        if (col)
#pragma unroll
            for (int v = 0; v < 2 * NV; ++v) D0[cd + v * DV] = 0.0;

        // A lane's place in the face passes: pass t takes RPW rows, the cells
        // rc = -1 .. BI of row t RPW + rjl on adjacent lanes, or CPW columns, the
        // cells tc = -1 .. BJ of column t CPW + til
        constexpr int RL = BI + 2, RPW = 64 / RL, NR = (BJ + RPW - 1) / RPW;
        constexpr int CL = BJ + 2, CPW = 64 / CL, NTH = (BI + CPW - 1) / CPW;
        constexpr PassSplit split = split_passes(NR + NTH, NT / 64, (NCOL + 63) / 64);
        const int lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
        int rc = lane % RL - 1, rjl = lane < RPW * RL ? lane / RL : BJ;
        int tc = lane % CL - 1, til = lane < CPW * CL ? lane / CL : BI;
        // the block's refluxed faces this column touches at r and theta
        int crf = (ci == 0 && (mk & 1)) || (ci == BI - 1 && (mk & 2)) || (cj == 0 && (mk & 4)) || (cj == BJ - 1 && (mk & 8));
        asm volatile("" : "+v"(rc), "+v"(tc), "+v"(rjl), "+v"(til), "+v"(cw), "+v"(cd), "+v"(crf));
        const unsigned long long ubase = (uintptr_t)(a.Ubase + (size_t)slot * NV * S::NC);
        const unsigned long long uout = (uintptr_t)(a.Uout + (size_t)slot * NV * S::NC);

        // What a thread needs from memory in the planes ahead is asked for early,
        // into registers.  A: the column's plane k+2 for the phi-face of plane k,
        // asked for at the end of plane k-1; B: its U_base of plane k, asked for
        // at the start of plane k and used after its barrier.  A thread without a
        // column: halo cells of plane k+1.
        double A[NV], B[NV], W2[NV], Fp[NV];
        auto load_A = [&](int k) {
            const Plane pl = phi_plane<S>(a, slot, nb.n4, nb.n5, k + 2);
            hp[0] += k + 1 < k1 ? hk[0] : 0;
            unsigned long long x = col ? pl.base + tb : hp[0];
            const int xs = col ? 8 * pl.sv : hv[0];
#pragma unroll
            for (int v = 0; v < NV; ++v, x += xs) A[v] = *(const AS_GLOBAL double *)x;
        };
        auto load_B = [&](int k) {
            hp[1] += k + 1 < k1 ? hk[1] : 0;
            unsigned long long y = col ? ubase + 8ll * k * NCOL + tb : hp[1];
            const int ys = col ? 8 * S::NC : hv[1];
#pragma unroll
            for (int v = 0; v < NV; ++v, y += ys) B[v] = *(const AS_GLOBAL double *)y;
        };
        load_A(k0);
        __syncthreads();

        // One barrier per plane: behind it a column thread updates its cell of
        // the plane whose faces are done, then the waves go on to the faces of
        // the next one, whose primitives were complete at the same barrier.
#pragma unroll 1
        for (int k = k0;; ++k) {
            if (k > k0 && col) {
                // update of cell (ci, cj, kc)
                const int kc = k - 1;
                double *const Wc = W0 + (kc & 1) * WB, *const Dc = D0 + (kc & 1) * DB;
                const LdsR &rr = sR[ci + 2];
                const LdsT &tt = sT[cj + 2];
                double w[NV], acc[NV];
#pragma unroll
                for (int v = 0; v < NV; ++v) w[v] = Wc[cw + v * WV];
#pragma unroll
                for (int v = 0; v < NV; ++v) acc[v] = Dc[cd + v * DV];
                const double rt = rr.rt, iw = sP[kc + 2].iw, kf = rt * tt.phf * iw;
#pragma unroll
                for (int v = 0; v < NV; ++v) {
                    Wc[cw + v * WV] = W2[v];         // own cell of plane kc+2, where plane kc's was
                    Dc[cd + v * DV] = 0.0;
                }
#pragma unroll
                for (int v = 0; v < NV; ++v) {
                    acc[v] = acc[v] + fma(-kf, Fp[v], kf * Fm[v]);
                    Fm[v] = Fp[v];
                }
                update_cell<NV>(a, gs, rr, tt, iw, adt, crf || (kc == 0 && (mk & 16)) || (kc == BK - 1 && (mk & 32)),
                                tid + NCOL * kc, w, acc, B, log);
                const unsigned long long uo = uout + 8ll * kc * NCOL;
#pragma unroll
                for (int v = 0; v < NV; ++v) st_at(uo, v * S::NC, tb, B[v]);
            }
            if (k == k1) break;
            double *const Wk = W0 + (k & 1) * WB, *const Wk1 = W0 + (~k & 1) * WB, *const Dk = D0 + (k & 1) * DB;
            load_B(k);

            // this wave's face passes.  Every lane goes through (those without a
            // cell, or whose face or difference is no use, on any values): each
            // reconstructs its cell's two face states, takes the upper one of the
            // cell below from its lane, and computes the flux at its lower face;
            // the flux at its upper face comes back from the lane above, and the
            // cell's difference goes to sD.
            const int ph = k % 3;
            const unsigned bs = (ph == 0 ? split.begin[0] : ph == 1 ? split.begin[1] : split.begin[2]) >> (4 * wave);
            const int t0 = bs & 15, t1 = (bs >> 4) & 15;
#pragma unroll 1
            for (int t = t0; t < t1 && t < NR; ++t) {            // r
                const int j = t * RPW + rjl;
                const bool act = j < BJ;
                const int at = act ? (j + 2) * PI + rc + 1 : 0;
                double wm[NV], w0[NV], wp[NV], lo[NV], hi[NV], L[NV], fx[NV];
#pragma unroll
                for (int v = 0; v < NV; ++v) {
                    wm[v] = Wk[at + v * WV];
                    w0[v] = Wk[at + v * WV + 1];
                    wp[v] = Wk[at + v * WV + 2];
                }
                const LdsR &m = sR[rc + 2];
                reconstruct<LIM, NV>(wm, w0, wp, m.im, m.ip, m.ic, m.hm, m.hp, lo, hi);
#pragma unroll
                for (int v = 0; v < NV; ++v) L[v] = shr1(hi[v]);
                rusanov<0, NV>(L, lo, fx, gs);
                const double ap = m.ap, am = m.am;
#pragma unroll
                for (int v = 0; v < NV; ++v) L[v] = fma(-ap, shl1(fx[v]), am * fx[v]);
                if (act && rc >= 0 && rc < BI)
#pragma unroll
                    for (int v = 0; v < NV; ++v) lds_add(Dk + j * DI + rc + v * DV, L[v]);
                if (act && (rc == 0 || rc == BI)) {      // raw flux at a coarse-fine face, for the reflux
                    const int r = rc == 0 ? fr0 : fr1;
                    if (r >= 0)
                        for (int v = 0; v < NV; ++v)
                            a.freg[(size_t)r * a.reg_stride + ((size_t)v * BK + k) * BJ + j] = fx[v];
                }
            }
#pragma unroll 1
            for (int t = t0 > NR ? t0 - NR : 0; t < t1 - NR; ++t) {    // theta
                const int i = t * CPW + til;
                const bool act = i < BI;
                const int at = act ? (tc + 1) * PI + i + 2 : 0;
                double wm[NV], w0[NV], wp[NV], lo[NV], hi[NV], L[NV], fx[NV];
#pragma unroll
                for (int v = 0; v < NV; ++v) {
                    wm[v] = Wk[at + v * WV];
                    w0[v] = Wk[at + v * WV + PI];
                    wp[v] = Wk[at + v * WV + 2 * PI];
                }
                const LdsT &m = sT[tc + 2];
                reconstruct<LIM, NV>(wm, w0, wp, m.im, m.ip, m.ic, m.hm, m.hp, lo, hi);
#pragma unroll
                for (int v = 0; v < NV; ++v) L[v] = shr1(hi[v]);
                rusanov<1, NV>(L, lo, fx, gs);
                const double rt = sR[act ? i + 2 : 0].rt, thp = rt * m.thp, thm = rt * m.thm;
#pragma unroll
                for (int v = 0; v < NV; ++v) L[v] = fma(-thp, shl1(fx[v]), thm * fx[v]);
                if (act && tc >= 0 && tc < BJ)
#pragma unroll
                    for (int v = 0; v < NV; ++v) lds_add(Dk + tc * DI + i + v * DV, L[v]);
                if (act && (tc == 0 || tc == BJ)) {
                    const int r = tc == 0 ? fr2 : fr3;
                    if (r >= 0)
                        for (int v = 0; v < NV; ++v)
                            a.freg[(size_t)r * a.reg_stride + ((size_t)v * BK + k) * BI + i] = fx[v];
                }
            }

            // phi-face k+1/2 of the column: cells k, k+1 (LDS) and k+2 (memory)
            if (col) {
                double lo1[NV], hi1[NV], w0[NV], w1[NV];
                cons_to_prim<false, NV>(A, W2, gs);
#pragma unroll
                for (int v = 0; v < NV; ++v) {
                    w0[v] = Wk[cw + v * WV];
                    w1[v] = Wk1[cw + v * WV];
                }
                const LdsP &m = sP[k + 3];
                reconstruct<LIM, NV>(w0, w1, W2, m.im, m.ip, m.ic, m.hm, m.hp, lo1, hi1);
                rusanov<2, NV>(wL, lo1, Fp, gs);
                if (k == BK - 1 && fr5 >= 0) {
                    int r = fr5;
                    asm volatile("" : "+s"(r));     // its addresses are formed here, not kept through the loop
                    for (int v = 0; v < NV; ++v) st_at((uintptr_t)(a.freg + (size_t)r * a.reg_stride), v * NCOL, tb, Fp[v]);
                }
#pragma unroll
                for (int v = 0; v < NV; ++v) wL[v] = hi1[v];
            } else if (k + 1 < k1) {
                // the other threads turn the halo of plane k+1 into primitives
#pragma unroll
                for (int h = 0; h < HIT; ++h)
                    if (hw[h] >= 0) {
                        double w[NV];
                        cons_to_prim<false, NV>(h == 0 ? A : B, w, gs);
#pragma unroll
                        for (int v = 0; v < NV; ++v) Wk1[hw[h] + v * WV] = w[v];
                    }
            }
            if (k + 1 < k1) load_A(k + 1);
            __syncthreads();
        }
        end_item<NT>(a, slot, mem, part, ks, log, sred);
    }
}

// ---------------------------------------------------------------------------
// the same stage for short work lists
// ---------------------------------------------------------------------------
// k_stage marches: a work-group does the planes of its part one after another,
// which costs latency where the list does not fill the chip.  k_tile does KZ
// planes of a block at once, with the same face states, fluxes and sums, hence
// the same bits: the rows of cells along r and theta, then along phi, are
// passes of one wave each, straight from memory (64 / (B + 4) rows a wave, halo
// cells included, neighbours passed between lanes); the differences are added
// in LDS, the phi ones behind a barrier, and after another one every thread
// updates cells.  It executes about 1.3 times the instructions (the phi rows of
// KZ cells carry four halo cells), but no wave waits for another's plane, and
// four waves a SIMD hide each other's latency (128 VGPRs: up to 19 values are
// spilled and read back once per work item, none in the passes' loops).

// Measured (stage launch, k_stage with its default split, with its best one,
// k_tile): 8 blocks of 12^3 21.5, 16.0, 14.8 us, 40 of them 25, 21.1, 20, 80 31,
// 26.2, 26, 160 45, 36.4, 40, 320 71, 64.4, 69, 512 84, 84.2, 97; 1,024 blocks of
// 4^3 42 and 24 (default, k_tile), 48 of 16 x 12 x 12 27 and 29.
constexpr int TT = 512;      // threads per work-group of k_tile

// Rows along D of planes k0 .. k0 + KZ - 1, and how many go into a pass.
template <int BI, int BJ, int KZ, int D>
struct TileRows {
    static constexpr int B = D == 0 ? BI : D == 1 ? BJ : KZ;                 // cells of a row
    static constexpr int X = D == 0 ? BJ : D == 1 ? BI : BI * BJ;            // rows per plane (phi: in all)
    static constexpr int RL = B + 4, RPW = 64 / RL, NROW = D == 2 ? X : X * KZ, NP = (NROW + RPW - 1) / RPW;
};

// Passes first, first + step, ... over the rows along D.
template <int BI, int BJ, int BK, int NV, int LIM, int KZ, int D>
DEV void tile_passes(const KArgs &a, int slot, int nlo, int nhi, int flo, int fhi, const Gas &gs, int k0, int first,
                     int step, int lane, const LdsR *sR, const LdsT *sT, const LdsP *sP, double *D0)
{
    using S = Shape<BI, BJ, BK, NV>;
    using T = TileRows<BI, BJ, KZ, D>;
    constexpr int PL = BI * BJ, DI = tile_pitch(BI), DK = BJ * DI + 2, DV = KZ * DK;
    constexpr int ext = S::dim(D), st = D == 0 ? 1 : D == 1 ? BI : PL;      // the block along D: cells, stride
    const unsigned long long own = (uintptr_t)(a.U + (size_t)slot * NV * S::NC);
    const FaceMap mlo = face_map<S>(a, slot, nlo, D, 0), mhi = face_map<S>(a, slot, nhi, D, 1);
    const int c = lane % T::RL - 2, rl = lane < T::RPW * T::RL ? lane / T::RL : T::NROW;
    const int cd = D == 2 ? k0 + c : c;
    // the lane's cell: in the block, or behind its lower or upper face
    const bool below = cd < 0, above = cd >= ext;
    const unsigned long long base = below ? (uintptr_t)mlo.base : above ? (uintptr_t)mhi.base : own;
    const int off = below ? (cd + 2) * mlo.sl : above ? (cd - ext) * mhi.sl : st * cd;
    const int sx = D == 2 ? 1 : below ? mlo.sa : above ? mhi.sa : D == 0 ? BI : 1;
    const int sk = D == 2 ? 0 : below ? mlo.sk : above ? mhi.sk : PL;
    const long long sv = 8 * (below ? mlo.sv : above ? mhi.sv : S::NC);
#pragma unroll 1
    for (int p = first; p < T::NP; p += step) {
        const int row = p * T::RPW + rl;
        const bool act = row < T::NROW;
        const int x = act ? row % T::X : 0, kk = act ? row / T::X : 0;
        unsigned long long ad = base + 8ll * (off + x * sx + (k0 + kk) * sk);
        double u[NV], w[NV], wm[NV], wp[NV], lo[NV], hi[NV], fx[NV];
#pragma unroll
        for (int v = 0; v < NV; ++v, ad += sv) u[v] = *(const AS_GLOBAL double *)ad;
        cons_to_prim<false, NV>(u, w, gs);
#pragma unroll
        for (int v = 0; v < NV; ++v) {
            wm[v] = shr1(w[v]);
            wp[v] = shl1(w[v]);
        }
        double fm, fp;
        if (D == 0) {
            const LdsR &m = sR[c + 2];
            reconstruct<LIM, NV>(wm, w, wp, m.im, m.ip, m.ic, m.hm, m.hp, lo, hi);
            fm = m.am;
            fp = m.ap;
        } else if (D == 1) {
            const LdsT &m = sT[c + 2];
            reconstruct<LIM, NV>(wm, w, wp, m.im, m.ip, m.ic, m.hm, m.hp, lo, hi);
            const double rt = sR[x + 2].rt;
            fm = rt * m.thm;
            fp = rt * m.thp;
        } else {
            const LdsP &m = sP[c + 2];
            reconstruct<LIM, NV>(wm, w, wp, m.im, m.ip, m.ic, m.hm, m.hp, lo, hi);
            fm = fp = sR[x % BI + 2].rt * sT[x / BI + 2].phf * m.iw;
        }
#pragma unroll
        for (int v = 0; v < NV; ++v) hi[v] = shr1(hi[v]);
        rusanov<D, NV>(hi, lo, fx, gs);
#pragma unroll
        for (int v = 0; v < NV; ++v) lo[v] = fma(-fp, shl1(fx[v]), fm * fx[v]);
        if (act && c >= 0 && c < T::B) {
            double *const d = D0 + (D == 0 ? kk * DK + x * DI + c : D == 1 ? kk * DK + c * DI + x : c * DK + x / BI * DI + x % BI);
#pragma unroll
            for (int v = 0; v < NV; ++v) lds_add(d + v * DV, lo[v]);
        }
        // raw flux at a coarse-fine face of the block, for the reflux
        if (act && (cd == 0 || cd == ext) && c >= 0 && c <= T::B) {
            const int r = cd == 0 ? flo : fhi;
            if (r >= 0) {
                constexpr int FB = D == 2 ? 1 : BK;
                double *const f = a.freg + (size_t)r * a.reg_stride + (D == 2 ? x : (k0 + kk) * T::X + x);
                for (int v = 0; v < NV; ++v) f[v * T::X * FB] = fx[v];
            }
        }
    }
}

template <int BI, int BJ, int BK, int NV, int LIM, int KZ>
__global__ void __launch_bounds__(TT) __attribute__((amdgpu_waves_per_eu(4, 4)))
k_tile(KArgs a)
{
    using S = Shape<BI, BJ, BK, NV>;
    static_assert(BK % KZ == 0 && BK / KZ <= KSPLIT_MAX, "planes per work-group");
    constexpr int PL = BI * BJ, DI = tile_pitch(BI), DK = BJ * DI + 2, DV = KZ * DK, PARTS = BK / KZ, NW = TT / 64;
    __shared__ double sD[NV * DV];
    __shared__ LdsR sR[BI + 4];
    __shared__ LdsT sT[BJ + 4];
    __shared__ LdsP sP[KZ + 4];
    __shared__ double sred[NW];
    const Gas gs = a.gas;
    const int nwork = *in_const(a.nitems) * PARTS;
    for (int wi = blockIdx.x; wi < nwork; wi += gridDim.x) {
        const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
        const int it = wi / PARTS, part = wi % PARTS, k0 = part * KZ;
        const int slot = in_const(a.items)[it];
        const AS_CONST BlockDesc *const bd = in_const(a.desc) + slot;
        const int mem = bd->member, mk = bd->reflux_mask;
        const double dt = in_const(a.dt)[mem];
        if (dt <= 0.0) continue;                 // member finished: state stays in place
        const double adt = a.alpha * dt;
        const AS_CONST LevelGeo *const lg = in_const(a.geo) + bd->level;
        __syncthreads();                         // the LDS of the item before is done with
        load_tables<BI, BJ, LIM>(a, lg, bd->org[0], bd->org[1], bd->org[2], k0, KZ + 4, tid, sR, sT, sP);
        for (int q = tid; q < NV * DV; q += TT) sD[q] = 0.0;
        __syncthreads();
        tile_passes<BI, BJ, BK, NV, LIM, KZ, 0>(a, slot, bd->nbr[0], bd->nbr[1], bd->freg[0], bd->freg[1], gs, k0, wave, NW,
                                                lane, sR, sT, sP, sD);
        // the theta passes go on where the r passes ended among the waves
        tile_passes<BI, BJ, BK, NV, LIM, KZ, 1>(a, slot, bd->nbr[2], bd->nbr[3], bd->freg[2], bd->freg[3], gs, k0,
                                                (wave + NW - TileRows<BI, BJ, KZ, 0>::NP % NW) % NW, NW, lane, sR, sT, sP, sD);
        __syncthreads();
        tile_passes<BI, BJ, BK, NV, LIM, KZ, 2>(a, slot, bd->nbr[4], bd->nbr[5], bd->freg[4], bd->freg[5], gs, k0, wave, NW,
                                                lane, sR, sT, sP, sD);
        __syncthreads();
        CellLog log;
        const unsigned long long own = (uintptr_t)(a.U + (size_t)slot * NV * S::NC + (size_t)k0 * PL);
        const unsigned long long ubase = (uintptr_t)(a.Ubase + (size_t)slot * NV * S::NC + (size_t)k0 * PL);
        const unsigned long long uout = (uintptr_t)(a.Uout + (size_t)slot * NV * S::NC + (size_t)k0 * PL);
#pragma unroll 1
        for (int q = tid; q < PL * KZ; q += TT) {
            const int i = q % BI, j = q / BI % BJ, kk = q / PL, k = k0 + kk;
            double u[NV], w[NV], acc[NV];
#pragma unroll
            for (int v = 0; v < NV; ++v) u[v] = ld_at(own, v * S::NC, 8u * q);
            cons_to_prim<false, NV>(u, w, gs);
#pragma unroll
            for (int v = 0; v < NV; ++v) u[v] = ld_at(ubase, v * S::NC, 8u * q);
#pragma unroll
            for (int v = 0; v < NV; ++v) acc[v] = sD[kk * DK + j * DI + i + v * DV];
            const bool refluxed = (i == 0 && (mk & 1)) || (i == BI - 1 && (mk & 2)) || (j == 0 && (mk & 4)) ||
                                  (j == BJ - 1 && (mk & 8)) || (k == 0 && (mk & 16)) || (k == BK - 1 && (mk & 32));
            update_cell<NV>(a, gs, sR[i + 2], sT[j + 2], sP[kk + 2].iw, adt, refluxed, q + k0 * PL, w, acc, u, log);
#pragma unroll
            for (int v = 0; v < NV; ++v) st_at(uout, v * S::NC, 8u * q, u[v]);
        }
        end_item<TT>(a, slot, mem, part, PARTS, log, sred);
    }
}

// ---------------------------------------------------------------------------
// instantiations and launch
// ---------------------------------------------------------------------------
// the other limiters are built for two waves per SIMD only; the tracer (NV =
// 9) with two waves per SIMD where two work-groups' LDS fits a CU (one on
// planes of more than 160 cells), every limiter
template <int BI, int BJ, int BK, int NV>
void launch_stage(dim3 g, hipStream_t s, const KArgs &a, int waves, int limiter)
{
    if constexpr (NV > 8) {
        constexpr int W9 = BI * BJ > 160 ? 1 : 2;
        if (limiter == LIM_MINMOD) hipLaunchKernelGGL((k_stage<BI, BJ, BK, NV, W9, LIM_MINMOD>), g, dim3(NT), 0, s, a);
        else if (limiter == LIM_VANLEER)
            hipLaunchKernelGGL((k_stage<BI, BJ, BK, NV, W9, LIM_VANLEER>), g, dim3(NT), 0, s, a);
        else hipLaunchKernelGGL((k_stage<BI, BJ, BK, NV, W9, LIM_MC>), g, dim3(NT), 0, s, a);
    } else {
        if (limiter == LIM_MINMOD) hipLaunchKernelGGL((k_stage<BI, BJ, BK, NV, 2, LIM_MINMOD>), g, dim3(NT), 0, s, a);
        else if (limiter == LIM_VANLEER)
            hipLaunchKernelGGL((k_stage<BI, BJ, BK, NV, 2, LIM_VANLEER>), g, dim3(NT), 0, s, a);
        else if (waves == 1) hipLaunchKernelGGL((k_stage<BI, BJ, BK, NV, 1, LIM_MC>), g, dim3(NT), 0, s, a);
        else hipLaunchKernelGGL((k_stage<BI, BJ, BK, NV, 2, LIM_MC>), g, dim3(NT), 0, s, a);
    }
}

// kz planes of a block per work-group: 1, 2 or, on planes of up to TILE4_PLANE
// cells, 4
template <int BI, int BJ, int BK, int NV, int LIM>
void launch_tile_lim(dim3 g, hipStream_t s, const KArgs &a, int kz)
{
    if (kz == 1) hipLaunchKernelGGL((k_tile<BI, BJ, BK, NV, LIM, 1>), g, dim3(TT), 0, s, a);
    else if (kz == 2) hipLaunchKernelGGL((k_tile<BI, BJ, BK, NV, LIM, 2>), g, dim3(TT), 0, s, a);
    else if constexpr (BI * BJ <= TILE4_PLANE) hipLaunchKernelGGL((k_tile<BI, BJ, BK, NV, LIM, 4>), g, dim3(TT), 0, s, a);
}
template <int BI, int BJ, int BK, int NV>
void launch_tile(dim3 g, hipStream_t s, const KArgs &a, int kz, int limiter)
{
    if (limiter == LIM_MINMOD) launch_tile_lim<BI, BJ, BK, NV, LIM_MINMOD>(g, s, a, kz);
    else if (limiter == LIM_VANLEER) launch_tile_lim<BI, BJ, BK, NV, LIM_VANLEER>(g, s, a, kz);
    else launch_tile_lim<BI, BJ, BK, NV, LIM_MC>(g, s, a, kz);
}

#define IC_INSTANTIATE(BI, BJ, BK)                                                                  \
    template void launch_tile<BI, BJ, BK, 8>(dim3, hipStream_t, const KArgs &, int, int);          \
    template void launch_tile<BI, BJ, BK, 9>(dim3, hipStream_t, const KArgs &, int, int);          \
    template __global__ void k_stage<BI, BJ, BK, 8, 1, LIM_MC>(KArgs);                             \
    template __global__ void k_stage<BI, BJ, BK, 8, 2, LIM_MC>(KArgs);                             \
    template __global__ void k_stage<BI, BJ, BK, 8, 2, LIM_MINMOD>(KArgs);                         \
    template __global__ void k_stage<BI, BJ, BK, 8, 2, LIM_VANLEER>(KArgs);                        \
    template void launch_stage<BI, BJ, BK, 8>(dim3, hipStream_t, const KArgs &, int, int);         \
    template void launch_stage<BI, BJ, BK, 9>(dim3, hipStream_t, const KArgs &, int, int);

#include "shapes.inc"
#undef IC_INSTANTIATE
