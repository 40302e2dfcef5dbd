// Pair kernels: the physical force F(R^n) (the do_force work of section 2.1) and the
// exact Hessian-vector product H(R^n) v that replaces the finite-difference term of
// eq. (5), for every pair bead of every path of a call in one launch (in two when only
// bead 1 needs energies: see launch_pair_e).
//
// Work unit: one wave per 8-atom i-cluster (8 consecutive slots of one column).
//   1. Lane-parallel over the x-y column stencil: keep columns whose rectangle lies
//      within the search radius of the cluster's bounding box, and per column the
//      cluster range covering the z window [zlo - r, zhi + r] (two ranges when the
//      window wraps around the box).
//   2. Candidate clusters are listed in LDS; the positions of 8 of them (64 atoms) are
//      loaded per step, one atom per lane, converted to FP32 coordinates relative to the
//      i-cluster's box centre (exact integer minimum image, then one rounding) and tested
//      against the search radius around the i-cluster's bounding box.  The slots of the
//      survivors are compacted (ballot + mbcnt) into a per-wave LDS list.
//   3. Every 64 listed slots: the atoms are gathered, one per lane, converted and written
//      to a 64-entry LDS ring, and 8 steps of 8 j-atoms x 8 i-atoms (lane = 8*i + j)
//      evaluate the pair terms; each lane accumulates a partial sum for its i atom.
//   4. Partial sums are reduced over the 8 j lanes.
//   The force pass records each cluster's neighbour list (one record per candidate
//   cluster with survivors); the Hessian pass of the same bead replays it instead of
//   steps 1-2: the records' atom masks give the slot list directly.
//   What bounds the kernels is the issue time of vector instructions, with LDS (active 62%
//   of the time in the force kernel, 52% in the Hessian) and instruction fetch (0.38 per CU
//   and cycle; two CUs share a cache) not far behind, at clocks that the power limit sets
//   (1.75 to 2.2 GHz).  On gfx950 instruction rates differ: FP32 add, multiply and fma, 32-bit
//   integer add and bitwise operations on vector registers take 2 cycles per wave and SIMD;
//   the same with a scalar-register operand, and compares, conversions, shifts, min / max,
//   three-operand integer operations, DPP forms and v_mbcnt 4; rsq, rcp and exp 8 (timed
//   in loops of independent instructions, 8 waves per SIMD).  Only survivors are therefore
//   converted, charged and written to the ring, all 64 lanes at work: of the candidates
//   tested, and of the atoms of recorded clusters, only about 58% survive (150,000-atom
//   workload), and the ring writes and conversions of the idle lanes cost as much.
// Launch: a flat grid (one workgroup per W clusters, k_pair) or, as a plan option, a
// persistent grid over per-XCD work queues (k_pair_q); both run the same per-wave body.
// Energies are a template parameter, so that kernels that need none take fewer
// registers and hold more waves per SIMD (PAIR_WAVES).
//
// Two variants:
//   N3 = 1 (opt-in): Newton's third law.  A wave takes only clusters with a larger
//      index than its own, so every pair of distinct clusters is evaluated once.  The
//      j-side contribution of a step is summed over the 8 i lanes (lane exchanges) and
//      added to its ring entry by one lane, and, once per EB entries, flushed to a
//      slot-order FP32 buffer with one global atomic per entry and component; i-sums are
//      added the same way.  The own cluster is one 8 x 8 block evaluated from both
//      sides.  Summation order depends on scheduling.
//   N3 = 0 (default): every pair evaluated from both sides; no atomics; run-to-run
//      reproducible for a given binning.  Results go straight to original atom order.
//      Measured on MI355X (150,000 atoms, 15 beads), this is the faster variant: the
//      global flush of the j-side sums (three float atomics per ring entry) costs more
//      than the pair work it saves.
//
// Pair terms, d = x_j - x_i, r = |d|, shifted-force LJ + reaction field:
//   g = phi_sf'(r)/r = G6 r^-8 + qq (2 k_rf - r^-3) + C1 r^-1,   G6 = a12 r^-6 + a6,
//       C1 = -phi'(r_c) = csf + qq crf1
//   h = (phi'' - phi_sf'/r)/r^2 = (b12 r^-6 + b6) r^-10 + 3 qq r^-5 - C1 r^-3,
//       where b12 r^-6 + b6 = -8 (0.75 a12 r^-6 + G6) (b12 = -14 a12, b6 = -8 a6), so
//       the Hessian kernel reads one table entry {a12, a6, csf, 0.75 a12} per pair
//   F_i += g d,   (H v)_i += g (v_i - v_j) + h (d . (v_i - v_j)) d   (j: the opposite)
//
// Ewald variant (EL = 1, systems with particle-mesh Ewald): the reaction-field terms
// become the Ewald real-space term qq psi(r), psi = erfc(beta r)/r, shifted-force at r_c
// (C1 = csf + qq crf1 with crf1 = -psi'(r_c)), and excluded partners within r_c carry
// the correction qq (erfc(beta r) - 1)/r = -qq erf(beta r)/r instead of nothing.  With
// E = erfc(beta r) (minus 1 for excluded pairs) and D = 2 beta/sqrt(pi) exp(-beta^2 r^2):
//   g_el = -(D r^-2 + E r^-3),   h_el = (2 beta^2 D + 3 D r^-2 + 3 E r^-3) r^-2.
// erfc(x) = exp(-x^2) erfcx(x) with erfcx a polynomial in t = 1/(1 + x/2) fitted on
// 0 <= x <= 6 (coefficients from erfc_fit.py next to this package; relative error below
// 4e-7 in FP32), so E and D share one exponential.
#include <algorithm>
#include <atomic>
#include <type_traits>

#include "device_common.h"
#include "launch.h"

namespace mop {

// Ring entries evaluated per batch: one per lane of the wave that gathers them.
constexpr int EB = RING;
static_assert(EB == 64, "evaluation batch");

// Ring of j-atoms, one per wave in LDS.  Full-shell kernels keep entries as float4 {x, y,
// z, q} followed by float4 {w, v_x, v_y, v_z} (Hessian) or a float {w} (force), so a step
// reads a j-atom with one or two 16-byte loads.  Integers are stored as float bits: w is
// the packed 16 * exclusion key + LJ type of the system's key table, or (Ewald kernels, see
// XSKIP) the byte offset of the type in a table row, with the packed key as one more float
// that only batches with excluded pairs read.  The Newton-3 kernels keep one array per
// field [field][entry], F_* below.
typedef float v4f __attribute__((ext_vector_type(4)));

constexpr int F_X = 0, F_Y = 1, F_Z = 2, F_Q = 3, F_K = 4, F_S = 5, F_J = 6;

// Table entries per type pair in LDS, 16 bytes apart: the force kernels keep
// {a12, a6, csf, e0lj} for the nt^2 pairs followed by {b12, b6, c12, c6} (energies);
// the Hessian kernel keeps {a12, a6, csf, 0.75 a12}.
template <int MODE>
constexpr int TAB_COPIES = MODE == 1 ? 1 : 2;

// erfcx(x) = exp(x^2) erfc(x) for 0 <= x <= 6.
__device__ __forceinline__ float erfc_ex2(float x) {
    const float t = __builtin_amdgcn_rcpf(fmaf(0.5f, x, 1.0f));
    float p = -3.256256573e-02f;
    p = fmaf(p, t, 2.505454269e-01f);
    p = fmaf(p, t, -6.964120320e-01f);
    p = fmaf(p, t, 7.776858691e-01f);
    p = fmaf(p, t, -2.269658047e-01f);
    p = fmaf(p, t, 3.915052002e-01f);
    p = fmaf(p, t, 2.504345553e-01f);
    p = fmaf(p, t, 2.859732478e-01f);
    p = fmaf(p, t, -2.038257043e-04f);
    return p;
}

// 32-bit words of LDS per wave: ring, candidate clusters (16 more, so that chunks can be
// read whole and ahead), slots of survivors, survivor masks of 64 candidate clusters.
constexpr int SLOTS = 128;  // power of two, at least 63 + 64
// Bit map (hash of the cluster index) of the clusters that hold an excluded partner of the
// i-cluster, itself among them: at most 33 of 4,096 bits set.  Candidates from other
// clusters cannot be excluded (XSKIP kernels).
constexpr int XMAP = 128;   // words (XSKIP kernels)
// The flag of such a cluster: bit 23 of its index in the candidate list, which makes it bit
// 26 of a listed slot and bit 31 of a neighbour-list record.  Layouts of 2^26 slots or more
// have no room for it (and no lists), and keys that repeat or leave wide gaps no map to the
// atoms; there every batch is tested.
constexpr int XFLAG = 1 << 23;
constexpr int XSLOT = XFLAG * CLUSTER;
template <class F>
constexpr int WAVE_LDS = F::NF * RING + (CLIST + 16) + SLOTS + 16 + F::X;

// Kernels that skip the exclusion test in batches without excluded pairs.  About 3 of 4
// batches are such.  The Ewald kernels then save the test, the selects between pair term
// and correction and the self test: 10.8 -> 10.3 ms per call on the 150,000-atom workload.
// The reaction-field kernels would save a subtraction and a compare per step and were 2-4%
// slower with it: their VALU time then falls below what LDS and instruction fetch take.
template <int N3, int EL>
constexpr bool XSKIP = N3 == 0 && EL == 1;

template <int MODE, int N3, int EL>
struct Fields {
    static constexpr int V = F_J + 3;  // v_j (Newton-3 HVP)
    static constexpr int K = MODE == 1 ? 8 : 5;  // packed key of XSKIP kernels
    static constexpr int NF = N3 ? (MODE == 1 ? V + 3 : V) : K + (XSKIP<N3, EL> ? 1 : 0);
    static constexpr int X = XSKIP<N3, EL> ? XMAP : 0;
};

struct IAtom {
    float x, y, z;  // relative to the box centre, or (EX) raw fixed-point bits
    float q, vx, vy, vz;
    uint32_t kp;  // 16 * (key + 2) + 15, from the packed word 16 * key + type
    int tiN;
    bool v;
};

struct PairK {
    float sx, sy, sz, rc2, krf2, crf1, krf, crf, e0rf, beta, c2b, b2x2;
    float krf2_3, crf1_3;  // krf2 / 3, crf1 / 3 (Hessian kernel: charges carried as 3 q_j)
};

// The reaction-field Hessian kernel keeps 3 q_j in its ring, so that the 3 qq of h needs no
// multiply; g and C1 then use constants divided by 3.
template <int MODE, int N3, int EL>
constexpr bool THREE_Q = MODE == 1 && N3 == 0 && EL == 0;

// One pair term for lane atom I and j-atom (jx, jy, jz): coordinates relative to the
// box centre, or (EX) raw fixed-point bits.  The contribution to atom i (force: g d;
// HVP: g (v_i - v_j) + h (d . (v_i - v_j)) d) is added to (ax, ay, az) with fused
// multiply-adds; with T_OUT it is also returned in t (for the j side).  tabrow points
// at the type-table row of atom i.
// Everything after the cutoff test runs only in the lanes of pairs that interact (58% on
// the 150,000-atom workload): no selects on the results, and the idle lanes draw no
// power, which the kernels are short of (they run at 1.8-2.1 GHz of the GPU's 2.4).
// Every fused multiply-add is written out (contraction is off), so that the variants of
// the kernels round alike, but for cube_first.
// toff: byte offset of type j in the table row (XSKIP kernels; the others take the type
// from kj); EXCL: the pair may be excluded (kj is read).
// cube_first (force, reaction field; the first step of a full batch in kernels with
// energies): r^-3 is rounded before it is taken from 2 k_rf.  It gains nothing: so the
// compiler formed that step when it chose the fused operations itself, and trajectories and
// gradients of earlier builds are reproduced only with it (without, gradients move by 3e-9 to
// 4e-8, their error against 64 bits by nothing).  Forces of a kernel with energies differ in
// the last bits from those of one without: bead_forces with and without energies, and a
// path's beads after the first when its launch is large enough to be split (launch_pair_e).
template <int MODE, bool EX, bool WANTE, bool T_OUT, int EL, bool Q3, bool EXCL>
__device__ __forceinline__ void pair_term(const IAtom& I, const PairK& P, const float4* tabrow,
                                          int ntab,
                                          float jx, float jy, float jz,
                                          float qj, uint32_t toff, uint32_t kj, float vjx, float vjy,
                                          float vjz, bool valid, float& ax, float& ay,
                                          float& az, float& tx, float& ty, float& tz,
                                          float& en, bool cube_first = false) {
#pragma clang fp contract(off)
    float dx, dy, dz;
    if (EX) {
        dx = (float)(int)(__float_as_uint(jx) - __float_as_uint(I.x)) * P.sx;
        dy = (float)(int)(__float_as_uint(jy) - __float_as_uint(I.y)) * P.sy;
        dz = (float)(int)(__float_as_uint(jz) - __float_as_uint(I.z)) * P.sz;
    } else {
        dx = jx - I.x;
        dy = jy - I.y;
        dz = jz - I.z;
    }
    const float r2 = fmaf(dx, dx, fmaf(dy, dy, dz * dz));
    // kj = 16 key_j + type_j, so I.kp - kj = 16 (key_i - key_j + 2) + 15 - type_j (keys
    // below 2^27, no wrap-around): it lies in [0, 79] exactly when |key_i - key_j| <= 2
    // (same molecule within two chain positions), and in [32, 47] for the atom itself
    const uint32_t kd = I.kp - kj;
    const bool exc = EXCL && kd <= 79u;
    // Ewald: excluded partners carry a correction, the atom itself nothing
    const bool act = !EXCL || (EL == 1 ? kd - 32u > 15u : !exc);
    if (T_OUT) tx = ty = tz = 0.0f;
    if (valid & I.v & act & (r2 < P.rc2)) {
        const float rinv = __builtin_amdgcn_rsqf(r2);
        const float rinv2 = rinv * rinv;
        const float rinv3 = rinv2 * rinv;
        const float rinv6 = rinv3 * rinv3;
        const float4* tp = XSKIP<T_OUT, EL>
                               ? reinterpret_cast<const float4*>(reinterpret_cast<const char*>(tabrow) + toff)
                               : tabrow + (kj & 15u);
        const float4 T = *tp;
        const float qq = I.q * qj;  // 3 q_i q_j when Q3
        const float C1 = fmaf(qq, Q3 ? P.crf1_3 : P.crf1, T.z);
        const float G6 = fmaf(T.x, rinv6, T.y);
        const float rinv8 = rinv6 * rinv2;
        float g, E = 0.0f, D = 0.0f, r = 0.0f;
        if (EL == 0) {
            g = G6 * rinv8;
            g = fmaf(qq, Q3 ? fmaf(rinv3, -1.0f / 3.0f, P.krf2_3)
                            : (cube_first ? P.krf2 - rinv3 : fmaf(-rinv, rinv2, P.krf2)), g);
            g = fmaf(C1, rinv, g);
        } else {
            r = r2 * rinv;
            const float bx = P.beta * r;
            const float ex2 = __expf(-bx * bx);
            const float ecx = erfc_ex2(bx);
            D = P.c2b * ex2;
            E = exc ? fmaf(ex2, ecx, -1.0f) : ex2 * ecx;
            const float ge = -fmaf(D, rinv2, E * rinv3);
            const float gs = fmaf(G6, rinv8, C1 * rinv);
            g = exc ? qq * ge : fmaf(qq, ge, gs);
        }
        if (MODE == 0) {
            if (T_OUT) {
                tx = g * dx;
                ty = g * dy;
                tz = g * dz;
                ax += tx;
                ay += ty;
                az += tz;
            } else {
                ax = fmaf(g, dx, ax);
                ay = fmaf(g, dy, ay);
                az = fmaf(g, dz, az);
            }
            if (WANTE) {
                const float4 T2 = tp[ntab];
                if (EL == 0) r = r2 * rinv;
                float e = fmaf(T2.z, rinv6, -T2.w) * rinv6;
                const float eel = EL == 0 ? fmaf(P.crf1, r, (fmaf(P.krf, r2, rinv) - P.crf) + P.e0rf)
                                          : fmaf(E, rinv, fmaf(P.crf1, r, P.e0rf));
                e = fmaf(qq, eel, e);
                e += fmaf(T.z, r, T.w);
                en = EL == 1 && exc ? qq * E * rinv : e;
            }
        } else {
            const float h6 = fmaf(T.w, rinv6, G6);
            float h;
            if (EL == 0) {
                // h = r^-5 (3 qq - 8 h6 r^-5) - C1 r^-3
                const float rinv5 = rinv3 * rinv2;
                h = fmaf(h6 * rinv5, -8.0f, Q3 ? qq : 3.0f * qq);
                h = fmaf(rinv5, h, -(C1 * rinv3));
            } else {
                h = h6 * (rinv8 * (-8.0f * rinv2));
                const float he = fmaf(P.b2x2, D, 3.0f * fmaf(D, rinv2, E * rinv3)) * rinv2;
                h = fmaf(-C1, rinv3, h);
                h = exc ? qq * he : fmaf(qq, he, h);
            }
            const float dvx = I.vx - vjx, dvy = I.vy - vjy, dvz = I.vz - vjz;
            const float sd = fmaf(dx, dvx, fmaf(dy, dvy, dz * dvz));
            const float hs = h * sd;
            if (T_OUT) {
                tx = fmaf(g, dvx, hs * dx);
                ty = fmaf(g, dvy, hs * dy);
                tz = fmaf(g, dvz, hs * dz);
                ax += tx;
                ay += ty;
                az += tz;
            } else {
                ax = fmaf(g, dvx, fmaf(hs, dx, ax));
                ay = fmaf(g, dvy, fmaf(hs, dy, ay));
                az = fmaf(g, dvz, fmaf(hs, dz, az));
            }
        }
    }
}

// Copy segment p's pair table(s) to LDS: threads t0, t0 + stride, ... of the caller's group.
template <int MODE>
__device__ __forceinline__ void load_table(const SegDev* __restrict__ sg, float4* s_tab, int t0, int stride) {
    const int nt = sg->s.nt;
    for (int t = t0; t < nt * nt; t += stride) {
        if (MODE == 1) {
            s_tab[t] = sg->s.tabh[t];
        } else {
            s_tab[t] = sg->s.tab[t];
            s_tab[nt * nt + t] = sg->s.tab2[t];
        }
    }
}

// The work of one wave: i-cluster gw of path p (bead bead0 + gw / cpb, cluster gw % cpb),
// with the path's table at s_tab and the wave's own WAVE_LDS words of LDS at ring.
// ENERGY: the kernel can sum pair energies (of bead energy_bead, or of every bead for -2);
// kernels without it need fewer registers.
template <int MODE, int N3, int EL, int ENERGY>
__device__ __forceinline__ void pair_wave(const SegDev* __restrict__ segs, const Launch& L,
                                          char* __restrict__ ws, int outsel, int energy_bead,
                                          int lists, int bead0, int p, int gw, const float4* s_tab,
                                          float* ring) {
    using FL = Fields<MODE, N3, EL>;
    constexpr int NF = FL::NF, FV = FL::V, FK = FL::K;
    int* clist = reinterpret_cast<int*>(ring) + NF * RING;
    int* slist = clist + CLIST + 16;
    unsigned long long* smask = reinterpret_cast<unsigned long long*>(slist + SLOTS);
    unsigned* xmap = reinterpret_cast<unsigned*>(slist + SLOTS) + 16;
    const SegDev* __restrict__ sg = segs + p;
    const int nt = sg->s.nt;
    const int lane = threadIdx.x & 63;
    const int cpb = sg->s.cpb;
    const int bl = gw / cpb, c = gw - bl * cpb;
    if (bl >= L.nb[p]) return;
    const int b = bead0 + bl;
    const int S = sg->s.S, Q = sg->s.Q, ncol = sg->s.ncol, nzb = sg->s.nzb;
    const int ncx = sg->s.ncx, ncy = sg->s.ncy;
    const uint4* __restrict__ upos = wsp<const uint4>(ws, sg->o_upos) + (size_t)b * S;
    const int2* __restrict__ umeta = wsp<const int2>(ws, sg->o_umeta) + (size_t)b * S;
    const int* __restrict__ colstart = wsp<const int>(ws, sg->o_colstart) + (size_t)b * (ncol + 1);
    const int* __restrict__ binoff = wsp<const int>(ws, sg->o_binoff) + (size_t)b * ncol * (nzb + 1);
    const float4* __restrict__ vs = wsp<const float4>(ws, sg->o_vs) + (size_t)b * S;
    float* __restrict__ fsx = wsp<float>(ws, sg->o_fs) + (size_t)b * 3 * S;
    float* __restrict__ fsy = fsx + S;
    float* __restrict__ fsz = fsy + S;
    const int nslots = colstart[ncol];
    if (c * CLUSTER >= nslots) return;

    const bool wantE = MODE == 0 && ENERGY && (energy_bead == -2 || energy_bead == b);
    PairK P;
    P.sx = sg->s.sc[0];
    P.sy = sg->s.sc[1];
    P.sz = sg->s.sc[2];
    P.rc2 = sg->s.rc2;
    P.krf2 = sg->s.krf2;
    P.crf1 = sg->s.crf1;
    P.krf = sg->s.krf;
    P.crf = sg->s.crf;
    P.e0rf = sg->s.e0rf;
    P.beta = sg->s.ew_beta;
    P.c2b = sg->s.ew_c2b;
    P.b2x2 = sg->s.ew_b2x2;
    P.krf2_3 = sg->s.krf2 * (1.0f / 3.0f);
    P.crf1_3 = sg->s.crf1 * (1.0f / 3.0f);
    // a scalar operand would halve the rate of the instructions that read it
    if (MODE == 0 && !ENERGY) asm("" : "+v"(P.krf2), "+v"(P.crf1));
    constexpr float QSC = THREE_Q<MODE, N3, EL> ? 3.0f : 1.0f;
    float sx = P.sx, sy = P.sy, sz = P.sz;
    if (MODE == 0 && !ENERGY) asm("" : "+v"(sx), "+v"(sy), "+v"(sz));  // as above
    const float rcs = sg->s.rcs, rcs2 = sg->s.rcs2;

    // ---- the i-cluster ------------------------------------------------------------
    const int isub = lane >> 3, jslot = lane & 7;
    const int si = c * CLUSTER + isub;
    const uint4 ui = upos[si];
    const int2 mi = umeta[si];
    // first reference point: the cluster's middle atom (atoms of a cluster are z-sorted
    // inside one column)
    const uint4 ref = upos[c * CLUSTER + 3];
    IAtom I;
    I.v = mi.x != DUMMY_KEY;
    I.q = __uint_as_float(ui.w);
    I.kp = (uint32_t)(mi.x - mi.y) + 47u;
    I.tiN = mi.y * nt;
    const float4* tabrow = s_tab + I.tiN;
    const int ntab = nt * nt;
    I.vx = I.vy = I.vz = 0.0f;
    if (MODE == 1) {
        const float4 v4 = vs[si];
        I.vx = v4.x;
        I.vy = v4.y;
        I.vz = v4.z;
    }
    // bounding box relative to the reference atom, then to its own centre
    float lox, hix, loy, hiy, loz, hiz;
    auto bbox = [&](float x, float y, float z) __attribute__((always_inline)) {
        lox = I.v ? x : 3.0e38f;
        hix = I.v ? x : -3.0e38f;
        loy = I.v ? y : 3.0e38f;
        hiy = I.v ? y : -3.0e38f;
        loz = I.v ? z : 3.0e38f;
        hiz = I.v ? z : -3.0e38f;
        auto step = [&](auto mc) __attribute__((always_inline)) {
            constexpr int M = decltype(mc)::value;
            lox = fminf(lox, lane_xor<M>(lox));
            hix = fmaxf(hix, lane_xor<M>(hix));
            loy = fminf(loy, lane_xor<M>(loy));
            hiy = fmaxf(hiy, lane_xor<M>(hiy));
            loz = fminf(loz, lane_xor<M>(loz));
            hiz = fmaxf(hiz, lane_xor<M>(hiz));
        };
        step(std::integral_constant<int, 8>{});
        step(std::integral_constant<int, 16>{});
        step(std::integral_constant<int, 32>{});
    };
    bbox((float)(int)(ui.x - ref.x) * sx, (float)(int)(ui.y - ref.y) * sy,
         (float)(int)(ui.z - ref.z) * sz);
    // re-reference to the box centre uc: the image of an atom nearest the centre is the
    // one nearest the box, which keeps the candidate test conservative in small boxes.
    // The shifted bounds may differ from the atoms' new coordinates by an ulp, which the
    // search-radius margin absorbs.
    const int ocx = (int)rintf(0.5f * (lox + hix) / sx);
    const int ocy = (int)rintf(0.5f * (loy + hiy) / sy);
    const int ocz = (int)rintf(0.5f * (loz + hiz) / sz);
    const uint32_t ucx = ref.x + (uint32_t)ocx, ucy = ref.y + (uint32_t)ocy, ucz = ref.z + (uint32_t)ocz;
    {
        const float fx = (float)ocx * sx, fy = (float)ocy * sy, fz = (float)ocz * sz;
        lox -= fx;
        hix -= fx;
        loy -= fy;
        hiy -= fy;
        loz -= fz;
        hiz -= fz;
    }
    // Coordinates relative to the reference give exact pair differences when
    // max(|lo|, |hi|) + search radius < L/2 along every axis: for a pair within the
    // cutoff, (image of i) + d then lies within L/2 of the reference, so it is the image
    // of j that the relative coordinate picks.  Otherwise each pair difference is taken
    // from the fixed-point coordinates (small boxes, sparse columns).
    const bool exact_l = (fmaxf(-lox, hix) + rcs >= 0.5f * sg->s.Lf[0]) ||
                       (fmaxf(-loy, hiy) + rcs >= 0.5f * sg->s.Lf[1]) ||
                       (fmaxf(-loz, hiz) + rcs >= 0.5f * sg->s.Lf[2]);
    const bool exact = __builtin_amdgcn_readfirstlane((int)exact_l) != 0;  // uniform
    if (exact) {
        I.x = __uint_as_float(ui.x);
        I.y = __uint_as_float(ui.y);
        I.z = __uint_as_float(ui.z);
    } else {
        I.x = (float)(int)(ui.x - ucx) * sx;
        I.y = (float)(int)(ui.y - ucy) * sy;
        I.z = (float)(int)(ui.z - ucz) * sz;
    }

    float ax = 0.f, ay = 0.f, az = 0.f;
    float eacc = 0.0f;
    double eacc64 = 0.0;
    int wp = 0, rp = 0;  // slots listed / gathered (uniform); rp stays a multiple of 64
    int wr = 0;          // neighbour-list records written (force pass)

    float4* ring4 = reinterpret_cast<float4*>(ring);

    // neighbour lists (full-shell kernels): the force pass records the slots that pass
    // the search, the Hessian pass of the same bead replays them
    const int lcap = sg->s.lcap;
    const bool rec = !N3 && MODE == 0 && (lists & LISTS_RECORD) && lcap > 0;
    const bool rpl = !N3 && (lists & LISTS_REPLAY) && lcap > 0;
    int* __restrict__ nl = nullptr;
    int* __restrict__ nlc = nullptr;
    if (rec || rpl) {
        nl = wsp<int>(ws, sg->o_nl) + ((size_t)b * cpb + c) * lcap;
        nlc = wsp<int>(ws, sg->o_nlc) + (size_t)b * cpb + c;
    }

    // ---- own cluster (N3): one 8 x 8 block, both sides, weight 1/2 for energies ----
    if (N3) {
        const int sj = c * CLUSTER + jslot;
        const uint4 uj = upos[sj];
        const int2 mj = umeta[sj];
        float jx, jy, jz, vjx = 0.f, vjy = 0.f, vjz = 0.f;
        if (exact) {
            jx = __uint_as_float(uj.x);
            jy = __uint_as_float(uj.y);
            jz = __uint_as_float(uj.z);
        } else {
            jx = (float)(int)(uj.x - ucx) * sx;
            jy = (float)(int)(uj.y - ucy) * sy;
            jz = (float)(int)(uj.z - ucz) * sz;
        }
        if (MODE == 1) {
            const float4 v4 = vs[sj];
            vjx = v4.x;
            vjy = v4.y;
            vjz = v4.z;
        }
        float tx, ty, tz, en = 0.f;
        const bool vj = mj.x != DUMMY_KEY;
        const float qj = __uint_as_float(uj.w);
        if (exact) {
            if (wantE)
                pair_term<MODE, true, true, false, EL, false, true>(I, P, tabrow, ntab, jx, jy, jz, qj, 0u, (uint32_t)mj.x, vjx,
                                            vjy, vjz, vj, ax, ay, az, tx, ty, tz, en);
            else
                pair_term<MODE, true, false, false, EL, false, true>(I, P, tabrow, ntab, jx, jy, jz, qj, 0u, (uint32_t)mj.x, vjx,
                                             vjy, vjz, vj, ax, ay, az, tx, ty, tz, en);
        } else {
            if (wantE)
                pair_term<MODE, false, true, false, EL, false, true>(I, P, tabrow, ntab, jx, jy, jz, qj, 0u, (uint32_t)mj.x, vjx,
                                             vjy, vjz, vj, ax, ay, az, tx, ty, tz, en);
            else
                pair_term<MODE, false, false, false, EL, false, true>(I, P, tabrow, ntab, jx, jy, jz, qj, 0u, (uint32_t)mj.x, vjx,
                                              vjy, vjz, vj, ax, ay, az, tx, ty, tz, en);
        }
        eacc += 0.5f * en;
    }

    // ---- 8 j-atoms x 8 i-atoms per step from ring entries [0, count) ----------------
    // Every field of every step is one immediate offset from the same address.  Entries
    // past the count of a partial batch are zero.
    // EXCL: the batch may hold excluded partners.
    auto eval_t = [&]<bool EX, bool WE, bool FULL, bool EXCL>(int count) __attribute__((always_inline)) {
        float* rb = ring + jslot;
        const int nsteps = FULL ? EB / 8 : (count + 7) >> 3;
#pragma unroll
        for (int s = 0; s < nsteps; ++s) {
            const int o = s * 8;
            float jx, jy, jz, qj, vjx = 0.f, vjy = 0.f, vjz = 0.f;
            uint32_t kj = 0u, toff = 0u;
            if (N3) {
                jx = rb[F_X * RING + o];
                jy = rb[F_Y * RING + o];
                jz = rb[F_Z * RING + o];
                qj = rb[F_Q * RING + o];
                kj = __float_as_uint(rb[F_K * RING + o]);
                if (MODE == 1) {
                    vjx = rb[FV * RING + o];
                    vjy = rb[(FV + 1) * RING + o];
                    vjz = rb[(FV + 2) * RING + o];
                }
            } else {
                // the empty asm keeps the reads 16 bytes wide and here: their parts would
                // otherwise sink into the masked region of pair_term as reads of their own
                v4f a = *reinterpret_cast<const v4f*>(ring4 + o + jslot);
                asm volatile("" : "+v"(a));
                jx = a[0];
                jy = a[1];
                jz = a[2];
                qj = a[3];
                if (MODE == 1) {
                    v4f w = *reinterpret_cast<const v4f*>(ring4 + RING + o + jslot);
                    asm volatile("" : "+v"(w));
                    toff = kj = __float_as_uint(w[0]);
                    vjx = w[1];
                    vjy = w[2];
                    vjz = w[3];
                } else {
                    toff = kj = __float_as_uint(ring[4 * RING + o + jslot]);
                }
                if (XSKIP<N3, EL> && EXCL) kj = __float_as_uint(ring[FK * RING + o + jslot]);
            }
            const bool valid = FULL || o + jslot < count;
            float tx, ty, tz, en = 0.f;
            pair_term<MODE, EX, WE, N3 == 1, EL, THREE_Q<MODE, N3, EL>, EXCL>(
                I, P, tabrow, ntab, jx, jy, jz, qj, toff, kj, vjx, vjy,
                                             vjz, valid, ax, ay, az, tx, ty, tz, en,
                                             ENERGY && FULL && s == 0);
            if (WE) eacc += N3 ? en : 0.5f * en;
            if (N3) {
                // sum the j side over the 8 i lanes (lanes 8 apart), then the 8 lanes of
                // i-atom 0 add it to their ring entries: one plain LDS update per entry
                tx += lane_xor<8>(tx);
                ty += lane_xor<8>(ty);
                tz += lane_xor<8>(tz);
                tx += lane_xor<16>(tx);
                ty += lane_xor<16>(ty);
                tz += lane_xor<16>(tz);
                tx += lane_xor<32>(tx);
                ty += lane_xor<32>(ty);
                tz += lane_xor<32>(tz);
                if (lane < 8) {
                    rb[(F_J + 0) * RING + o] += tx;
                    rb[(F_J + 1) * RING + o] += ty;
                    rb[(F_J + 2) * RING + o] += tz;
                }
            }
        }
        if (WE) {  // FP32 partial of at most 64 pair terms per lane, summed in FP64
            eacc64 += (double)eacc;
            eacc = 0.0f;
        }
        if (N3) {
            // j-side sums of this chunk (stored with the sign of the i side) go to the
            // slot-order buffer, one entry per lane
            wave_sync();
            if (FULL || lane < count) {
                const int slot = __float_as_int(ring[F_S * RING + lane]);
                unsafeAtomicAdd(fsx + slot, -ring[(F_J + 0) * RING + lane]);
                unsafeAtomicAdd(fsy + slot, -ring[(F_J + 1) * RING + lane]);
                unsafeAtomicAdd(fsz + slot, -ring[(F_J + 2) * RING + lane]);
            }
        }
    };
    auto eval_x = [&]<bool FULL, bool EXCL>(int count) __attribute__((always_inline)) {
        if (exact) {
            if (wantE) eval_t.template operator()<true, true, FULL, EXCL>(count);
            else eval_t.template operator()<true, false, FULL, EXCL>(count);
        } else {
            if (wantE) eval_t.template operator()<false, true, FULL, EXCL>(count);
            else eval_t.template operator()<false, false, FULL, EXCL>(count);
        }
    };
    auto eval = [&](bool excl) __attribute__((always_inline)) {
        if (!XSKIP<N3, EL> || excl) eval_x.template operator()<true, true>(64);
        else eval_x.template operator()<true, false>(64);
    };

    // ---- the batch of listed slots in flight ----------------------------------------
    // gather() starts the loads of the next n (<= 64) listed atoms, one per lane;
    // to_ring() converts them and writes them to the ring.
    const bool flags = XSKIP<N3, EL> && S < XSLOT && sg->s.nkey > 0;
    const int slot_bits = flags ? XSLOT - 1 : ~0;
    int gs = 0;
    bool gx = false;  // the batch may hold excluded partners
    int2 gk = make_int2(0, 0);
    uint4 gu = make_uint4(0u, 0u, 0u, 0u);
    float4 gv = make_float4(0.f, 0.f, 0.f, 0.f);
    auto gather = [&](int n) __attribute__((always_inline)) {
        const int sl = slist[(rp & (SLOTS - 1)) + lane];
        gs = lane < n ? sl : 0;  // lanes past the list load slot 0 (always present)
        gx = !flags || __builtin_amdgcn_ballot_w64((gs & XSLOT) != 0) != 0ull;
        gs &= slot_bits;
        gu = upos[(uint32_t)gs];
        if (MODE == 1) gv = vs[(uint32_t)gs];  // .w: the packed key
        else if (XSKIP<N3, EL>) gk = umeta[(uint32_t)gs];
        else gk.x = umeta[(uint32_t)gs].x;
    };
    auto to_ring = [&](int n) __attribute__((always_inline)) {
        float jx, jy, jz;
        if (exact) {
            jx = __uint_as_float(gu.x);
            jy = __uint_as_float(gu.y);
            jz = __uint_as_float(gu.z);
        } else {
            jx = (float)(int)(gu.x - ucx) * sx;
            jy = (float)(int)(gu.y - ucy) * sy;
            jz = (float)(int)(gu.z - ucz) * sz;
        }
        float jq = QSC * __uint_as_float(gu.w);
        float jk = MODE == 1 ? gv.w : __int_as_float(gk.x);
        float jt = jk;  // the entry's word
        if (XSKIP<N3, EL>) jt = __int_as_float(MODE == 1 ? (__float_as_int(gv.w) & 15) << 4 : gk.y << 4);
        float vx = gv.x, vy = gv.y, vz = gv.z;
        if (n < 64) {
            const bool v = lane < n;
            jx = v ? jx : 0.0f;
            jy = v ? jy : 0.0f;
            jz = v ? jz : 0.0f;
            jq = v ? jq : 0.0f;
            jk = v ? jk : 0.0f;
            jt = v ? jt : 0.0f;
            vx = v ? vx : 0.0f;
            vy = v ? vy : 0.0f;
            vz = v ? vz : 0.0f;
        }
        if (N3) {
            float* re = ring + lane;
            re[F_X * RING] = jx;
            re[F_Y * RING] = jy;
            re[F_Z * RING] = jz;
            re[F_Q * RING] = jq;
            re[F_K * RING] = jk;
            re[F_S * RING] = __int_as_float(gs);
            re[(F_J + 0) * RING] = 0.0f;
            re[(F_J + 1) * RING] = 0.0f;
            re[(F_J + 2) * RING] = 0.0f;
            if (MODE == 1) {
                re[FV * RING] = vx;
                re[(FV + 1) * RING] = vy;
                re[(FV + 2) * RING] = vz;
            }
        } else {
            ring4[lane] = make_float4(jx, jy, jz, jq);
            if (MODE == 1) ring4[RING + lane] = make_float4(jt, vx, vy, vz);
            else ring[4 * RING + lane] = jt;
            if (XSKIP<N3, EL>) ring[FK * RING + lane] = jk;
        }
    };

    // Appends the slots of the lanes in m to the list.
    auto append = [&](unsigned long long m, int slot) __attribute__((always_inline)) {
        const int pos = __builtin_amdgcn_mbcnt_hi((unsigned)(m >> 32),
                                                  __builtin_amdgcn_mbcnt_lo((unsigned)m, (unsigned)wp));
        wave_sync();  // the gather's reads of the list come first
        if (__builtin_amdgcn_inverse_ballot_w64(m)) slist[pos & (SLOTS - 1)] = slot;
        wave_sync();
        wp += (int)__popcll(m);
    };
    // mask of the lanes 0 .. 8 n - 1 (n >= 1)
    auto lanes8 = [](int n) __attribute__((always_inline)) {
        return n >= 8 ? ~0ull : (1ull << (8 * n)) - 1ull;
    };

    const int sub = lane >> 3, atom = lane & 7;

    // ---- 64 listed slots: gather them, evaluate the batch gathered before -------------
    int cur = 0;  // entries of the batch in flight
    auto batch = [&]() __attribute__((always_inline)) {
        if (cur > 0) to_ring(64);
        const bool x = gx;
        gather(64);
        rp += 64;
        wave_sync();
        if (cur > 0) eval(x);
        wave_sync();  // reads of the ring are done before it is overwritten
        cur = 64;
    };

    // ---- replay of a recorded list: 64 records at a time through LDS, 8 (up to 64 atoms)
    // per chunk.  Lane l takes atom l & 7 of record l >> 3 and keeps it when the record's
    // mask has its bit: the slots are listed in the order the search listed them, so every
    // sum is the search's.  The next 64 records are read ahead.
    bool searched = true;
    if (rpl) {
        const int cnt = *nlc;
        if (cnt <= lcap) {
            searched = false;
            uint32_t nr = lane < cnt ? (uint32_t)nl[lane] : 0u;
            for (int k0 = 0; k0 < cnt; k0 += 64) {
                clist[lane] = (int)nr;
                const int kn = k0 + 64 + lane;
                nr = kn < cnt ? (uint32_t)nl[kn] : 0u;
                wave_sync();
                const int nc = min(64, cnt - k0);
                for (int q = 0; q < nc; q += 8) {
                    const uint32_t r = (uint32_t)clist[q + sub];
                    append(__builtin_amdgcn_ballot_w64((r & (1u << atom)) != 0u), (int)((r >> 8) << 3) | atom);
                    if (wp - rp >= 64) batch();
                }
                wave_sync();
            }
        }
    }

    // ---- search ---------------------------------------------------------------------
    // State: clusters [tq, T) of clist still to test.
    const int lst = sg->s.nst, nst = !searched ? 0 : lst > 0 ? lst : sg->s.wx * sg->s.wy;
    int k0 = 0, skip = 0, T = 0, tq = 0;
    if (flags && nst > 0) {
        // excluded partners: key differences of up to 2; lane 8 i + j looks up the j-th of
        // atom i (j < 4), lane 4 the cluster itself
        reinterpret_cast<uint2*>(xmap)[lane] = make_uint2(0u, 0u);
        const int k = (mi.x >> 4) + (jslot < 2 ? jslot - 2 : jslot - 1);
        int cl = lane == 4 ? c : -1;
        if (I.v && jslot < 4 && k >= 0 && k < sg->s.nkey) {
            const int a = sg->s.kmap[k];
            if (a >= 0) cl = wsp<const int>(ws, sg->o_slotof)[(size_t)b * sg->s.Q + a] >> 3;
        }
        wave_sync();
        if (cl >= 0) atomicOr(xmap + ((cl >> 5) & (XMAP - 1)), 1u << (cl & 31));
        wave_sync();
    }
    uint4 nu = make_uint4(0u, 0u, 0u, 0u);
    int nslot = 0;
    // Positions of the chunk of 8 candidate clusters at clist[q] (one chunk ahead of use).
    auto load_chunk = [&](int q) __attribute__((always_inline)) {
        nslot = (clist[q + sub] << 3) | atom;
        nu = upos[(uint32_t)(nslot & slot_bits)];
    };
    // Cluster ranges [a0, a1) and [b0, b1) of stencil column k of this lane (empty past the
    // stencil).  Everything derived from the box is computed here, on its own copy of the
    // bounds: hoisted out of the search it would hold a dozen registers through it.
    auto columns = [&](int k, int& a0, int& a1, int& b0, int& b1) __attribute__((always_inline)) {
        a0 = a1 = b0 = b1 = 0;
        float qlx = lox, qhx = hix, qly = loy, qhy = hiy, qlz = loz, qhz = hiz;
        uint32_t qux = ucx, quy = ucy, quz = ucz;
        asm volatile("" : "+v"(qlx), "+v"(qhx), "+v"(qly), "+v"(qhy), "+v"(qlz), "+v"(qhz));
        asm volatile("" : "+v"(qux), "+v"(quy), "+v"(quz));
        // z window of candidate atoms of a column whose rectangle is (gx, gy) away from the
        // bounding box: |z - box| < sqrt(rcs^2 - gx^2 - gy^2), in z bins (per lane)
        const float Lz = sg->s.Lf[2];
        // reciprocals instead of divisions: a z bound off by one fixed-point unit, or a
        // column image chosen either way at an exact half-box tie (both images then lie at
        // the same distance), changes no test
        const float isz = sg->s.isz;
        auto zwindow = [&](float g2, bool& fullz, bool& zwrap, int& zb0, int& zb1)
                           __attribute__((always_inline)) {
            const float hz = sqrtf(fmaxf(rcs2 - g2, 0.0f));
            fullz = (qhz - qlz + 2.0f * hz) >= Lz;
            zb0 = 0;
            zb1 = nzb - 1;
            zwrap = false;
            if (!fullz) {
                const long long dlo = (long long)floorf((qlz - hz) * isz);
                const long long dhi = (long long)ceilf((qhz + hz) * isz);
                const uint32_t zlo = quz + (uint32_t)dlo;
                const uint32_t zhi = quz + (uint32_t)dhi;
                zb0 = fixed_bin(zlo, nzb);
                zb1 = fixed_bin(zhi, nzb);
                zwrap = zlo > zhi;
                if (zwrap && zb1 + 1 >= zb0) fullz = true;
            }
        };
        const float bcx = 0.5f * (qlx + qhx), bhx = 0.5f * (qhx - qlx);
        const float bcy = 0.5f * (qly + qhy), bhy = 0.5f * (qhy - qly);
        const float xref = (float)qux * sx, yref = (float)quy * sy;
        const float Lx = sg->s.Lf[0], Ly = sg->s.Lf[1];
        const float iLx = sg->s.iL[0], iLy = sg->s.iL[1];
        const float cwx = sg->s.cw[0], cwy = sg->s.cw[1];
        // the column of the i-cluster: its reference atom's as it was binned
        const uint4 ref =
            (MODE == 0 && (lists & KEPT_BINS) ? reinterpret_cast<const uint4*>(vs) : upos)[c * CLUSTER + 3];
        const int cx = fixed_bin(ref.x, ncx), cy = fixed_bin(ref.y, ncy);
        if (k < nst) {
            // stencil half widths are below the column counts (else the stencil spans
            // every column), so one wrap suffices
            int jxc, jyc;
            if (lst > 0) {
                jxc = cx + sg->s.st[k][0];
                jyc = cy + sg->s.st[k][1];
            } else {
                const int wy = sg->s.wy, ox = k / wy, oy = k - ox * wy;
                jxc = sg->s.allx ? ox : cx + ox - sg->s.rx;
                jyc = sg->s.ally ? oy : cy + oy - sg->s.ry;
            }
            jxc += jxc < 0 ? ncx : (jxc >= ncx ? -ncx : 0);
            jyc += jyc < 0 ? ncy : (jyc >= ncy ? -ncy : 0);
            float dxc = ((float)jxc + 0.5f) * cwx - xref;
            dxc -= Lx * rintf(dxc * iLx);
            dxc -= bcx;
            dxc -= Lx * rintf(dxc * iLx);
            float dyc = ((float)jyc + 0.5f) * cwy - yref;
            dyc -= Ly * rintf(dyc * iLy);
            dyc -= bcy;
            dyc -= Ly * rintf(dyc * iLy);
            const float gx = fmaxf(0.0f, fabsf(dxc) - 0.5f * cwx - bhx);
            const float gy = fmaxf(0.0f, fabsf(dyc) - 0.5f * cwy - bhy);
            const int col = jxc * ncy + jyc;
            if (gx * gx + gy * gy < rcs2) {
                bool fullz, zwrap;
                int zb0, zb1;
                zwindow(gx * gx + gy * gy, fullz, zwrap, zb0, zb1);
                const int base = colstart[col];
                const int* bo = binoff + (size_t)col * (nzb + 1);
                const int cnt = bo[nzb];
                if (cnt > 0) {
                    if (fullz) {
                        a0 = base >> 3;
                        a1 = (base + cnt + 7) >> 3;
                    } else if (!zwrap) {
                        a0 = (base + bo[zb0]) >> 3;
                        a1 = (base + bo[zb1 + 1] + 7) >> 3;
                    } else {
                        a0 = (base + bo[zb0]) >> 3;
                        a1 = (base + cnt + 7) >> 3;
                        b0 = base >> 3;
                        b1 = (base + bo[zb1 + 1] + 7) >> 3;
                        if (b1 > a0) b1 = a0;  // never list a cluster twice
                    }
                    if (N3) {  // only clusters after the own one
                        a0 = max(a0, c + 1);
                        b0 = max(b0, c + 1);
                    }
                    if (a1 < a0) a1 = a0;
                    if (b1 < b0) b1 = b0;
                }
            }
        }
    };
    // Lists the next up to CLIST candidate clusters; false when there are none left.  The
    // clusters of 64 columns that did not fit are listed by later calls, which find their
    // ranges again (k0: first of the 64 columns, skip: their clusters listed so far).
    auto refill = [&]() __attribute__((always_inline)) {
        while (k0 < nst) {
            int a0, a1, b0, b1;
            columns(k0 + lane, a0, a1, b0, b1);
            const int la = a1 - a0, len = la + (b1 - b0);
            const int incl = wave_incl_scan(len);
            const int total = __builtin_amdgcn_readlane(incl, 63);
            T = min(total - skip, CLIST);
            const int at = incl - len - skip;  // list position of this column's first cluster
            const int t1 = min(len, T - at);
            wave_sync();  // the previous list has been consumed
            // Each cluster range marks its first list position with its number (2 lane, the
            // second range of a column 2 lane + 1; ranges follow one another in that order);
            // a running maximum over the positions then gives the range of each, and the
            // clusters of a range are consecutive.  The marks' bases wait in the ring, which
            // holds no batch here.
            int* base = reinterpret_cast<int*>(ring);
            reinterpret_cast<int4*>(clist)[lane] = make_int4(0, 0, 0, 0);
            wave_sync();
            base[2 * lane] = a0 - at;
            base[2 * lane + 1] = b0 - at - la;
            if (la > 0 && at + la > 0 && at < T) clist[max(at, 0)] = 2 * lane;
            if (len > la && at + len > 0 && at + la < T) clist[max(at + la, 0)] = 2 * lane + 1;
            wave_sync();
            int last = 0;
            for (int g = 0; g < T; g += 64) {
                const int own = max(wave_incl_max(clist[g + lane]), last);
                last = __builtin_amdgcn_readlane(own, 63);
                int cl = base[own] + g + lane;
                if (flags && (xmap[(cl >> 5) & (XMAP - 1)] >> (cl & 31)) & 1u) cl |= XFLAG;
                clist[g + lane] = cl;
            }
            wave_sync();
            skip += T;
            if (skip >= total) {
                k0 += 64;
                skip = 0;
            }
            if (T == 0) continue;
            if (lane < 16) clist[T + lane] = 0;  // the last chunk read whole, and one more
            wave_sync();
            tq = 0;
            load_chunk(0);
            return true;
        }
        return false;
    };
    // Tests the chunk of 8 candidate clusters (64 atoms) at clist[tq] and lists the slots
    // of its survivors.
    auto search_chunk = [&]() __attribute__((always_inline)) {
        const uint4 uj = nu;
        const int slot = nslot;
        load_chunk(tq + 8);  // past the list: cluster 0, unused
        const float jx = (float)(int)(uj.x - ucx);
        const float jy = (float)(int)(uj.y - ucy);
        const float jz = (float)(int)(uj.z - ucz);
        const float ex = fmaxf(fmaxf(fmaf(-sx, jx, lox), fmaf(sx, jx, -hix)), 0.0f);
        const float ey = fmaxf(fmaxf(fmaf(-sy, jy, loy), fmaf(sy, jy, -hiy)), 0.0f);
        const float ez = fmaxf(fmaxf(fmaf(-sz, jz, loz), fmaf(sz, jz, -hiz)), 0.0f);
        const unsigned long long m =
            __builtin_amdgcn_ballot_w64((uj.w != PAD_W) & (fmaf(ex, ex, fmaf(ey, ey, ez * ez)) < rcs2)) &
            lanes8(T - tq);
        if (rec) {
            // masks of 64 candidate clusters (a byte each) gather in LDS; then one record
            // per cluster with a survivor, in candidate order: cluster index << 8 | mask
            if (lane == 0) smask[(tq >> 3) & 7] = m;
            if ((tq & 56) == 56 || tq + 8 >= T) {
                wave_sync();
                const int k = (tq & ~63) + lane;
                const uint32_t mk = reinterpret_cast<const unsigned char*>(smask)[lane];
                const bool has = (k < T) & (mk != 0u);
                const unsigned long long nzm = __builtin_amdgcn_ballot_w64(has);
                const int pos = __builtin_amdgcn_mbcnt_hi(
                    (unsigned)(nzm >> 32), __builtin_amdgcn_mbcnt_lo((unsigned)nzm, (unsigned)wr));
                if (has && pos < lcap) nl[pos] = (int)(((uint32_t)clist[k] << 8) | mk);
                wr += (int)__popcll(nzm);
                wave_sync();
            }
        }
        append(m, slot);
        tq += 8;
    };

    while (refill()) {
        for (; tq < T;) {
            search_chunk();
            if (wp - rp >= 64) batch();
        }
    }
    // ---- the batch in flight and the remaining slots ----------------------------------
    {
        const int n = wp - rp;
        if (cur > 0) {
            to_ring(64);
            const bool x = gx;
            if (n > 0) gather(n);
            wave_sync();
            eval(x);
            wave_sync();
        } else if (n > 0) {
            gather(n);
        }
        if (n > 0) {
            to_ring(n);
            wave_sync();
            eval_x.template operator()<false, true>(n);
        }
    }
    if (rec && lane == 0) *nlc = wr;

    // ---- reduce over the 8 j lanes of each i atom and store ------------------------
    ax += lane_xor<1>(ax);
    ay += lane_xor<1>(ay);
    az += lane_xor<1>(az);
    ax += lane_xor<2>(ax);
    ay += lane_xor<2>(ay);
    az += lane_xor<2>(az);
    ax += lane_xor<4>(ax);
    ay += lane_xor<4>(ay);
    az += lane_xor<4>(az);
    if (jslot == 0 && I.v) {
        if (N3) {
            unsafeAtomicAdd(fsx + si, ax);
            unsafeAtomicAdd(fsy + si, ay);
            unsafeAtomicAdd(fsz + si, az);
        } else {
            const int oi = wsp<const int>(ws, sg->o_orig)[(size_t)b * S + si];
            size_t o = sg->o_f32;
            if (MODE == 1 || outsel == 1) o = sg->o_hv32;
            else if (outsel == 2) o = sg->o_f32m;
            wsp<float4>(ws, o)[(size_t)b * Q + oi] = make_float4(ax, ay, az, 0.0f);
        }
    }
    if (wantE) {
        eacc64 += (double)eacc;
        eacc64 += lane_xor<1>(eacc64);
        eacc64 += lane_xor<2>(eacc64);
        eacc64 += lane_xor<4>(eacc64);
        eacc64 += lane_xor<8>(eacc64);
        eacc64 += lane_xor<16>(eacc64);
        eacc64 += lane_xor<32>(eacc64);
        if (lane == 0) wsp<double>(ws, sg->o_epart)[(size_t)b * cpb + c] = eacc64;
    }
}

// Waves per SIMD the pair kernels are compiled for (register budget 512 / waves, in
// steps of 8): 6 (80 registers) for the reaction-field force kernel without energies and
// the full-shell reaction-field Hessian kernel, 4 (128) for the Newton-3 force kernel with
// energies, 5 (96) for the rest.  A few set-up values spill (16 to 36 bytes per lane in the
// flat kernels, none of them read per step; 5 waves without spills: +5%).  Measured per
// veff_grad call on the 150,000-atom workload against 4 waves (128
// registers): -7.5% with reaction field, -1.5% with particle-mesh
// Ewald (whose mesh kernels on the second stream need room beside the pair kernels).  The
// wave index is made scalar (readfirstlane) and the lane exchanges use swizzles
// (lane_xor), so that per-wave pointers and shuffle bounds take no vector registers.
template <int MODE, int N3, int EL, int WE>
constexpr int PAIR_WAVES = EL == 0 && N3 == 0 && (MODE == 1 || WE == 0) ? 6 : (N3 && WE ? 4 : 5);

// One workgroup per PW i-clusters; consecutive workgroups of the logical order
// (neighbouring clusters) go to one XCD (workgroups are dealt to the 8 XCDs in turn).
// The launch covers beads bead0 .. bead0 + L.nb[p] - 1 of every path p.
template <int MODE, int PW, int N3, int EL, int WE>
__global__ void __launch_bounds__(64 * PW, (PAIR_WAVES<MODE, N3, EL, WE>))
    k_pair(const SegDev* __restrict__ segs, Launch L, char* __restrict__ ws, int outsel,
           int energy_bead, int lists, int bead0) {
    extern __shared__ float4 s_dyn[];
    const int nblk = L.pf[L.nseg];
    const int per = (nblk + 7) >> 3;
    const int lblk = (int)(blockIdx.x & 7) * per + (int)(blockIdx.x >> 3);
    if (lblk >= nblk) return;
    const int p = find_seg(L, lblk);
    float4* s_tab = s_dyn;
    float* s_ring = reinterpret_cast<float*>(s_dyn + TAB_COPIES<MODE> * L.ntmax * L.ntmax);
    load_table<MODE>(segs + p, s_tab, threadIdx.x, 64 * PW);
    __syncthreads();  // the only block barrier: waves are independent from here on
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);  // uniform: scalar indices
    pair_wave<MODE, N3, EL, WE>(segs, L, ws, outsel, energy_bead, lists, bead0, p,
                                (lblk - L.pf[p]) * PW + wave, s_tab, s_ring + wave * WAVE_LDS<Fields<MODE, N3, EL>>);
}

// Persistent form: as many workgroups as the GPU holds at once, each taking logical blocks
// of PW i-clusters (the flat form's workgroups) from its XCD's queue until the queue is
// empty; XCD x owns logical blocks x*per .. (x+1)*per - 1, taken in order.  One block
// barrier per logical block: the taken index goes through two alternating LDS words, so a
// word is rewritten only after every wave has passed the barrier that follows its next
// read.  The path's table is reloaded only when the path changes.  queue: 8 counters, zero
// before the launch.  A block's results do not depend on which workgroup computes it:
// results equal k_pair's.
template <int MODE, int PW, int N3, int EL, int WE>
__global__ void __launch_bounds__(64 * PW, (PAIR_WAVES<MODE, N3, EL, WE>))
    k_pair_q(const SegDev* __restrict__ segs, Launch L, char* __restrict__ ws, int outsel,
             int energy_bead, int lists, int bead0, int* __restrict__ queue) {
    extern __shared__ float4 s_dyn[];
    __shared__ int s_next[2];
    const int nblk = L.pf[L.nseg];
    const int per = (nblk + 7) >> 3;
    const int x = (int)(blockIdx.x & 7);
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);  // uniform: scalar indices
    float4* s_tab = s_dyn;
    float* s_ring = reinterpret_cast<float*>(s_dyn + TAB_COPIES<MODE> * L.ntmax * L.ntmax);
    int cur = -1;
    for (int it = 0;; it ^= 1) {
        if (threadIdx.x == 0) s_next[it] = atomicAdd(queue + x, 1);
        __syncthreads();  // also: every wave is done with the previous block (and table)
        const int k = s_next[it];
        const int lblk = x * per + k;
        if (k >= per || lblk >= nblk) break;
        const int p = find_seg(L, lblk);
        if (p != cur) {
            load_table<MODE>(segs + p, s_tab, threadIdx.x, 64 * PW);
            __syncthreads();
            cur = p;
        }
        pair_wave<MODE, N3, EL, WE>(segs, L, ws, outsel, energy_bead, lists, bead0, p,
                                    (lblk - L.pf[p]) * PW + wave, s_tab, s_ring + wave * WAVE_LDS<Fields<MODE, N3, EL>>);
    }
}

__global__ void k_queue_reset(int* queue) { queue[threadIdx.x] = 0; }

// Slot-order sums of the Newton-3 kernel to original atom order (float4), clearing the
// slot-order buffer for the next pass.
__global__ void __launch_bounds__(EWB) k_unsort(const SegDev* __restrict__ segs, Launch L, char* ws,
                                                int outsel) {
    const int blk = blockIdx.x;
    const int p = find_seg(L, blk);
    const SegDev& sg = segs[p];
    const int local = blk - L.pf[p];
    const int b = local / sg.bpb;
    const int i = (local - b * sg.bpb) * EWB + threadIdx.x;
    const int Q = sg.s.Q, S = sg.s.S;
    if (i >= Q) return;
    const int slot = wsp<const int>(ws, sg.o_slotof)[(size_t)b * Q + i];
    float* f = wsp<float>(ws, sg.o_fs) + (size_t)b * 3 * S + slot;
    const float4 v = make_float4(f[0], f[S], f[2 * S], 0.0f);
    f[0] = 0.0f;
    f[S] = 0.0f;
    f[2 * S] = 0.0f;
    size_t o = sg.o_f32;
    if (outsel == 1) o = sg.o_hv32;
    else if (outsel == 2) o = sg.o_f32m;
    wsp<float4>(ws, o)[(size_t)b * Q + i] = v;
}

// Beads bead0 .. bead0 + base.nb[p] - 1 of every path p.
template <int MODE, int PW, int N3, int EL, int WE>
static void launch_pair_t(const SegDev* dsegs, const SegDev* hsegs, const Launch& base, char* ws,
                          int outsel, int energy_bead, int lists, int bead0, bool persistent,
                          hipStream_t st) {
    Launch L = base;
    L.pf[0] = 0;
    L.ntmax = 1;
    for (int p = 0; p < base.nseg; ++p) {
        L.pf[p + 1] = L.pf[p] + (base.nb[p] * hsegs[p].s.cpb + PW - 1) / PW;
        L.ntmax = std::max(L.ntmax, hsegs[p].s.nt);
    }
    const int nblk = L.pf[base.nseg];
    if (nblk == 0) return;
    const size_t tab = TAB_COPIES<MODE> * (size_t)L.ntmax * L.ntmax * sizeof(float4);
    const size_t wlds = (size_t)WAVE_LDS<Fields<MODE, N3, EL>> * sizeof(float);
    if (persistent) {
        // a grid of what the GPU holds at once: a multiple of 8 workgroups (one set per XCD
        // queue), no more workgroups than logical blocks
        const size_t lds = tab + PW * wlds;
        // CU count and resident workgroups per CU, cached per kernel as (lds << 32 | occ)
        static std::atomic<int> ncu_c{0};
        static std::atomic<unsigned long long> occ_c{0};
        int ncu = ncu_c.load(std::memory_order_relaxed);
        if (ncu <= 0) {
            int dev = 0;
            if (hipGetDevice(&dev) != hipSuccess ||
                hipDeviceGetAttribute(&ncu, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess ||
                ncu <= 0)
                ncu = 256;
            ncu_c.store(ncu, std::memory_order_relaxed);
        }
        unsigned long long oc = occ_c.load(std::memory_order_relaxed);
        int occ = (int)(oc & 0xFFFFFFFFull);
        if (occ <= 0 || (oc >> 32) != lds) {
            if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&occ, k_pair_q<MODE, PW, N3, EL, WE>, 64 * PW,
                                                            lds) != hipSuccess ||
                occ <= 0)
                occ = 1;
            occ_c.store(((unsigned long long)lds << 32) | (unsigned)occ, std::memory_order_relaxed);
        }
        const int per = (nblk + 7) / 8;
        const int wg = std::max(1, std::min(per, occ * ncu / 8));
        int* queue = reinterpret_cast<int*>(ws + WS_QUEUE);
        hipLaunchKernelGGL(k_queue_reset, dim3(1), dim3(8), 0, st, queue);
        hipLaunchKernelGGL((k_pair_q<MODE, PW, N3, EL, WE>), dim3(8 * wg), dim3(64 * PW), lds, st, dsegs,
                           L, ws, outsel, energy_bead, lists, bead0, queue);
        return;
    }
    hipLaunchKernelGGL((k_pair<MODE, PW, N3, EL, WE>), dim3(8 * ((nblk + 7) / 8)), dim3(64 * PW),
                       tab + PW * wlds, st, dsegs, L, ws, outsel, energy_bead, lists, bead0);
}

// Waves (i-clusters) of a pair launch over every bead of base.
static long long pair_waves(const SegDev* hsegs, const Launch& base) {
    long long n = 0;
    for (int p = 0; p < base.nseg; ++p) n += (long long)base.nb[p] * hsegs[p].s.cpb;
    return n;
}
constexpr long long SPLIT_MIN_WAVES = 16384;  // about 2 rounds of the GPU's resident waves

template <int MODE, int PW, int N3, int EL>
static void launch_pair_e(const SegDev* dsegs, const SegDev* hsegs, const Launch& base, char* ws,
                          int outsel, int energy_bead, int lists, bool pq, hipStream_t st) {
    if constexpr (MODE == 1) {
        launch_pair_t<MODE, PW, N3, EL, 0>(dsegs, hsegs, base, ws, outsel, energy_bead, lists, 0, pq, st);
    } else if (energy_bead == -1) {
        launch_pair_t<MODE, PW, N3, EL, 0>(dsegs, hsegs, base, ws, outsel, energy_bead, lists, 0, pq, st);
    } else if (energy_bead == 0 && pair_waves(hsegs, base) >= SPLIT_MIN_WAVES) {
        // bead 0 of every path with energies, the other beads without (reaction field: 6 waves
        // per SIMD instead of 5; Ewald: no spilled registers, and mesh kernels that found no
        // room beside the pair kernel run while the chip drains between the two launches:
        // 9.43 -> 9.38 ms per call at 150,000 atoms x 16 beads; cutting the passes into 3 to 8
        // launches gave 0.5% more.  Launches too small to fill the GPU gain nothing from a
        // second one)
        Launch L0 = base, L1 = base;
        for (int p = 0; p < base.nseg; ++p) {
            L0.nb[p] = std::min(base.nb[p], 1);
            L1.nb[p] = base.nb[p] - L0.nb[p];
        }
        launch_pair_t<MODE, PW, N3, EL, 1>(dsegs, hsegs, L0, ws, outsel, energy_bead, lists, 0, pq, st);
        launch_pair_t<MODE, PW, N3, EL, 0>(dsegs, hsegs, L1, ws, outsel, energy_bead, lists, 1, pq, st);
    } else {
        launch_pair_t<MODE, PW, N3, EL, 1>(dsegs, hsegs, base, ws, outsel, energy_bead, lists, 0, pq, st);
    }
}

template <int MODE, int N3, int EL>
static void launch_pair_w(const SegDev* dsegs, const SegDev* hsegs, const Launch& base, char* ws,
                          int outsel, int energy_bead, int waves, int lists, hipStream_t st) {
    const bool pq = (waves & WAVES_PERSISTENT) != 0;
    switch (waves & ~WAVES_PERSISTENT) {
        case 1: launch_pair_e<MODE, 1, N3, EL>(dsegs, hsegs, base, ws, outsel, energy_bead, lists, pq, st); break;
        case 2: launch_pair_e<MODE, 2, N3, EL>(dsegs, hsegs, base, ws, outsel, energy_bead, lists, pq, st); break;
        case 8: launch_pair_e<MODE, 8, N3, EL>(dsegs, hsegs, base, ws, outsel, energy_bead, lists, pq, st); break;
        default: launch_pair_e<MODE, 4, N3, EL>(dsegs, hsegs, base, ws, outsel, energy_bead, lists, pq, st); break;
    }
}

void run_pair(const SegDev* dsegs, const SegDev* hsegs, const Launch& base, char* ws, int mode,
              int outsel, int energy_bead, int waves, int newton3, hipStream_t st, int lists) {
    if (mode == 1) outsel = 1;
    // Ewald systems: full-shell kernels only (the host rejects Newton-3 plans for them;
    // a launch holds one path then)
    if (hsegs[0].s.elec == 1) {
        if (mode == 0) launch_pair_w<0, 0, 1>(dsegs, hsegs, base, ws, outsel, energy_bead, waves, lists, st);
        else launch_pair_w<1, 0, 1>(dsegs, hsegs, base, ws, outsel, energy_bead, waves, lists, st);
        return;
    }
    if (newton3) {
        lists &= KEPT_BINS;
        if (mode == 0) launch_pair_w<0, 1, 0>(dsegs, hsegs, base, ws, outsel, energy_bead, waves, lists, st);
        else launch_pair_w<1, 1, 0>(dsegs, hsegs, base, ws, outsel, energy_bead, waves, lists, st);
        Launch L = base;
        L.pf[0] = 0;
        for (int p = 0; p < base.nseg; ++p) L.pf[p + 1] = L.pf[p] + base.nb[p] * hsegs[p].bpb;
        if (L.pf[base.nseg] > 0)
            hipLaunchKernelGGL(k_unsort, dim3(L.pf[base.nseg]), dim3(EWB), 0, st, dsegs, L, ws, outsel);
    } else {
        if (mode == 0) launch_pair_w<0, 0, 0>(dsegs, hsegs, base, ws, outsel, energy_bead, waves, lists, st);
        else launch_pair_w<1, 0, 0>(dsegs, hsegs, base, ws, outsel, energy_bead, waves, lists, st);
    }
}

}  // namespace mop
