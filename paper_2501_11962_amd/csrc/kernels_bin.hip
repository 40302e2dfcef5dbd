// Binning of every pair bead of every path of a call into the column/cluster layout.
//
// Per bead: wrap coordinates into 32-bit fixed point, histogram atoms over
// (column, z bin), scan bins inside each column, scan padded column counts, scatter
// atoms into slot order, and fill each column's padding slots.  The counting sort
// replaces the pair search of the physical force routine (do_force, section 2.1).
// Inside a bin atoms are ordered by index (the histogram's atomic ranks only reserve
// places), so the slot order, and with it every pair sum, is the same on every call.
// HBM-bound, O(Q) per bead.
#include <algorithm>

#include "bin_forms.h"
#include "device_common.h"
#include "launch.h"

namespace mop {

// Zero the bin histograms, the slot-order pair sums (newton3) and (zero_dmax) the per-bead
// max |d|^2 of every segment.
__global__ void __launch_bounds__(EWB) k_zero(const SegDev* __restrict__ segs, Launch L, char* ws,
                                              int zero_dmax, int newton3) {
    const int blk = blockIdx.x;
    const int p = find_seg(L, blk);
    const SegDev& sg = segs[p];
    const size_t idx = (size_t)(blk - L.pf[p]) * EWB + threadIdx.x;
    const size_t n1 = (size_t)L.nb[p] * sg.s.ncol * sg.s.nzb;
    const size_t n2 = newton3 ? (size_t)L.nb[p] * 3 * sg.s.S : 0;
    if (idx < n1) {
        wsp<int>(ws, sg.o_bincnt)[idx] = 0;
    } else if (idx - n1 < n2) {
        wsp<float>(ws, sg.o_fs)[idx - n1] = 0.0f;
    } else if (zero_dmax && idx - n1 - n2 < (size_t)sg.maxN) {
        wsp<unsigned long long>(ws, sg.o_dmax)[idx - n1 - n2] = 0ull;
    }
}

// Fixed-point coordinates, bin key and rank inside the bin.  fdsign != 0 bins the
// displaced configuration R^b + fdsign * eps_b d^b of the finite-difference term.
__global__ void __launch_bounds__(EWB) k_bin_count(const SegDev* __restrict__ segs, Launch L,
                                                   char* ws, const double* __restrict__ R,
                                                   int fdsign, double fdh) {
    const int blk = blockIdx.x;
    const int p = find_seg(L, blk);
    const SegDev& sg = segs[p];
    const int local = blk - L.pf[p];
    const int b = local / sg.bpb;
    const int i = (local - b * sg.bpb) * EWB + threadIdx.x;
    const int Q = sg.s.Q;
    if (i >= Q) return;
    const double* r = R + sg.roff + ((size_t)b * Q + i) * 3;
    double x = r[0], y = r[1], z = r[2];
    if (fdsign != 0) {
        const double m2 = __longlong_as_double(
            (long long)wsp<unsigned long long>(ws, sg.o_dmax)[b]);
        const double eps = m2 > 0.0 ? fdsign * fdh / sqrt(m2) : 0.0;
        const double* d = wsp<const double>(ws, sg.o_d64) + ((size_t)b * Q + i) * 3;
        x += eps * d[0];
        y += eps * d[1];
        z += eps * d[2];
    }
    const uint32_t ux = to_fixed(x, sg.s.L[0]), uy = to_fixed(y, sg.s.L[1]), uz = to_fixed(z, sg.s.L[2]);
    const int col = fixed_bin(ux, sg.s.ncx) * sg.s.ncy + fixed_bin(uy, sg.s.ncy);
    const int key = col * sg.s.nzb + fixed_bin(uz, sg.s.nzb);
    int* cnt = wsp<int>(ws, sg.o_bincnt) + (size_t)b * sg.s.ncol * sg.s.nzb;
    const int rank = atomicAdd(cnt + key, 1);
    wsp<uint4>(ws, sg.o_atomu)[(size_t)b * Q + i] = make_uint4(ux, uy, uz, (uint32_t)key);
    wsp<int>(ws, sg.o_rank)[(size_t)b * Q + i] = rank;
}

// Exclusive scan of the z bins of each column; column totals.  One wave per column:
// each lane sums a run of consecutive bins, a wave scan places the runs.
__global__ void __launch_bounds__(EWB) k_bin_colscan(const SegDev* __restrict__ segs, Launch L, char* ws) {
    const int blk = blockIdx.x;
    const int p = find_seg(L, blk);
    const SegDev& sg = segs[p];
    const int t = (blk - L.pf[p]) * (EWB / 64) + (threadIdx.x >> 6);  // column of this wave
    const int lane = threadIdx.x & 63;
    const int ncol = sg.s.ncol, nzb = sg.s.nzb;
    if (t >= L.nb[p] * ncol) return;
    const int b = t / ncol, col = t - b * ncol;
    const int* cnt = wsp<const int>(ws, sg.o_bincnt) + ((size_t)b * ncol + col) * nzb;
    int* off = wsp<int>(ws, sg.o_binoff) + ((size_t)b * ncol + col) * (nzb + 1);
    const int per = (nzb + 63) >> 6;
    const int z0 = min(lane * per, nzb), z1 = min(z0 + per, nzb);
    int sum = 0;
    for (int z = z0; z < z1; ++z) sum += cnt[z];
    const int incl = wave_incl_scan(sum);
    int run = incl - sum;
    for (int z = z0; z < z1; ++z) {
        off[z] = run;
        run += cnt[z];
    }
    if (lane == 63) {
        off[nzb] = incl;
        wsp<int>(ws, sg.o_colcnt)[(size_t)b * ncol + col] = incl;
    }
}

// Exclusive scan of the padded (multiple of 8) column counts of one bead per block.
constexpr int CSB = 1024;
__global__ void __launch_bounds__(CSB) k_bin_colstart(const SegDev* __restrict__ segs, Launch L, char* ws) {
    __shared__ int sh[CSB];
    const int blk = blockIdx.x;
    const int p = find_seg(L, blk);
    const SegDev& sg = segs[p];
    const int b = blk - L.pf[p];
    const int ncol = sg.s.ncol;
    const int* cc = wsp<const int>(ws, sg.o_colcnt) + (size_t)b * ncol;
    int* cs = wsp<int>(ws, sg.o_colstart) + (size_t)b * (ncol + 1);
    const int per = (ncol + CSB - 1) / CSB;
    const int c0 = threadIdx.x * per, c1 = min(ncol, c0 + per);
    int sum = 0;
    for (int c = c0; c < c1; ++c) sum += (cc[c] + 7) & ~7;
    sh[threadIdx.x] = sum;
    __syncthreads();
    for (int d = 1; d < CSB; d <<= 1) {
        const int v = threadIdx.x >= d ? sh[threadIdx.x - d] : 0;
        __syncthreads();
        sh[threadIdx.x] += v;
        __syncthreads();
    }
    int run = sh[threadIdx.x] - sum;
    for (int c = c0; c < c1; ++c) {
        cs[c] = run;
        run += (cc[c] + 7) & ~7;
    }
    if (threadIdx.x == CSB - 1) cs[ncol] = sh[CSB - 1];
}

// Atom i's bin: first slot and atom count.
__device__ __forceinline__ void bin_range(const SegDev& sg, char* ws, int b, int key, int& first,
                                          int& count) {
    const int ncol = sg.s.ncol, nzb = sg.s.nzb;
    const int col = key / nzb, zb = key - col * nzb;
    const int* bo = wsp<const int>(ws, sg.o_binoff) + ((size_t)b * ncol + col) * (nzb + 1);
    first = wsp<const int>(ws, sg.o_colstart)[(size_t)b * (ncol + 1) + col] + bo[zb];
    count = bo[zb + 1] - bo[zb];
}

// Reserve places: the atoms of each bin in the order of their atomic ranks.
__global__ void __launch_bounds__(EWB) k_bin_scatter(const SegDev* __restrict__ segs, Launch L, char* ws) {
    const int blk = xcd_block(L.pf[L.nseg]);
    if (blk < 0) return;
    const int p = find_seg(L, blk);
    const SegDev& sg = segs[p];
    const int local = blk - L.pf[p];
    const int b = local / sg.bpb;
    const int i = (local - b * sg.bpb) * EWB + threadIdx.x;
    const int Q = sg.s.Q;
    if (i >= Q) return;
    const int key = (int)wsp<const uint4>(ws, sg.o_atomu)[(size_t)b * Q + i].w;
    int first, count;
    bin_range(sg, ws, b, key, first, count);
    wsp<int>(ws, sg.o_tmpo)[(size_t)b * sg.s.S + first + wsp<const int>(ws, sg.o_rank)[(size_t)b * Q + i]] = i;
}

// Place each atom at its bin's first slot plus the number of atoms of the bin with a
// smaller index.
__global__ void __launch_bounds__(EWB) k_bin_place(const SegDev* __restrict__ segs, Launch L, char* ws) {
    const int blk = xcd_block(L.pf[L.nseg]);
    if (blk < 0) return;
    const int p = find_seg(L, blk);
    const SegDev& sg = segs[p];
    const int local = blk - L.pf[p];
    const int b = local / sg.bpb;
    const int i = (local - b * sg.bpb) * EWB + threadIdx.x;
    const int Q = sg.s.Q, S = sg.s.S;
    if (i >= Q) return;
    const uint4 u = wsp<const uint4>(ws, sg.o_atomu)[(size_t)b * Q + i];
    int first, count;
    bin_range(sg, ws, b, (int)u.w, first, count);
    const int* tmpo = wsp<const int>(ws, sg.o_tmpo) + (size_t)b * S + first;
    int r = 0;
    for (int k = 0; k < count; ++k) r += tmpo[k] < i;
    const int slot = first + r;
    wsp<uint4>(ws, sg.o_upos)[(size_t)b * S + slot] =
        make_uint4(u.x, u.y, u.z, __float_as_uint(sg.s.qs[i]));
    wsp<int2>(ws, sg.o_umeta)[(size_t)b * S + slot] = make_int2(sg.s.key[i], sg.s.type[i]);
    wsp<int>(ws, sg.o_orig)[(size_t)b * S + slot] = i;
    wsp<int>(ws, sg.o_slotof)[(size_t)b * Q + i] = slot;
}

// Padding slots of each column: position of the column's last atom, PAD_W, DUMMY_KEY
// (displaced: its position as binned too).
__global__ void __launch_bounds__(EWB) k_bin_pad(const SegDev* __restrict__ segs, Launch L, char* ws,
                                                 int displaced) {
    const int blk = blockIdx.x;
    const int p = find_seg(L, blk);
    const SegDev& sg = segs[p];
    const int t = (blk - L.pf[p]) * EWB + threadIdx.x;
    const int ncol = sg.s.ncol, S = sg.s.S;
    if (t >= L.nb[p] * ncol) return;
    const int b = t / ncol, col = t - b * ncol;
    const int n = wsp<const int>(ws, sg.o_colcnt)[(size_t)b * ncol + col];
    const int pad = (n + 7) & ~7;
    if (pad == n) return;
    const int base = wsp<const int>(ws, sg.o_colstart)[(size_t)b * (ncol + 1) + col];
    uint4* up = wsp<uint4>(ws, sg.o_upos) + (size_t)b * S;
    int2* um = wsp<int2>(ws, sg.o_umeta) + (size_t)b * S;
    int* og = wsp<int>(ws, sg.o_orig) + (size_t)b * S;
    uint4* vs = wsp<uint4>(ws, sg.o_vs) + (size_t)b * S;
    const uint4 last = up[base + n - 1];
    for (int k = n; k < pad; ++k) {
        up[base + k] = make_uint4(last.x, last.y, last.z, PAD_W);
        um[base + k] = make_int2(DUMMY_KEY, 0);
        og[base + k] = -1;
        if (displaced) vs[base + k] = vs[base + n - 1];
    }
}

// Shared-bin finite differences: the displaced coordinates R^b + fdsign eps_b d^b written
// into the slots the binning of R gave each atom (no new sort).  R's own go to vs, which only
// exact gradients read otherwise: the pair search takes a cluster's column from them, as a
// displaced atom may lie in the next one.
__global__ void __launch_bounds__(EWB) k_bin_displace(const SegDev* __restrict__ segs, Launch L,
                                                      char* ws, const double* __restrict__ R,
                                                      int fdsign, double fdh) {
    const int blk = blockIdx.x;
    const int p = find_seg(L, blk);
    const SegDev& sg = segs[p];
    const int local = blk - L.pf[p];
    const int b = local / sg.bpb;
    const int i = (local - b * sg.bpb) * EWB + threadIdx.x;
    const int Q = sg.s.Q;
    if (i >= Q) return;
    const double* r = R + sg.roff + ((size_t)b * Q + i) * 3;
    const double m2 = __longlong_as_double((long long)wsp<unsigned long long>(ws, sg.o_dmax)[b]);
    const double eps = m2 > 0.0 ? fdsign * fdh / sqrt(m2) : 0.0;
    const double* d = wsp<const double>(ws, sg.o_d64) + ((size_t)b * Q + i) * 3;
    const int slot = wsp<const int>(ws, sg.o_slotof)[(size_t)b * Q + i];
    wsp<uint4>(ws, sg.o_upos)[(size_t)b * sg.s.S + slot] =
        make_uint4(to_fixed(r[0] + eps * d[0], sg.s.L[0]), to_fixed(r[1] + eps * d[1], sg.s.L[1]),
                   to_fixed(r[2] + eps * d[2], sg.s.L[2]), __float_as_uint(sg.s.qs[i]));
    wsp<uint4>(ws, sg.o_vs)[(size_t)b * sg.s.S + slot] =
        make_uint4(to_fixed(r[0], sg.s.L[0]), to_fixed(r[1], sg.s.L[1]), to_fixed(r[2], sg.s.L[2]), 0u);
}

// Overlap check of a binned configuration: sets ST_OVERLAP in the status word, which leads
// the workspace, when a non-excluded pair lies closer than OVERLAP_R (the same FP32
// difference of fixed-point coordinates the pair kernels form).  Each pair is looked for
// from one of its atoms:
//   same column: slots are in the order of the z bins, so the partners of slot si are the
//     slots after it up to the bin of u_z + d (in most cases the one or two that share
//     its bin); past the top of the box, the column's first bins too;
//   neighbouring columns: only for an atom within d of its column's upper x or y face
//     (d is far below a column width), over the bins from u_z - d to u_z + d.
// Looking through the bins around every atom instead (two columns per axis, bin bounds
// read first) took 61 us for 15 beads of 150,000 atoms and 17 of the 28 us of the
// one-workgroup binning of 3,000.
// Past 16 partners a thread stops at its first hit: the status has no more to say, and where a
// run has diverged (coordinates that are not finite share one bin) every pair would be tested,
// one after another: 5,349 atoms x 2 beads 2506 us a gradient, now 806; 3,000 x 2, where
// k_bin_bead does the same, 1834 and 968.
// pos(slot) and key(slot) read a slot; first(col, zb) and end(col, zb) give a bin's slots.
template <class Pos, class Key, class First, class End>
__device__ __forceinline__ bool overlaps(const SysDev& s, int si, uint32_t ux, uint32_t uy, uint32_t uz,
                                         int nslots, Pos pos, Key key, First first, End end) {
    const int ncx = s.ncx, ncy = s.ncy, nzb = s.nzb;
    const uint32_t d0 = s.ovr[0], d1 = s.ovr[1], d2 = s.ovr[2];
    bool hit = false;
    auto test = [&](int sj, const uint4& uj) __attribute__((always_inline)) {
        const float dx = (float)(int)(uj.x - ux) * s.sc[0];
        const float dy = (float)(int)(uj.y - uy) * s.sc[1];
        const float dz = (float)(int)(uj.z - uz) * s.sc[2];
        const float r2 = fmaf(dx, dx, fmaf(dy, dy, dz * dz));
        if (r2 < OVERLAP_R2) hit |= abs((key(si) >> 4) - (key(sj) >> 4)) > 2;
    };
    const int cx = fixed_bin(ux, ncx), cy = fixed_bin(uy, ncy);
    // upper end of the z bins to look through; all of them after a wrap (d < box height)
    const uint32_t zt = uz + d2;
    const int zb1 = zt < uz ? nzb - 1 : fixed_bin(zt, nzb);
    int sj = si + 1;
    auto column = [&](int end, bool first_hit) __attribute__((always_inline)) {
        for (; sj < end && !(first_hit && hit); ++sj) {
            const uint4 uj = pos(sj);
            if (uj.w == PAD_W || fixed_bin(uj.z, nzb) > zb1 || fixed_bin(uj.x, ncx) != cx ||
                fixed_bin(uj.y, ncy) != cy)
                return;
            test(sj, uj);
        }
    };
    // the few partners of most atoms without a look at what was found (35 against 42 us at
    // 150,000 atoms x 15 beads)
    const int few = min(nslots, si + 17);
    column(few, false);
    if (sj == few) column(nslots, true);
    auto bins = [&](int col, int za, int zb) __attribute__((always_inline)) {  // za .. zb, wrapping
        for (int z = za;; z = z + 1 == nzb ? 0 : z + 1) {
            const int e = end(col, z);
            for (int sj = first(col, z); sj < e; ++sj)
                if (sj != si) test(sj, pos(sj));
            if (z == zb) break;
        }
    };
    if (zt < uz) bins(cx * ncy + cy, 0, fixed_bin(zt, nzb));
    const int x1 = fixed_bin(ux + d0, ncx), y1 = fixed_bin(uy + d1, ncy);
    if (x1 != cx || y1 != cy) {
        const int y0 = fixed_bin(uy - d1, ncy), z0 = fixed_bin(uz - d2, nzb), z1 = fixed_bin(zt, nzb);
        if (y1 != cy) bins(cx * ncy + y1, z0, z1);
        if (x1 != cx) {
            bins(x1 * ncy + cy, z0, z1);
            if (y1 != cy) bins(x1 * ncy + y1, z0, z1);
            if (y0 != cy && y0 != y1) bins(x1 * ncy + y0, z0, z1);
        }
    }
    return hit;
}

__global__ void __launch_bounds__(EWB) k_overlap(const SegDev* __restrict__ segs, Launch L, char* ws) {
    const int blk = xcd_block(L.pf[L.nseg]);
    if (blk < 0) return;
    const int p = find_seg(L, blk);
    const SegDev& sg = segs[p];
    const int local = blk - L.pf[p];
    const int S = sg.s.S, nzb = sg.s.nzb;
    const int bps = (S + EWB - 1) / EWB;  // blocks per bead (slot order)
    const int b = local / bps;
    const int si = (local - b * bps) * EWB + threadIdx.x;
    const int* cs = wsp<const int>(ws, sg.o_colstart) + (size_t)b * (sg.s.ncol + 1);
    const int ns = cs[sg.s.ncol];
    if (si >= ns) return;  // slots past the last column hold no atom
    const uint4* up = wsp<const uint4>(ws, sg.o_upos) + (size_t)b * S;
    const int2* um = wsp<const int2>(ws, sg.o_umeta) + (size_t)b * S;
    const int* bo = wsp<const int>(ws, sg.o_binoff) + (size_t)b * sg.s.ncol * (nzb + 1);
    const uint4 ui = up[si];
    if (ui.w == PAD_W) return;
    const bool hit = overlaps(
        sg.s, si, ui.x, ui.y, ui.z, ns, [&](int sj) { return up[sj]; }, [&](int sj) { return um[sj].x; },
        [&](int col, int z) { return cs[col] + bo[(size_t)col * (nzb + 1) + z]; },
        [&](int col, int z) { return cs[col] + bo[(size_t)col * (nzb + 1) + z + 1]; });
    if (hit) atomicOr(reinterpret_cast<int*>(ws), ST_OVERLAP);
}

// ---- one bead per workgroup ---------------------------------------------------------
// The whole binning of a bead in one workgroup whose bin counts and reserved places fit the
// LDS: the eight kernels above cost a launch and a trip through memory each, which is what
// bounds them on small systems (3-5 us each; 27 of the 58 us of a gradient of 256 atoms x
// 32 beads), and global atomics bound the counting on larger ones.  Same slots, same arrays.
//   J > 0    atoms per thread at most (Q <= 1024 J), kept in registers, positions in LDS.
//            The overlap check is done here too: pairs of one bin while the bin is ordered,
//            then the few atoms within OVERLAP_R of an upper bin face against the bins
//            beyond it, as a list of (atom, bin) tasks spread over all threads.
//   J == 0   more atoms: coordinates and ranks wait in the workspace; k_overlap follows
constexpr int FB = 1024;           // threads
constexpr int FUSED_COLS = 1024;   // columns at most (one per thread in the column scan)
constexpr size_t FUSED_LDS = 144 * 1024;

constexpr int TASKS = 2048;        // overlap tasks held (more are done where they arise)

static size_t fused_lds(const SysDev& s, bool regs) {
    const size_t bins = (size_t)s.ncol * s.nzb;
    return bins * 4 + (((size_t)s.S * 2 + 3) & ~(size_t)3) + (regs ? (size_t)s.Q * 12 + TASKS * 4 : 0);
}
constexpr int FUSED_J = 4;
static bool fused_regs(const SysDev& s) {
    return s.Q <= FB * FUSED_J && s.ncol <= FUSED_COLS && (size_t)s.ncol * s.nzb <= 65536 &&
           fused_lds(s, true) <= FUSED_LDS;
}
static bool fused_any(const SysDev& s) {
    return s.Q <= 65535 && s.ncol <= FUSED_COLS && fused_lds(s, false) <= FUSED_LDS;
}

template <int J>
__global__ void __launch_bounds__(FB) k_bin_bead(const SegDev* __restrict__ segs, Launch L, char* ws,
                                                 const double* __restrict__ R, int fdsign, double fdh,
                                                 int newton3) {
    extern __shared__ int s_bin[];  // counts, then offsets inside the column
    __shared__ int s_cnt[FUSED_COLS], s_start[FUSED_COLS + 1], s_wave[FB / 64], s_ntask;
    constexpr bool REGS = J > 0;
    constexpr int NJ = REGS ? J : 1;
    const int p = find_seg(L, blockIdx.x);
    const SegDev& sg = segs[p];
    const int b = (int)blockIdx.x - L.pf[p];
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int Q = sg.s.Q, S = sg.s.S, ncol = sg.s.ncol, nzb = sg.s.nzb, ncx = sg.s.ncx, ncy = sg.s.ncy;
    const int nbin = ncol * nzb;
    unsigned short* s_tmp = reinterpret_cast<unsigned short*>(s_bin + nbin);
    uint32_t* s_x = reinterpret_cast<uint32_t*>(s_tmp + ((S + 1) & ~1));
    uint32_t *s_y = s_x + Q, *s_z = s_y + Q, *s_task = s_z + Q;  // (J > 0) by atom
    uint4* upos = wsp<uint4>(ws, sg.o_upos) + (size_t)b * S;
    int2* umeta = wsp<int2>(ws, sg.o_umeta) + (size_t)b * S;
    int* orig = wsp<int>(ws, sg.o_orig) + (size_t)b * S;
    int* slotof = wsp<int>(ws, sg.o_slotof) + (size_t)b * Q;
    uint4* atomu = wsp<uint4>(ws, sg.o_atomu) + (size_t)b * Q;
    int* rankg = wsp<int>(ws, sg.o_rank) + (size_t)b * Q;
    int* binoff = wsp<int>(ws, sg.o_binoff) + (size_t)b * ncol * (nzb + 1);
    int* colstart = wsp<int>(ws, sg.o_colstart) + (size_t)b * (ncol + 1);

    double eps = 0.0;
    const double* dis = nullptr;
    if (fdsign != 0) {
        const double m2 = __longlong_as_double((long long)wsp<unsigned long long>(ws, sg.o_dmax)[b]);
        eps = m2 > 0.0 ? fdsign * fdh / sqrt(m2) : 0.0;
        dis = wsp<const double>(ws, sg.o_d64) + (size_t)b * Q * 3;
    } else if (tid == 0) {
        wsp<unsigned long long>(ws, sg.o_dmax)[b] = 0ull;
    }
    for (int t = tid; t < nbin; t += FB) s_bin[t] = 0;
    if (tid == 0) s_ntask = 0;
    if (newton3) {  // the slot-order pair sums of the Newton-3 kernels
        float* fs = wsp<float>(ws, sg.o_fs) + (size_t)b * 3 * S;
        for (int t = tid; t < 3 * S; t += FB) fs[t] = 0.0f;
    }
    __syncthreads();

    // counts and ranks.  .w: column << 20 | z bin (z bins are below 2^16 here)
    uint4 u[NJ];
    int rk[NJ];
    const double* Rb = R + sg.roff + (size_t)b * Q * 3;
    auto count = [&](int i, uint4& v, int& rank) __attribute__((always_inline)) {
        double x = Rb[3 * (size_t)i], y = Rb[3 * (size_t)i + 1], z = Rb[3 * (size_t)i + 2];
        if (fdsign != 0) {
            x += eps * dis[3 * (size_t)i];
            y += eps * dis[3 * (size_t)i + 1];
            z += eps * dis[3 * (size_t)i + 2];
        }
        v.x = to_fixed(x, sg.s.L[0]);
        v.y = to_fixed(y, sg.s.L[1]);
        v.z = to_fixed(z, sg.s.L[2]);
        const int col = fixed_bin(v.x, ncx) * ncy + fixed_bin(v.y, ncy), zb = fixed_bin(v.z, nzb);
        v.w = ((uint32_t)col << 20) | (uint32_t)zb;
        rank = atomicAdd(s_bin + col * nzb + zb, 1);
    };
    if constexpr (REGS) {
#pragma unroll
        for (int j = 0; j < NJ; ++j)
            if (tid + j * FB < Q) {
                const int i = tid + j * FB;
                count(i, u[j], rk[j]);
                s_x[i] = u[j].x;
                s_y[i] = u[j].y;
                s_z[i] = u[j].z;
            }
    } else {
        for (int i = tid; i < Q; i += FB) {
            count(i, u[0], rk[0]);
            atomu[i] = u[0];
            rankg[i] = rk[0];
        }
    }
    __syncthreads();

    // z-bin offsets inside each column, one wave per column
    const int per = (nzb + 63) >> 6;
    for (int col = wave; col < ncol; col += FB / 64) {
        int* cnt = s_bin + col * nzb;
        int* off = binoff + (size_t)col * (nzb + 1);
        const int z0 = min(lane * per, nzb), z1 = min(z0 + per, nzb);
        int sum = 0;
        for (int z = z0; z < z1; ++z) sum += cnt[z];
        const int incl = wave_incl_scan(sum);
        int run = incl - sum;
        for (int z = z0; z < z1; ++z) {
            const int c = cnt[z];
            cnt[z] = run;
            off[z] = run;
            run += c;
        }
        if (lane == 63) {
            off[nzb] = incl;
            s_cnt[col] = incl;
            wsp<int>(ws, sg.o_colcnt)[(size_t)b * ncol + col] = incl;
        }
    }
    __syncthreads();
    // first slot of each column (counts padded to whole clusters)
    {
        const int v = tid < ncol ? (s_cnt[tid] + 7) & ~7 : 0;
        const int incl = wave_incl_scan(v);
        if (lane == 63) s_wave[wave] = incl;
        __syncthreads();
        int base = 0;
        for (int k = 0; k < wave; ++k) base += s_wave[k];
        if (tid < ncol) {
            s_start[tid] = base + incl - v;
            colstart[tid] = base + incl - v;
        }
        if (tid == FB - 1) {
            s_start[ncol] = base + incl;
            colstart[ncol] = base + incl;
        }
    }
    __syncthreads();
    // reserve places in rank order, then place each atom after the atoms of its bin with a
    // smaller index
    auto first_of = [&](uint32_t w) __attribute__((always_inline)) {
        const int col = (int)(w >> 20), zb = (int)(w & 0xFFFFFu);
        return s_start[col] + s_bin[col * nzb + zb];
    };
    if constexpr (REGS) {
#pragma unroll
        for (int j = 0; j < NJ; ++j)
            if (tid + j * FB < Q) s_tmp[first_of(u[j].w) + rk[j]] = (unsigned short)(tid + j * FB);
    } else {
        for (int i = tid; i < Q; i += FB) s_tmp[first_of(atomu[i].w) + rankg[i]] = (unsigned short)i;
    }
    __syncthreads();
    bool hit = false;
    // atoms i and k closer than OVERLAP_R (see k_overlap) and not excluded (J > 0)
    auto near = [&](int i, const uint4& v, int k) __attribute__((always_inline)) {
        const float dx = (float)(int)(s_x[k] - v.x) * sg.s.sc[0];
        const float dy = (float)(int)(s_y[k] - v.y) * sg.s.sc[1];
        const float dz = (float)(int)(s_z[k] - v.z) * sg.s.sc[2];
        if (fmaf(dx, dx, fmaf(dy, dy, dz * dz)) < OVERLAP_R2)
            hit |= abs((sg.s.key[i] >> 4) - (sg.s.key[k] >> 4)) > 2;
    };
    auto bin_end = [&](int bin) __attribute__((always_inline)) {
        const int col = bin / nzb;
        return bin - col * nzb + 1 < nzb ? s_bin[bin + 1] : s_cnt[col];
    };
    auto place = [&](int i, const uint4& v) __attribute__((always_inline)) {
        const int col = (int)(v.w >> 20), zb = (int)(v.w & 0xFFFFFu);
        const int off = s_bin[col * nzb + zb];
        const int n = (zb + 1 < nzb ? s_bin[col * nzb + zb + 1] : s_cnt[col]) - off;
        const int first = s_start[col] + off;
        int r = 0, k = 0;
        auto ranks = [&](int end, bool first_hit) __attribute__((always_inline)) {
            for (; k < end; ++k) {
                const int o = s_tmp[first + k];
                r += o < i;
                if (REGS && o > i && !(first_hit && hit)) near(i, v, o);
            }
        };
        ranks(min(n, 16), false);  // as in overlaps()
        ranks(n, true);
        const int slot = first + r;
        upos[slot] = make_uint4(v.x, v.y, v.z, __float_as_uint(sg.s.qs[i]));
        umeta[slot] = make_int2(sg.s.key[i], sg.s.type[i]);
        orig[slot] = i;
        slotof[i] = slot;
    };
    // (J > 0) atom i against every atom of a bin
    auto scan_bin = [&](int i, const uint4& v, int bin) __attribute__((always_inline)) {
        const int base = s_start[bin / nzb], e = base + bin_end(bin);
        for (int k = base + s_bin[bin]; k < e; ++k)
            if ((int)s_tmp[k] != i) near(i, v, s_tmp[k]);
    };
    // (J > 0) the bins beyond the upper faces that atom i is near (every pair of bins is
    // looked at from the lower one; x-y neighbours over the bins of u_z -/+ d)
    auto faces = [&](int i, const uint4& v) __attribute__((always_inline)) {
        const int cx = fixed_bin(v.x, ncx), cy = fixed_bin(v.y, ncy), zb = (int)(v.w & 0xFFFFFu);
        auto add = [&](int col, int za, int ze) {
            for (int z = za;; z = z + 1 == nzb ? 0 : z + 1) {
                const int bin = col * nzb + z;
                const int t = atomicAdd(&s_ntask, 1);
                if (t < TASKS) s_task[t] = (uint32_t)i << 16 | (uint32_t)bin;
                else scan_bin(i, v, bin);
                if (z == ze) break;
            }
        };
        const uint32_t* d = sg.s.ovr;
        const int z1 = fixed_bin(v.z + d[2], nzb);
        if (z1 != zb) add(cx * ncy + cy, zb + 1 == nzb ? 0 : zb + 1, z1);
        const int x1 = fixed_bin(v.x + d[0], ncx), y1 = fixed_bin(v.y + d[1], ncy);
        if (x1 != cx || y1 != cy) {
            const int y0 = fixed_bin(v.y - d[1], ncy), z0 = fixed_bin(v.z - d[2], nzb);
            if (y1 != cy) add(cx * ncy + y1, z0, z1);
            if (x1 != cx) {
                add(x1 * ncy + cy, z0, z1);
                if (y1 != cy) add(x1 * ncy + y1, z0, z1);
                if (y0 != cy && y0 != y1) add(x1 * ncy + y0, z0, z1);
            }
        }
    };
    if constexpr (REGS) {
#pragma unroll
        for (int j = 0; j < NJ; ++j)
            if (tid + j * FB < Q) {
                place(tid + j * FB, u[j]);
                faces(tid + j * FB, u[j]);
            }
    } else {
        for (int i = tid; i < Q; i += FB) place(i, atomu[i]);
    }
    __syncthreads();
    if (REGS) {
        for (int t = tid; t < min(s_ntask, TASKS) && !hit; t += FB) {
            const int i = (int)(s_task[t] >> 16);
            scan_bin(i, make_uint4(s_x[i], s_y[i], s_z[i], 0u), (int)(s_task[t] & 0xFFFFu));
        }
        if (hit) atomicOr(reinterpret_cast<int*>(ws), ST_OVERLAP);
    }
    // padding slots of each column
    if (tid < ncol) {
        const int n = s_cnt[tid], base = s_start[tid], pad = (n + 7) & ~7;
        if (pad > n) {
            const uint4 last = upos[base + n - 1];
            for (int k = base + n; k < base + pad; ++k) {
                upos[k] = make_uint4(last.x, last.y, last.z, PAD_W);
                umeta[k] = make_int2(DUMMY_KEY, 0);
                orig[k] = -1;
            }
        }
    }
}

void run_displace(const SegDev* dsegs, const SegDev* hsegs, const Launch& base, char* ws,
                  const double* R, int fdsign, double fdh, hipStream_t st) {
    Launch La = base;
    La.pf[0] = 0;
    for (int p = 0; p < base.nseg; ++p) La.pf[p + 1] = La.pf[p] + base.nb[p] * hsegs[p].bpb;
    hipLaunchKernelGGL(k_bin_displace, dim3(La.pf[base.nseg]), dim3(EWB), 0, st, dsegs, La, ws, R,
                       fdsign, fdh);
    Launch Lc = base;
    Lc.pf[0] = 0;
    for (int p = 0; p < base.nseg; ++p)
        Lc.pf[p + 1] = Lc.pf[p] + (base.nb[p] * hsegs[p].s.ncol + EWB - 1) / EWB;
    hipLaunchKernelGGL(k_bin_pad, dim3(Lc.pf[base.nseg]), dim3(EWB), 0, st, dsegs, Lc, ws, 1);
}

template <int J>
static void launch_bead(const SegDev* dsegs, const SegDev* hsegs, const Launch& base, const char* which,
                        char* ws, const double* R, int fdsign, double fdh, int newton3, hipStream_t st) {
    Launch L = base;
    L.pf[0] = 0;
    size_t lds = 0;
    for (int p = 0; p < base.nseg; ++p) {
        const bool mine = which[p] == (J > 0 ? 1 : 2);
        L.pf[p + 1] = L.pf[p] + (mine ? base.nb[p] : 0);
        if (mine) lds = std::max(lds, fused_lds(hsegs[p].s, J > 0));
    }
    if (L.pf[base.nseg] == 0) return;
    hipLaunchKernelGGL(k_bin_bead<J>, dim3(L.pf[base.nseg]), dim3(FB), lds, st, dsegs, L, ws, R, fdsign, fdh,
                       newton3);
}

static void bin_general(const SegDev* dsegs, const SegDev* hsegs, const Launch& base, char* ws,
                        const double* R, int fdsign, double fdh, int newton3, hipStream_t st);

static void launch_overlap(const SegDev* dsegs, const SegDev* hsegs, const Launch& base, char* ws,
                           hipStream_t st) {
    Launch L = base;  // one thread per slot
    L.pf[0] = 0;
    for (int p = 0; p < base.nseg; ++p)
        L.pf[p + 1] = L.pf[p] + base.nb[p] * ((hsegs[p].s.S + EWB - 1) / EWB);
    if (L.pf[base.nseg] > 0)
        hipLaunchKernelGGL(k_overlap, dim3(xcd_grid(L.pf[base.nseg])), dim3(EWB), 0, st, dsegs, L, ws);
}

void run_binning(const SegDev* dsegs, const SegDev* hsegs, const Launch& base, char* ws,
                 const double* R, int fdsign, double fdh, int newton3, hipStream_t st) {
    // one workgroup per bead (k_bin_bead) or eight kernels over all beads
    BinPath path[MAXSEG];
    for (int p = 0; p < base.nseg; ++p) {
        const SysDev& s = hsegs[p].s;
        path[p] = {s.Q, base.nb[p], fused_regs(s), fused_any(s), 0};
    }
    choose_bin_forms(path, base.nseg);
    char which[MAXSEG] = {};
    Launch G = base, O = base;  // beads binned by the eight kernels / with the overlap check apart
    bool rest = false, one = false, two = false;
    for (int p = 0; p < base.nseg; ++p) {
        which[p] = (char)path[p].form;
        if (which[p]) G.nb[p] = 0;
        if (which[p] == 1) O.nb[p] = 0;
        one = one || which[p] == 1;
        two = two || which[p] == 2;
        rest = rest || (!which[p] && base.nb[p] > 0);
    }
    if (one) launch_bead<FUSED_J>(dsegs, hsegs, base, which, ws, R, fdsign, fdh, newton3, st);
    if (two) launch_bead<0>(dsegs, hsegs, base, which, ws, R, fdsign, fdh, newton3, st);
    if (rest) bin_general(dsegs, hsegs, G, ws, R, fdsign, fdh, newton3, st);
    launch_overlap(dsegs, hsegs, O, ws, st);
}

static void bin_general(const SegDev* dsegs, const SegDev* hsegs, const Launch& base, char* ws,
                        const double* R, int fdsign, double fdh, int newton3, hipStream_t st) {
    Launch L = base;
    // zero histograms (+ max |d|^2 when not binning a displaced configuration)
    L.pf[0] = 0;
    for (int p = 0; p < base.nseg; ++p) {
        const size_t n = (size_t)base.nb[p] * hsegs[p].s.ncol * hsegs[p].s.nzb +
                         (newton3 ? (size_t)base.nb[p] * 3 * hsegs[p].s.S : 0) +
                         (fdsign == 0 ? hsegs[p].maxN : 0);
        L.pf[p + 1] = L.pf[p] + (int)((n + EWB - 1) / EWB);
    }
    if (L.pf[base.nseg] > 0) hipLaunchKernelGGL(k_zero, dim3(L.pf[base.nseg]), dim3(EWB), 0, st, dsegs, L, ws,
                                                 fdsign == 0 ? 1 : 0, newton3);
    // atoms
    Launch La = base;
    La.pf[0] = 0;
    for (int p = 0; p < base.nseg; ++p) La.pf[p + 1] = La.pf[p] + base.nb[p] * hsegs[p].bpb;
    hipLaunchKernelGGL(k_bin_count, dim3(La.pf[base.nseg]), dim3(EWB), 0, st, dsegs, La, ws, R, fdsign, fdh);
    // columns
    Launch Lc = base;
    Lc.pf[0] = 0;
    for (int p = 0; p < base.nseg; ++p)
        Lc.pf[p + 1] = Lc.pf[p] + (base.nb[p] * hsegs[p].s.ncol + EWB - 1) / EWB;
    Launch Lw = base;  // one wave per column
    Lw.pf[0] = 0;
    for (int p = 0; p < base.nseg; ++p)
        Lw.pf[p + 1] = Lw.pf[p] + (base.nb[p] * hsegs[p].s.ncol + EWB / 64 - 1) / (EWB / 64);
    hipLaunchKernelGGL(k_bin_colscan, dim3(Lw.pf[base.nseg]), dim3(EWB), 0, st, dsegs, Lw, ws);
    Launch Lb = base;
    Lb.pf[0] = 0;
    for (int p = 0; p < base.nseg; ++p) Lb.pf[p + 1] = Lb.pf[p] + base.nb[p];
    hipLaunchKernelGGL(k_bin_colstart, dim3(Lb.pf[base.nseg]), dim3(CSB), 0, st, dsegs, Lb, ws);
    hipLaunchKernelGGL(k_bin_scatter, dim3(xcd_grid(La.pf[base.nseg])), dim3(EWB), 0, st, dsegs, La, ws);
    hipLaunchKernelGGL(k_bin_place, dim3(xcd_grid(La.pf[base.nseg])), dim3(EWB), 0, st, dsegs, La, ws);
    hipLaunchKernelGGL(k_bin_pad, dim3(Lc.pf[base.nseg]), dim3(EWB), 0, st, dsegs, Lc, ws, 0);
}

}  // namespace mop
