// How the pair beads of a call are binned: the choice between the forms of kernels_bin.hip.
// Host code without any include of its own.
#pragma once

namespace mop {

// One path of a call.
struct BinPath {
    long long atoms;   // per bead
    long long beads;   // pair beads
    bool regs, lds;    // a bead fits one workgroup: atoms in registers / only its bins in LDS
    int form;          // result: 0 eight kernels, 1 one workgroup with registers, 2 without
};

// With its atoms in registers one workgroup per bead (form 1) is faster for any number of
// beads: 24 against 47 us for 64 beads of 3,000 atoms, 10 against 25 for one of 256.  Beyond,
// the workgroups of form 2 run side by side and take about 12 us + 3.4 ns per atom of the
// largest bead among them; the eight kernels (form 0) 28 us + 0.086 ns per atom of all their
// beads (measured from 5,000 x 1 to 30,000 x 32; 140 against 221 us for 96 beads of 22,999).
// The launches of a call follow one another, so the two add.  Paths that could take form 2 do
// so up to the size that makes the sum least: for a single path, where 3.4 ns per atom are
// less than 16 us + 0.086 ns per atom and bead.  Costs in picoseconds.
inline void choose_bin_forms(BinPath* path, int n) {
    long long general = 0, either = 0;   // atoms of the beads that must / may use form 0
    bool must = false;
    for (int p = 0; p < n; ++p) {
        BinPath& b = path[p];
        b.form = b.regs ? 1 : 0;
        if (b.regs || b.beads == 0) continue;
        if (b.lds) either += b.atoms * b.beads;
        else must = true, general += b.atoms * b.beads;
    }
    long long best = 0, limit = 0;   // largest bead of form 2 (0: none)
    for (int k = -1; k < n; ++k) {
        const long long top = k < 0 ? 0 : path[k].atoms;
        if (k >= 0 && (path[k].regs || !path[k].lds || path[k].beads == 0)) continue;
        long long rest = general + either;
        bool all = !must;
        for (int p = 0; p < n; ++p) {
            const BinPath& b = path[p];
            if (b.regs || !b.lds || b.beads == 0) continue;
            if (b.atoms <= top) rest -= b.atoms * b.beads;
            else all = false;
        }
        const long long cost = (top > 0 ? 12000000 + 3400 * top : 0) + (all ? 0 : 28000000) + 86 * rest;
        if (k < 0 || cost < best) best = cost, limit = top;
    }
    for (int p = 0; p < n; ++p)
        if (!path[p].regs && path[p].lds && path[p].atoms <= limit) path[p].form = 2;
}

}  // namespace mop
