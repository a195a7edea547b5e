// Sizes of the pair-product contraction, shared by the host tables and the
// kernels.
//
// For prisms B_q[r][(k,t)] = tau_r(t, ij) lam_r(k, m), and the value and the
// zeta derivative share the triangle factor T, so with the operators 0 (value),
// o (d/dxi1) and e (d/dxi2 - d/dxi1 / 2) on the triangle functions
//   A[(k,t)][(k',t')] = sum_ij sum_{r,s in {0,o,e}} T_r(t,ij) T_s(t',ij) G_rs^{kk'}(ij),
// where G holds the zeta sums: a product of a fixed table, over pairs (t, t')
// and (ij, r, s), with an element's G, whose columns are the pairs (k, k').
// Two symmetries cut the table into four independent blocks ("classes"):
// exchanging t and t' (G split into its parts symmetric and antisymmetric in
// r, s), and the reflection that swaps the barycentric coordinates lambda0 and
// lambda1, under which the lattice, the rule's points and the operators (0, e
// even, o odd) are invariant (points folded into pairs, sums and differences
// of the two points' W).  Rows are the orbits of the pairs (t, t') under
// both; the four classes' results give the orbit's (up to) four entries.
#pragma once

namespace feint {

// classes: 0 even symmetric, 1 even antisymmetric, 2 odd symmetric, 3 odd antisymmetric
struct PairDims {
    int nk, nt, fx, rf;               // line functions, triangle functions, fixed ones, reflected pairs of them
    int nfull, rows;                  // orbits of four pairs, all orbits
    int nij, npair, nself, sets;      // triangle points, reflected pairs of them, fixed ones, both
};

constexpr int pair_self_points(int p, int rule) {
    // collapsed: the middle of an odd number of points per line, on every line;
    // symmetric rule: the centroid and one point of each 3-orbit
    return rule == 0 ? ((p + 1) % 2 ? p + 1 : 0)
                     : (p == 1 ? 1 : p == 2 ? 2 : p == 3 ? 2 : p == 4 ? 4 : p == 5 ? 3 : p == 6 ? 5 : 6);
}
constexpr int pair_tri_points(int p, int rule) {
    return rule == 0 ? (p + 1) * (p + 1)
                     : (p == 1 ? 3 : p == 2 ? 6 : p == 3 ? 12 : p == 4 ? 16 : p == 5 ? 25 : p == 6 ? 33 : 42);
}
constexpr PairDims pair_dims(int p, int rule) {
    PairDims d{};
    d.nk = p + 1;
    d.nt = (p + 1) * (p + 2) / 2;
    d.fx = p / 2 + 1;
    d.rf = (d.nt - d.fx) / 2;
    const int nff = d.fx * (d.fx - 1) / 2;
    d.nfull = (d.nt * d.nt - d.fx - 2 * (nff + 2 * d.rf)) / 4;
    d.rows = d.nfull + 2 * d.rf + nff + d.fx;
    d.nij = pair_tri_points(p, rule);
    d.nself = pair_self_points(p, rule);
    d.npair = (d.nij - d.nself) / 2;
    d.sets = d.npair + d.nself;
    return d;
}
// Orbits are ordered: of four pairs, (t,t), (t, reflected t), (f,f') and (f,f) of
// fixed functions f; a class's rows that are not identically zero come first.
constexpr int pair_rows(int p, int cls) {
    const PairDims d = pair_dims(p, 0);
    return cls == 0 ? d.rows : cls == 1 ? d.rows - d.fx : cls == 2 ? d.nfull + d.rf : d.nfull + 2 * d.rf;
}
constexpr int pair_tiles(int p, int cls) { return (pair_rows(p, cls) + 15) / 16; }
// Contraction rows of a class, type by type: (0,o) (0,e) (0,0) (o,o) (e,e) (o,e), in the
// antisymmetric classes (0,o) (0,e) (o,e); per type the pairs of points, then
// the fixed points if the type's parity is the class's.
constexpr int pair_k(int p, int rule, int cls) {
    const PairDims d = pair_dims(p, rule);
    return cls == 0 ? 6 * d.npair + 4 * d.nself : cls == 1 ? 3 * d.npair + d.nself : cls == 2 ? 6 * d.npair + 2 * d.nself
                                                                                         : 3 * d.npair + 2 * d.nself;
}
// The same in blocks of g rows.
constexpr int pair_kb(int p, int rule, int cls, int g) { return (pair_k(p, rule, cls) + g - 1) / g; }
// Table offset of a class, in blocks of g rows x 16 orbits.
constexpr int pair_off(int p, int rule, int cls, int g) {
    int o = 0;
    for (int c = 0; c < cls; ++c) o += pair_tiles(p, c) * pair_kb(p, rule, c, g);
    return o;
}

}  // namespace feint
