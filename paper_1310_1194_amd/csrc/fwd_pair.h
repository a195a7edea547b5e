// Forward integration of prisms as products of pairs of triangle functions
// (the sizes, symmetries and classes are described in pair_dims.h).
//
// A workgroup takes EPB elements at a time:
//   1. W_q of every point in FP64, a pair of reflected points in neighbouring
//      lanes; their sums and differences (rows "even" and "odd" of E) into LDS.
//   2. per parity, the zeta sums G of every pair of points as small matrix
//      products: E (rows: type and pair of points, K: zeta point) times the
//      products of line factors (K x 16 columns (k, k'), held in registers).
//      On the vector ALU the same sums read E nine 16-byte LDS rows per zeta
//      point and lane and were bound by that (61k of 440k cycles per element
//      at p = 7 in FP64).
//   3. the symmetric and the antisymmetric product of the parity: table
//      fragments (16 orbits x K, from L2) times G (K x 16 columns, from LDS).
//      A wave keeps the four classes' tiles of its orbits in registers, so the
//      table is read once per workgroup and pass over the columns.
//   4. sums and differences of the four classes give the (up to) four entries
//      of each orbit, scattered through LDS so that A leaves in whole rows.
// The grid covers the device once; a workgroup goes on to further elements, whose
// inputs it fetches during the products of the present ones.
// Against the contraction per triangle point (K = 4 rows per point, tiles of
// 16 over the triangle functions, Z values formed on the vector ALU) the
// matrix work is 3.1x less at p = 7 (75 -> 24 MFLOP per element counted with the
// padding of 36 functions to 48), 4x at p = 5, 2x at p = 4, and none is spent on
// forming operands from the table.
// Bound by the matrix cores in FP64 at p = 7 (busy 65 % of the cycles; 53 % at p = 4,
// in FP32 59 % at p = 6, in bf16x3 31 % at p = 4), elsewhere by the latency of an
// element's phases, which overlap only with other workgroups' (p = 4: a quarter
// fewer workgroups per CU leave each phase as long as it was).  What shortened them:
// the table's first steps fetched before the barrier and PD steps ahead, what an
// element's first phases read held in LDS (a global load there waits for the
// stores of the element before), places and E rows looked up instead of formed,
// A stored in 16-byte pieces: p = 4 bf16x3 1.77 -> 1.57 ms, p = 5 FP32 1.86 -> 1.59,
// p = 7 bf16x3 2.88 -> 2.06; in fp16 the largest |E| by a wave's maximum instead of 64
// LDS atomics on one word, its scale from the exponent instead of a logarithm: p = 4
// 2.29 -> 1.74.
// Collapsed rule, ms, the best other kernel -> this one
// (131072 elements at p = 3, 4, 32768 at p = 5, 16384 at p = 6, 7):
//   FP64    p = 3 1.80 -> 0.85, 4 4.83 -> 3.88, 5 7.19 -> 3.00, 6 7.15 -> 4.59, 7 21.8 -> 8.31
//   FP32    p = 3 0.98 -> 0.51, 4 2.93 -> 2.19, 5 3.86 -> 1.59, 6 5.06 -> 2.31, 7 12.4 -> 4.27
//   bf16x3  p = 2 0.83 -> 0.54, 3 1.41 -> 0.48, 4 2.67 -> 1.61, 5 2.56 -> 1.02, 6 2.76 -> 1.32, 7 6.44 -> 2.02
//   fp16x3  p = 2 1.00 -> 0.60, 3 1.42 -> 0.51, 4 2.78 -> 1.74, 5 3.18 -> 1.02, 6 3.76 -> 1.37, 7 7.31 -> 2.07
// and from p = 3 at every smaller batch (one element: p = 7 FP64 0.13 against 0.40, p = 4
// 0.015 against 0.025).  At p = 2 the number of elements decides (fwd_registry.h); in FP64
// (262144 elements 0.82 of the kernel of lanes per element against 0.93) and in FP32 on the
// symmetric rule this one is not compiled.
// Errors against 64 bits are smaller in FP32 and the split forms (FP32 p = 7 1.9e-7, was
// 3.1e-7; bf16x3 p = 4 2.3e-6, was 4.3e-6: fewer terms are summed per entry), in FP64 the
// same to 2 % (p = 7 4.87e-15, was 4.82e-15).
#pragma once
#include "fwd_kernels.h"
#include "pair_dims.h"

namespace feint {

template <int FORM> struct PairForm { typedef float T; static constexpr int GK = 32; };
template <> struct PairForm<F64> { typedef double T; static constexpr int GK = 16; };
template <> struct PairForm<F32> { typedef float T; static constexpr int GK = 16; };

// The value of the neighbouring lane (lane ^ 1).
__device__ inline double lane_swap(double v) {
    const uint2 u = __builtin_bit_cast(uint2, v);
    const uint2 w = {(unsigned)__builtin_amdgcn_mov_dpp((int)u.x, 0xB1, 0xF, 0xF, true),
                     (unsigned)__builtin_amdgcn_mov_dpp((int)u.y, 0xB1, 0xF, 0xF, true)};
    return __builtin_bit_cast(double, w);
}

__device__ inline float lane_swap(float v) {
    return __int_as_float(__builtin_amdgcn_mov_dpp(__float_as_int(v), 0xB1, 0xF, 0xF, true));
}
__device__ inline uint32_t wave_max(uint32_t v) {
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) {
        const uint32_t w = (uint32_t)__shfl_xor((int)v, o, 64);
        v = w > v ? w : v;
    }
    return v;
}

// The thread's index, opaque to the optimiser: what is computed from it in a phase
// of the loop over elements is not carried, in registers or scratch, through
// the others.
__device__ inline int phase_tid() {
    int t = threadIdx.x;
    asm volatile("" : "+v"(t));
    return t;
}

// A value that no kernel in flight writes, at a uniform address: read through the
// scalar cache.  (A vector load in one branch makes the compiler wait, where the
// branches meet, for every vector memory operation before it, stores of A included.)
template <class I> __device__ inline I uniform_load(const I *p) {
    return *(const __attribute__((address_space(4))) I *)(uintptr_t)p;
}
__device__ inline int64_t pair_elem(const FwdParams &prm, int64_t slot) {
    return prm.perm ? (int64_t)uniform_load(prm.perm + slot) : slot;
}

// An element's inputs as staged in LDS: the edge vectors v1-v0, v2-v0, v4-v3, v5-v3,
// v3-v0, v4-v1, v5-v2, then D, beta, c, f of the element or of its six vertices.
// A value is fetched as two numbers whose difference is staged, so that nothing
// waits for the loads before the store.
__device__ inline double2 pair_edge(const FwdParams &prm, int64_t e, int i) {
    const int edge = i / 3, d = i - 3 * edge, hi = 0x5435421 >> (4 * edge) & 7, lo = 0x2103300 >> (4 * edge) & 7;
    const double *x = prm.coords + 18 * e + d;
    return {x[3 * hi], x[3 * lo]};
}
// The Jacobian's cofactor rows in the operators o, e and d/dzeta; returns det J.
__device__ inline double pair_cofactors(const double *in, const double *pt, double co[3], double ce[3], double cz[3]) {
    const double t = 0.5 * (1.0 + pt[2]), s = 0.5 * (1.0 - pt[2]);
    const double h0 = 0.5 * (1.0 - pt[0] - pt[1]), h1 = 0.5 * pt[0], h2 = 0.5 * pt[1];
    double a[3], b[3], c[3];
#pragma unroll
    for (int d = 0; d < 3; ++d) {
        a[d] = s * in[d] + t * in[6 + d];
        b[d] = s * in[3 + d] + t * in[9 + d];
        c[d] = h0 * in[12 + d] + h1 * in[15 + d] + h2 * in[18 + d];
    }
    co[0] = b[1] * c[2] - b[2] * c[1]; co[1] = b[2] * c[0] - b[0] * c[2]; co[2] = b[0] * c[1] - b[1] * c[0];
    ce[0] = c[1] * a[2] - c[2] * a[1]; ce[1] = c[2] * a[0] - c[0] * a[2]; ce[2] = c[0] * a[1] - c[1] * a[0];
    cz[0] = a[1] * b[2] - a[2] * b[1]; cz[1] = a[2] * b[0] - a[0] * b[2]; cz[2] = a[0] * b[1] - a[1] * b[0];
    const double det = a[0] * co[0] + a[1] * co[1] + a[2] * co[2];
#pragma unroll
    for (int d = 0; d < 3; ++d) co[d] += 0.5 * ce[d];       // d/dxi1 = o, d/dxi2 = e + o / 2
    return det;
}
// Entries of W_q at a point, in the operators 0, o, e and 3 = d/dzeta:
// 0o o3 3o, 0e e3 3e, 00 03 33, oo, ee, oe+eo, oe-eo, and w det J f.
// With C = det J K the cofactors, w det J K D K^T = (w / det J) C D C^T: K is not formed.
constexpr int PAIR_ENTRIES = 14;
template <class Coef>
__device__ inline void pair_entries(const Coef &E, double w, double det, const double co[3], const double ce[3], const double cz[3],
                                    double v[PAIR_ENTRIES]) {
    const double wd = w * det, q = w / det;
    v[6] = wd * E.c;
    v[13] = wd * E.f;
const double be[3] = {w * E.be[0], w * E.be[1], w * E.be[2]};
    auto dot = [](const double *a, const double *b) { return a[0] * b[0] + a[1] * b[1] + a[2] * b[2]; };
    v[0] = dot(co, be); v[3] = dot(ce, be); v[7] = dot(cz, be);
    auto times_D = [&](const double *a, double m[3]) {
        const double x = q * a[0], y = q * a[1], z = q * a[2];
#pragma unroll
        for (int d = 0; d < 3; ++d) m[d] = x * E.D[d] + y * E.D[3 + d] + z * E.D[6 + d];
    };
    double mo[3], me[3], mz[3];
    times_D(co, mo); times_D(ce, me); times_D(cz, mz);
    v[1] = dot(mo, cz); v[2] = dot(mz, co); v[4] = dot(me, cz); v[5] = dot(mz, ce); v[8] = dot(mz, cz);
    v[9] = dot(mo, co); v[10] = dot(me, ce);
    const double oe = dot(mo, ce), eo = dot(me, co);
    v[11] = oe + eo; v[12] = oe - eo;
}
template <class Geo> struct PairInputs {
    static constexpr int EDGES = 21, MAX = EDGES + 6 * 14;
    __device__ static int count(const FwdParams &prm) { return prm.fD ? MAX : EDGES + 14; }
    __device__ static double2 fetch(const FwdParams &prm, int64_t e, int i) {
        if (i < EDGES) return pair_edge(prm, e, i);
        i -= EDGES;
        if (prm.fD)
            return {i < 54 ? prm.fD[54 * e + i] : i < 72 ? prm.fbeta[18 * e + i - 54] : i < 78 ? prm.fc[6 * e + i - 72] : prm.ff[6 * e + i - 78], 0.0};
        return {i < 9 ? prm.D[9 * e + i] : i < 12 ? prm.beta[3 * e + i - 9] : i < 13 ? prm.c[e] : prm.f[e], 0.0};
    }
    struct Coef { double D[9], be[3], c, f; };
    // Returns det J.  The coefficients are read once the edges are done with (both at
    // once cost 28 more registers).
    __device__ static double block(const FwdParams &prm, const double *in, const double *pt, double v[PAIR_ENTRIES]) {
        double co[3], ce[3], cz[3];
        const double det = pair_cofactors(in, pt, co, ce, cz);
        __builtin_amdgcn_sched_barrier(0);
        in += EDGES;
        Coef E;
        if (!prm.fD) {
#pragma unroll
            for (int i = 0; i < 9; ++i) E.D[i] = in[i];
#pragma unroll
            for (int i = 0; i < 3; ++i) E.be[i] = in[9 + i];
            E.c = in[12];
            E.f = in[13];
        } else {
            const double t = 0.5 * (1.0 + pt[2]), s = 0.5 * (1.0 - pt[2]), l0 = 1.0 - pt[0] - pt[1];
#pragma unroll
            for (int i = 0; i < 9; ++i) E.D[i] = 0.0;
#pragma unroll
            for (int i = 0; i < 3; ++i) E.be[i] = 0.0;
            E.c = 0.0;
            E.f = 0.0;
#pragma unroll 1
            for (int a = 0; a < 6; ++a) {
                const double Na = (a % 3 == 0 ? l0 : (a % 3 == 1 ? pt[0] : pt[1])) * (a < 3 ? s : t);
#pragma unroll
                for (int i = 0; i < 9; ++i) E.D[i] += Na * in[9 * a + i];
#pragma unroll
                for (int i = 0; i < 3; ++i) E.be[i] += Na * in[54 + 3 * a + i];
                E.c += Na * in[72 + a];
                E.f += Na * in[78 + a];
            }
        }
        pair_entries(E, pt[3], det, co, ce, cz, v);
        return det;
    }
};
template <> struct PairInputs<PrismLaplaceGeo> {
    static constexpr int EDGES = 21, MAX = EDGES;
    __device__ static int count(const FwdParams &) { return EDGES; }
    __device__ static double2 fetch(const FwdParams &prm, int64_t e, int i) { return pair_edge(prm, e, i); }
    __device__ static double block(const FwdParams &, const double *in, const double *pt, double v[PAIR_ENTRIES]) {
        double co[3], ce[3], cz[3];
        const double det = pair_cofactors(in, pt, co, ce, cz), q = pt[3] / det;
        auto dot = [](const double *a, const double *b) { return a[0] * b[0] + a[1] * b[1] + a[2] * b[2]; };
        v[0] = v[3] = v[6] = v[7] = v[12] = v[13] = 0.0;
        const double so[3] = {q * co[0], q * co[1], q * co[2]}, sz[3] = {q * cz[0], q * cz[1], q * cz[2]};
        const double se[3] = {q * ce[0], q * ce[1], q * ce[2]};
        v[1] = v[2] = dot(so, cz); v[4] = v[5] = dot(se, cz); v[8] = dot(sz, cz);
        v[9] = dot(so, co); v[10] = dot(se, ce); v[11] = 2.0 * dot(so, ce);
        return det;
    }
};

// EPB elements per workgroup of NW waves; a wave takes every WT-th tile of 16
// orbits and CT / (NW / WT) tiles of 16 columns; EPB = 1: KPP values of k per
// pass over the columns; KS values of k per round through the LDS copy of A.
template <int P, int FORM, int R, class Geo, int EPB, int NW, int WT, int KPP, int KS>
struct KP {
    typedef PairForm<FORM> PF;
    typedef PairInputs<Geo> In;
    static constexpr int EPB_ = EPB, NW_ = NW;
    typedef typename PF::T T;
    typedef typename AccT<T>::type V4;
    typedef T V2 __attribute__((ext_vector_type(2)));
    // The load vector's sums: in FP64 at p = 2 in FP32, as in the kernel of lanes per element
    // (b is then rounded once; summed in FP32, entries were up to 22 times that rounding off).
    typedef std::conditional_t<P == 2 && FORM == F32, double, T> LT;
    typedef typename AccT<LT>::type VL4;
    typedef LT VL2 __attribute__((ext_vector_type(2)));
    static constexpr bool SPLIT = FORM == BF16X3 || FORM == FP16X3;
    static constexpr PairDims D = pair_dims(P, R);
    static constexpr int NK = D.nk, NT = D.nt, N = NT * NK, NIJ = D.nij, NQ = NIJ * NK;
    static constexpr int S = D.sets, NPAIR = D.npair;
    static constexpr int NTHR = NW * 64, GK = PF::GK;
    static constexpr int PASSES = c_cdiv(NK, KPP);
    static constexpr int NCOL = EPB * KPP * NK, CT = c_cdiv(NCOL, 16);
    static constexpr int WC = NW / WT, CTW = CT / WC;
    static constexpr int TPW = c_cdiv(pair_tiles(P, 0), WT);
    static constexpr int NE = PAIR_ENTRIES;                   // rows of E
    static constexpr int NS = N % 2 ? N : N + 1;              // row of the LDS copy of A: an odd stride spreads the banks
    static_assert(N == c_nshp(P) && CTW * WC == CT && NW % WT == 0, "pair kernel shape");
    static_assert(NS != N || EPB == 1, "one copy of A with unpadded rows");
    static_assert(EPB == 1 || (PASSES == 1 && NK * NK <= 16 && EPB * NK <= 16), "several elements: one pass, a column tile each");
    static constexpr int kb(int cls) { return pair_kb(P, R, cls, GK); }
    static constexpr int mx(int a, int b) { return a > b ? a : b; }
    // LDS, in bytes: G of the symmetric and antisymmetric class, E; the load vector's
    // zeta sums and the copy of A lie over what is no longer read
    static constexpr int GB = 16 * (int)sizeof(T);            // bytes per contraction row and column tile
    // rows of a class in LDS: whole blocks, in FP64 half blocks
    static constexpr int gr(int cls) { return FORM == F64 ? (pair_k(P, R, cls) + 7) / 8 * 8 : kb(cls) * GK; }
    static constexpr int GS = CT * mx(gr(0), gr(2)) * GB, GA = CT * mx(gr(1), gr(3)) * GB;
    static constexpr int GALL = GS + GA;
    static constexpr int EP = EPB * (NE - 1) * NK * S;        // E of a parity; w det J f of both follows
    static constexpr int EB = (2 * EP * (int)sizeof(T) + 2 * EPB * NK * S * (int)sizeof(LT) + 15) / 16 * 16;
    static constexpr int HT = c_cdiv(S, 16);                  // blocks of 16 sets
    static constexpr int HC = EPB * NK;                       // columns of the load vector's sums
    static constexpr int HB = 2 * HT * 16 * HC * (int)sizeof(LT);
    static constexpr bool OVER = HB <= EP * (int)sizeof(T);   // the load vector's sums lie over the even E
    static_assert(OVER || PASSES == 1, "E of every pass");
    static constexpr int VW = 16 / (int)sizeof(T);            // values of a 16-byte store
    static constexpr int ST = (EPB * KS * NT * NS + (NS == N ? VW : 0)) * (int)sizeof(T);
    static constexpr int ZR = 16 * (c_cdiv(pair_k(P, R, 0), 16) + c_cdiv(pair_k(P, R, 1), 16) + c_cdiv(pair_k(P, R, 2), 16) + c_cdiv(pair_k(P, R, 3), 16));
    static constexpr int EOFF = PASSES == 1 ? GALL : mx(GALL, (ST + 15) / 16 * 16);
    static constexpr int LOFF = EOFF + 2 * EP * (int)sizeof(T), HOFF = OVER ? EOFF : EOFF + EB;
    static constexpr int LDS = mx(EOFF + EB + (OVER ? 0 : HB), ST);
    struct alignas(16) Smem {
        char raw[(LDS + 15) / 16 * 16];
        double in[EPB][In::MAX];
        uint2 place[pair_rows(P, 0)];                         // where an orbit's entries lie in the copy of A
        double tri[2 * S][3], line[NK][2];                    // points: xi1, xi2, weight; zeta, weight
        T lam[2][NK * NK];                                    // line factors and their derivatives
        LT lamL[sizeof(LT) != sizeof(T) ? NK * NK : 1];       // line factors for the load vector, where not the same
        uint16_t zrow[ZR];                                    // contraction rows: place in E, kind
        uint32_t wmax[EPB];                                   // fp16: bits of the largest |E| of the element
    };

    // Element of slot0 + el, el varying over the lanes.
    __device__ static int64_t element(const FwdParams &prm, int64_t slot0, int el) {
        if (EPB == 1) return pair_elem(prm, slot0);
        if (!prm.perm) return slot0 + el;
        int e = uniform_load(prm.perm + slot0);
#pragma unroll
        for (int i = 1; i < EPB; ++i) {
            const int x = uniform_load(prm.perm + (slot0 + i < prm.ne ? slot0 + i : slot0));
            e = el == i ? x : e;
        }
        return e;
    }
    // ---- inputs ------------------------------------------------------------------
    static constexpr int NF = c_cdiv(EPB * In::MAX, NTHR);    // values fetched per thread
    __device__ static void fetch(const FwdParams &prm, int64_t slot0, double2 (&v)[NF]) {
        const int tid = phase_tid();
        const int cnt = In::count(prm);
#pragma unroll
        for (int f = 0; f < NF; ++f) {
            const int x = tid + f * NTHR, el = EPB == 1 ? 0 : x / cnt;
            if (el < EPB && x < EPB * cnt && slot0 + el < prm.ne) v[f] = In::fetch(prm, element(prm, slot0, el), x - el * cnt);
        }
    }
    __device__ static void store_inputs(const FwdParams &prm, const double2 (&v)[NF], Smem &sm) {
        const int tid = phase_tid();
        const int cnt = In::count(prm);
        __builtin_amdgcn_s_waitcnt(0x0F70);                   // the loads, for every path from here on
#pragma unroll
        for (int f = 0; f < NF; ++f) {
            const int x = tid + f * NTHR, el = EPB == 1 ? 0 : x / cnt;
            if (el < EPB && x < EPB * cnt) sm.in[el][x - el * cnt] = v[f].x - v[f].y;
        }
    }

    // ---- 1: E ------------------------------------------------------------------
    static constexpr bool odd_entry(int x) { return x <= 2 || x == 11 || x == 12; }     // types 0o and oe

    // One point per lane, the two points of a pair in neighbouring lanes (both
    // lanes of a fixed point hold it): task = (el, m, set, side), side fastest.
    static constexpr int TASKS = 2 * S * NK;
    __device__ static void points(const FwdParams &prm, int64_t slot0, Smem &sm) {
        const int tid = phase_tid();
        T *E = (T *)(sm.raw + EOFF);
#pragma unroll 1
        for (int first = tid & ~63; first < EPB * TASKS; first += NTHR) {
            const int task = first + (tid & 63);
            const int el0 = EPB == 1 ? 0 : task / TASKS;
            const bool live = task < EPB * TASKS && slot0 + el0 < prm.ne;
            const int el = live ? el0 : 0, rest = live ? task - el0 * TASKS : 0;
            const int m = rest / (2 * S), set = (rest - m * 2 * S) >> 1, side = rest & 1;
            const double *tp = sm.tri[rest - m * 2 * S];
            const double pt[4] = {tp[0], tp[1], sm.line[m][0], tp[2] * sm.line[m][1]};
            double v[NE];
            const double det = In::block(prm, sm.in[el], pt, v);
            if (live && !(det > 0.0) && prm.status) atomicOr(prm.status, 1u);
            if (live && prm.xq) {
                const int64_t e = element(prm, slot0, el);
                const int q = m * NIJ + prm.ppts[2 * set + side];
                double x[3];
                prism_map(prm.coords + 18 * e, pt[0], pt[1], pt[2], x);
#pragma unroll
                for (int c = 0; c < 3; ++c) prm.xq[(e * NQ + q) * 3 + c] = x[c];
            }
            // even classes (row 0, written by side 0) take the sums of the entries even under
            // the reflection and the differences of the odd ones, odd classes (row 1, side 1) the
            // others; a fixed point is its own partner with half its weight
            const double sg = side == 0 ? 1.0 : -1.0;
            T *row = E + side * EP + (el * (NE - 1) * NK + m) * S + set;
            float big = 0.0f;
#pragma unroll
            for (int x = 0; x < NE; ++x) {
                const double o = lane_swap(v[x]), y = odd_entry(x) ? fma(-sg, o, v[x]) : fma(sg, v[x], o);
                if (FORM == FP16X3 && x < 13) big = fmaxf(big, fabsf((float)y));
                if (x < NE - 1) {
                    if (live) row[x * NK * S] = (T)y;
                } else if (Geo::LOAD && live) {
                    ((LT *)(sm.raw + LOFF))[((side * EPB + el) * NK + m) * S + set] = (LT)y;
                }
            }
            if (FORM == FP16X3) {
                // one LDS atomic per wave and element (a wave's points are of one or two elements)
#pragma unroll 1
                for (int x = first / TASKS; x <= (first + 63) / TASKS && x < EPB; ++x) {
                    const uint32_t m = wave_max(live && el0 == x ? __float_as_uint(big) : 0u);
                    if ((tid & 63) == 0) atomicMax(&sm.wmax[x], m);
                }
            }
        }
    }

    // ---- 2: G ------------------------------------------------------------------
    // Contraction rows: types 0o 0e 00 oo ee oe (antisymmetric: 0o 0e oe), each over
    // every set, or over the pairs only where the type's parity is not the class's.
    static constexpr int rows_of(int par, int y) { return ((y == 0 || y == 5) == (par == 1)) ? S : NPAIR; }
    // G is kept in blocks of 16 rows as the zeta products leave them in registers:
    // lane (g, n), value v is row 4 v + g of column n, which is the second operand
    // of the products' step v (the split forms take two blocks per step).
    // At: offset of this lane's values of element el, column tile j, in a class's first block.
    static constexpr int GV = SPLIT ? 8 : FORM == F64 ? 2 : 4;
    __device__ static int column_at(int el, int j, int rows, int lane) {
        if constexpr (EPB == 1) return j * rows * 16 + lane * GV;
        const int c = el * NK * NK + (lane & 15);
        return (c >> 4) * rows * 16 + ((lane & 48) + (c & 15)) * GV;
    }
    // Row of a lane of a tile: its set, and the first x of its entries of E.
    static constexpr int zoff(int cls) { return cls == 0 ? 0 : zoff(cls - 1) + 16 * c_cdiv(pair_k(P, R, cls - 1), 16); }
    template <int CLS> __device__ static void zeta_rows(Smem &sm) {
        constexpr int PAR = CLS / 2;
        constexpr bool SYM = CLS % 2 == 0;
        constexpr int N0 = rows_of(PAR, 0), N1 = rows_of(PAR, 1), N2 = rows_of(PAR, 2), N3 = rows_of(PAR, 3), N4 = rows_of(PAR, 4);
        constexpr int K = pair_k(P, R, CLS), Z = zoff(CLS);
        for (int i = threadIdx.x; i < c_cdiv(K, 16) * 16; i += NTHR) {
            const int i16 = i & 15, r = FORM == F64 ? i : (i & ~15) + 4 * (i16 & 3) + (i16 >> 2);
            int set = r < K ? r : K - 1, x = 0;
            if (set >= N0) { set -= N0; x = 3; }
            if (x == 3 && set >= N1) { set -= N1; x = SYM ? 6 : 12; }
            if (x == 6 && set >= N2) { set -= N2; x = 9; }
            if (x == 9 && set >= N3) { set -= N3; x = 10; }
            if (x == 10 && set >= N4) { set -= N4; x = 11; }
            sm.zrow[Z + i] = (uint16_t)((x * NK * S + set) | (x < 9 ? 0x4000 : 0) | (x == 6 ? 0x8000 : 0));
        }
    }
    // What the loop over elements reads unchanged.
    __device__ static void start(const FwdParams &prm, Smem &sm) {
        static_assert(NE * NK * S < 0x4000, "places in E");
        static_for<0, 4>([&](auto c) { zeta_rows<decltype(c)::value>(sm); });
        for (int i = threadIdx.x; i < pair_rows(P, 0); i += NTHR) {
            const uint32_t w = prm.potab[i], t = w & 0xFF, u = w >> 8 & 0xFF, rt = w >> 16 & 0xFF, ru = w >> 24;
            static_assert(NT * NS * PLACE <= 0x10000, "places in the copy of A");
            sm.place[i] = uint2{(t * NS + u) * PLACE | (u * NS + t) * PLACE << 16, (rt * NS + ru) * PLACE | (ru * NS + rt) * PLACE << 16};
        }
        // the points' weights are products of a triangle's and a line's
        for (int i = threadIdx.x; i < 2 * S; i += NTHR) {
            sm.tri[i][0] = prm.pqw[4 * i]; sm.tri[i][1] = prm.pqw[4 * i + 1]; sm.tri[i][2] = prm.pqw[4 * i + 3];
        }
        if (threadIdx.x < NK) {
            const double *q = prm.pqw + 4 * 2 * S * threadIdx.x;
            sm.line[threadIdx.x][0] = q[2];
            sm.line[threadIdx.x][1] = q[3] / prm.pqw[3];
        }
        const T *lam = sizeof(T) == 8 ? (const T *)(const void *)prm.lam : (const T *)(const void *)prm.lam32;
        for (int i = threadIdx.x; i < NK * NK; i += NTHR) {
            sm.lam[0][i] = lam[i];
            sm.lam[1][i] = lam[3 * NK * NK + i];
            if constexpr (sizeof(LT) != sizeof(T)) sm.lamL[i] = prm.lam[i];
        }
        if (FORM == FP16X3 && threadIdx.x < EPB) sm.wmax[threadIdx.x] = 0;
    }
    static constexpr int PLACE = sizeof(T) == 8 ? 1 : 4;      // unit of a place: value, byte
    __device__ static T &placed(T *at, uint32_t place) {
        return sizeof(T) == 8 ? at[place] : *(T *)((char *)at + place);
    }
    template <int CLS> __device__ static void put(char *g, int at, int tile, V4 v, float sc) {
        constexpr int KB = kb(CLS), TILES = c_cdiv(pair_k(P, R, CLS), 16);
        if constexpr (FORM == F64) {
            T *q = (T *)g + at + tile * 256;
            *(V2 *)q = V2{v[0], v[1]};
            if (gr(CLS) % 16 == 0 || tile < TILES - 1) *(V2 *)(q + 128) = V2{v[2], v[3]};
        } else if constexpr (FORM == F32) {
            *(V4 *)((T *)g + at + tile * 256) = v;
        } else {
            typedef typename SplitT<FORM>::scal H;
            typedef H H4 __attribute__((ext_vector_type(4)));
            H *q = (H *)g + at + (tile >> 1) * 512 + (tile & 1) * 4;
            if (FORM == FP16X3) v *= sc;
            const H4 h = __builtin_convertvector(v, H4);
            V4 l;
            if constexpr (FORM == BF16X3) {                   // a bf16 value is the upper half of its float
                const uint2 u = __builtin_bit_cast(uint2, h);
                l = v - V4{__uint_as_float(u.x << 16), __uint_as_float(u.x & 0xFFFF0000u), __uint_as_float(u.y << 16), __uint_as_float(u.y & 0xFFFF0000u)};
            } else {
                l = v - __builtin_convertvector(h, V4);
            }
            *(H4 *)q = h;
            *(H4 *)(q + CT * KB * 512) = __builtin_convertvector(l, H4);
            if (TILES % 2 && tile == TILES - 1) {              // the rest of the last step: zero
                *(H4 *)(q + 4) = H4{0, 0, 0, 0};
                *(H4 *)(q + 4 + CT * KB * 512) = H4{0, 0, 0, 0};
            }
        }
    }
    // fp16: the power of two that puts the bound on |G| of an element in [2^13, 2^14)
    __device__ static float scale(const FwdParams &prm, const Smem &sm, int el) {
        const double m = (double)__uint_as_float(sm.wmax[el]) * prm.pair_gz;
        if (!(m > 0.0) || !(m < 1e300)) return 1.0f;
        const int ex = 13 - ((int)(__builtin_bit_cast(uint2, m).y >> 20) - 1023);
        return __uint_as_float((uint32_t)((ex < -60 ? -60 : (ex > 60 ? 60 : ex)) + 127) << 23);
    }
    // Products of line factors of a column tile, as the second operand: lane (g, n)
    // holds zeta points 4 s + g of column n (zero past the last point).
    static constexpr int KZ = c_cdiv(NK, 4);
    static constexpr int CTE = EPB == 1 ? CT : 1;
    struct Lines { T ll[KZ], ld[KZ], dl[KZ], dd[KZ]; };
    __device__ static void load_lines(const Smem &sm, int col0, Lines &l) {
        const int lane = phase_tid() & 63, c = col0 + (lane & 15), cc = c < NK * NK ? c : 0, k = cc / NK, kp = cc - k * NK;
#pragma unroll
        for (int s = 0; s < KZ; ++s) {
            const int m = 4 * s + (lane >> 4), mm = m < NK ? m : 0;
            const T on = m < NK ? (T)1 : (T)0;
            const T a = on * sm.lam[0][k * NK + mm], da = on * sm.lam[1][k * NK + mm], b = sm.lam[0][kp * NK + mm], db = sm.lam[1][kp * NK + mm];
            l.ll[s] = a * b; l.ld[s] = a * db; l.dl[s] = da * b; l.dd[s] = da * db;
        }
    }
    __device__ static void lines(const Smem &sm, int k0, Lines (&l)[CTE]) {
#pragma unroll
        for (int j = 0; j < CTE; ++j) load_lines(sm, k0 * NK + j * 16, l[j]);
    }
    // A task is a tile of 16 contraction rows for every column tile of one element:
    // its rows of E are read once.
    template <int PAR>
    __device__ static void zeta(const FwdParams &prm, int k0, const Lines (&l)[CTE], Smem &sm) {
        constexpr int C0 = 2 * PAR, C1 = 2 * PAR + 1;
        constexpr int N0 = rows_of(PAR, 0), N1 = N0 + rows_of(PAR, 1), N2 = N1 + rows_of(PAR, 2), N3 = N2 + rows_of(PAR, 3);
        constexpr int N4 = N3 + rows_of(PAR, 4), KS0 = pair_k(P, R, C0), KS1 = pair_k(P, R, C1);
        static_assert(KS0 == N4 + rows_of(PAR, 5) && KS1 == N1 + rows_of(PAR, 5), "contraction rows");
        // tiles of 16 rows: those of 0o and 0e alone serve both classes
        constexpr int BOTH = N1 / 16, TS = c_cdiv(KS0, 16), TA = c_cdiv(KS1, 16), TT = TS + TA - BOTH;
        constexpr int Z0 = zoff(C0), Z1 = zoff(C1);
        char *gs = sm.raw, *ga = sm.raw + GS;
        const int tid = phase_tid(), lane = tid & 63, i16 = lane & 15, g4 = lane >> 4;
        float sc = FORM == FP16X3 && EPB == 1 ? scale(prm, sm, 0) : 1.0f;
#pragma unroll 1
        for (int id = wave_uniform(tid >> 6); id < EPB * TT; id += NW) {
            const int el = EPB == 1 ? 0 : id / TT, task = id - el * TT;
            if (FORM == FP16X3 && EPB > 1) sc = scale(prm, sm, el);
            const bool sym = task < TS, anti = task < BOTH || !sym;
            const int tile = sym ? task : task - (TS - BOTH);
            const uint32_t zr = sm.zrow[(sym ? Z0 : Z1) + tile * 16 + i16];
            const bool x9 = zr & 0x4000, x6 = zr & 0x8000;
            const T *E = (const T *)(sm.raw + EOFF) + PAR * EP + el * (NE - 1) * NK * S + (zr & 0x3FFF);
            auto at = [&](int d, int s) {
                const int m = 4 * s + g4;
                return E[(m < NK ? m : NK - 1) * S + d * NK * S];
            };
            // which products the tile's rows take: those of 0o and 0e (L l', l L') and of 00 (L l', l l');
            // each kind is straight-line code, with independent chains of products
            const bool mixed = tile * 16 < N1, zz = sym && tile * 16 + 15 >= N1 && tile * 16 < N2;
            auto form = [&](auto mx, auto zx) {
                constexpr bool MX = decltype(mx)::value, ZX = decltype(zx)::value;
                T a0[KZ], a1[KZ], a2[KZ];
#pragma unroll
                for (int s = 0; s < KZ; ++s) {
                    a0[s] = at(0, s);
                    if (MX || ZX) {
                        const T u = at(1, s), w = at(2, s);
                        a1[s] = x9 ? u : (T)0;
                        a2[s] = x9 ? w : (T)0;
                    }
                }
                V4 p[CTE], q[CTE], w[CTE];
#pragma unroll
                for (int j = 0; j < CTE; ++j) p[j] = q[j] = w[j] = V4{0, 0, 0, 0};
#pragma unroll
                for (int s = 0; s < KZ; ++s) {
#pragma unroll
                    for (int j = 0; j < CTE; ++j) p[j] = mfma4(a0[s], l[j].ll[s], p[j]);
                    if (MX || ZX) {
#pragma unroll
                        for (int j = 0; j < CTE; ++j) q[j] = mfma4(a1[s], l[j].ld[s], q[j]);
                    }
                    if (MX) {
#pragma unroll
                        for (int j = 0; j < CTE; ++j) w[j] = mfma4(ZX && x6 ? (T)0 : a2[s], l[j].dl[s], w[j]);
                    }
                    if (ZX) {
#pragma unroll
                        for (int j = 0; j < CTE; ++j) w[j] = mfma4(MX && !x6 ? (T)0 : a2[s], l[j].dd[s], w[j]);
                    }
                }
#pragma unroll
                for (int j = 0; j < CTE; ++j) {
                    if (MX || ZX) p[j] += w[j];
                    if (EPB == 1 || i16 < NK * NK) {
                        if (sym) put<C0>(gs, column_at(el, j, gr(C0), lane), tile, MX || ZX ? p[j] + q[j] : p[j], sc);
                        if (anti) put<C1>(ga, column_at(el, j, gr(C1), lane), tile, MX || ZX ? p[j] - q[j] : p[j], sc);
                    }
                }
            };
            if (!mixed && !zz) form(ic<0>{}, ic<0>{});
            else if (!zz) form(ic<1>{}, ic<0>{});
            else if (mixed) form(ic<1>{}, ic<1>{});
            else form(ic<0>{}, ic<1>{});
        }
        if (Geo::LOAD && PAR == 1 && k0 + KPP >= NK) load_sums(sm);
    }

    // ---- load vector ------------------------------------------------------------
    // b[(k,t)] = sum over the sets of T(t) H(k), H = sum_m L_k w det J f, by halves
    // for the sum and the difference of a pair of points; both sums on the matrix
    // cores, the columns being k of every element.
    // Taken when the even E is no longer read: they lie over it.
    __device__ static void load_sums(Smem &sm) {
        LT *H = (LT *)(sm.raw + HOFF);
        const LT *L = sizeof(LT) != sizeof(T) ? sm.lamL : (const LT *)(const void *)sm.lam[0];
        const int tid = phase_tid(), lane = tid & 63, i16 = lane & 15, g4 = lane >> 4;
#pragma unroll 1
        for (int id = NW - 1 - wave_uniform(tid >> 6); id < 2 * EPB * HT; id += NW) {
            const int par = id / (EPB * HT), el = id / HT - par * EPB, tile = id % HT, k = i16 < NK ? i16 : 0;
            const int row = tile * 16 + (sizeof(LT) == 8 ? i16 : 4 * (i16 & 3) + (i16 >> 2)), set = row < S ? row : S - 1;
            const LT *E = (const LT *)(sm.raw + LOFF) + (par * EPB + el) * NK * S + set;
            VL4 p = {0, 0, 0, 0};
#pragma unroll
            for (int s = 0; s < KZ; ++s) {
                const int m = 4 * s + g4, mm = m < NK ? m : 0;
                const LT lk = m < NK ? L[k * NK + mm] : (LT)0;
                p = mfma4(E[mm * S], lk, p);
            }
            if (i16 < NK) {
                LT *q = H + (par * HT + tile) * 16 * HC + (g4 * HC + el * NK + i16) * (sizeof(LT) == 8 ? 2 : 4);
                if constexpr (sizeof(LT) == 8) {
                    *(VL2 *)q = VL2{p[0], p[1]};
                    *(VL2 *)(q + 8 * HC) = VL2{p[2], p[3]};
                } else {
                    *(VL4 *)q = p;
                }
            }
        }
    }
    __device__ static void load_vector(const FwdParams &prm, int64_t slot0, int wave, Smem &sm) {
        const LT *H = (const LT *)(sm.raw + HOFF);
        const LT *bt = sizeof(LT) == 8 ? (const LT *)(const void *)prm.pbt64 : (const LT *)(const void *)prm.pbt32;
        const int lane = phase_tid() & 63, i16 = lane & 15, hl = (lane >> 4) * HC + (i16 < HC ? i16 : 0);
#pragma unroll 1
        for (int tile = NW - 1 - wave; tile < c_cdiv(NT, 16); tile += NW) {
            VL4 v = {0, 0, 0, 0};
            const LT *A = bt + tile * 2 * HT * 256;
#pragma unroll
            for (int b = 0; b < 2 * HT; ++b) {
                if constexpr (sizeof(LT) == 8) {
#pragma unroll
                    for (int h = 0; h < 2; ++h) {
                        const VL2 x = *(const VL2 *)(A + (2 * b + h) * 128 + 2 * lane), y = *(const VL2 *)(H + (2 * b + h) * 8 * HC + 2 * hl);
                        v = mfma4(x[0], y[0], v);
                        v = mfma4(x[1], y[1], v);
                    }
                } else {
                    const VL4 x = *(const VL4 *)(A + b * 256 + 4 * lane), y = *(const VL4 *)(H + b * 16 * HC + 4 * hl);
#pragma unroll
                    for (int u = 0; u < 4; ++u) v = mfma4(x[u], y[u], v);
                }
            }
            const int el = i16 / NK, k = i16 - el * NK;
            if (el >= EPB || slot0 + el >= prm.ne) continue;
            const int64_t e = element(prm, slot0, el);
            T *bo = (T *)prm.b + (EPB == 1 && prm.offb ? uniform_load(prm.offb + e) : offb_of(prm, e, N)) + k * NT;
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                const int t = tile * 16 + acc_row<LT>(lane, r);
                if (t < NT) bo[t] = (T)v[r];
            }
        }
    }

    // ---- 3: products ------------------------------------------------------------
    // The table's first steps of a class are fetched before the class's G is complete,
    // the others PD steps ahead.
    static constexpr int PD = FORM == F64 || TPW <= 2 ? 2 : 1;
    static constexpr int PV = SPLIT ? 2 : 1;                  // vectors per tile and step
    static constexpr int KW = SPLIT ? 32 : FORM == F64 ? 8 : 16;                           // rows per step
    static constexpr int steps(int cls) { return c_cdiv(pair_k(P, R, cls), KW); }
    template <int F, bool = true> struct Frag { typedef typename SplitT<F>::vec V; };
    template <bool B> struct Frag<F64, B> { typedef V2 V; };
    template <bool B> struct Frag<F32, B> { typedef V4 V; };
    typedef typename Frag<FORM>::V FV;
    struct Ahead { FV a[PD][TPW][PV]; };
    template <int CLS> static constexpr int stride() { return (SPLIT ? 2 * kb(CLS) : kb(CLS) * GK / KW) * 64; }   // vectors per tile
    template <int CLS> __device__ static const FV *table(const FwdParams &prm) {
        return (const FV *)prm.pairA + (size_t)(SPLIT ? pair_off(P, R, CLS, GK) * 2 : pair_off(P, R, CLS, GK) * GK / KW) * 64 + (phase_tid() & 63);
    }
    template <int CLS> __device__ static void ahead(const FwdParams &prm, int wt, Ahead &h) {
        constexpr int TL = pair_tiles(P, CLS), NA = c_cdiv(TL, WT);
        const FV *A = table<CLS>(prm);
#pragma unroll
        for (int b = 0; b < PD; ++b)
            if (b < steps(CLS)) {
#pragma unroll
                for (int i = 0; i < NA; ++i) {
                    const int t = wt + i * WT < TL ? wt + i * WT : TL - 1;
#pragma unroll
                    for (int v = 0; v < PV; ++v) h.a[b][i][v] = A[t * stride<CLS>() + (PV * b + v) * 64];
                }
            }
    }
    template <int CLS, int NA>
    __device__ static void product(const FwdParams &prm, const char *g, int wt, int ct0, Ahead &h, V4 (&acc)[TPW][CTW]) {
        constexpr int STEPS = steps(CLS), ST1 = stride<CLS>(), KB = kb(CLS);
        constexpr int GVS = gr(CLS) / KW;                     // steps of G per column tile (not the split forms)
        constexpr int TAIL = c_cdiv(pair_k(P, R, CLS) - (STEPS - 1) * KW, 4);              // steps of 4 rows in the last one
        const FV *A = table<CLS>(prm) + wt * ST1;
        const FV *B = (const FV *)g + ct0 * (SPLIT ? KB : GVS) * 64 + (phase_tid() & 63);
        auto step = [&](int b8, int slot, bool more, int nv) {
            if constexpr (!SPLIT) {
                FV b[CTW];
#pragma unroll
                for (int j = 0; j < CTW; ++j) b[j] = B[(j * GVS + b8) * 64];
#pragma unroll
                for (int v = 0; v < KW / 4; ++v)
                    if (v < nv) {
#pragma unroll
                        for (int i = 0; i < NA; ++i)
#pragma unroll
                            for (int j = 0; j < CTW; ++j) acc[i][j] = mfma4(h.a[slot][i][0][v], b[j][v], acc[i][j]);
                    }
            } else {
                FV bh[CTW], bl[CTW];
#pragma unroll
                for (int j = 0; j < CTW; ++j) { bh[j] = B[(j * KB + b8) * 64]; bl[j] = B[(j * KB + b8 + CT * KB) * 64]; }
#pragma unroll
                for (int i = 0; i < NA; ++i)
#pragma unroll
                    for (int j = 0; j < CTW; ++j) acc[i][j] = mfma32(h.a[slot][i][0], bl[j], acc[i][j]);
#pragma unroll
                for (int i = 0; i < NA; ++i)
#pragma unroll
                    for (int j = 0; j < CTW; ++j) acc[i][j] = mfma32(h.a[slot][i][PV - 1], bh[j], acc[i][j]);
#pragma unroll
                for (int i = 0; i < NA; ++i)
#pragma unroll
                    for (int j = 0; j < CTW; ++j) acc[i][j] = mfma32(h.a[slot][i][0], bh[j], acc[i][j]);
            }
            if (more) {
#pragma unroll
                for (int i = 0; i < NA; ++i)
#pragma unroll
                    for (int v = 0; v < PV; ++v) h.a[slot][i][v] = A[i * WT * ST1 + (PV * (b8 + PD) + v) * 64];
            }
        };
        // whole rounds of PD steps that fetch as many, then the rest
        constexpr int ROUNDS = STEPS > PD ? (STEPS - PD) / PD : 0;
#pragma unroll 1
        for (int r = 0; r < ROUNDS; ++r)
#pragma unroll
            for (int u = 0; u < PD; ++u) step(r * PD + u, u, true, KW / 4);
        static_for<ROUNDS * PD, STEPS>([&](auto b) {
            constexpr int b8 = decltype(b)::value;
            step(b8, b8 % PD, b8 + PD < STEPS, b8 == STEPS - 1 ? TAIL : KW / 4);
        });
        // Fetched for a tile that this wave does not have: taken here, as the wait for these
        // registers' next use would else wait for the stores of A too.
#pragma unroll
        for (int b = 0; b < PD; ++b)
            if (b < STEPS) {
#pragma unroll
                for (int i = NA; i < c_cdiv(pair_tiles(P, CLS), WT); ++i)
#pragma unroll
                    for (int v = 0; v < PV; ++v) asm volatile("" : : "v"(h.a[b][i][v]));
            }
    }
    // The class's tiles of this wave are a prefix of its list.
    template <int CLS>
    __device__ static void products(const FwdParams &prm, const char *g, int wt, int ct0, Ahead &h, V4 (&acc)[TPW][CTW]) {
        constexpr int TL = pair_tiles(P, CLS);
        static_for<1, TPW + 1>([&](auto n) {
            constexpr int NA = decltype(n)::value;
            // some wave has NA tiles: wt + (NA - 1) WT < TL <= wt + NA WT
            if constexpr ((NA - 1) * WT < TL && TL <= WT - 1 + NA * WT)
                if (wt + (NA - 1) * WT < TL && TL <= wt + NA * WT) product<CLS, NA>(prm, g, wt, ct0, h, acc);
        });
    }
    // Whether any wave has an i-th tile in a class: where none has, the class adds nothing.
    static constexpr bool has(int cls, int i) { return i * WT < pair_tiles(P, cls); }
    static constexpr bool odd(int i) { return has(2, i) || has(3, i); }
    static constexpr bool anti(int i) { return has(1, i) || has(3, i); }
    __device__ static void zero(V4 (&acc)[TPW][CTW]) {
#pragma unroll
        for (int i = 0; i < TPW; ++i)
#pragma unroll
            for (int j = 0; j < CTW; ++j) acc[i][j] = V4{0, 0, 0, 0};
    }
    // Both products of a parity, from G's formation; s = sum, d = difference of the two.
    template <int PAR>
    __device__ static void parity(const FwdParams &prm, int k0, int wt, int ct0, V4 (&s)[TPW][CTW], V4 (&d)[TPW][CTW],
                                  const Lines (&l)[CTE], Smem &sm) {
        Ahead h;
        zeta<PAR>(prm, k0, l, sm);
        ahead<2 * PAR>(prm, wt, h);
        __syncthreads();
        zero(s);
        products<2 * PAR>(prm, sm.raw, wt, ct0, h, s);
        ahead<2 * PAR + 1>(prm, wt, h);
        zero(d);
        products<2 * PAR + 1>(prm, sm.raw + GS, wt, ct0, h, d);
#pragma unroll
        for (int i = 0; i < TPW; ++i)
            if (has(2 * PAR + 1, i)) {
#pragma unroll
                for (int j = 0; j < CTW; ++j) {
                    const V4 x = s[i][j], y = d[i][j];
                    s[i][j] = x + y;
                    d[i][j] = x - y;
                }
            }
    }

    // ---- 4: A -------------------------------------------------------------------
    __device__ static T *out(const FwdParams &prm, int64_t slot, int k) {
        const int64_t e = pair_elem(prm, slot);
        return (T *)prm.A + (prm.offA ? uniform_load(prm.offA + e) : e * (int64_t)N * N) + (size_t)k * NT * N;
    }
    // values between the last 16-byte boundary and p
    __device__ static int head(const T *p) { return (int)((uintptr_t)p / sizeof(T) % VW); }
    // cnt values of the copy, whole rows, to A: in 16-byte pieces (8 bytes where only
    // pairs divide a row).
    __device__ static void copy_out(T *Ao, const T *src, int cnt, int tid) {
        if constexpr (NS == N) {
            typedef T VT __attribute__((ext_vector_type(VW)));
            const int h = head(Ao), end = h + cnt;
            Ao -= h;
            for (int q = tid * VW; q < end; q += NTHR * VW) {
                if (q >= h && q + VW <= end) {
                    *(VT *)(Ao + q) = *(const VT *)(src + q);
                } else {
#pragma unroll
                    for (int i = 0; i < VW; ++i)
                        if (q + i >= h && q + i < end) Ao[q + i] = src[q + i];
                }
            }
        } else {
            constexpr int VN = N % VW == 0 ? VW : 2, NV = N / VN, INV = ((1 << 20) + NV - 1) / NV;
            static_assert(N % VN == 0 && KS * NT * NV * (NV - 1) < 1 << 20, "row of a piece");
            typedef T VT __attribute__((ext_vector_type(VN)));
            if ((uintptr_t)Ao % sizeof(VT) == 0) {
#pragma unroll 4
                for (int q = tid; q < cnt / VN; q += NTHR) {
                    const T *x = src + q * VN + (__umul24(q, INV) >> 20);
                    VT v;
#pragma unroll
                    for (int i = 0; i < VN; ++i) v[i] = x[i];
                    *(VT *)(Ao + q * VN) = v;
                }
            } else {
                for (int x = tid; x < cnt; x += NTHR) Ao[x] = src[x + x / N];
            }
        }
    }

    // ---- one group of elements ----------------------------------------------------
    // slot0's inputs are in sm.in; those of next0 are there at the end.
    __device__ static void group(const FwdParams &prm, int64_t slot0, int64_t next0, int wave, Smem &sm) {
        const int tid = phase_tid();
        const int lane = tid & 63;
        const int wt = wave % WT, ct0 = wave / WT * CTW;
        points(prm, slot0, sm);
        double2 nx[NF];
        if (next0 < prm.ne) fetch(prm, next0, nx);
        Lines l[CTE];
        if (PASSES == 1) lines(sm, 0, l);
        __syncthreads();
#pragma unroll 1
        for (int k0 = 0; k0 < NK; k0 += KPP) {
            V4 es[TPW][CTW], ed[TPW][CTW], os[TPW][CTW], od[TPW][CTW];
            if (PASSES > 1) lines(sm, k0, l);
            parity<0>(prm, k0, wt, ct0, es, ed, l, sm);
            if (k0 == 0) {
                if (next0 < prm.ne) store_inputs(prm, nx, sm);
            }
            __syncthreads();
            parity<1>(prm, k0, wt, ct0, os, od, l, sm);
            if (Geo::LOAD && k0 + KPP >= NK) load_vector(prm, slot0, wave, sm);
            // the four entries of an orbit
#pragma unroll
            for (int i = 0; i < TPW; ++i)
#pragma unroll
                for (int j = 0; j < CTW; ++j) {
                    if (!odd(i)) continue;
                    const V4 x = es[i][j], y = has(1, i) ? ed[i][j] : x, z = os[i][j], w = has(3, i) ? od[i][j] : z;
                    es[i][j] = x + z; os[i][j] = x - z;
                    if (anti(i)) { ed[i][j] = y + w; od[i][j] = y - w; }
                }
            // the places of the wave's orbits, all read before the first write waits for LDS
            uint2 place[TPW][4];
#pragma unroll
            for (int i = 0; i < TPW; ++i)
#pragma unroll
                for (int r = 0; r < 4; ++r) {
                    const int o = (wt + i * WT) * 16 + acc_row<T>(lane, r);
                    place[i][r] = sm.place[o < pair_rows(P, 0) ? o : 0];
                }
            __syncthreads();
#pragma unroll 1
            for (int kr = 0; kr < KPP && k0 + kr < NK; kr += KS) {
                if (kr > 0) __syncthreads();
                // one element: the copy starts where A's 16-byte pieces do, if its rows are not padded
                T *st = (T *)sm.raw;
                if (NS == N) st += head(out(prm, slot0, k0 + kr));
#pragma unroll
                for (int j = 0; j < CTW; ++j) {
                    const int c = (ct0 + j) * 16 + (lane & 15);
                    const int el = EPB == 1 ? 0 : c / (NK * NK), cc = c - el * NK * NK, kk = cc / NK;
                    if (EPB > 1 ? el >= EPB : kk >= KPP || k0 + kk >= NK) continue;      // no column
                    if (kk < kr || kk >= kr + KS) continue;                              // another round's
                    T *at = st + (EPB == 1 ? 0 : el * NT * NK * NS) + (kk - kr) * NT * NS + (cc - kk * NK) * NT;
                    const T un = FORM == FP16X3 ? (T)ldexpf(1.0f / scale(prm, sm, el), -prm.pair_shift) : (T)1;
#pragma unroll
                    for (int i = 0; i < TPW; ++i) {
                        if (wt + i * WT >= pair_tiles(P, 0)) break;
#pragma unroll
                        for (int r = 0; r < 4; ++r) {
                            const int o = (wt + i * WT) * 16 + acc_row<T>(lane, r);
                            if ((wt + i * WT + 1) * 16 > pair_rows(P, 0) && o >= pair_rows(P, 0)) continue;
                            uint2 pl = place[i][r];
                            asm volatile("" : "+v"(pl.x), "+v"(pl.y));     // unpacked here, not kept unpacked across the rounds
                            const T e0 = es[i][j][r], e1 = anti(i) ? ed[i][j][r] : e0;
                            const T e2 = odd(i) ? os[i][j][r] : e0, e3 = !odd(i) ? e1 : anti(i) ? od[i][j][r] : e2;
                            placed(at, pl.x & 0xFFFF) = FORM == FP16X3 ? e0 * un : e0;
                            placed(at, pl.x >> 16) = FORM == FP16X3 ? e1 * un : e1;
                            placed(at, pl.y & 0xFFFF) = FORM == FP16X3 ? e2 * un : e2;
                            placed(at, pl.y >> 16) = FORM == FP16X3 ? e3 * un : e3;
                        }
                    }
                }
                __syncthreads();
                const int ks = NK - k0 - kr < KS ? NK - k0 - kr : KS;
                for (int el = 0; el < EPB && slot0 + el < prm.ne; ++el)
                    copy_out(out(prm, slot0 + el, k0 + kr), (const T *)sm.raw + el * NT * NK * NS, ks * NT * N, tid);
            }
            if (FORM == FP16X3 && k0 + KPP >= NK && tid < EPB) sm.wmax[tid] = 0;
            __syncthreads();
        }
    }
    // Groups first, first + step, ... of EPB slots.
    __device__ static void run(const FwdParams &prm, int64_t first, int64_t step, Smem &sm) {
        const int64_t groups = (prm.ne + EPB - 1) / EPB;
        if (first >= groups) return;
        start(prm, sm);
        double2 v[NF];
        fetch(prm, first * EPB, v);
        store_inputs(prm, v, sm);
        __syncthreads();
#pragma unroll 1
        for (int64_t g = first; g < groups; g += step) {
            // the wave's share of the orbits turns with the group: the last tiles are uneven
            const int wave = (wave_uniform(threadIdx.x >> 6) + (int)(g & 1023)) % NW;
            group(prm, g * EPB, (g + step) * EPB, wave, sm);
        }
    }
};

// Waves that do not divide over the four SIMDs cost most (p = 4: five for the five
// tiles of orbits 7.1 ms against 4.1 with four in FP64; p = 6: seven for 14 tiles
// 3.4 against 2.5 in FP32), then workgroups per CU count: the shapes are the
// fastest of those that fit.
// Shapes per degree and form: elements per workgroup, waves, waves over the
// orbits, values of k per pass and per round, waves per SIMD asked of the
// register allocator.
template <int P, int FORM> struct PairShape;
#define FEINT_PAIR_SHAPE(P, FORM, EPB_, NW_, WT_, KPP_, KS_, W_)                                        \
    template <> struct PairShape<P, FORM> {                                                              \
        static constexpr int EPB = EPB_, NW = NW_, WT = WT_, KPP = KPP_, KS = KS_, W = W_;                \
    };
FEINT_PAIR_SHAPE(3, F64, 1, 2, 2, 4, 4, 4)
FEINT_PAIR_SHAPE(4, F64, 1, 4, 4, 5, 5, 3)
FEINT_PAIR_SHAPE(5, F64, 1, 4, 4, 2, 1, 3)
FEINT_PAIR_SHAPE(6, F64, 1, 8, 8, 4, 1, 2)
FEINT_PAIR_SHAPE(7, F64, 1, 8, 8, 4, 1, 2)
FEINT_PAIR_SHAPE(3, F32, 4, 4, 2, 4, 4, 4)
FEINT_PAIR_SHAPE(4, F32, 1, 4, 4, 5, 5, 4)
FEINT_PAIR_SHAPE(5, F32, 1, 4, 4, 6, 3, 3)
FEINT_PAIR_SHAPE(6, F32, 1, 8, 8, 4, 2, 4)
FEINT_PAIR_SHAPE(7, F32, 1, 8, 8, 8, 2, 2)
FEINT_PAIR_SHAPE(2, F32, 3, 2, 1, 3, 3, 4)
FEINT_PAIR_SHAPE(2, BF16X3, 3, 2, 1, 3, 3, 4)
FEINT_PAIR_SHAPE(3, BF16X3, 2, 2, 1, 4, 4, 3)
FEINT_PAIR_SHAPE(4, BF16X3, 1, 4, 4, 5, 5, 4)
FEINT_PAIR_SHAPE(5, BF16X3, 1, 4, 4, 6, 2, 3)
FEINT_PAIR_SHAPE(6, BF16X3, 1, 8, 8, 4, 2, 4)
FEINT_PAIR_SHAPE(7, BF16X3, 1, 8, 8, 8, 2, 2)
template <int P> struct PairShape<P, FP16X3> : PairShape<P, BF16X3> {};

template <int P, int FORM, int R = 0, class Geo = PrismGeo, class S = PairShape<P, FORM>>
using KPOf = KP<P, FORM, R, Geo, S::EPB, S::NW, S::WT, S::KPP, S::KS>;

template <class K, int NW, int MINW>
__global__ __launch_bounds__(NW * 64, MINW) void fwd_pair(FwdParams prm) {
    __shared__ typename K::Smem sm;
    K::run(prm, blockIdx.x, gridDim.x, sm);
}

}  // namespace feint
