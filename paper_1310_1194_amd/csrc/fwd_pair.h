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
// Bound by the matrix cores in FP64 at p = 7 (58 % of an element's time in the
// products, which then run at their peak rate), elsewhere by the phases that do
// not overlap with them.  Collapsed rule, ms, the best other kernel -> this one
// (131072 elements at p = 3, 4, 32768 at p = 5, 16384 at p = 6, 7):
//   FP64    p = 3 1.80 -> 1.09, 4 4.83 -> 4.13, 5 7.19 -> 3.31, 6 7.15 -> 4.83, 7 21.8 -> 8.39
//   FP32    p = 3 0.98 -> 0.61, 4 2.93 -> 2.45, 5 3.86 -> 1.86, 6 5.06 -> 2.70, 7 12.4 -> 4.76
//   bf16x3  p = 2 0.83 -> 0.71, 3 1.41 -> 0.63, 4 2.67 -> 1.89, 5 2.56 -> 1.58, 6 2.76 -> 2.09, 7 6.44 -> 2.88
//   fp16x3  p = 2 1.00 -> 0.99, 3 1.42 -> 1.01, 4 2.78 -> 2.46, 5 3.18 -> 2.00, 6 3.76 -> 2.24, 7 7.31 -> 3.37
// At p = 2 in FP64 and FP32 the kernel of lanes per element is faster (0.86
// against 1.17 ms, 0.56 against 0.70 on 262144 elements) and this one is not compiled.
// Errors against 64 bits are no larger in any form (FP32 p = 7 1.9e-7, was 3.1e-7;
// bf16x3 p = 4 2.3e-6, was 4.3e-6): fewer terms are summed per entry.
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

// The thread's index, opaque to the optimiser: what is computed from it in a phase
// of the loop over elements is not carried, in registers or scratch, through
// the others.
__device__ inline int phase_tid() {
    int t = threadIdx.x;
    asm volatile("" : "+v"(t));
    return t;
}

// An element's inputs as staged in LDS: vertices, then D, beta, c, f of the
// element or of its six vertices.
template <class Geo> struct PairInputs {
    static constexpr int MAX = 18 + 6 * 14;
    __device__ static int count(const FwdParams &prm) { return prm.fD ? MAX : 32; }
    __device__ static double fetch(const FwdParams &prm, int64_t e, int i) {
        if (i < 18) return prm.coords[18 * e + i];
        i -= 18;
        if (prm.fD)
            return i < 54 ? prm.fD[54 * e + i] : i < 72 ? prm.fbeta[18 * e + i - 54] : i < 78 ? prm.fc[6 * e + i - 72] : prm.ff[6 * e + i - 78];
        return i < 9 ? prm.D[9 * e + i] : i < 12 ? prm.beta[3 * e + i - 9] : i < 13 ? prm.c[e] : prm.f[e];
    }
    struct Coef { double D[9], be[3], c, f; };
    // W_q and w det J f at a point; returns det J.  The coefficients are read once
    // the vertices are done with (both at once cost 28 more registers).
    __device__ static double block(const FwdParams &prm, const double *in, const double *pt, double W[16], double &sf) {
        double X[18], K[9];
#pragma unroll
        for (int i = 0; i < 18; ++i) X[i] = in[i];
        const double det = prism_jacobian(X, pt[0], pt[1], pt[2], K);
        __builtin_amdgcn_sched_barrier(0);
        in += 18;
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
        fused_block(E, K, pt[3] * det, W, sf);
        return det;
    }
};
template <> struct PairInputs<PrismLaplaceGeo> {
    static constexpr int MAX = 18;
    __device__ static int count(const FwdParams &) { return 18; }
    __device__ static double fetch(const FwdParams &prm, int64_t e, int i) { return prm.coords[18 * e + i]; }
    __device__ static double block(const FwdParams &, const double *in, const double *pt, double W[16], double &sf) {
        double X[18], K[9];
#pragma unroll
        for (int i = 0; i < 18; ++i) X[i] = in[i];
        const double det = prism_jacobian(X, pt[0], pt[1], pt[2], K);
        laplace_block(K, pt[3] * det, W);
        sf = 0.0;
        return det;
    }
};

// EPB elements per workgroup of NW waves; a wave takes every WT-th tile of 16
// orbits and CT / (NW / WT) tiles of 16 columns; EPB = 1: KPP values of k per
// pass over the columns; KS values of k per round through the LDS copy of A;
// SC: the symmetric and the antisymmetric G one after the other in the same LDS.
template <int P, int FORM, int R, class Geo, int EPB, int NW, int WT, int KPP, int KS, bool SC = false>
struct KP {
    typedef PairForm<FORM> PF;
    typedef PairInputs<Geo> In;
    static constexpr int EPB_ = EPB, NW_ = NW;
    typedef typename PF::T T;
    typedef typename AccT<T>::type V4;
    typedef T V2 __attribute__((ext_vector_type(2)));
    static constexpr bool SPLIT = FORM == BF16X3 || FORM == FP16X3;
    static constexpr PairDims D = pair_dims(P, R);
    static constexpr int NK = D.nk, NT = D.nt, N = NT * NK, NIJ = D.nij, NQ = NIJ * NK;
    static constexpr int S = D.sets, NPAIR = D.npair;
    static constexpr int NTHR = NW * 64, GK = PF::GK;
    static constexpr int PASSES = c_cdiv(NK, KPP);
    static constexpr int NCOL = EPB * KPP * NK, CT = c_cdiv(NCOL, 16);
    static constexpr int WC = NW / WT, CTW = CT / WC;
    static constexpr int TPW = c_cdiv(pair_tiles(P, 0), WT);
    static constexpr int NE = 14;                             // rows of E: 13 entries of W and w det J f
    static constexpr int NS = N % 2 ? N : N + 1;              // row of the LDS copy of A: an odd stride spreads the banks
    static_assert(N == c_nshp(P) && CTW * WC == CT && NW % WT == 0, "pair kernel shape");
    static_assert(EPB == 1 || (PASSES == 1 && NK * NK <= 16 && EPB * NK <= 16), "several elements: one pass, a column tile each");
    static constexpr int kb(int cls) { return pair_kb(P, R, cls, GK); }
    static constexpr int mx(int a, int b) { return a > b ? a : b; }
    // LDS, in bytes: G of the symmetric and antisymmetric class, E, the load
    // vector's zeta sums; the copy of A lies over what is no longer read
    static constexpr int GB = 16 * (int)sizeof(T);            // bytes per contraction row and column tile
    // rows of a class in LDS: whole blocks, in FP64 half blocks
    static constexpr int gr(int cls) { return FORM == F64 ? (pair_k(P, R, cls) + 7) / 8 * 8 : kb(cls) * GK; }
    static constexpr int GS = CT * mx(gr(0), gr(2)) * GB, GA = CT * mx(gr(1), gr(3)) * GB;
    static constexpr int GALL = SC ? mx(GS, GA) : GS + GA;
    static constexpr int GAOFF = SC ? 0 : GS;
    static constexpr int EB = (EPB * 2 * NE * NK * S * (int)sizeof(T) + 15) / 16 * 16;
    static constexpr int HT = c_cdiv(S, 16);                  // blocks of 16 sets
    static constexpr int HB = Geo::LOAD ? 2 * HT * 256 * (int)sizeof(T) : 0;
    static constexpr int ST = EPB * KS * NT * NS * (int)sizeof(T);
    static constexpr int EOFF = PASSES == 1 ? GALL : mx(GALL, (ST + 15) / 16 * 16);
    static constexpr int HOFF = EOFF + EB;
    static constexpr int LDS = mx(HOFF + HB, ST);
    struct alignas(16) Smem {
        char raw[(LDS + 15) / 16 * 16];
        double in[EPB][In::MAX];
        uint32_t wmax[EPB];                                   // fp16: bits of the largest |E| of the element
    };

    // ---- inputs ------------------------------------------------------------------
    static constexpr int NF = c_cdiv(EPB * In::MAX, NTHR);    // values fetched per thread
    __device__ static void fetch(const FwdParams &prm, int64_t slot0, double (&v)[NF]) {
        const int tid = phase_tid();
        const int cnt = In::count(prm);
#pragma unroll
        for (int f = 0; f < NF; ++f) {
            const int x = tid + f * NTHR, el = EPB == 1 ? 0 : x / cnt;
            if (el < EPB && x < EPB * cnt && slot0 + el < prm.ne) v[f] = In::fetch(prm, elem_of(prm, slot0 + el), x - el * cnt);
        }
    }
    __device__ static void store_inputs(const FwdParams &prm, const double (&v)[NF], Smem &sm) {
        const int tid = phase_tid();
        const int cnt = In::count(prm);
#pragma unroll
        for (int f = 0; f < NF; ++f) {
            const int x = tid + f * NTHR, el = EPB == 1 ? 0 : x / cnt;
            if (el < EPB && x < EPB * cnt) sm.in[el][x - el * cnt] = v[f];
        }
    }

    // ---- 1: E ------------------------------------------------------------------
    // entries of E: 0o o3 3o, 0e e3 3e, 00 03 33, oo, ee, oe+eo, oe-eo, w det J f
    __device__ static void entries(const double W[16], double sf, double v[NE]) {
        // operators o = d1, e = d2 - d1/2: row o is W[1] + W[2]/2, likewise the columns
        const double r11 = W[5] + 0.5 * W[9], r12 = W[6] + 0.5 * W[10], e1 = W[9] + 0.5 * W[10];
        v[0] = W[1] + 0.5 * W[2]; v[1] = W[7] + 0.5 * W[11]; v[2] = W[13] + 0.5 * W[14];
        v[3] = W[2]; v[4] = W[11]; v[5] = W[14];
        v[6] = W[0]; v[7] = W[3]; v[8] = W[15];
        v[9] = r11 + 0.5 * r12; v[10] = W[10]; v[11] = r12 + e1; v[12] = r12 - e1;
        v[13] = sf;
    }
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
            const double *qp = prm.pqw + 4 * rest;
            const double pt[4] = {qp[0], qp[1], qp[2], qp[3]};
            double W[16], sf, v[NE];
            const double det = In::block(prm, sm.in[el], pt, W, sf);
            if (live && !(det > 0.0) && prm.status) atomicOr(prm.status, 1u);
            if (live && prm.xq) {
                const int64_t e = elem_of(prm, slot0 + el);
                const int q = m * NIJ + prm.ppts[2 * set + side];
                double x[3];
                prism_map(sm.in[el], pt[0], pt[1], pt[2], x);
#pragma unroll
                for (int c = 0; c < 3; ++c) prm.xq[(e * NQ + q) * 3 + c] = x[c];
            }
            entries(W, sf, v);
            // even classes (row 0, written by side 0) take the sums of the entries even under
            // the reflection and the differences of the odd ones, odd classes (row 1, side 1) the
            // others; a fixed point its entries
            const bool fixed = set >= NPAIR;
            T *row = E + ((el * 2 + side) * NE * NK + m) * S + set;
            float big = 0.0f;
#pragma unroll
            for (int x = 0; x < NE; ++x) {
                const double o = lane_swap(v[x]);
                const double y = fixed ? v[x] : side == 0 ? (odd_entry(x) ? v[x] - o : v[x] + o) : (odd_entry(x) ? o + v[x] : o - v[x]);
                if (FORM == FP16X3 && x < 13) big = fmaxf(big, fabsf((float)y));
                if (live) row[x * NK * S] = (T)y;
            }
            if (FORM == FP16X3 && live) atomicMax(&sm.wmax[el], __float_as_uint(big));
        }
    }

    // ---- 2: G ------------------------------------------------------------------
    // Contraction rows: types 0o 0e 00 oo ee oe (antisymmetric: 0o 0e oe), each over
    // every set, or over the pairs only where the type's parity is not the class's.
    static constexpr int rows_of(int par, int y) { return ((y == 0 || y == 5) == (par == 1)) ? S : NPAIR; }
    // G is kept in blocks of 16 rows as the zeta products leave them in registers:
    // lane (g, n), value v is row 4 v + g of column n, which is the second operand
    // of the products' step v (the split forms take two blocks per step).
    // At: offset of lane (g, column c) in a class's first block.
    __device__ static int column_at(int c, int rows) {
        const int g4 = (phase_tid() & 63) >> 4;
        return (c >> 4) * rows * 16 + (g4 * 16 + (c & 15)) * (SPLIT ? 8 : FORM == F64 ? 2 : 4);
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
            const V4 l = v - __builtin_convertvector(h, V4);
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
        return pow2_scale((double)__uint_as_float(sm.wmax[el]) * prm.pair_gz);
    }
    // Products of line factors of a column tile, as the second operand: lane (g, n)
    // holds zeta points 4 s + g of column n (zero past the last point).
    static constexpr int KZ = c_cdiv(NK, 4);
    static constexpr int CTE = EPB == 1 ? CT : 1;
    struct Lines { T ll[KZ], ld[KZ], dl[KZ], dd[KZ]; };
    __device__ static void load_lines(const FwdParams &prm, int col0, Lines &l) {
        const T *lam = sizeof(T) == 8 ? (const T *)(const void *)prm.lam : (const T *)(const void *)prm.lam32;
        const int lane = phase_tid() & 63, c = col0 + (lane & 15), cc = c < NK * NK ? c : 0, k = cc / NK, kp = cc - k * NK;
#pragma unroll
        for (int s = 0; s < KZ; ++s) {
            const int m = 4 * s + (lane >> 4), mm = m < NK ? m : 0;
            const T on = m < NK ? (T)1 : (T)0;
            const T a = on * lam[k * NK + mm], da = on * lam[(3 * NK + k) * NK + mm], b = lam[kp * NK + mm], db = lam[(3 * NK + kp) * NK + mm];
            l.ll[s] = a * b; l.ld[s] = a * db; l.dl[s] = da * b; l.dd[s] = da * db;
        }
    }
    __device__ static void lines(const FwdParams &prm, int k0, Lines (&l)[CTE]) {
#pragma unroll
        for (int j = 0; j < CTE; ++j) load_lines(prm, k0 * NK + j * 16, l[j]);
    }
    // A task is a tile of 16 contraction rows for every column tile of one element:
    // its rows of E are read once.
    template <int PAR, bool SYM, bool ANTI>
    __device__ static void zeta(const FwdParams &prm, int k0, const Lines (&l)[CTE], Smem &sm) {
        constexpr int C0 = 2 * PAR, C1 = 2 * PAR + 1;
        constexpr int N0 = rows_of(PAR, 0), N1 = N0 + rows_of(PAR, 1), N2 = N1 + rows_of(PAR, 2), N3 = N2 + rows_of(PAR, 3);
        constexpr int N4 = N3 + rows_of(PAR, 4), KS0 = pair_k(P, R, C0), KS1 = pair_k(P, R, C1);
        static_assert(KS0 == N4 + rows_of(PAR, 5) && KS1 == N1 + rows_of(PAR, 5), "contraction rows");
        // tiles of 16 rows: those of 0o and 0e alone serve both classes
        constexpr int BOTH = SYM && ANTI ? N1 / 16 : 0, TS = SYM ? c_cdiv(KS0, 16) : 0, TA = ANTI ? c_cdiv(KS1, 16) : 0;
        constexpr int TT = BOTH + (SYM ? TS - BOTH : 0) + (ANTI ? TA - BOTH : 0);
        char *gs = sm.raw, *ga = sm.raw + GAOFF;
        const int tid = phase_tid(), lane = tid & 63, i16 = lane & 15, g4 = lane >> 4;
        float sc = FORM == FP16X3 && EPB == 1 ? scale(prm, sm, 0) : 1.0f;
#pragma unroll 1
        for (int id = wave_uniform(tid >> 6); id < EPB * TT; id += NW) {
            const int el = EPB == 1 ? 0 : id / TT, task = id - el * TT;
            if (FORM == FP16X3 && EPB > 1) sc = scale(prm, sm, el);
            const bool sym = SYM && task < TS, anti = ANTI && (task < BOTH || !sym);
            const int tile = sym ? task : task - (SYM ? TS - BOTH : 0);
            // the row of this lane, its first entry x and its set
            const int last = sym ? KS0 - 1 : KS1 - 1, r0 = tile * 16 + 4 * (i16 & 3) + (i16 >> 2);
            int set = FORM == F64 ? tile * 16 + i16 : r0, x = 0;
            set = set < last ? set : last;
            if (set >= N0) { set -= N0; x = 3; }
            if (x == 3 && set >= N1 - N0) { set -= N1 - N0; x = sym ? 6 : 12; }
            if (SYM) {
                if (x == 6 && set >= N2 - N1) { set -= N2 - N1; x = 9; }
                if (x == 9 && set >= N3 - N2) { set -= N3 - N2; x = 10; }
                if (x == 10 && set >= N4 - N3) { set -= N4 - N3; x = 11; }
            }
            const T *E = (const T *)(sm.raw + EOFF) + ((el * 2 + PAR) * NE + x) * NK * S + set;
            auto at = [&](int d, int s) {
                const int m = 4 * s + g4;
                return E[(d * NK + (m < NK ? m : NK - 1)) * S];
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
                        a1[s] = x < 9 ? u : (T)0;
                        a2[s] = x < 9 ? w : (T)0;
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
                        for (int j = 0; j < CTE; ++j) w[j] = mfma4(ZX && x == 6 ? (T)0 : a2[s], l[j].dl[s], w[j]);
                    }
                    if (ZX) {
#pragma unroll
                        for (int j = 0; j < CTE; ++j) w[j] = mfma4(MX && x != 6 ? (T)0 : a2[s], l[j].dd[s], w[j]);
                    }
                }
#pragma unroll
                for (int j = 0; j < CTE; ++j) {
                    if (MX || ZX) p[j] += w[j];
                    const int c = EPB == 1 ? j * 16 + i16 : el * NK * NK + i16;
                    if (EPB == 1 || i16 < NK * NK) {
                        if (sym) put<C0>(gs, column_at(c, gr(C0)), tile, MX || ZX ? p[j] + q[j] : p[j], sc);
                        if (anti) put<C1>(ga, column_at(c, gr(C1)), tile, MX || ZX ? p[j] - q[j] : p[j], sc);
                    }
                }
            };
            if (!mixed && !zz) form(ic<0>{}, ic<0>{});
            else if (!zz) form(ic<1>{}, ic<0>{});
            else if (mixed) form(ic<1>{}, ic<1>{});
            else form(ic<0>{}, ic<1>{});
        }
        if (Geo::LOAD && SYM && k0 == 0) load_sums<PAR>(prm, sm);
    }

    // ---- load vector ------------------------------------------------------------
    // b[(k,t)] = sum over the sets of T(t) H(k), H = sum_m L_k w det J f, by halves
    // for the sum and the difference of a pair of points; both sums on the matrix
    // cores, the columns being k of every element.
    template <int PAR> __device__ static void load_sums(const FwdParams &prm, Smem &sm) {
        T *H = (T *)(sm.raw + HOFF);
        const T *lam = sizeof(T) == 8 ? (const T *)(const void *)prm.lam : (const T *)(const void *)prm.lam32;
        const int tid = phase_tid(), lane = tid & 63, i16 = lane & 15, g4 = lane >> 4;
#pragma unroll 1
        for (int id = NW - 1 - wave_uniform(tid >> 6); id < EPB * HT; id += NW) {
            const int el = id / HT, tile = id - el * HT, k = i16 < NK ? i16 : 0;
            const int row = tile * 16 + (FORM == F64 ? i16 : 4 * (i16 & 3) + (i16 >> 2)), set = row < S ? row : S - 1;
            const T *E = (const T *)(sm.raw + EOFF) + ((el * 2 + PAR) * NE + 13) * NK * S + set;
            V4 p = {0, 0, 0, 0};
#pragma unroll
            for (int s = 0; s < KZ; ++s) {
                const int m = 4 * s + g4, mm = m < NK ? m : 0;
                const T lk = m < NK ? lam[k * NK + mm] : (T)0;
                p = mfma4(E[mm * S], lk, p);
            }
            if (i16 < NK) {
                T *q = H + (PAR * HT + tile) * 256 + (g4 * 16 + el * NK + i16) * (FORM == F64 ? 2 : 4);
                if constexpr (FORM == F64) {
                    *(V2 *)q = V2{p[0], p[1]};
                    *(V2 *)(q + 128) = V2{p[2], p[3]};
                } else {
                    *(V4 *)q = p;
                }
            }
        }
    }
    __device__ static void load_vector(const FwdParams &prm, int64_t slot0, int wave, Smem &sm) {
        const T *H = (const T *)(sm.raw + HOFF);
        const T *bt = sizeof(T) == 8 ? (const T *)(const void *)prm.pbt64 : (const T *)(const void *)prm.pbt32;
        const int lane = phase_tid() & 63, i16 = lane & 15;
#pragma unroll 1
        for (int tile = NW - 1 - wave; tile < c_cdiv(NT, 16); tile += NW) {
            V4 v = {0, 0, 0, 0};
            const T *A = bt + tile * 2 * HT * 256;
#pragma unroll
            for (int b = 0; b < 2 * HT; ++b) {
                if constexpr (FORM == F64) {
#pragma unroll
                    for (int h = 0; h < 2; ++h) {
                        const V2 x = *(const V2 *)(A + (2 * b + h) * 128 + 2 * lane), y = *(const V2 *)(H + (2 * b + h) * 128 + 2 * lane);
                        v = mfma4(x[0], y[0], v);
                        v = mfma4(x[1], y[1], v);
                    }
                } else {
                    const V4 x = *(const V4 *)(A + b * 256 + 4 * lane), y = *(const V4 *)(H + b * 256 + 4 * lane);
#pragma unroll
                    for (int u = 0; u < 4; ++u) v = mfma4(x[u], y[u], v);
                }
            }
            const int el = i16 / NK, k = i16 - el * NK;
            if (el >= EPB || slot0 + el >= prm.ne) continue;
            T *bo = (T *)prm.b + offb_of(prm, elem_of(prm, slot0 + el), N) + k * NT;
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                const int t = tile * 16 + acc_row<T>(lane, r);
                if (t < NT) bo[t] = v[r];
            }
        }
    }

    // ---- 3: products ------------------------------------------------------------
    template <int CLS, int NA>
    __device__ static void product(const FwdParams &prm, const char *g, int wt, int ct0, V4 (&acc)[TPW][CTW]) {
        const int tid = phase_tid();
        constexpr int KB = kb(CLS);
        const int lane = tid & 63;
        if constexpr (!SPLIT) {
            // steps of VW x 4 rows; rows past the last step of the class are not taken
            constexpr int VW = FORM == F64 ? 2 : 4, KV = KB * 4 / VW, GV = gr(CLS) / (4 * VW), STEPS = c_cdiv(pair_k(P, R, CLS), 4 * VW);
            constexpr int TAIL = c_cdiv(pair_k(P, R, CLS) - (STEPS - 1) * 4 * VW, 4);      // steps in the last of them
            typedef T VT __attribute__((ext_vector_type(VW)));
            const VT *A = (const VT *)prm.pairA + (size_t)(pair_off(P, R, CLS, GK) * 4 / VW + wt * KV) * 64 + lane;
            const VT *B = (const VT *)g + ct0 * GV * 64 + lane;
            VT a[NA];
#pragma unroll
            for (int i = 0; i < NA; ++i) a[i] = A[i * WT * KV * 64];
            auto step = [&](int b8, int nv) {
                VT an[NA], b[CTW];
                const int nx = b8 + 1 < STEPS ? b8 + 1 : b8;
#pragma unroll
                for (int i = 0; i < NA; ++i) an[i] = A[(i * WT * KV + nx) * 64];
#pragma unroll
                for (int j = 0; j < CTW; ++j) b[j] = B[(j * GV + b8) * 64];
#pragma unroll
                for (int v = 0; v < VW; ++v)
                    if (v < nv) {
#pragma unroll
                        for (int i = 0; i < NA; ++i)
#pragma unroll
                            for (int j = 0; j < CTW; ++j) acc[i][j] = mfma4(a[i][v], b[j][v], acc[i][j]);
                    }
#pragma unroll
                for (int i = 0; i < NA; ++i) a[i] = an[i];
            };
#pragma unroll 2
            for (int b8 = 0; b8 + 1 < STEPS; ++b8) step(b8, VW);
            step(STEPS - 1, TAIL);
        } else {
            typedef typename SplitT<FORM>::vec HV;
            const HV *A = (const HV *)prm.pairA + (size_t)(pair_off(P, R, CLS, GK) + wt * KB) * 128 + lane;
            const HV *B = (const HV *)g + ct0 * KB * 64 + lane;
            HV ah[NA], al[NA];
#pragma unroll
            for (int i = 0; i < NA; ++i) { ah[i] = A[i * WT * KB * 128]; al[i] = A[i * WT * KB * 128 + 64]; }
#pragma unroll
            for (int b8 = 0; b8 < KB; ++b8) {
                HV nh[NA], nl[NA], bh[CTW], bl[CTW];
                const int nx = b8 + 1 < KB ? b8 + 1 : b8;
#pragma unroll
                for (int i = 0; i < NA; ++i) { nh[i] = A[(i * WT * KB + nx) * 128]; nl[i] = A[(i * WT * KB + nx) * 128 + 64]; }
#pragma unroll
                for (int j = 0; j < CTW; ++j) { bh[j] = B[(j * KB + b8) * 64]; bl[j] = B[(j * KB + b8 + CT * KB) * 64]; }
#pragma unroll
                for (int i = 0; i < NA; ++i)
#pragma unroll
                    for (int j = 0; j < CTW; ++j) acc[i][j] = mfma32(ah[i], bl[j], acc[i][j]);
#pragma unroll
                for (int i = 0; i < NA; ++i)
#pragma unroll
                    for (int j = 0; j < CTW; ++j) acc[i][j] = mfma32(al[i], bh[j], acc[i][j]);
#pragma unroll
                for (int i = 0; i < NA; ++i)
#pragma unroll
                    for (int j = 0; j < CTW; ++j) acc[i][j] = mfma32(ah[i], bh[j], acc[i][j]);
#pragma unroll
                for (int i = 0; i < NA; ++i) { ah[i] = nh[i]; al[i] = nl[i]; }
            }
        }
    }
    // The class's tiles of this wave are a prefix of its list.
    template <int CLS>
    __device__ static void products(const FwdParams &prm, const char *g, int wt, int ct0, V4 (&acc)[TPW][CTW]) {
        constexpr int TL = pair_tiles(P, CLS);
        static_for<1, TPW + 1>([&](auto n) {
            constexpr int NA = decltype(n)::value;
            // some wave has NA tiles: wt + (NA - 1) WT < TL <= wt + NA WT
            if constexpr ((NA - 1) * WT < TL && TL <= WT - 1 + NA * WT)
                if (wt + (NA - 1) * WT < TL && TL <= wt + NA * WT) product<CLS, NA>(prm, g, wt, ct0, acc);
        });
    }
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
        zeta<PAR, true, !SC>(prm, k0, l, sm);
        __syncthreads();
        zero(s);
        products<2 * PAR>(prm, sm.raw, wt, ct0, s);
        if (SC) {
            __syncthreads();
            zeta<PAR, false, true>(prm, k0, l, sm);
            __syncthreads();
        }
        zero(d);
        products<2 * PAR + 1>(prm, sm.raw + GAOFF, wt, ct0, d);
#pragma unroll
        for (int i = 0; i < TPW; ++i)
#pragma unroll
            for (int j = 0; j < CTW; ++j) {
                const V4 x = s[i][j], y = d[i][j];
                s[i][j] = x + y;
                d[i][j] = x - y;
            }
    }

    // ---- one group of elements ----------------------------------------------------
    // slot0's inputs are in sm.in; those of next0 are there at the end.
    __device__ static void group(const FwdParams &prm, int64_t slot0, int64_t next0, int wave, Smem &sm) {
        const int tid = phase_tid();
        const int lane = tid & 63;
        const int wt = wave % WT, ct0 = wave / WT * CTW;
        points(prm, slot0, sm);
        double nx[NF];
        if (next0 < prm.ne) fetch(prm, next0, nx);
        Lines l[CTE];
        if (PASSES == 1) lines(prm, 0, l);
        __syncthreads();
#pragma unroll 1
        for (int k0 = 0; k0 < NK; k0 += KPP) {
            V4 es[TPW][CTW], ed[TPW][CTW], os[TPW][CTW], od[TPW][CTW];
            if (PASSES > 1) lines(prm, k0, l);
            parity<0>(prm, k0, wt, ct0, es, ed, l, sm);
            if (k0 == 0) {
                if (next0 < prm.ne) store_inputs(prm, nx, sm);
            }
            __syncthreads();
            parity<1>(prm, k0, wt, ct0, os, od, l, sm);
            if (Geo::LOAD && k0 == 0) load_vector(prm, slot0, wave, sm);
            // the four entries of an orbit
#pragma unroll
            for (int i = 0; i < TPW; ++i)
#pragma unroll
                for (int j = 0; j < CTW; ++j) {
                    const V4 x = es[i][j], y = ed[i][j], z = os[i][j], w = od[i][j];
                    es[i][j] = x + z; os[i][j] = x - z;
                    ed[i][j] = y + w; od[i][j] = y - w;
                }
            __syncthreads();
            T *st = (T *)sm.raw;
            // (t, t', reflected t, reflected t') of the wave's orbits, a byte each
            uint32_t place[TPW][4];
#pragma unroll
            for (int i = 0; i < TPW; ++i)
#pragma unroll
                for (int r = 0; r < 4; ++r) place[i][r] = wt + i * WT < pair_tiles(P, 0) ? prm.potab[(wt + i * WT) * 16 + acc_row<T>(lane, r)] : 0u;
#pragma unroll 1
            for (int kr = 0; kr < KPP && k0 + kr < NK; kr += KS) {
                if (kr > 0) __syncthreads();
#pragma unroll
                for (int j = 0; j < CTW; ++j) {
                    const int c = (ct0 + j) * 16 + (lane & 15);
                    const int el = EPB == 1 ? 0 : c / (NK * NK), cc = c - el * NK * NK, kk = cc / NK;
                    if (EPB > 1 ? el >= EPB : kk >= KPP || k0 + kk >= NK) continue;      // no column
                    if (kk < kr || kk >= kr + KS) continue;                              // another round's
                    T *at = st + (EPB == 1 ? 0 : el * NT * NK * NS) + (kk - kr) * NT * NS + (cc - kk * NK) * NT;
                    const T un = FORM == FP16X3 ? (T)(ldexpf(1.0f, -prm.pair_shift) / scale(prm, sm, el)) : (T)1;
#pragma unroll
                    for (int i = 0; i < TPW; ++i) {
                        if (wt + i * WT >= pair_tiles(P, 0)) break;
#pragma unroll
                        for (int r = 0; r < 4; ++r) {
                            uint32_t o = place[i][r];
                            asm volatile("" : "+v"(o));      // the four addresses are formed here, not kept across the rounds
                            if ((wt + i * WT + 1) * 16 > pair_rows(P, 0) && o == 0xFFFFFFFFu) continue;
                            const int t = o & 0xFF, u = o >> 8 & 0xFF, rt = o >> 16 & 0xFF, ru = o >> 24;
                            at[__umul24(t, NS) + u] = FORM == FP16X3 ? es[i][j][r] * un : es[i][j][r];
                            at[__umul24(u, NS) + t] = FORM == FP16X3 ? ed[i][j][r] * un : ed[i][j][r];
                            at[__umul24(rt, NS) + ru] = FORM == FP16X3 ? os[i][j][r] * un : os[i][j][r];
                            at[__umul24(ru, NS) + rt] = FORM == FP16X3 ? od[i][j][r] * un : od[i][j][r];
                        }
                    }
                }
                __syncthreads();
                const int ks = NK - k0 - kr < KS ? NK - k0 - kr : KS;
                for (int el = 0; el < EPB && slot0 + el < prm.ne; ++el) {
                    T *Ao = (T *)prm.A + offA_of(prm, elem_of(prm, slot0 + el), N) + (size_t)(k0 + kr) * NT * N;
                    const T *src = st + el * NT * NK * NS;
                    const int cnt = ks * NT * N;
#pragma unroll 8
                    for (int x = tid; x < cnt; x += NTHR) Ao[x] = src[NS == N ? x : x + x / N];
                }
            }
            if (FORM == FP16X3 && k0 + KPP >= NK && tid < EPB) sm.wmax[tid] = 0;
            __syncthreads();
        }
    }
    // Groups first, first + step, ... of EPB slots.
    __device__ static void run(const FwdParams &prm, int64_t first, int64_t step, Smem &sm) {
        const int64_t groups = (prm.ne + EPB - 1) / EPB;
        if (first >= groups) return;
        if (FORM == FP16X3 && threadIdx.x < EPB) sm.wmax[threadIdx.x] = 0;
        double v[NF];
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

// Shapes per degree and form: elements per workgroup, waves, waves over the
// orbits, values of k per pass and per round, SC, waves per SIMD asked of the
// register allocator.
template <int P, int FORM> struct PairShape;
#define FEINT_PAIR_SHAPE(P, FORM, EPB_, NW_, WT_, KPP_, KS_, SC_, W_)                                   \
    template <> struct PairShape<P, FORM> {                                                              \
        static constexpr int EPB = EPB_, NW = NW_, WT = WT_, KPP = KPP_, KS = KS_, W = W_;                \
        static constexpr bool SC = SC_;                                                                  \
    };
FEINT_PAIR_SHAPE(3, F64, 4, 4, 2, 4, 4, false, 2)
FEINT_PAIR_SHAPE(4, F64, 1, 4, 4, 5, 5, false, 3)
FEINT_PAIR_SHAPE(5, F64, 1, 4, 4, 6, 3, true, 2)
FEINT_PAIR_SHAPE(6, F64, 1, 8, 8, 4, 1, false, 2)
FEINT_PAIR_SHAPE(7, F64, 1, 8, 8, 4, 1, false, 2)
FEINT_PAIR_SHAPE(3, F32, 4, 4, 2, 4, 4, false, 4)
FEINT_PAIR_SHAPE(4, F32, 1, 4, 4, 5, 5, false, 4)
FEINT_PAIR_SHAPE(5, F32, 1, 4, 4, 6, 3, false, 3)
FEINT_PAIR_SHAPE(6, F32, 1, 4, 4, 4, 2, false, 2)
FEINT_PAIR_SHAPE(7, F32, 1, 8, 8, 8, 2, false, 2)
FEINT_PAIR_SHAPE(2, BF16X3, 5, 3, 1, 3, 3, false, 4)
FEINT_PAIR_SHAPE(3, BF16X3, 4, 4, 2, 4, 4, false, 4)
FEINT_PAIR_SHAPE(4, BF16X3, 1, 4, 4, 5, 5, false, 4)
FEINT_PAIR_SHAPE(5, BF16X3, 1, 4, 4, 6, 3, false, 3)
FEINT_PAIR_SHAPE(6, BF16X3, 1, 4, 4, 4, 2, false, 2)
FEINT_PAIR_SHAPE(7, BF16X3, 1, 8, 8, 8, 2, false, 2)
template <int P> struct PairShape<P, FP16X3> : PairShape<P, BF16X3> {};

template <int P, int FORM, int R = 0, class Geo = PrismGeo, class S = PairShape<P, FORM>>
using KPOf = KP<P, FORM, R, Geo, S::EPB, S::NW, S::WT, S::KPP, S::KS, S::SC>;

template <class K, int NW, int MINW>
__global__ __launch_bounds__(NW * 64, MINW) void fwd_pair(FwdParams prm) {
    __shared__ typename K::Smem sm;
    K::run(prm, blockIdx.x, gridDim.x, sm);
}

}  // namespace feint
