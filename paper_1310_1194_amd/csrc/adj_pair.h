// Adjoint on prisms, FP64, through the products of pairs of triangle functions
// (fwd_pair.h, pair_dims.h) run backwards:
//   1. dL/dA of 16 orbits at a time, for every column (k, k'): the sums and
//      differences of an orbit's four entries are the four classes' values; they
//      go to LDS as first operands, two chunks of orbits alternating.
//   2. per class, (columns x orbits) times the transposed table (orbits x
//      contraction rows, from L2): the zeta sums' gradients.  An element's waves
//      share the contraction rows and keep their tiles over all orbits, so G is
//      read once and the table once per element.
//   3. the accumulators are, lane for lane, the second operand of the zeta sums
//      run backwards (products of line factors x columns): the gradients of E,
//      into LDS over the spent chunks.
//   4. a point per lane: its W's gradient from the rows "even" and "odd" of E, then
//      the chain rule to the 32 inputs, summed over the element's waves.
// Collapsed rule, ms, best other kernel -> this one (131072, 65536, 16384, 8192,
// 4001 elements at p = 3..7): 2.73 -> 1.36, 6.05 -> 2.62, 5.67 -> 1.90, 7.90 -> 2.82,
// 8.73 -> 2.54; one element 0.039 -> 0.025 at p = 4, 0.17 -> 0.14 at p = 7.
// At p = 7 the matrix cores are busy 55 % of the cycles, and 12.4 GB pass L2 for the 2.66 GB
// of G: an orbit's entries (t, t') and (t', t) lie in different rows and 16 orbits take
// about four lines of 128 bytes for each they fill.  That is 4.9 TB/s, what a large copy
// reaches, so either may be the bound: passes over 32 or 16 columns at a time, whose
// rows of G stay in L2, took 2.77 and 3.62 ms against 2.65, but read the table again
// per pass.  The next chunk's table under way over the barrier gave 2.81 -> 2.56.  Orbits are ordered by patches of 8 x 4 (t, t'): 3.05
// ms row by row, 2.88 (4 x 4: 2.88, 8 x 8: 2.89, 16 x 16: 2.97).
// Against KFA2 the matrix work is 4.6x less at p = 7 (with 16-padded tiles of
// triangle functions, the unused three quarters of its second product) and no
// operand is combined from line factors on the vector ALU.
#pragma once
#include "fwd_kernels.h"
#include "pair_dims.h"

namespace feint {

// WPE waves per element (half of them on each parity), EPW elements per workgroup.
template <int P, int R, int WPE, int EPW>
struct AdjPair {
    typedef Adj<P, double, 1, 1, R> Chain;
    typedef f64x4 V4;
    typedef double V2 __attribute__((ext_vector_type(2)));
    static constexpr int WPE_ = WPE;
    static constexpr PairDims D = pair_dims(P, R);
    static constexpr int NK = D.nk, NT = D.nt, N = NT * NK, NIJ = D.nij, NQ = NIJ * NK, S = D.sets, NPAIR = D.npair;
    static constexpr int NW = WPE * EPW, NTHR = NW * 64, NTE = WPE * 64;
    static constexpr int CT = c_cdiv(NK * NK, 16);            // column tiles
    static constexpr int CHUNKS = pair_tiles(P, 0);
    static constexpr int WH = WPE / 2;                        // waves per parity
    static_assert(WPE % 2 == 0, "both parities");
    static constexpr int tiles(int cls) { return c_cdiv(pair_k(P, R, cls), 16); }
    static constexpr int mx(int a, int b) { return a > b ? a : b; }
    // tiles of a class per wave: dealt in turn over a parity's waves, symmetric first
    static constexpr int TSW = c_cdiv(mx(tiles(0), tiles(2)), WH), TAW = c_cdiv(mx(tiles(1), tiles(3)), WH);
    // line products are stacked TS to a tile of 16 rows (a type's NK zeta points each)
    static constexpr int TS = 16 / NK < 4 ? 16 / NK : 4, SETS_L = c_cdiv(4, TS);
    // gradients of E: 12 slots of a parity's symmetric class (0o 0e 00 by L L', L l', and l L' or
    // l l'; oo ee oe), 7 of the antisymmetric one
    static constexpr int SLOTS = 19;
    static constexpr int CHUNK = 4 * CT * 256;                // doubles: [class][column tile][half][64][2]
    static constexpr int EBUF = 2 * SLOTS * NK * S;
    static constexpr int AREA = mx(2 * CHUNK, EBUF);
    struct alignas(16) Smem {
        double a[EPW][AREA];
        double u[EPW][NIJ * NK];                              // sum_t g[k][t] T(t, ij)
        double red[NW][32];
    };

    // ---- 1 -----------------------------------------------------------------------
    static constexpr int PP = c_cdiv(16 * CT * 16, NTE);      // (orbit, column) pairs per thread
    __device__ static void fetch(const AdjParams &prm, const double *G, int ch, int t0, double (&v)[PP][4]) {
#pragma unroll
        for (int i = 0; i < PP; ++i) {
            const int x = t0 + i * NTE, o = x & 15, c = x >> 4, k = c / NK, kp = c - k * NK;
            const uint32_t w = prm.potab[ch * 16 + o];
            const bool on = c < NK * NK && w != 0xFFFFFFFFu;
            const int a = w & 0xFF, b = w >> 8 & 0xFF, ra = w >> 16 & 0xFF, rb = w >> 24;
            const double *g = G + (on ? k * NT * N + kp * NT : 0);
#pragma unroll
            for (int m = 0; m < 4; ++m) v[i][m] = 0.0;
            if (on) {
                v[i][0] = g[a * N + b]; v[i][1] = g[b * N + a];
                v[i][2] = g[ra * N + rb]; v[i][3] = g[rb * N + ra];
            }
        }
    }
    __device__ static void store(double *buf, int t0, const double (&v)[PP][4]) {
#pragma unroll
        for (int i = 0; i < PP; ++i) {
            const int x = t0 + i * NTE, o = x & 15, c = x >> 4;
            if ((16 * CT * 16) % NTE != 0 && c >= CT * 16) continue;
            double *q = buf + (c >> 4) * 256 + (o >> 3) * 128 + ((o & 3) * 16 + (c & 15)) * 2 + (o >> 2 & 1);
            const double s0 = v[i][0] + v[i][1], d0 = v[i][0] - v[i][1], s1 = v[i][2] + v[i][3], d1 = v[i][2] - v[i][3];
            q[0] = s0 + s1;
            q[CT * 256] = d0 + d1;
            q[2 * CT * 256] = s0 - s1;
            q[3 * CT * 256] = d0 - d1;
        }
    }

    // ---- 2 -----------------------------------------------------------------------
    // A chunk's table fragments for the wave's tiles of one class: tile j is class
    // tile first + j WH.
    template <int CLS, int NTL>
    __device__ static void table(const AdjParams &prm, int ch, int first, V2 (&b)[NTL][2]) {
        if (ch >= pair_tiles(P, CLS)) return;
        constexpr int TL = tiles(CLS), OB = pair_tiles(P, CLS) * 2;       // half chunks of the class
        constexpr int OFF = [] { int o = 0; for (int c = 0; c < CLS; ++c) o += tiles(c) * pair_tiles(P, c) * 2; return o; }();
        const V2 *B = (const V2 *)prm.padj + (size_t)(OFF + first * OB + 2 * ch) * 64 + (threadIdx.x & 63);
#pragma unroll
        for (int j = 0; j < NTL; ++j)
#pragma unroll
            for (int h = 0; h < 2; ++h)
                if (first + j * WH < TL) b[j][h] = B[(j * WH * OB + h) * 64];
    }
    template <int CLS, int NTL>
    __device__ static void product(const double *buf, int ch, int first, const V2 (&b)[NTL][2], V4 (&acc)[NTL][CT]) {
        if (ch >= pair_tiles(P, CLS)) return;
        constexpr int TL = tiles(CLS);
        const V2 *A = (const V2 *)(buf + CLS * CT * 256) + (threadIdx.x & 63);
#pragma unroll
        for (int h = 0; h < 2; ++h) {
            V2 a[CT];
#pragma unroll
            for (int c = 0; c < CT; ++c) a[c] = A[(c * 2 + h) * 64];
#pragma unroll
            for (int u = 0; u < 2; ++u)
#pragma unroll
                for (int j = 0; j < NTL; ++j)
                    if (first + j * WH < TL) {
#pragma unroll
                        for (int c = 0; c < CT; ++c) acc[j][c] = mfma4(a[c][u], b[j][h][u], acc[j][c]);
                    }
        }
    }

    // ---- 3 -----------------------------------------------------------------------
    static constexpr int rows_of(int par, int y) { return ((y == 0 || y == 5) == (par == 1)) ? S : NPAIR; }
    // The tiles' sums over the columns by products of line factors; every tile's before the
    // first is written (written tile by tile, p = 7 took 2.88 ms).
    template <int CLS, int NTL, int J0, int GT>
    __device__ static void backward(const AdjParams &prm, int first, const V4 (&acc)[NTL][CT], V4 (&p)[GT][SETS_L]) {
        constexpr int PAR = CLS / 2, ANTI = CLS & 1, TL = tiles(CLS);
        constexpr int N1 = rows_of(PAR, 0) + rows_of(PAR, 1), N2 = N1 + rows_of(PAR, 2);
        const double *lines = prm.plines + (threadIdx.x & 63);
#pragma unroll
        for (int j = 0; j < GT; ++j) {
            const int tile = first + (J0 + j) * WH;
            if (tile >= TL) continue;
            // rows of 0o, 0e or 00 among the tile's
            const bool mixed = tile * 16 < (ANTI ? N1 : N2);
#pragma unroll
            for (int c = 0; c < CT; ++c)
#pragma unroll
                for (int r = 0; r < 4; ++r) {
                    p[j][0] = mfma4(lines[(c * 4 + r) * 64], acc[J0 + j][c][r], p[j][0]);
                    if (mixed) {
#pragma unroll
                        for (int q = 1; q < SETS_L; ++q) p[j][q] = mfma4(lines[((q * CT + c) * 4 + r) * 64], acc[J0 + j][c][r], p[j][q]);
                    }
                }
        }
    }
    template <int CLS, int J0, int GT>
    __device__ static void gradients(double *Ebuf, int first, const V4 (&p)[GT][SETS_L]) {
        constexpr int PAR = CLS / 2, ANTI = CLS & 1, TL = tiles(CLS);
        constexpr int N0 = rows_of(PAR, 0), N1 = N0 + rows_of(PAR, 1), N2 = N1 + rows_of(PAR, 2), N3 = N2 + rows_of(PAR, 3);
        constexpr int N4 = N3 + rows_of(PAR, 4), K = pair_k(P, R, CLS);
        const int lane = threadIdx.x & 63, i16 = lane & 15;
#pragma unroll
        for (int j = 0; j < GT; ++j) {
            const int tile = first + (J0 + j) * WH;
            if (tile >= TL) continue;
            // the column's type y and set
            const int kap = tile * 16 + i16;
            int set = kap, y = 0;
            if (set >= N0) { set -= N0; y = 1; }
            if (y == 1 && set >= N1 - N0) { set -= N1 - N0; y = ANTI ? 5 : 2; }
            if (!ANTI) {
                if (y == 2 && set >= N2 - N1) { set -= N2 - N1; y = 3; }
                if (y == 3 && set >= N3 - N2) { set -= N3 - N2; y = 4; }
                if (y == 4 && set >= N4 - N3) { set -= N4 - N3; y = 5; }
            }
            const int slot = ANTI ? (y < 2 ? 12 + 3 * y : 18) : (y < 3 ? 3 * y : 6 + y);
            if (kap >= K) continue;
#pragma unroll
            for (int q = 0; q < SETS_L; ++q)
#pragma unroll
                for (int r = 0; r < 4; ++r) {
                    const int row = acc_row<double>(lane, r), d = q * TS + row / NK, m = row % NK;      // d: ll, ld, dl, dd
                    const bool on = row < TS * NK && (d == 0 || (d == 1 && y < 3) || (d == 2 && y < 2) || (d == 3 && y == 2));
                    if (on) Ebuf[((PAR * SLOTS + slot + (d == 0 ? 0 : d == 1 ? 1 : 2)) * NK + m) * S + set] = p[j][q][r];
                }
        }
    }

    template <int CLS, int NTL> __device__ static void sums(const AdjParams &prm, double *Ebuf, int first, const V4 (&acc)[NTL][CT]) {
        constexpr int GT = P <= 4 ? 1 : NTL;                  // tiles at a time: at p = 4 all of them spill
        static_for<0, NTL / GT>([&](auto gi) {
            constexpr int J0 = decltype(gi)::value * GT;
            V4 p[GT][SETS_L];
#pragma unroll
            for (int j = 0; j < GT; ++j)
#pragma unroll
                for (int q = 0; q < SETS_L; ++q) p[j][q] = V4{0, 0, 0, 0};
            backward<CLS, NTL, J0, GT>(prm, first, acc, p);
            gradients<CLS, J0, GT>(Ebuf, first, p);
        });
    }

    // ---- 4 -----------------------------------------------------------------------
    // Gradient with respect to the entries of one row of E (fwd_pair.h) of a parity.
    __device__ static void row(const double *e, int par, int set, double v[13]) {
        auto at = [&](int slot) { return e[slot * NK * S]; };
        const bool all = set < NPAIR;                         // a fixed point enters a parity's own types only
        const bool o = all || par == 1, z = all || par == 0;  // types 0o oe; 0e 00 oo ee
        v[0] = o ? at(0) + at(12) : 0.0;
        v[1] = o ? at(1) - at(13) : 0.0;
        v[2] = o ? at(2) + at(14) : 0.0;
        v[3] = z ? at(3) + at(15) : 0.0;
        v[4] = z ? at(4) - at(16) : 0.0;
        v[5] = z ? at(5) + at(17) : 0.0;
        v[6] = z ? at(6) : 0.0;
        v[7] = z ? at(7) : 0.0;
        v[8] = z ? at(8) : 0.0;
        v[9] = z ? at(9) : 0.0;
        v[10] = z ? at(10) : 0.0;
        v[11] = o ? at(11) : 0.0;
        v[12] = o ? at(18) : 0.0;
    }
    __device__ static bool odd_entry(int x) { return x <= 2 || x == 11 || x == 12; }

    __device__ static void zero(V4 (&s)[TSW][CT], V4 (&a)[TAW][CT]) {
#pragma unroll
        for (int c = 0; c < CT; ++c) {
#pragma unroll
            for (int j = 0; j < TSW; ++j) s[j][c] = V4{0, 0, 0, 0};
#pragma unroll
            for (int j = 0; j < TAW; ++j) a[j][c] = V4{0, 0, 0, 0};
        }
    }
    // The chunks of one parity's waves.
    template <int PAR>
    __device__ static void half(const AdjParams &prm, const double *G, int idx, int t0, bool live, double *buf) {
        V4 s[TSW][CT], a[TAW][CT];
        zero(s, a);
        constexpr int TSY = tiles(2 * PAR);
        const int fa = ((idx - TSY) % WH + WH) % WH;          // the antisymmetric tiles go on where the symmetric ones end
        double v[PP][4];
        if (live) fetch(prm, G, 0, t0, v);
        V2 bs[TSW][2], ba[TAW][2];
        if (live) {
            table<2 * PAR, TSW>(prm, 0, idx, bs);
            table<2 * PAR + 1, TAW>(prm, 0, fa, ba);
            store(buf, t0, v);
        }
        __syncthreads();
#pragma unroll 1
        for (int ch = 0; ch < CHUNKS; ++ch) {
            const double *now = buf + (ch & 1) * CHUNK;
            if (live) {
                if (ch + 1 < CHUNKS) fetch(prm, G, ch + 1, t0, v);
                product<2 * PAR, TSW>(now, ch, idx, bs, s);
                product<2 * PAR + 1, TAW>(now, ch, fa, ba, a);
                // the next chunk's table is under way over the barrier
                if (ch + 1 < CHUNKS) {
                    table<2 * PAR, TSW>(prm, ch + 1, idx, bs);
                    table<2 * PAR + 1, TAW>(prm, ch + 1, fa, ba);
                    store(buf + ((ch + 1) & 1) * CHUNK, t0, v);
                }
            }
            __syncthreads();
        }
        if (live) {
            sums<2 * PAR, TSW>(prm, buf, idx, s);
            sums<2 * PAR + 1, TAW>(prm, buf, fa, a);
        }
    }
    __device__ static void load_sums(const AdjParams &prm, int64_t e, int wv, double *u) {
        constexpr int TPD = c_pad16(NT);
        const int lane = threadIdx.x & 63, i16 = lane & 15, g4 = lane >> 4;
        const double *g = (const double *)prm.g + e * N;
        for (int tile = wv; tile < c_cdiv(NIJ, 16); tile += WPE) {
            const int ij = tile * 16 + i16 < NIJ ? tile * 16 + i16 : NIJ - 1, k = i16 < NK ? i16 : 0;
            const double *tau = (const double *)prm.tau + (size_t)ij * 4 * TPD;
            V4 p = {0, 0, 0, 0};
#pragma unroll
            for (int s = 0; s < c_cdiv(NT, 4); ++s) {
                const int t = 4 * s + g4, tt = t < NT ? t : 0;
                p = mfma4(t < NT ? tau[tt] : 0.0, t < NT ? g[k * NT + tt] : 0.0, p);
            }
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                const int row = tile * 16 + acc_row<double>(lane, r);
                if (row < NIJ && i16 < NK) u[row * NK + i16] = p[r];
            }
        }
    }
    __device__ static void run(const AdjParams &prm, int64_t first, Smem &sm) {
        const int wave = wave_uniform(threadIdx.x >> 6), lane = threadIdx.x & 63;
        const int el = wave / WPE, wv = wave - el * WPE, t0 = wv * 64 + lane;
        const bool live = first + el < prm.ne;
        const int64_t e = live ? first + el : first;
        const double *G = (const double *)prm.G + e * (int64_t)N * N;
        double *buf = sm.a[el];
        if (live) load_sums(prm, e, wv, sm.u[el]);
        // the waves of the two parities run different code with the same barriers
        if (wv / WH == 0) half<0>(prm, G, wv % WH, t0, live, buf);
        else half<1>(prm, G, wv % WH, t0, live, buf);
        __syncthreads();
        double gacc = 0.0;
        if (live) {
            ElemIn E;
            load_elem(prm.coords, prm.D, prm.beta, prm.c, prm.f, e, E);
            constexpr int TASKS = 2 * S * NK;
#pragma unroll 1
            for (int x0 = wv * 64; x0 < TASKS; x0 += NTE) {
                double gr[32];
#pragma unroll
                for (int k = 0; k < 32; ++k) gr[k] = 0.0;
                const int task = x0 + lane, m = task / (2 * S), set = (task - m * 2 * S) >> 1, side = task & 1;
                if (task < TASKS && !(set >= NPAIR && side)) {
                    double v[13], w[13];
                    row(buf + m * S + set, 0, set, v);
                    row(buf + (SLOTS * NK + m) * S + set, 1, set, w);
                    // the second point of a pair enters the differences with the other sign
#pragma unroll
                    for (int x = 0; x < 13; ++x) v[x] = side == 0 ? v[x] + w[x] : odd_entry(x) ? w[x] - v[x] : v[x] - w[x];
                    const double Sq[16] = {v[6], v[0], 0.5 * v[0] + v[3], v[7],
                                           0.0, v[9], 0.5 * v[9] + v[11] + v[12], v[1],
                                           0.0, 0.5 * v[9] + v[11] - v[12], 0.25 * v[9] + v[10] + v[11], 0.5 * v[1] + v[4],
                                           0.0, v[2], 0.5 * v[2] + v[5], v[8]};
                    const int ij = prm.ppts[2 * set + side];
                    double tau = 0.0;
#pragma unroll
                    for (int k = 0; k < NK; ++k) tau += ((const double *)prm.lamT)[k * NK + m] * sm.u[el][ij * NK + k];
                    Chain::template chain_rule<true>(prm, E, m * NIJ + ij, Sq, false, e, gr, tau);
                }
                gacc += Chain::reduce_scatter32(gr, lane);
            }
        }
        if ((lane & 1) == 0) sm.red[wave][lane >> 1] = gacc;
        __syncthreads();
        if (live && wv == 0 && lane < 32) {
            // component c: vertices 0..17, D 18..26, beta 27..29, c 30, f 31
            const int c = lane;
            double g = 0.0;
#pragma unroll
            for (int w = 0; w < WPE; ++w) g += sm.red[el * WPE + w][c];
            double *dst = c < 18 ? prm.dX + 18 * e + c
                        : c < 27 ? prm.dD + 9 * e + (c - 18)
                        : c < 30 ? prm.dbeta + 3 * e + (c - 27)
                        : c == 30 ? prm.dc + e : prm.df + e;
            *dst = g;
        }
    }
};

template <class K, int MINW>
__global__ __launch_bounds__(K::NTHR, MINW) void adj_pair(AdjParams prm) {
    __shared__ typename K::Smem sm;
    K::run(prm, (int64_t)blockIdx.x * (K::NW / K::WPE_), sm);
}

}  // namespace feint
