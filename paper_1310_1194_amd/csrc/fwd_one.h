// Forward integration of prisms of degree 1 from moments, two lanes per element, one for
// each zeta point.
//
// At p = 1 the triangle functions are the barycentric coordinates l_t, so that with
// the operators o = d/dxi1 and e = d/dxi2 - d/dxi1 / 2 (fwd_pair.h)
//   T_o(t) = (-1, 1, 0), T_e(t) = (-1/2, -1/2, 1) for every point:
// of W's entries only sums over the triangle's points are needed, of those that meet
// two derivatives as they are, one derivative times l_t, none times l_t l_t'.  Per
// zeta point 40 accumulators and as many multiply-adds per point instead of 222, and
// one combination with the line factors, added over the two lanes.  W_q itself takes
// its cofactors from two edge vectors and their cross product per zeta point and the
// third edge vector per triangle point.  (One lane for both zeta points spilled: the
// inputs stay live over the combination of the first.)
// The wave's matrices go through LDS, 16 bytes of 144-byte rows at a time (an odd
// number of them: no bank conflicts), and leave as one contiguous block.
// 524288 elements, us, one lane per element point by point -> this one: FP32 79 -> 59 (3.7
// TB/s), FP64 118 -> 78; coefficients per vertex 1430 -> 300, 834 -> 318; one element level.
// Two waves per SIMD: with three the registers spill (112 us).
#pragma once
#include "fwd_pair.h"

namespace feint {

template <typename T, int R>
struct KM {
    typedef PrismGeo G;
    static constexpr int N = 6, NIJ = pair_tri_points(1, R), NQ = 2 * NIJ;
    static constexpr int EPI = 32, NBLK = 1, VL = 16 / (int)sizeof(T), PIECES = N * N / VL;
    typedef T VT __attribute__((ext_vector_type(VL)));
    struct alignas(16) Smem { T a[4][EPI * N * N]; };

    __device__ static void run(const FwdParams &prm, int64_t group, int, int wave, Smem &sm) {
        const int lane = threadIdx.x & 63, m = lane & 1;
        const int64_t first = group * EPI, slot = first + (lane >> 1);
        const bool act = slot < prm.ne;
        const int64_t e = act ? elem_of(prm, slot) : 0;
        ElemIn E;
        G::load(prm, e, E);
        const double *qw = uniform_ptr(prm.qw), *lam = uniform_ptr(prm.lam);
        VT *mine = (VT *)(sm.a[wave] + (lane >> 1) * N * N);
        const double ze = m ? qw[4 * NIJ + 2] : qw[2], t = 0.5 * (1.0 + ze), s = 0.5 * (1.0 - ze);
        double a[3], b[3], cz[3], g[9];
#pragma unroll
        for (int d = 0; d < 3; ++d) {
            a[d] = s * (E.X[3 + d] - E.X[d]) + t * (E.X[12 + d] - E.X[9 + d]);
            b[d] = s * (E.X[6 + d] - E.X[d]) + t * (E.X[15 + d] - E.X[9 + d]);
            g[d] = 0.5 * (E.X[9 + d] - E.X[d]); g[3 + d] = 0.5 * (E.X[12 + d] - E.X[3 + d]); g[6 + d] = 0.5 * (E.X[15 + d] - E.X[6 + d]);
        }
        cz[0] = a[1] * b[2] - a[2] * b[1]; cz[1] = a[2] * b[0] - a[0] * b[2]; cz[2] = a[0] * b[1] - a[1] * b[0];
        // sums over the triangle's points: oo, ee, oe+eo, oe-eo; l_t times 0o 0e, o3 e3, 3o 3e;
        // l_t l_t' times 00, 03
        T f[4], m0[2][3], ms[2][3], m3[2][3], p[6], q[6], s33[6];
        double h[3];
#pragma unroll
        for (int i = 0; i < 4; ++i) f[i] = (T)0;
#pragma unroll
        for (int i = 0; i < 3; ++i) {
            m0[0][i] = m0[1][i] = ms[0][i] = ms[1][i] = m3[0][i] = m3[1][i] = (T)0;
            h[i] = 0.0;
        }
#pragma unroll
        for (int i = 0; i < 6; ++i) p[i] = q[i] = s33[i] = (T)0;
#pragma unroll 1
        for (int ij = 0; ij < NIJ; ++ij) {
            const double qp[4] = {qw[4 * ij], qw[4 * ij + 1], ze, m ? qw[4 * (NIJ + ij) + 3] : qw[4 * ij + 3]};
            G::coeffs(prm, e, qp, E);
            const double l[3] = {1.0 - qp[0] - qp[1], qp[0], qp[1]};
            double c[3], co[3], ce[3];
#pragma unroll
            for (int d = 0; d < 3; ++d)
                c[d] = l[0] * g[d] + l[1] * g[3 + d] + l[2] * g[6 + d];
            co[0] = b[1] * c[2] - b[2] * c[1]; co[1] = b[2] * c[0] - b[0] * c[2]; co[2] = b[0] * c[1] - b[1] * c[0];
            ce[0] = c[1] * a[2] - c[2] * a[1]; ce[1] = c[2] * a[0] - c[0] * a[2]; ce[2] = c[0] * a[1] - c[1] * a[0];
            const double det = c[0] * cz[0] + c[1] * cz[1] + c[2] * cz[2];
            if (act && !(det > 0.0) && prm.status) atomicOr(prm.status, 1u);
            if (act && prm.xq) {
                double x[3];
                prism_map(prm.coords + 18 * e, qp[0], qp[1], qp[2], x);
#pragma unroll
                for (int d = 0; d < 3; ++d) prm.xq[(e * NQ + m * NIJ + ij) * 3 + d] = x[d];
            }
#pragma unroll
            for (int d = 0; d < 3; ++d) co[d] += 0.5 * ce[d];
            double v[PAIR_ENTRIES];
            pair_entries(E, qp[3], det, co, ce, cz, v);
            f[0] += (T)v[9]; f[1] += (T)v[10]; f[2] += (T)v[11]; f[3] += (T)v[12];
            T lt[3];
#pragma unroll
            for (int i = 0; i < 3; ++i) {
                lt[i] = (T)l[i];
                m0[0][i] += lt[i] * (T)v[0]; m0[1][i] += lt[i] * (T)v[3];
                ms[0][i] += lt[i] * (T)v[1]; ms[1][i] += lt[i] * (T)v[4];
                m3[0][i] += lt[i] * (T)v[2]; m3[1][i] += lt[i] * (T)v[5];
                h[i] = __builtin_fma(l[i], v[13], h[i]);
            }
#pragma unroll
            for (int i = 0, k = 0; i < 3; ++i)
#pragma unroll
                for (int j = i; j < 3; ++j, ++k) {
                    const T ll = lt[i] * lt[j];
                    p[k] += ll * (T)v[6]; q[k] += ll * (T)v[7]; s33[k] += ll * (T)v[8];
                }
        }
        // A(k t, k' t') = sum over m of L_k L_k' P + L_k l_k' Q + l_k L_k' R + l_k l_k' S
        const T foe = (T)0.5 * (f[2] + f[3]), feo = (T)0.5 * (f[2] - f[3]);
        T A[N * N], L[2], dl[2];
        double bj[N];
#pragma unroll
        for (int k = 0; k < 2; ++k) {
            const double x = m ? lam[k * 2 + 1] : lam[k * 2];
            L[k] = (T)x;
            dl[k] = (T)(m ? lam[(6 + k) * 2 + 1] : lam[(6 + k) * 2]);
#pragma unroll
            for (int i = 0; i < 3; ++i) {
                bj[k * 3 + i] = x * h[i];
                bj[k * 3 + i] += lane_swap(bj[k * 3 + i]);
            }
        }
        constexpr T half = (T)0.5;
        auto oe = [](int t, T o, T e) { return t == 0 ? -o - half * e : t == 1 ? o - half * e : e; };      // T_o(t) o + T_e(t) e
#pragma unroll
        for (int i = 0; i < 3; ++i)
#pragma unroll
            for (int j = 0; j < 3; ++j) {
                const int k6 = i <= j ? (i == 0 ? j : i == 1 ? 2 + j : 5) : (j == 0 ? i : j == 1 ? 2 + i : 5);
                const T P = p[k6] + oe(j, m0[0][i], m0[1][i]) + oe(i, oe(j, f[0], foe), oe(j, feo, f[1]));
                const T Q = q[k6] + oe(i, ms[0][j], ms[1][j]), Rr = oe(j, m3[0][i], m3[1][i]);
#pragma unroll
                for (int k = 0; k < 2; ++k)
#pragma unroll
                    for (int kp = 0; kp < 2; ++kp) {
                        const T x = L[k] * L[kp] * P + L[k] * dl[kp] * Q + dl[k] * L[kp] * Rr + dl[k] * dl[kp] * s33[k6];
                        A[(k * 3 + i) * N + kp * 3 + j] = x + lane_swap(x);
                    }
            }
        // each lane of the pair stores every other piece
#pragma unroll
        for (int x = 0; x < PIECES; ++x) {
            VT w;
#pragma unroll
            for (int i = 0; i < VL; ++i) w[i] = A[x * VL + i];
            if ((x & 1) == m) mine[x] = w;
        }
        const int nact = (int)(prm.ne - first < EPI ? prm.ne - first : EPI);
        T *Ao = (T *)prm.A + first * (N * N);
        if (!prm.perm && !prm.offA && (uintptr_t)Ao % 16 == 0) {
            wave_sync();
            const VT *src = (const VT *)sm.a[wave];
            for (int x = lane; x < nact * PIECES; x += 64) ((VT *)Ao)[x] = src[x];
        } else if (act) {
            wave_sync();
            Ao = (T *)prm.A + offA_of(prm, e, N);
#pragma unroll
            for (int x = 0; x < PIECES; ++x) {
                const VT w = mine[x];
                if ((x & 1) == m)
#pragma unroll
                    for (int i = 0; i < VL; ++i) Ao[x * VL + i] = w[i];
            }
        }
        if (act) {
            T *bout = (T *)prm.b + offb_of(prm, e, N);
#pragma unroll
            for (int i = 0; i < 3; ++i) bout[m * 3 + i] = (T)(m ? bj[3 + i] : bj[i]);
        }
    }
};

}  // namespace feint
