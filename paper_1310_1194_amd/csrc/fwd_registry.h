// Launch helpers that instantiate the forward kernels for a list of tile
// shapes of one form.
#pragma once
#include <atomic>

#include "fwd_kernels.h"
#include "fwd_staged.h"
#include "fwd_valu.h"
#include "fwd_pipe.h"
#include "fwd_sc.h"
#include "fwd_fact.h"
#include "fwd_ymfma.h"
#include "fwd_hsf.h"
#include "fwd_tref.h"
#include "fwd_one.h"
#include "fwd_pair.h"

namespace feint {

template <class KER, int MINW>
void launch_direct(const FwdParams &prm, hipStream_t s) {
    const int64_t items = items_for<KER>(prm.ne);
    const int64_t blocks = (items + 3) / 4;
    hipLaunchKernelGGL((fwd_direct<KER, MINW>), dim3((unsigned)blocks), dim3(256), 0, s, prm);
}

template <class KER, int MINW>
void launch_coop(const FwdParams &prm, hipStream_t s) {
    const int64_t items = items_for<KER>(prm.ne);
    const int64_t blocks = (items + 3) / 4;
    hipLaunchKernelGGL((fwd_coop<KER, MINW>), dim3((unsigned)blocks), dim3(256), 0, s, prm);
}

template <class KER, int MINW>
void launch_staged(const FwdParams &prm, hipStream_t s) {
    const int64_t items = items_for<KER>(prm.ne);
    const int64_t blocks = (items + 3) / 4;
    hipLaunchKernelGGL((fwd_staged<KER, MINW>), dim3((unsigned)blocks), dim3(256), 0, s, prm);
}

template <class KER>
int64_t items_of(int64_t ne) { return items_for<KER>(ne); }

// U: unstaged (each wave reads the table through L2); S: LDS-staged.
// W: minimum waves per SIMD asked of the register allocator.  R: quadrature
// rule (0 = collapsed Gauss, 1 = symmetric triangle rule x Gauss in zeta);
// the forms without _R compile the collapsed rule.
#define FEINT_K4U_R(P, T, TM, TN, W, R) \
    FwdVariant{TM, TN, 0, W, &launch_direct<K4<P, T, TM, TN, R>, W>, &items_of<K4<P, T, TM, TN, R>>}
#define FEINT_K4S_R(P, T, TM, TN, SP, W, R) \
    FwdVariant{TM, TN, 1, W, &launch_staged<K4S<P, T, TM, TN, SP, R>, W>, &items_of<K4S<P, T, TM, TN, SP, R>>}
#define FEINT_K32U_R(P, F, TM, TN, W, R) \
    FwdVariant{TM, TN, 0, W, &launch_direct<K32<P, F, TM, TN, R>, W>, &items_of<K32<P, F, TM, TN, R>>}
// V: vector-ALU kernel, LPE lanes per element (tm = 0, tn = LPE, staged = 3).
#define FEINT_KV_R(P, T, LPE, W, R) \
    FwdVariant{0, LPE, 3, W, &launch_direct<KV<P, T, LPE, R>, W>, &items_of<KV<P, T, LPE, R>>}
// E: one element per lane, vector ALU (p = 1; tm = 0, tn = 1 lane per element, staged = 3); two
// waves per SIMD are not marked ("v1"): "v1o2" is M.
#define FEINT_KE_R(P, T, W, R) \
    FwdVariant{0, 1, 3, (W) == 2 ? 1 : (W), &launch_direct<KE<P, T, R>, W>, &items_of<KE<P, T, R>>}
#define FEINT_KE(P, T, W) FEINT_KE_R(P, T, W, 0)
// M: prisms of degree 1 from moments, two lanes per element ("v1o2").
#define FEINT_KM(T, W, R) FwdVariant{0, 1, 3, W, &launch_direct<KM<T, R>, W>, &items_of<KM<T, R>>}
// R: tetrahedra from reference matrices (staged = 11): one element per lane.
#define FEINT_KT(P, T, R, W) FwdVariant{R, 1, 11, W, &launch_direct<KT<P, T, R>, W>, &items_of<KT<P, T, R>>}
#define FEINT_KTS(P, T, W) FwdVariant{1, 2, 11, W, &launch_direct<KT<P, T, 1, true>, W>, &items_of<KT<P, T, 1, true>>}
#define FEINT_KTE(P, T, E, S, W) \
    FwdVariant{1, (S ? 2 : 1) + 4 * E, 11, W, &launch_direct<KT<P, T, 1, S, E>, W>, &items_of<KT<P, T, 1, S, E>>}
// L: staged stores of whole lines, E elements per wave ("ref2s")
#define FEINT_KTL(P, T, E, W) FwdVariant{2, 2 + 4 * E, 11, W, &launch_direct<KT<P, T, 1, 2, E>, W>, &items_of<KT<P, T, 1, 2, E>>}
// B: these for outputs past 256 MB, the staged kernel of 16 elements per wave for others.
// Whole lines pay where the matrices leave the last-level cache (256 MB) before their
// neighbours complete the lines that they share: p = 4 FP32, us, staged -> whole lines,
// 49 MB 29 -> 31, 490 MB 188 -> 135, 1.9 GB 726 -> 521; p = 3 FP32 160 MB 40 -> 53, 1.3 GB
// 474 -> 348; p = 4 FP64 98 MB 35 -> 43, 980 MB 343 -> 268.  Where n^2 values are whole
// lines (p = 5, 7) staged stores are as good or better at every size.
template <class SMALL, class LARGE, int MINW>
void launch_by_output(const FwdParams &prm, hipStream_t s) {
    if (prm.ne * LARGE::N2 * LARGE::VALUE > (int64_t)256 << 20) launch_direct<LARGE, MINW>(prm, s);
    else launch_direct<SMALL, MINW>(prm, s);
}
#define FEINT_KTB(P, T, E, W)                                                                                       \
    FwdVariant{2, 2 + 4 * E, 11, W, &launch_by_output<KT<P, T, 1, 1, 16>, KT<P, T, 1, 2, E>, W>, &items_of<KT<P, T, 1, 1, 16>>}
#define FEINT_KE_G(P, T, W, GEO) \
    FwdVariant{0, 1, 3, W, &launch_direct<KE<P, T, 0, GEO>, W>, &items_of<KE<P, T, 0, GEO>>}
// P: software-pipelined split kernel (staged = 4).
#define FEINT_K32P_R(P, F, TM, TN, W, R) \
    FwdVariant{TM, TN, 4, W, &launch_direct<K32P<P, F, TM, TN, R>, W>, &items_of<K32P<P, F, TM, TN, R>>}
#define FEINT_K32S_R(P, F, TM, TN, SY, W, R) \
    FwdVariant{TM, TN, 1 + !(SY), W, &launch_staged<K32S<P, F, TM, TN, SY, R>, W>, \
               &items_of<K32S<P, F, TM, TN, SY, R>>}

// Y: split kernel whose Y = W_q B_q is formed on the matrix cores (staged = 7).
// CH: 1 points in chunks of 64, 0 the element's points at once.
#define FEINT_K32Y_R(P, F, TM, TN, W, R, CH)                                                  \
    FwdVariant{TM, TN, 7, W, &launch_direct<K32Y<P, F, TM, TN, R, CH>, W>, \
               &items_of<K32Y<P, F, TM, TN, R, CH>>}
#define FEINT_K32Y(P, F, TM, TN, W, CH) FEINT_K32Y_R(P, F, TM, TN, W, 0, CH)

// C: shape functions computed at each point, no B table (staged = 5).
#define FEINT_KSC_R(P, T, TM, TN, W, R) \
    FwdVariant{TM, TN, 5, W, &launch_direct<KSC<P, T, TM, TN, R>, W>, &items_of<KSC<P, T, TM, TN, R>>}

// Hexahedra: the 16x16x4 kernel with the hexahedral geometry.
#define FEINT_K4U_HEX(P, T, TM, TN, W) \
    FwdVariant{TM, TN, 0, W, &launch_direct<K4<P, T, TM, TN, 0, HexGeo>, W>, &items_of<K4<P, T, TM, TN, 0, HexGeo>>}

// Tetrahedra: the 16x16x4 kernel with the affine tetrahedral geometry.
#define FEINT_K4U_TET(P, T, TM, TN, W) \
    FwdVariant{TM, TN, 0, W, &launch_direct<K4<P, T, TM, TN, 0, TetGeo>, W>, &items_of<K4<P, T, TM, TN, 0, TetGeo>>}

// Split forms on hexahedra and tetrahedra: the 16x16x32 kernel with their geometry.
#define FEINT_K32U_G(P, F, TM, TN, W, GEO) \
    FwdVariant{TM, TN, 0, W, &launch_direct<K32<P, F, TM, TN, 0, GEO>, W>, &items_of<K32<P, F, TM, TN, 0, GEO>>}

// Vector-ALU kernel on hexahedra and tetrahedra (low degree).
#define FEINT_KV_G(P, T, LPE, W, GEO) \
    FwdVariant{0, LPE, 3, W, &launch_direct<KV<P, T, LPE, 0, GEO>, W>, &items_of<KV<P, T, LPE, 0, GEO>>}

// F: contraction per triangle point (tensor factors of B, staged = 6):
// TMK row blocks k and TN column tiles per wave.
#define FEINT_KF_R(P, T, TMK, TN, W, R) \
    FwdVariant{TMK, TN, 6, W, &launch_direct<KF<P, T, TMK, TN, R>, W>, &items_of<KF<P, T, TMK, TN, R>>}
// the same, two waves per element sharing its point blocks through LDS (staged = 13)
#define FEINT_KF2_R(P, T, TMK, TN, W, R) \
    FwdVariant{TMK, TN, 13, W, &launch_coop<KF2<P, T, TMK, TN, R>, W>, &items_of<KF2<P, T, TMK, TN, R>>}
#define FEINT_KF2(P, T, TMK, TN, W) FEINT_KF2_R(P, T, TMK, TN, W, 0)
// the split forms of it with the zeta sums taken first and shared through LDS (staged = 15)
#define FEINT_KF2G_R(P, TMK, TN, W, R) \
    FwdVariant{TMK, TN, 15, W, &launch_coop<KF2G<P, TMK, TN, R>, W>, &items_of<KF2G<P, TMK, TN, R>>}
#define FEINT_KF2G(P, TMK, TN, W) FEINT_KF2G_R(P, TMK, TN, W, 0)
#define FEINT_KF2GH_R(P, TMK, TN, W, R)                                                            \
    FwdVariant{TMK, TN, 15, W, &launch_coop<KF2G<P, TMK, TN, R, PrismGeo, FP16X3>, W>,          \
               &items_of<KF2G<P, TMK, TN, R, PrismGeo, FP16X3>>}
#define FEINT_KF2GH(P, TMK, TN, W) FEINT_KF2GH_R(P, TMK, TN, W, 0)
// FP64 / FP32 with the zeta sums taken first (staged = 16)
#define FEINT_KF2Z_R(P, T, TMK, TN, IJB, W, R)                                                     \
    FwdVariant{TMK, TN, 16, W, &launch_coop<KF2Z<P, T, TMK, TN, IJB, R>, W>,                    \
               &items_of<KF2Z<P, T, TMK, TN, IJB, R>>}
#define FEINT_KF2Z(P, T, TMK, TN, IJB, W) FEINT_KF2Z_R(P, T, TMK, TN, IJB, W, 0)
#define FEINT_KF_HEX(P, T, TMK, TN, W)                                        \
    FwdVariant{TMK, TN, 6, W, &launch_direct<KF<P, T, TMK, TN, 0, HexGeo>, W>, \
               &items_of<KF<P, T, TMK, TN, 0, HexGeo>>}

// H: hexahedra by sum factorisation in all three directions (staged = 8): EPW
// elements per workgroup of NTH threads (tm = EPW, tn = NTH / 64 waves), W waves
// per SIMD asked of the register allocator; KHR forms W_q again in every pass of
// the slots (staged = 9).
#define FEINT_KH(P, T, NTH, EPW, W) \
    FwdVariant{EPW, (NTH) / 64, 8, W, &launch_hsf<P, T, NTH, EPW, false, W>, &items_hsf<EPW>}
#define FEINT_KHR(P, T, NTH, EPW, W) \
    FwdVariant{EPW, (NTH) / 64, 9, W, &launch_hsf<P, T, NTH, EPW, true, W>, &items_hsf<EPW>}
// KHL: W_q formed again per pass, and the last pass reading T2 from LDS where it
// is used (fewer registers: two waves per SIMD in FP64 at p >= 5; staged = 10)
#define FEINT_KHL(P, T, NTH, EPW, W) \
    FwdVariant{EPW, (NTH) / 64, 10, W, &launch_hsf<P, T, NTH, EPW, true, W, true>, &items_hsf<EPW>}

// PP: products of pairs of triangle functions (staged = 17)
// as many workgroups as the current device holds at once, each going on to further elements
// (asked once per device: the answer depends on the kernel and the device alone)
template <class K, int MINW>
int64_t pair_grid() {
    constexpr int DEVICES = 16;
    static std::atomic<int> known[DEVICES];
    int dev = 0, cus = 0, n = 0;
    if (hipGetDevice(&dev) != hipSuccess) return 1;
    if (dev < DEVICES)
        if (const int v = known[dev].load(std::memory_order_relaxed)) return v;
    if (hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess || cus < 1 ||
        hipOccupancyMaxActiveBlocksPerMultiprocessor(&n, fwd_pair<K, K::NW_, MINW>, K::NW_ * 64, 0) != hipSuccess || n < 1)
        return 1;                                      // the launch reports the error
    if (dev < DEVICES) known[dev].store(cus * n, std::memory_order_relaxed);
    return (int64_t)cus * n;
}
template <class K, int MINW>
void launch_pair(const FwdParams &prm, hipStream_t s) {
    const int64_t groups = (prm.ne + K::EPB_ - 1) / K::EPB_, most = pair_grid<K, MINW>();
    hipLaunchKernelGGL((fwd_pair<K, K::NW_, MINW>), dim3((unsigned)(groups < most ? groups : most)), dim3(K::NW_ * 64), 0, s, prm);
}
template <class K>
int64_t items_pair(int64_t ne) { return (ne + K::EPB_ - 1) / K::EPB_ * 4; }
#define FEINT_KPG(P, F, R, GEO)                                                                        \
    FwdVariant{PairShape<P, F>::EPB, PairShape<P, F>::NW, 17, PairShape<P, F>::W,                      \
               &launch_pair<KPOf<P, F, R, GEO>, PairShape<P, F>::W>, &items_pair<KPOf<P, F, R, GEO>>}
#define FEINT_KP(P, F) FEINT_KPG(P, F, 0, PrismGeo)

// Two kernels at p = 2 by the number of elements: FEW up to LINE of them (with
// coefficients at the vertices at any number, if FIELDS), MANY past it ("2x2so4":
// "2x2s", then "0x2fo4"; "v18o4": "0x2fo4", then "v18o2").  At p = 2 an
// element of the pair products passes six barriers for little work; a batch of a few
// elements per CU waits for them, and where the rule has few points the kernels that
// form W_q once per element and need no barrier are as fast at any size.  us, pair
// products against the other (200001 elements unless stated):
//   FP32 collapsed, lanes per element: 300 elements 10.8, 16.5, 16000 38, 39, 32000 69, 64, 408, 368; coefficients
//     at the vertices 12.3, 20.4, 45, 56, 83, 98, 500, 624.  Symmetric rule: 300 10.9, 11.2, 4000 14.8, 12.8, 379,
//     262; 12.0, 12.3, 17.9, 15.2, 480, 350: lanes per element at every size.
//   bf16x3 collapsed, staged products: 1000 11.2, 10.8, 2000 11.5, 11.5, 384, 633; vertices 13.4, 10.5, 13.7, 14.3, 478, 944;
//     symmetric 1000 11.0, 11.0, 4000 14.4, 13.6, 8000 20.2, 22.2, 370, 427; 13.3, 10.1, 17.5, 15.2, 25.8, 25.2, 471, 619.
//   fp16x3 collapsed: 1000 12.6, 10.7, 2000 12.9, 13.1, 448, 755; vertices 15.0, 12.9, 15.3, 17.0, 537, 1081;
//     symmetric 1000 12.2, 11.0, 2000 12.3, 11.7, 4000 16.1, 19.1, 424, 652; 14.6, 11.7, 14.8, 15.5, 18.7, 25.4, 517, 986.
template <auto FEW, auto MANY, int LINE, bool FIELDS>
void launch_by_count(const FwdParams &prm, hipStream_t s) {
    if (prm.ne <= LINE || (FIELDS && prm.fD)) FEW(prm, s);
    else MANY(prm, s);
}
#define FEINT_P2_F32                                                                                        \
    FwdVariant{0, 18, 3, 4, &launch_by_count<&launch_pair<KPOf<2, F32>, PairShape<2, F32>::W>,              \
                                             &launch_direct<KV<2, float, 18>, 2>, 16384, true>,             \
               &items_of<KV<2, float, 18>>}
#define FEINT_P2_SPLIT(F, R, LINE)                                                                          \
    FwdVariant{2, 2, 1, 4, &launch_by_count<&launch_staged<K32S<2, F, 2, 2, true, R>, 1>,                  \
                                             &launch_pair<KPOf<2, F, R>, PairShape<2, F>::W>, LINE, false>, \
               &items_of<K32S<2, F, 2, 2, true, R>>}

#define FEINT_K4U(P, T, TM, TN, W) FEINT_K4U_R(P, T, TM, TN, W, 0)
#define FEINT_KSC(P, T, TM, TN, W) FEINT_KSC_R(P, T, TM, TN, W, 0)
#define FEINT_K4S(P, T, TM, TN, SP, W) FEINT_K4S_R(P, T, TM, TN, SP, W, 0)
#define FEINT_K32U(P, F, TM, TN, W) FEINT_K32U_R(P, F, TM, TN, W, 0)
#define FEINT_KV(P, T, LPE, W) FEINT_KV_R(P, T, LPE, W, 0)
#define FEINT_K32P(P, F, TM, TN, W) FEINT_K32P_R(P, F, TM, TN, W, 0)
#define FEINT_K32S(P, F, TM, TN, SY, W) FEINT_K32S_R(P, F, TM, TN, SY, W, 0)

}  // namespace feint
