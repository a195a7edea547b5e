// Global assembly of element matrices and load vectors into a CSR matrix
// (Sec. 2: the global matrix is the sum of the element matrices placed
// through the element-to-global numbering; elements of one colour share no
// global entry, so a colour is assembled without atomics).
//
// Set-up, once per mesh, on the host (threads over rows / elements):
//   * node -> element incidence from the caller's dof map,
//   * the CSR pattern: row i holds every dof that shares an element with i,
//     columns ascending,
//   * the position map: for entry (a, b) of element e, the offset of column
//     dofs[e][b] inside row dofs[e][a] (uint16: a row of a degree-p prism mesh
//     holds at most (2p+1)^3 <= 3375 columns),
//   * a greedy colouring: each element takes the smallest colour not used by
//     an element sharing one of its dofs,
//   * every dof's rows of element matrices, in the order of their elements' colours.
// Per assembly, on the device, one launch over the rows of the global matrix:
// G lanes clear (or read, when accumulating) a row in LDS, add the element rows
// one after the other, values[row_ptr[dofs[e][a]] + pos[e][a][b]] += A_e[a][b],
// and write the row; rhs[dofs[e][a]] += b_e[a] likewise.  The order of the sums is
// that of the colours: no atomics, the same bits in every run.
// Near the memory's rate: 32768 elements at p = 3 in FP64 take 0.275 ms, in which 0.77 GB are
// read and 0.32 written past L2 (3.9 TB/s; a large copy 4.7), where A, pos and the lists are 0.53
// GB: element rows of 320 bytes, and of 80 in pos, touch 2.5 to 3.5 lines of 128 that other
// workgroups' rows share.  Rows of more values than LDS holds (1024; 512 at p = 2, 128 at p =
// 1) are taken in pieces, side by side, that each read the row's element rows.  A launch per
// colour, one wave per element, read and wrote each value once per colour that
// meets it and took 13 to 16 launches and two fills: 0.67 ms; 512 elements 0.23 and here
// 0.009; p = 7, 512 elements, 15.2 and 0.24.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <atomic>
#include <cstdio>
#include <cstring>
#include <thread>
#include <vector>

#include "capi_internal.h"
#include "device_common.h"
#include "tables.h"

struct feint_asm_plan {
    int dev = 0;
    int64_t ne = 0, ndof = 0, nnz = 0;
    int n = 0, ncolors = 0, max_row = 0;
    std::vector<int32_t> color_of;        // host: colour of every element
    // device buffers (one allocation)
    void *base = nullptr;
    int64_t *row_ptr = nullptr;   // [ndof + 1]
    int32_t *col_idx = nullptr;   // [nnz]
    int64_t *inc_ptr = nullptr;   // [ndof + 1]
    void *inc = nullptr;          // [ne * n] rows e * n + a of the element matrices, dof by dof: uint32, or int64 if wide
    bool wide = false;
    int64_t *more = nullptr;      // [nmore] pieces of long rows past the first (row, piece << 32)
    int64_t nmore = 0;
    uint16_t *pos = nullptr;      // [ne][n][n]
};

namespace feint {
namespace {

template <typename F>
void parallel_for(int64_t n, F fn) {
    unsigned nt = std::thread::hardware_concurrency();
    nt = nt == 0 ? 4 : (nt > 64 ? 64 : nt);
    if (n < 4096) nt = 1;
    std::vector<std::thread> th;
    for (unsigned t = 0; t < nt; ++t)
        th.emplace_back([&, t]() {
            const int64_t lo = n * t / nt, hi = n * (t + 1) / nt;
            fn(lo, hi, t);
        });
    for (auto &x : th) x.join();
}

// Values of a row of the global matrix in LDS at a time, by the lanes that take it: 8 KB per
// wave at most (FP64).
constexpr int asm_lanes(int n) { return n <= 8 ? 8 : n <= 32 ? 32 : 64; }
constexpr int asm_cap(int n) { return 16 * asm_lanes(n); }

// G lanes take R rows of the global matrix, one after the other, the first cap values of
// each; longer rows have their further pieces of cap values in `more` (row, piece << 32), each
// taken by G lanes of its own (the first blocks).  CH steps of G lanes cover a row of an
// element matrix.  The R rows' element rows are one list: U of it are fetched while U are
// added, also across the ends of rows, so that no row waits for its own first loads.
// (A dof of many elements: the pieces taken one after the other by the same lanes were 157 ms
// for a fan of 4000 elements at p = 1, where a launch per colour took 15; here 1.3.)
template <typename T, typename I, int G, int CH, int U, int R>
__global__ __launch_bounds__(256) void assemble_rows(const T *__restrict__ A, const T *__restrict__ b,
                                                     const int64_t *__restrict__ inc_ptr, const I *__restrict__ inc,
                                                     const int64_t *__restrict__ row_ptr, const uint16_t *__restrict__ pos,
                                                     const int64_t *__restrict__ more, int64_t nmore, int n, int64_t ndof,
                                                     int cap, int accumulate, T *values, T *rhs) {
    static_assert(R < G, "a lane per row and the end of the last");
    constexpr int GROUPS = 256 / G;
    extern __shared__ __align__(16) char lds[];
    const int lane = threadIdx.x % G, grp = threadIdx.x / G;
    T *row = (T *)lds + grp * cap;
    const int64_t pieces = (nmore + GROUPS - 1) / GROUPS;             // blocks
    int64_t i0;
    int c0 = 0, nr = 1;
    if (blockIdx.x < pieces) {
        i0 = (int64_t)blockIdx.x * GROUPS + grp;
        if (i0 >= nmore) return;
        const int64_t x = more[i0];
        c0 = (int)(x >> 32) * cap;
        i0 = x & 0xFFFFFFFF;
    } else {
        i0 = ((blockIdx.x - pieces) * GROUPS + grp) * R;
        if (i0 >= ndof) return;
        nr = ndof - i0 < R ? (int)(ndof - i0) : R;
    }
    // lane r: where row r begins in the list and in the values
    const int64_t ip = inc_ptr[i0 + (lane < nr ? lane : nr)], rp = row_ptr[i0 + (lane < nr ? lane : nr)];
    const int64_t k0 = __shfl(ip, 0, G), v0 = __shfl(rp, 0, G);
    const int st = (int)(ip - k0), en = __shfl(st, lane < nr ? lane + 1 : nr, G), total = __shfl(st, nr, G);
    const int at0 = (int)(rp - v0);
    T sum = accumulate && c0 == 0 && lane < nr ? rhs[i0 + lane] : (T)0;
    int r = -1, end = 0, m = 0;                               // the row at hand, its end in the list, its values in LDS
    T *out = values;
    auto close = [&] {
        wave_sync();
        for (int j = lane; j < m; j += G) out[j] = row[j];
    };
    auto open = [&] {
        ++r;
        end = __shfl(st, r + 1, G);
        const int a = __shfl(at0, r, G), len = __shfl(at0, r + 1, G) - a - c0;
        m = len < cap ? len : cap;
        out = values + v0 + a + c0;
        wave_sync();
        for (int j = lane; j < m; j += G) row[j] = accumulate ? out[j] : (T)0;
        wave_sync();
    };
    for (int xb = 0; xb < total; xb += G) {
        const int xn = total - xb < G ? total - xb : G;
        const int64_t mine = lane < xn ? (int64_t)inc[k0 + xb + lane] : 0;
        const T bm = c0 == 0 && lane < xn ? b[mine] : (T)0;
        struct Rows { T v[U][CH]; int at[U][CH]; } cur, nxt;
        auto fetch = [&](int x, Rows &f) {
#pragma unroll
            for (int u = 0; u < U; ++u) {
                const int64_t e = __shfl(mine, x + u < xn ? x + u : 0, G) * n;
#pragma unroll
                for (int h = 0; h < CH; ++h) {
                    const int j = h * G + lane;
                    const bool on = x + u < xn && j < n;
                    f.v[u][h] = on ? A[e + j] : (T)0;
                    f.at[u][h] = on ? pos[e + j] - c0 : -1;
                }
            }
        };
        fetch(0, cur);
        for (int x = 0; x < xn; x += U) {
            fetch(x + U, nxt);
#pragma unroll
            for (int u = 0; u < U; ++u) {
                if (x + u >= xn) break;
                while (xb + x + u == end) {
                    close();
                    open();
                }
#pragma unroll
                for (int h = 0; h < CH; ++h)
                    if ((unsigned)cur.at[u][h] < (unsigned)m) row[cur.at[u][h]] += cur.v[u][h];
                wave_sync();                                  // the next element's lanes meet other columns
            }
            cur = nxt;
        }
        if (c0 == 0)
            for (int x = 0; x < xn; ++x) {
                const T v = __shfl(bm, x, G);
                if (xb + x >= st && xb + x < en) sum += v;
            }
    }
    close();
    if (c0 == 0 && lane < nr && (en > st || !accumulate)) rhs[i0 + lane] = sum;
}

template <typename T, typename I, int G, int CH, int U, int R>
void launch_rows(const feint_asm_plan *pl, const void *A, const void *b, void *values, void *rhs, int accumulate, hipStream_t st) {
    constexpr int CAP = 16 * G, GROUPS = 256 / G;
    const int cap = pl->max_row < CAP ? pl->max_row : CAP;
    const int64_t blocks = (pl->ndof + GROUPS * R - 1) / (GROUPS * R) + (pl->nmore + GROUPS - 1) / GROUPS;
    hipLaunchKernelGGL((assemble_rows<T, I, G, CH, U, R>), dim3((unsigned)blocks), dim3(256), GROUPS * cap * sizeof(T), st,
                       (const T *)A, (const T *)b, pl->inc_ptr, (const I *)pl->inc, pl->row_ptr, pl->pos, pl->more, pl->nmore, pl->n,
                       pl->ndof, cap, accumulate, (T *)values, (T *)rhs);
}
// Lanes per row: the fewest of a power of two that hold a row of the element matrix, a
// wave from p = 3 on; loads in flight per lane about four.  Waves take four rows where
// these fill the device (1024 SIMDs of several waves), as the rows' first loads then
// overlap; fewer rows need the waves.  us with one row, with four, FP64, by dofs: p = 3 8125
// 9, 15, 34225 26, 30, 60025 42, 37, 117649 77, 62; p = 4 35937 35, 37, 55473 47, 45, 79233 63,
// 57; p = 5 35301 49, 41, 68921 116, 95; p = 6 60025 149, 131, 117649 289, 242; p = 7 24389 56,
// 68, 94221 289, 240.  FP32 alike to p = 5; p = 6 60025 56, 60, 117649 146, 138; p = 7 94221
// 152, 152, 287337 460, 401.
template <typename T, typename I>
void launch_rows(const feint_asm_plan *pl, const void *A, const void *b, void *values, void *rhs, int accumulate, hipStream_t st) {
    const bool few = pl->ndof < 65536;
    auto f = pl->n <= 8 ? launch_rows<T, I, 8, 1, 4, 1> : pl->n <= 32 ? launch_rows<T, I, 32, 1, 4, 2>
           : pl->n <= 64 ? (few ? launch_rows<T, I, 64, 1, 4, 1> : launch_rows<T, I, 64, 1, 4, 4>)
           : pl->n <= 128 ? (few ? launch_rows<T, I, 64, 2, 2, 1> : launch_rows<T, I, 64, 2, 2, 4>)
           : pl->n <= 256 ? (few ? launch_rows<T, I, 64, 4, 1, 1> : launch_rows<T, I, 64, 4, 1, 4>)
                          : (few ? launch_rows<T, I, 64, 5, 1, 1> : launch_rows<T, I, 64, 5, 1, 4>);
    static_assert(c_nshp(7) <= 5 * 64, "row of an element matrix");
    f(pl, A, b, values, rhs, accumulate, st);
}
template <typename T>
void launch_rows(const feint_asm_plan *pl, const void *A, const void *b, void *values, void *rhs, int accumulate, hipStream_t st) {
    if (pl->wide) launch_rows<T, int64_t>(pl, A, b, values, rhs, accumulate, st);
    else launch_rows<T, uint32_t>(pl, A, b, values, rhs, accumulate, st);
}

}  // namespace
}  // namespace feint

using namespace feint;

extern "C" {

feint_status feint_asm_plan_create(const int32_t *dofs, int64_t ne, int n, int64_t ndof, feint_asm_plan **out) {
    if (!out) return FEINT_ERR_INVALID_ARG;
    *out = nullptr;
    if (!dofs || ne <= 0 || ndof <= 0 || ndof >= (1LL << 31)) return FEINT_ERR_INVALID_ARG;
    bool known = false;
    for (int p = 1; p <= kMaxP; ++p) known |= c_nshp(p) == n;
    if (!known) return FEINT_ERR_INVALID_ARG;
    for (int64_t i = 0; i < ne * n; ++i)
        if (dofs[i] < 0 || dofs[i] >= ndof) return FEINT_ERR_INVALID_ARG;

    // node -> element incidence
    std::vector<int64_t> inc_ptr(ndof + 1, 0);
    for (int64_t i = 0; i < ne * n; ++i) inc_ptr[dofs[i] + 1]++;
    for (int64_t i = 0; i < ndof; ++i) inc_ptr[i + 1] += inc_ptr[i];
    std::vector<int32_t> inc(inc_ptr[ndof]);
    {
        std::vector<int64_t> fill(inc_ptr.begin(), inc_ptr.end() - 1);
        for (int64_t e = 0; e < ne; ++e)
            for (int a = 0; a < n; ++a) inc[fill[dofs[e * n + a]]++] = (int32_t)e;
    }

    // CSR pattern: row lengths, then the sorted columns
    std::vector<int64_t> row_ptr(ndof + 1, 0);
    std::atomic<bool> twice{false};         // a dof listed twice in one element is a bad map
    parallel_for(ndof, [&](int64_t lo, int64_t hi, unsigned) {
        std::vector<int32_t> seen;
        for (int64_t i = lo; i < hi; ++i) {
            seen.clear();
            for (int64_t k = inc_ptr[i]; k < inc_ptr[i + 1]; ++k) {
                if (k > inc_ptr[i] && inc[k] == inc[k - 1]) twice = true;
                const int32_t *de = dofs + (int64_t)inc[k] * n;
                seen.insert(seen.end(), de, de + n);
            }
            std::sort(seen.begin(), seen.end());
            row_ptr[i + 1] = std::unique(seen.begin(), seen.end()) - seen.begin();
        }
    });
    if (twice) return FEINT_ERR_INVALID_ARG;
    for (int64_t i = 0; i < ndof; ++i) {
        if (row_ptr[i + 1] > 65535) return FEINT_ERR_TOO_LARGE;
        row_ptr[i + 1] += row_ptr[i];
    }
    const int64_t nnz = row_ptr[ndof];
    std::vector<int32_t> col_idx(nnz);
    parallel_for(ndof, [&](int64_t lo, int64_t hi, unsigned) {
        std::vector<int32_t> seen;
        for (int64_t i = lo; i < hi; ++i) {
            seen.clear();
            for (int64_t k = inc_ptr[i]; k < inc_ptr[i + 1]; ++k) {
                const int32_t *de = dofs + (int64_t)inc[k] * n;
                seen.insert(seen.end(), de, de + n);
            }
            std::sort(seen.begin(), seen.end());
            const auto end = std::unique(seen.begin(), seen.end());
            std::copy(seen.begin(), end, col_idx.begin() + row_ptr[i]);
        }
    });

    // position map
    const int64_t nn = (int64_t)n * n;
    std::vector<uint16_t> pos(ne * nn);
    parallel_for(ne, [&](int64_t lo, int64_t hi, unsigned) {
        for (int64_t e = lo; e < hi; ++e)
            for (int a = 0; a < n; ++a) {
                const int32_t *c0 = col_idx.data() + row_ptr[dofs[e * n + a]];
                const int32_t *c1 = col_idx.data() + row_ptr[dofs[e * n + a] + 1];
                for (int b = 0; b < n; ++b)
                    pos[e * nn + (int64_t)a * n + b] = (uint16_t)(std::lower_bound(c0, c1, dofs[e * n + b]) - c0);
            }
    });

    // greedy colouring in element order
    std::vector<int32_t> color(ne, -1);
    std::vector<int64_t> used;          // used[c] == e: colour c taken by a neighbour of e
    int ncolors = 0;
    for (int64_t e = 0; e < ne; ++e) {
        for (int a = 0; a < n; ++a) {
            const int32_t g = dofs[e * n + a];
            for (int64_t k = inc_ptr[g]; k < inc_ptr[g + 1]; ++k) {
                const int32_t c = color[inc[k]];
                if (c >= 0) used[c] = e;
            }
        }
        int c = 0;
        while (c < ncolors && used[c] == e) ++c;
        if (c == ncolors) { ++ncolors; used.push_back(-1); }
        color[e] = c;
    }
    // every dof's element rows, by colour: in the place of its elements where 32 bits hold them
    const bool wide = ne * n > (int64_t)UINT32_MAX;
    std::vector<int64_t> rows(wide ? ne * n : 0);
    parallel_for(ndof, [&](int64_t lo, int64_t hi, unsigned) {
        std::vector<std::pair<int32_t, int32_t>> list;
        for (int64_t i = lo; i < hi; ++i) {
            list.clear();
            for (int64_t k = inc_ptr[i]; k < inc_ptr[i + 1]; ++k) list.push_back({color[inc[k]], inc[k]});
            std::sort(list.begin(), list.end());
            int64_t k = inc_ptr[i];
            for (const auto &x : list) {
                const int32_t *de = dofs + (int64_t)x.second * n;
                const int64_t r = (int64_t)x.second * n + (std::find(de, de + n, (int32_t)i) - de);
                if (wide) rows[k++] = r;
                else inc[k++] = (int32_t)(uint32_t)r;
            }
        }
    });

    // long rows, in pieces of what LDS holds at a time
    std::vector<int64_t> more;
    for (int64_t i = 0; i < ndof; ++i)
        for (int64_t c = 1; c * asm_cap(n) < row_ptr[i + 1] - row_ptr[i]; ++c) more.push_back(i | c << 32);

    // upload
    auto al = [](size_t b) { return (b + 255) / 256 * 256; };
    const size_t s_rp = al((ndof + 1) * 8), s_ci = al(nnz * 4), s_in = al(ne * n * (wide ? 8 : 4)),
                 s_mo = al(more.size() * 8), s_pos = al(ne * nn * 2);
    feint_asm_plan *pl = new feint_asm_plan;
    if (hipGetDevice(&pl->dev) != hipSuccess) { delete pl; return FEINT_ERR_HIP; }
    hipError_t err = hipMalloc(&pl->base, 2 * s_rp + s_ci + s_in + s_mo + s_pos);
    if (err != hipSuccess) { set_error("asm plan allocation", err); delete pl; return FEINT_ERR_HIP; }
    char *p = (char *)pl->base;
    pl->row_ptr = (int64_t *)p; p += s_rp;
    pl->col_idx = (int32_t *)p; p += s_ci;
    pl->inc_ptr = (int64_t *)p; p += s_rp;
    pl->inc = p; p += s_in;
    pl->wide = wide;
    pl->more = (int64_t *)p; p += s_mo;
    pl->nmore = (int64_t)more.size();
    pl->pos = (uint16_t *)p;
    const bool ok = hipMemcpy(pl->row_ptr, row_ptr.data(), (ndof + 1) * 8, hipMemcpyHostToDevice) == hipSuccess &&
                    hipMemcpy(pl->col_idx, col_idx.data(), nnz * 4, hipMemcpyHostToDevice) == hipSuccess &&
                    hipMemcpy(pl->inc_ptr, inc_ptr.data(), (ndof + 1) * 8, hipMemcpyHostToDevice) == hipSuccess &&
                    hipMemcpy(pl->inc, wide ? (const void *)rows.data() : inc.data(), ne * n * (wide ? 8 : 4), hipMemcpyHostToDevice) == hipSuccess &&
                    (more.empty() || hipMemcpy(pl->more, more.data(), more.size() * 8, hipMemcpyHostToDevice) == hipSuccess) &&
                    hipMemcpy(pl->pos, pos.data(), ne * nn * 2, hipMemcpyHostToDevice) == hipSuccess;
    if (!ok) {
        set_error("asm plan upload", hipGetLastError());
        (void)hipFree(pl->base);
        delete pl;
        return FEINT_ERR_HIP;
    }
    pl->ne = ne; pl->ndof = ndof; pl->nnz = nnz; pl->n = n; pl->ncolors = ncolors;
    for (int64_t i = 0; i < ndof; ++i) pl->max_row = std::max(pl->max_row, (int)(row_ptr[i + 1] - row_ptr[i]));
    pl->color_of = std::move(color);
    *out = pl;
    return FEINT_OK;
}

feint_status feint_asm_plan_info(const feint_asm_plan *pl, int64_t *nnz, int *ncolors) {
    if (!pl) return FEINT_ERR_INVALID_ARG;
    if (nnz) *nnz = pl->nnz;
    if (ncolors) *ncolors = pl->ncolors;
    return FEINT_OK;
}

feint_status feint_asm_plan_pattern(const feint_asm_plan *pl, int64_t *row_ptr, int32_t *col_idx, void *stream) {
    if (!pl || !row_ptr || !col_idx) return FEINT_ERR_INVALID_ARG;
    hipStream_t st = (hipStream_t)stream;
    hipError_t e = hipMemcpyAsync(row_ptr, pl->row_ptr, (pl->ndof + 1) * 8, hipMemcpyDeviceToDevice, st);
    if (e == hipSuccess) e = hipMemcpyAsync(col_idx, pl->col_idx, pl->nnz * 4, hipMemcpyDeviceToDevice, st);
    if (e != hipSuccess) { set_error("asm pattern copy", e); return FEINT_ERR_HIP; }
    return FEINT_OK;
}

feint_status feint_asm_plan_colors(const feint_asm_plan *pl, int32_t *color_of) {
    if (!pl || !color_of) return FEINT_ERR_INVALID_ARG;
    std::memcpy(color_of, pl->color_of.data(), pl->ne * sizeof(int32_t));
    return FEINT_OK;
}

feint_status feint_assemble(feint_asm_plan *pl, feint_form form, const void *A, const void *b, void *values,
                            void *rhs, int accumulate, void *stream) {
    if (!pl) return FEINT_ERR_INVALID_ARG;
    if (form != FEINT_FP64 && form != FEINT_FP32 && form != FEINT_BF16X3 && form != FEINT_FP16X3)
        return FEINT_ERR_UNSUPPORTED_FORM;
    if (!A || !b || !values || !rhs) return FEINT_ERR_INVALID_ARG;
    hipStream_t st = (hipStream_t)stream;
    (void)hipGetLastError();
    if (form == FEINT_FP64)
        launch_rows<double>(pl, A, b, values, rhs, accumulate, st);
    else
        launch_rows<float>(pl, A, b, values, rhs, accumulate, st);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) { set_error("assembly launch", e); return FEINT_ERR_HIP; }
    return FEINT_OK;
}

void feint_asm_plan_destroy(feint_asm_plan *pl) {
    if (!pl) return;
    int cur = 0;
    (void)hipGetDevice(&cur);
    (void)hipSetDevice(pl->dev);
    (void)hipDeviceSynchronize();
    (void)hipFree(pl->base);
    (void)hipSetDevice(cur);
    delete pl;
}

}  // extern "C"
