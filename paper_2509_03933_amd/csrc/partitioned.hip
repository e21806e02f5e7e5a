// Staged divide-and-conquer solve: three kernels per batch of systems.
//
// Stage A (k_stage_a): one lane per (system, partition) streams the partition
//   once, carrying only O(1) state: the modified Thomas recurrences of
//   tile.hip.h and the running products that turn the back recurrence of the
//   row-1 spike into a forward sum.  It writes the partition's two
//   unit-diagonal interface equations (6 values) to the reduced buffer, and
//   the recurrence's state (d^, a^, c^) at the first row of every segment of
//   kSeg interior rows to a workspace (k_stage_a_rows: of every interior row).
// Stage B (k_stage_b_pcr, k_stage_b_seq): the 2P-row interface system of every system of the
//   batch, FP64; parallel cyclic reduction across P consecutive lanes with
//   wavefront shuffles (P a power of two <= 64), otherwise one lane per system
//   eliminating the 2P rows in sequence.
// Stage C (k_stage_c): one lane per (system, partition) takes the segments
//   from the last to the first: the recurrence runs forward again over the
//   segment's rows from its kept state (the same operations, so the same d^,
//   a^, c^), into registers, and then backwards x_{m-1} and x_0 being
//   interface unknowns, x_j = d^_j - a^_j x_0 - c^_j x_{j+1}.  A segment's rows
//   are read before any of them is written, and a lane reads only rows that
//   it alone writes, so x may alias d.  k_stage_c_rows walks the partition
//   backwards over the kept d^, a^, c^ of every row instead.
//
// HBM-bound.  Reading the rows twice costs less than keeping their factors:
// per unknown (FP64, per-row coefficients) A reads 32 B, C reads 30 and
// writes 8, the kept states are 1.5 B written and 1.5 read: 73 B against 88
// with every row's d^, a^, c^ written by A and read by C (shared operator 25
// against 32, with a shift 27 against 64), and the workspace is a sixteenth.
// 131,072 per-row lines of 2048 rows (P = 8): 4.77 -> 3.97 ms (73 B: 4.9 TB/s).
// That holds where the lanes of a wavefront read adjacent elements.  Where they
// do not (contiguous rows: adjacent lanes are n elements apart, each row's read
// costs a line per lane) the inputs are read once and the factors, which the
// workspace holds in lane order, are read back instead: 32,768 lines of 1000
// contiguous rows, FP64 shared operator, 0.68 ms keeping rows, 1.93 keeping
// states; per-row 2.56 and 3.35 (stage_keeps_rows).
//
// Partition p of a system of n rows has m_p = floor(n/P) + (p < n mod P) rows
// starting at p*floor(n/P) + min(p, n mod P).  Every system's arithmetic is
// independent of how systems are batched, so results are bit-identical for
// any batch size, stream count or schedule.
#include <type_traits>

#include "tile.hip.h"
#include "partitioned.h"

namespace tdma {
namespace {

// Interior rows per segment: the state kept by Stage A every kSeg rows (24 B in
// FP64, each way) against the registers that hold a segment's inputs (8 per
// row).  131,072 per-row lines of 2048 rows: 4.03 ms at 16, 4.13 at 8.
constexpr int kSeg = 16;

struct PartRange {
    int64_t start;
    int m;
};

__device__ __forceinline__ PartRange part_range(int64_t n, int P, int p) {
    const int64_t q = n / P, r = n % P;
    PartRange pr;
    pr.start = p * q + (p < r ? p : r);
    pr.m = (int)(q + (p < r ? 1 : 0));
    return pr;
}

// Reduced-buffer layout: value v (0..5 = first a, c, d, last a, c, d) of
// partition p of batch-local system k at ((v*P + p) * nb + k).
__device__ __forceinline__ size_t red_at(int v, int p, int64_t k, int P, int64_t nb) {
    return ((size_t)v * P + p) * nb + k;
}

// One row of the matrix as Stage A and C read it: no a_0, no c_{n-1}, the
// system's shift on the diagonal.
template <typename T, bool LIKE_D, bool SHIFT>
struct RowReader {
    const T *A, *B, *C, *d;
    int64_t base, rs, n;
    T sh;
    __device__ __forceinline__ void load(int64_t r, T &a, T &b, T &c, T &dd) const {
        const int64_t idx = base + r * rs;
        dd = d[idx];
        if constexpr (LIKE_D) {
            a = A[idx]; b = B[idx]; c = C[idx];
        } else {
            a = A[r]; b = B[r]; c = C[r];
        }
    }
    __device__ __forceinline__ void fix(int64_t r, T &a, T &b, T &c) const {
        if constexpr (SHIFT) b += sh;
        if (r == 0) a = T(0);
        if (r == n - 1) c = T(0);
    }
};

template <typename T, bool LIKE_D, bool SHIFT>
__device__ __forceinline__ RowReader<T, LIKE_D, SHIFT> row_reader(const SysMap &map, const Coef &coef,
                                                                  const T *d, const dev::LaneSys &sys) {
    RowReader<T, LIKE_D, SHIFT> rd;
    rd.A = (const T *)coef.a;
    rd.B = (const T *)coef.b;
    rd.C = (const T *)coef.c;
    rd.d = d;
    rd.base = sys.base;
    rd.rs = map.row_stride;
    rd.n = map.n;
    rd.sh = T(0);
    if constexpr (SHIFT) rd.sh = ((const T *)coef.shift)[sys.id];
    return rd;
}

// The state of the recurrence at one row, and the step to the next row.
template <typename T>
struct RowState {
    T ah, ch, dh;
    __device__ __forceinline__ T pivot(T a, T b) const { return b - a * ch; }
    __device__ __forceinline__ void step(T a, T c, T dd, T ib) {
        const T ra = a * ib;
        dh = (dd - a * dh) * ib;
        ch = c * ib;
        ah = -ra * ah;
    }
};

// Kept states: segment g of partition p (state of its row 1 + g*kSeg) of
// batch-local system k at ((p*nseg + g) * nb + k); with a shared operator the
// same a^, c^ for every system, kept once ((p*nseg + g)).
template <typename T, bool LIKE_D, bool SHIFT>
__global__ void __launch_bounds__(256)
k_stage_a(SysMap map, Coef coef, const T *__restrict__ d, T *__restrict__ ws_d,
          T *__restrict__ ws_a, T *__restrict__ ws_c, double *__restrict__ red, int64_t k_begin,
          int64_t nb, int P, int nseg, int *err) {
    constexpr bool SHARED_FACTORS = !LIKE_D && !SHIFT;
    const int64_t kl = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    const int p = blockIdx.y;
    if (kl >= nb) return;
    const dev::LaneSys sys = dev::lane_system(map, k_begin + kl);
    const PartRange pr = part_range(map.n, P, p);
    const auto rd = row_reader<T, LIKE_D, SHIFT>(map, coef, d, sys);
    const int m = pr.m;
    bool bad = false;
    T a, b, c, dd;
    rd.load(pr.start, a, b, c, dd);
    rd.fix(pr.start, a, b, c);
    bad |= dev::bad_pivot(b);
    T ib = dev::recip(b);
    const T a0 = a * ib, c0 = c * ib, d0 = dd * ib;
    rd.load(pr.start + 1, a, b, c, dd);
    rd.fix(pr.start + 1, a, b, c);
    bad |= dev::bad_pivot(b);
    ib = dev::recip(b);
    RowState<T> st{a * ib, c * ib, dd * ib};
    T pi = T(1), dt1 = T(0), at1 = T(0);
    // the current row is final: fold it into the row-1 spike, then advance
    auto advance = [&](int64_t r, T ra, T rb, T rc, T rdd) {
        dt1 += pi * st.dh;
        at1 += pi * st.ah;
        pi = -st.ch * pi;
        rd.fix(r, ra, rb, rc);
        const T piv = st.pivot(ra, rb);
        bad |= dev::bad_pivot(piv);
        st.step(ra, rc, rdd, dev::recip(piv));
    };
    auto keep = [&](int64_t q) {
        ws_d[q * nb + kl] = st.dh;
        if constexpr (SHARED_FACTORS) {
            if (kl == 0) {
                ws_a[q] = st.ah;
                ws_c[q] = st.ch;
            }
        } else {
            ws_a[q * nb + kl] = st.ah;
            ws_c[q * nb + kl] = st.ch;
        }
    };
    // rows 2 .. m-1, a segment's loads in flight together
    int j = 1;
    int64_t g = (int64_t)p * nseg;
    for (; j + kSeg <= m - 1; j += kSeg, ++g) {
        T va[kSeg], vb[kSeg], vc[kSeg], vd[kSeg];
#pragma unroll
        for (int i = 0; i < kSeg; ++i) rd.load(pr.start + j + 1 + i, va[i], vb[i], vc[i], vd[i]);
        keep(g);
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int i = 0; i < kSeg; ++i) advance(pr.start + j + 1 + i, va[i], vb[i], vc[i], vd[i]);
    }
    if (j <= m - 2) keep(g);
    for (; j < m - 1; ++j) {
        rd.load(pr.start + j + 1, a, b, c, dd);
        advance(pr.start + j + 1, a, b, c, dd);
    }
    const T ct1 = -pi;
    const double den = 1.0 - (double)c0 * (double)at1;
    bad |= dev::bad_pivot(den);
    const double rho = dev::recip(den);
    red[red_at(0, p, kl, P, nb)] = rho * (double)a0;
    red[red_at(1, p, kl, P, nb)] = -rho * (double)c0 * (double)ct1;
    red[red_at(2, p, kl, P, nb)] = rho * ((double)d0 - (double)c0 * (double)dt1);
    red[red_at(3, p, kl, P, nb)] = (double)st.ah;
    red[red_at(4, p, kl, P, nb)] = (double)st.ch;
    red[red_at(5, p, kl, P, nb)] = (double)st.dh;
    if (bad) atomicOr(err, 1);
}

// Stage A that keeps every interior row's d^, a^, c^: row r of batch-local
// system k at r*nb + k (a^, c^ of a shared operator at r).
template <typename T, bool LIKE_D, bool SHIFT>
__global__ void __launch_bounds__(256)
k_stage_a_rows(SysMap map, Coef coef, const T *__restrict__ d, T *__restrict__ ws_d,
               T *__restrict__ ws_a, T *__restrict__ ws_c, double *__restrict__ red, int64_t k_begin,
               int64_t nb, int P, int *err) {
    constexpr bool SHARED_FACTORS = !LIKE_D && !SHIFT;
    const int64_t kl = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    const int p = blockIdx.y;
    if (kl >= nb) return;
    const dev::LaneSys sys = dev::lane_system(map, k_begin + kl);
    const int64_t n = map.n;
    const PartRange pr = part_range(n, P, p);
    const T *__restrict__ A = (const T *)coef.a;
    const T *__restrict__ B = (const T *)coef.b;
    const T *__restrict__ C = (const T *)coef.c;
    const int64_t rs = map.row_stride;
    T sh = T(0);
    if constexpr (SHIFT) sh = ((const T *)coef.shift)[sys.id];
    auto load = [&](int64_t r, T &a, T &b, T &c, T &dd) {
        const int64_t idx = sys.base + r * rs;
        dd = d[idx];
        if constexpr (LIKE_D) {
            a = A[idx]; b = B[idx]; c = C[idx];
        } else {
            a = A[r]; b = B[r]; c = C[r];
        }
        if constexpr (SHIFT) b += sh;
        if (r == 0) a = T(0);
        if (r == n - 1) c = T(0);
    };
    // factor storage: row r of batch-local system kl at r*nb + kl (coalesced)
    const bool store_factors = !SHARED_FACTORS || kl == 0;
    const int64_t fk = SHARED_FACTORS ? 0 : kl;
    const int64_t fstride = SHARED_FACTORS ? 1 : nb;
    bool bad = false;
    T a, b, c, dd;
    load(pr.start, a, b, c, dd);
    bad |= dev::bad_pivot(b);
    T ib = dev::recip(b);
    const T a0 = a * ib, c0 = c * ib, d0 = dd * ib;
    load(pr.start + 1, a, b, c, dd);
    bad |= dev::bad_pivot(b);
    ib = dev::recip(b);
    T ah = a * ib, ch = c * ib, dh = dd * ib;
    T pi = T(1), dt1 = T(0), at1 = T(0);
    const int m = pr.m;
#pragma unroll 4
    for (int j = 1; j < m - 1; ++j) {
        // row j is final: store it, fold it into the row-1 spike, then advance
        const int64_t r = pr.start + j;
        ws_d[r * nb + kl] = dh;
        if (store_factors) {
            ws_a[r * fstride + fk] = ah;
            ws_c[r * fstride + fk] = ch;
        }
        dt1 += pi * dh;
        at1 += pi * ah;
        pi = -ch * pi;
        load(r + 1, a, b, c, dd);
        const T piv = b - a * ch;
        bad |= dev::bad_pivot(piv);
        ib = dev::recip(piv);
        const T ra = a * ib;
        dh = (dd - a * dh) * ib;
        ch = c * ib;
        ah = -ra * ah;
    }
    const T ct1 = -pi;
    const double den = 1.0 - (double)c0 * (double)at1;
    bad |= dev::bad_pivot(den);
    const double rho = dev::recip(den);
    red[red_at(0, p, kl, P, nb)] = rho * (double)a0;
    red[red_at(1, p, kl, P, nb)] = -rho * (double)c0 * (double)ct1;
    red[red_at(2, p, kl, P, nb)] = rho * ((double)d0 - (double)c0 * (double)dt1);
    red[red_at(3, p, kl, P, nb)] = (double)ah;
    red[red_at(4, p, kl, P, nb)] = (double)ch;
    red[red_at(5, p, kl, P, nb)] = (double)dh;
    if (bad) atomicOr(err, 1);
}

// Stage B, PCR variant: P consecutive lanes per system (P power of two <= 64).
__global__ void __launch_bounds__(256)
k_stage_b_pcr(const double *red, double *X, int64_t nb, int P, int P_log2, int *err) {
    const int64_t t = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    const int64_t kl = t >> P_log2;
    const int p = (int)(t & (P - 1));
    const bool valid = kl < nb;
    const int64_t kk = valid ? kl : 0;
    double a0 = red[red_at(0, p, kk, P, nb)], c0 = red[red_at(1, p, kk, P, nb)];
    double d0 = red[red_at(2, p, kk, P, nb)], a1 = red[red_at(3, p, kk, P, nb)];
    double c1 = red[red_at(4, p, kk, P, nb)], d1 = red[red_at(5, p, kk, P, nb)];
    const int lane = threadIdx.x & 63;
    bool bad = false;
    for (int h = 1; h < 2 * P; h <<= 1) {
        if (h == 1) {
            const bool has_lo = p > 0, has_hi = p < P - 1;
            const int lo = has_lo ? lane - 1 : lane, hi = has_hi ? lane + 1 : lane;
            double am = __shfl(a1, lo), cm = __shfl(c1, lo), dm = __shfl(d1, lo);
            double ap = __shfl(a0, hi), cp = __shfl(c0, hi), dp = __shfl(d0, hi);
            if (!has_lo) { am = 0.0; cm = 0.0; dm = 0.0; }
            if (!has_hi) { ap = 0.0; cp = 0.0; dp = 0.0; }
            const double oa0 = a0, oc0 = c0, od0 = d0;
            dev::pcr_row(a0, c0, d0, am, cm, dm, a1, c1, d1, bad);
            dev::pcr_row(a1, c1, d1, oa0, oc0, od0, ap, cp, dp, bad);
        } else {
            const int dl = h >> 1;
            const bool has_lo = p >= dl, has_hi = p + dl < P;
            const int lo = has_lo ? lane - dl : lane, hi = has_hi ? lane + dl : lane;
            double la0 = __shfl(a0, lo), lc0 = __shfl(c0, lo), ld0 = __shfl(d0, lo);
            double la1 = __shfl(a1, lo), lc1 = __shfl(c1, lo), ld1 = __shfl(d1, lo);
            double ua0 = __shfl(a0, hi), uc0 = __shfl(c0, hi), ud0 = __shfl(d0, hi);
            double ua1 = __shfl(a1, hi), uc1 = __shfl(c1, hi), ud1 = __shfl(d1, hi);
            if (!has_lo) { la0 = lc0 = ld0 = la1 = lc1 = ld1 = 0.0; }
            if (!has_hi) { ua0 = uc0 = ud0 = ua1 = uc1 = ud1 = 0.0; }
            dev::pcr_row(a0, c0, d0, la0, lc0, ld0, ua0, uc0, ud0, bad);
            dev::pcr_row(a1, c1, d1, la1, lc1, ld1, ua1, uc1, ud1, bad);
        }
    }
    if (valid) {
        X[(size_t)(2 * p) * nb + kl] = d0;
        X[(size_t)(2 * p + 1) * nb + kl] = d1;
        if (bad) atomicOr(err, 1);
    }
}

// Stage B, sequential variant: one lane per system eliminates its 2P
// unit-diagonal interface rows top-down and substitutes bottom-up (any P).
__global__ void __launch_bounds__(256)
k_stage_b_seq(const double *red, double *X, double *scratch, int64_t nb, int P, int *err) {
    const int64_t kl = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (kl >= nb) return;
    const int R2 = 2 * P;
    bool bad = false;
    // forward: row i -> x_i + g_i x_{i+1} = e_i (g, e kept in scratch, row-major by system)
    double gp = 0.0, ep = 0.0;
    for (int i = 0; i < R2; ++i) {
        const int p = i >> 1, v = (i & 1) * 3;
        const double a = red[red_at(v, p, kl, P, nb)], c = red[red_at(v + 1, p, kl, P, nb)];
        const double dd = red[red_at(v + 2, p, kl, P, nb)];
        const double piv = 1.0 - (i > 0 ? a * gp : 0.0);
        bad |= dev::bad_pivot(piv);
        const double ib = 1.0 / piv;
        gp = c * ib;
        ep = (dd - (i > 0 ? a * ep : 0.0)) * ib;
        scratch[(size_t)i * nb + kl] = gp;
        X[(size_t)i * nb + kl] = ep;
    }
    double xn = X[(size_t)(R2 - 1) * nb + kl];
    for (int i = R2 - 2; i >= 0; --i) {
        xn = X[(size_t)i * nb + kl] - scratch[(size_t)i * nb + kl] * xn;
        X[(size_t)i * nb + kl] = xn;
    }
    if (bad) atomicOr(err, 1);
}

template <typename T, bool SHARED_FACTORS>
__global__ void __launch_bounds__(256)
k_stage_c_rows(SysMap map, T *__restrict__ x, const T *__restrict__ ws_d, const T *__restrict__ ws_a,
               const T *__restrict__ ws_c, const double *__restrict__ X, int64_t k_begin, int64_t nb,
               int P) {
    const int64_t kl = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    const int p = blockIdx.y;
    if (kl >= nb) return;
    const dev::LaneSys sys = dev::lane_system(map, k_begin + kl);
    const PartRange pr = part_range(map.n, P, p);
    const int64_t rs = map.row_stride;
    const T xf = (T)X[(size_t)(2 * p) * nb + kl];
    T xn = (T)X[(size_t)(2 * p + 1) * nb + kl];
    const int64_t fk = SHARED_FACTORS ? 0 : kl;
    const int64_t fstride = SHARED_FACTORS ? 1 : nb;
    x[sys.base + (pr.start + pr.m - 1) * rs] = xn;
#pragma unroll 4
    for (int j = pr.m - 2; j >= 1; --j) {
        const int64_t r = pr.start + j;
        xn = ws_d[r * nb + kl] - ws_a[r * fstride + fk] * xf - ws_c[r * fstride + fk] * xn;
        x[sys.base + r * rs] = xn;
    }
    x[sys.base + pr.start * rs] = xf;
}

// d and x may be the same array: no __restrict__ on either.
template <typename T, bool LIKE_D, bool SHIFT>
__global__ void __launch_bounds__(256)
k_stage_c(SysMap map, Coef coef, const T *d, T *x, const T *__restrict__ ws_d,
          const T *__restrict__ ws_a, const T *__restrict__ ws_c, const double *__restrict__ X,
          int64_t k_begin, int64_t nb, int P, int nseg) {
    constexpr bool SHARED_FACTORS = !LIKE_D && !SHIFT;
    const int64_t kl = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    const int p = blockIdx.y;
    if (kl >= nb) return;
    const dev::LaneSys sys = dev::lane_system(map, k_begin + kl);
    const PartRange pr = part_range(map.n, P, p);
    const auto rd = row_reader<T, LIKE_D, SHIFT>(map, coef, d, sys);
    const int m = pr.m;
    const T xf = (T)X[(size_t)(2 * p) * nb + kl];
    T xn = (T)X[(size_t)(2 * p + 1) * nb + kl];
    T *xl = x + sys.base + pr.start * rd.rs;   // the partition's row 0
    xl[(m - 1) * rd.rs] = xn;
    // segment g: rows j0 = 1 + g*kSeg .. j0 + len - 1 (all interior); FULL: len = kSeg
    auto segment = [&](int g, int len, auto full) {
        constexpr bool FULL = decltype(full)::value;
        const int j0 = 1 + g * kSeg;
        T va[kSeg], vb[kSeg], vc[kSeg], vd[kSeg];
#pragma unroll
        for (int i = 1; i < kSeg; ++i) {
            const int j = j0 + (FULL || i < len ? i : len - 1);
            rd.load(pr.start + j, va[i], vb[i], vc[i], vd[i]);
        }
        __builtin_amdgcn_sched_barrier(0);
        const int64_t q = (int64_t)p * nseg + g;
        RowState<T> st;
        st.dh = ws_d[q * nb + kl];
        st.ah = SHARED_FACTORS ? ws_a[q] : ws_a[q * nb + kl];
        st.ch = SHARED_FACTORS ? ws_c[q] : ws_c[q * nb + kl];
        // e_j = d^_j - a^_j x_0 and c^_j of the segment's rows
        vd[0] = st.dh - st.ah * xf;
        vc[0] = st.ch;
#pragma unroll
        for (int i = 1; i < kSeg; ++i) {
            rd.fix(pr.start + j0 + i, va[i], vb[i], vc[i]);
            st.step(va[i], vc[i], vd[i], dev::recip(st.pivot(va[i], vb[i])));
            vd[i] = st.dh - st.ah * xf;
            vc[i] = st.ch;
        }
#pragma unroll
        for (int i = kSeg - 1; i >= 0; --i) {
            if (FULL || i < len) {
                xn = vd[i] - vc[i] * xn;
                __builtin_nontemporal_store(xn, xl + (j0 + i) * rd.rs);
            }
        }
    };
    int g = (m - 2 + kSeg - 1) / kSeg - 1;
    if (g >= 0 && (m - 2) % kSeg != 0) {
        segment(g, (m - 2) % kSeg, std::false_type{});
        --g;
    }
    for (; g >= 0; --g) segment(g, kSeg, std::true_type{});
    xl[0] = xf;
}

#define TDMA_STAGE_DISPATCH(CALL)                                   \
    if (like_d && !shift) { CALL(true, false); }                    \
    else if (like_d) { CALL(true, true); }                          \
    else if (!shift) { CALL(false, false); }                        \
    else { CALL(false, true); }

template <typename T>
hipError_t launch_a_t(const SysMap &map, const Coef &coef, const void *d, const StageWs &w, int64_t k_begin,
                      int64_t nb, int P, int *err, hipStream_t st) {
    const dim3 grid((unsigned)((nb + 255) / 256), (unsigned)P);
    const bool like_d = coef.mode == TDMA_COEF_LIKE_D, shift = coef.shift != nullptr;
#define TDMA_A(LD, SH)                                                                            \
    if (w.keep_rows)                                                                              \
        hipLaunchKernelGGL((k_stage_a_rows<T, LD, SH>), grid, dim3(256), 0, st, map, coef,       \
                           (const T *)d, (T *)w.ws_d, (T *)w.ws_a, (T *)w.ws_c, w.red, k_begin,   \
                           nb, P, err);                                                           \
    else                                                                                          \
        hipLaunchKernelGGL((k_stage_a<T, LD, SH>), grid, dim3(256), 0, st, map, coef,             \
                           (const T *)d, (T *)w.ws_d, (T *)w.ws_a, (T *)w.ws_c, w.red, k_begin,   \
                           nb, P, w.nseg, err)
    TDMA_STAGE_DISPATCH(TDMA_A)
#undef TDMA_A
    return hipGetLastError();
}

template <typename T>
hipError_t launch_c_t(const SysMap &map, const Coef &coef, const void *d, void *x, const StageWs &w,
                      int64_t k_begin, int64_t nb, int P, hipStream_t st) {
    const dim3 grid((unsigned)((nb + 255) / 256), (unsigned)P);
    const bool like_d = coef.mode == TDMA_COEF_LIKE_D, shift = coef.shift != nullptr;
    if (w.keep_rows) {
        if (!like_d && !shift)
            hipLaunchKernelGGL((k_stage_c_rows<T, true>), grid, dim3(256), 0, st, map, (T *)x,
                               (const T *)w.ws_d, (const T *)w.ws_a, (const T *)w.ws_c, w.X, k_begin, nb, P);
        else
            hipLaunchKernelGGL((k_stage_c_rows<T, false>), grid, dim3(256), 0, st, map, (T *)x,
                               (const T *)w.ws_d, (const T *)w.ws_a, (const T *)w.ws_c, w.X, k_begin, nb, P);
        return hipGetLastError();
    }
#define TDMA_C(LD, SH)                                                                          \
    hipLaunchKernelGGL((k_stage_c<T, LD, SH>), grid, dim3(256), 0, st, map, coef, (const T *)d, \
                       (T *)x, (const T *)w.ws_d, (const T *)w.ws_a, (const T *)w.ws_c, w.X,    \
                       k_begin, nb, P, w.nseg)
    TDMA_STAGE_DISPATCH(TDMA_C)
#undef TDMA_C
    return hipGetLastError();
}

}  // namespace

// Whether the staged solve keeps every row's factors: where fewer than 64 bytes
// of consecutive systems are adjacent (FP64, 32,768 lines of 1000 rows, shared
// operator, runs of 2 systems: 0.43 ms keeping rows, 0.79 keeping states; FP32
// runs of 4: 0.23 and 0.30, of 8: 0.16 and 0.15 per-row at 250 rows), and where
// partitions have fewer than kSeg / 2 interior rows, whose segment reads and
// eliminates kSeg rows all the same (400,000 lines of 40 rows, 5 per partition:
// 0.27 ms keeping rows, 0.33 keeping states).  Few systems wait for their loads,
// not for memory's rate, and a segment's loads are in flight together: they keep
// states.  The line lies where the two meet, on contiguous lines of 5000 to
// 40,000 rows (time keeping rows over time keeping states): shared operator 512
// systems 0.92 to 1.31, 1000 0.73 to 1.06, 2000 0.51 to 0.68; with a shift 1000
// 0.85 to 1.32, 1500 0.75 to 1.07, 2000 0.72 to 0.92; per-row FP32 64 0.79 to
// 0.87, FP64 64 1.25 to 1.33, 128 0.87 to 1.19.
static bool stage_keeps_rows(const SysMap &map, size_t esz, int P, const Coef &coef) {
    const int64_t stride = map.nsys0 > 1 ? map.sys_stride0 : map.sys_stride1;
    const int64_t run = map.nsys0 > 1 ? map.nsys0 : map.nsys;
    const int64_t few = coef.mode == TDMA_COEF_LIKE_D ? (esz == 4 ? 64 : 160) : coef.shift ? 1280 : 768;
    if (map.nsys < few) return false;
    return stride != 1 || run * (int64_t)esz < 64 || map.n / P - 2 < kSeg / 2;
}

size_t stage_ws(int dtype, const SysMap &map, const Coef &coef, int64_t batch, int P, void *mem,
                StageWs *out) {
    const size_t esz = dtype == TDMA_F64 ? 8 : 4;
    const int64_t n = map.n;
    const auto al = [](size_t b) { return (b + 255) & ~(size_t)255; };
    const int64_t mmax = n / P + (n % P != 0);
    const int64_t nseg = mmax > 2 ? (mmax - 2 + kSeg - 1) / kSeg : 0;
    const bool shared_factors = coef.mode == TDMA_COEF_SHARED && coef.shift == nullptr;
    out->keep_rows = stage_keeps_rows(map, esz, P, coef);
    const size_t states = out->keep_rows ? (size_t)n : (size_t)P * nseg;
    const size_t d_bytes = al(states * batch * esz);
    const size_t f_bytes = shared_factors ? al(states * esz) : d_bytes;
    const size_t red_bytes = al((size_t)6 * P * batch * 8), x_bytes = al((size_t)2 * P * batch * 8);
    char *b = (char *)mem;
    out->nseg = (int)nseg;
    if (b) {
        out->ws_d = b;
        out->ws_a = b + d_bytes;
        out->ws_c = b + d_bytes + f_bytes;
        out->red = (double *)(b + d_bytes + 2 * f_bytes);
        out->X = (double *)(b + d_bytes + 2 * f_bytes + red_bytes);
        out->scratch = (double *)(b + d_bytes + 2 * f_bytes + red_bytes + x_bytes);
    }
    return d_bytes + 2 * f_bytes + red_bytes + 2 * x_bytes;
}

hipError_t launch_stage_a(int dtype, const SysMap &map, const Coef &coef, const void *d,
                          const StageWs &w, int64_t k_begin, int64_t nb, int P, int *err,
                          hipStream_t st) {
    if (nb <= 0) return hipSuccess;
    if (dtype == TDMA_F64) return launch_a_t<double>(map, coef, d, w, k_begin, nb, P, err, st);
    return launch_a_t<float>(map, coef, d, w, k_begin, nb, P, err, st);
}

hipError_t launch_stage_b(const StageWs &w, int64_t nb, int P, int *err, hipStream_t st) {
    if (nb <= 0) return hipSuccess;
    if (P <= 64 && (P & (P - 1)) == 0) {
        int P_log2 = 0;
        while ((1 << P_log2) < P) ++P_log2;
        const int64_t lanes = nb * P;
        hipLaunchKernelGGL(k_stage_b_pcr, dim3((unsigned)((lanes + 255) / 256)), dim3(256), 0, st,
                           w.red, w.X, nb, P, P_log2, err);
    } else {
        hipLaunchKernelGGL(k_stage_b_seq, dim3((unsigned)((nb + 255) / 256)), dim3(256), 0, st, w.red,
                           w.X, w.scratch, nb, P, err);
    }
    return hipGetLastError();
}

hipError_t launch_stage_c(int dtype, const SysMap &map, const Coef &coef, const void *d, void *x,
                          const StageWs &w, int64_t k_begin, int64_t nb, int P, hipStream_t st) {
    if (nb <= 0) return hipSuccess;
    if (dtype == TDMA_F64) return launch_c_t<double>(map, coef, d, x, w, k_begin, nb, P, st);
    return launch_c_t<float>(map, coef, d, x, w, k_begin, nb, P, st);
}

}  // namespace tdma
