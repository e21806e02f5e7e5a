// Per-row coefficients on strided layouts: every system has its own a, b, c
// beside its right-hand side d (the general batched system of Sec. 2; the
// per-row z-lines of a 3-D grid, rows 2^20 elements apart at 1024^3).
//
// Resident workgroups walk tiles of S systems x P partitions x M rows per
// lane.  S is as many systems as the lanes allow (16 to 128, so every row of a
// tile is a 128-byte line or more and each address translation serves that much;
// fewer with 64 partitions or few tiles); this is what the one-tile-per-block
// kernel (S = 8, 64-byte rows) cannot reach, because it holds all four inputs of
// every row.  Here a lane keeps three values per
// interior row, alpha_j = g_j a_j, gamma_j = g_j c_j and delta_j = g_j d_j
// (g_j the pivot reciprocal of plain Thomas on the rows 1..M-2 with x_0 as a
// boundary value), computed as the rows arrive:
//  Stage A consumes the rows in order through a window of W rows whose loads
//    are in flight (row j + W is issued when row j is consumed), runs the
//    modified Thomas recurrences of tile.hip.h with O(1) running state, and
//    forms the partition's two interface rows;
//  Stage B solves the 2P-row interface systems of the tile (iface_pcr);
//  Stage C re-solves the interior from the kept values with the interface
//    unknowns as boundaries: e_j = delta_j - alpha_j e_{j-1} from e_0 = x_0,
//    then x_j = e_j - gamma_j x_{j+1} from x_{M-1}, storing each row of x
//    as it is produced.  (The same substitution as in shifted.hip, with the
//    operator rows per system instead of shared.)
// The window's registers are free from the end of Stage A, so the next
// tile's first W rows are loaded there and arrive during Stages B and C.
// 40 B per unknown in FP64 (a, b, c, d in, x out), each read or written once.
// HBM-bound: 131,072 lines of 512 rows (32 systems, 256-byte tile rows) 0.55
// ms, 4.9 TB/s; 67,072 lines of 1000 rows (16 systems) 0.64 ms, 4.2 TB/s.
#include "tile.hip.h"
#include "walk.hip.h"

namespace tdma {
namespace {

// Lanes per workgroup: FP64 1024 at 16 rows per lane (128 registers), 512
// above (256 registers); FP32 1024.
template <typename T, int M>
constexpr int perrow_max_threads() { return M > 16 && sizeof(T) == 8 ? 512 : 1024; }

// How a system's n rows lie on P partitions of M row slots:
// kFull: P*M = n.  kUneven: n mod P partitions of floor(n/P) + 1 rows, the
// rest of floor(n/P), at most kSlack short of M; a partition's rows fill
// slots 0 .. cnt-2 and its last row slot M-1, and the slots between are
// passed over (the recurrences keep their state, nothing is stored).  kPad
// (explicit tiles far from full): partitions of M rows, the last ones with
// identity rows past the system's end.  kUneven asks only at its kSlack
// doubtful slots; kPad asks at every row, for its load, its row and its
// store, and spills (91 registers at 32 rows): 320,000 lines of 1000 rows
// (FP64) 3.75 ms with kPad, 2.95 with kUneven.
enum { kFull = 0, kPad = 1, kUneven = 2 };
constexpr int kSlack = 4;

// Where a lane's rows are: element offsets from the kernel's array
// arguments, stepped as integers (accesses stay global-memory instructions).
template <typename T>
struct RowArrays {
    const T *a, *b, *c, *d;
};

// The 4 inputs of one row at element offset `o`.
template <typename T>
__device__ __forceinline__ void load_row(const RowArrays<T> &in, int64_t o, T &a, T &b, T &c, T &d) {
    a = __builtin_nontemporal_load(in.a + o);
    b = __builtin_nontemporal_load(in.b + o);
    c = __builtin_nontemporal_load(in.c + o);
    d = __builtin_nontemporal_load(in.d + o);
}

// Row j of a lane as the matrix has it: identity rows past the system's end
// (jl = the system's last row counted from the lane's first slot; only kPad
// has slots past it), no a_0 (first = the lane's partition starts the system), no
// c_{n-1}.
template <typename T, int KIND>
__device__ __forceinline__ void fix_row(int j, int jl, bool first, T &a, T &b, T &c, T &d) {
    if (KIND == kPad && j > jl) {
        a = T(0); b = T(1); c = T(0); d = T(0);
    }
    if (j == 0 && first) a = T(0);
    if (j == jl) c = T(0);
}

// The window of rows whose loads are in flight.
template <typename T, int W>
struct Window {
    T a[W], b[W], c[W], d[W];
};

// Element offset of row j of a partition whose row 0 is at o0: rows past the
// system's last row jl (padding) read row jl again, a valid row of the
// system even when jl < 0 (a lane wholly past the end reads the system's
// last row).
template <int KIND>
__device__ __forceinline__ int64_t row_off(int64_t o0, int j, int jl, int64_t rs) {
    return o0 + (int64_t)(KIND != kPad || j <= jl ? j : jl) * rs;
}

// The first W rows of a partition into the window.
template <typename T, int W, int KIND>
__device__ __forceinline__ void load_window(const RowArrays<T> &in, int64_t o0, int jl, int64_t rs,
                                            Window<T, W> &win) {
    int64_t o = opaque(row_off<KIND>(o0, 0, jl, rs));
#pragma unroll
    for (int j = 0; j < W; ++j) {
        load_row(in, o, win.a[j], win.b[j], win.c[j], win.d[j]);
        o = opaque(o + (KIND != kPad || j + 1 <= jl ? rs : 0));
    }
}

// Stage A, B and C of one tile on the lane's M rows (row 0 at o0, next
// tile's row 0 at no); the window holds rows 0..W-1 of the tile on entry
// and rows 0..W-1 of the next tile on return.  cnt: the partition's rows
// (kUneven).  Every thread of the block calls it.
template <typename T, int M, int W, int KIND, int PQ>
__device__ __forceinline__ void perrow_solve(double *XC, int S, int s, int p, int P, int P_log2,
                                             int jl, int cnt, int64_t rs, const RowArrays<T> &in,
                                             Window<T, W> &win, int64_t o0, int64_t no, T *x,
                                             bool store, bool &bad) {
    static_assert(M >= kSlack + 4 && W >= 1 && W < M - kSlack, "unconditional slots for the window");
    // the same for every tile: re-read through a register barrier so the
    // per-row comparisons with it are made where they are used, not hoisted
    // out of the walk and kept live across it
    if (KIND == kPad) jl = opaque(jl);
    if (KIND == kUneven) cnt = opaque(cnt);
    // slots that may be passed over, and whether slot j holds a row
    auto maybe = [](int j) { return KIND == kUneven && j >= M - 1 - kSlack && j < M - 1; };
    auto have = [&](int j) { return !maybe(j) || j < cnt - 1; };
    const bool first = p == 0;
    T al[M], ga[M], de[M];
    // rows are consumed in order; row j + W goes into the slot row j frees,
    // its offset stepped from the previous one
    int64_t lo = opaque(row_off<KIND>(o0, W, jl, rs));
    auto take = [&](int j, T &a, T &b, T &c, T &d) {
        const int sl = j % W;
        a = win.a[sl]; b = win.b[sl]; c = win.c[sl]; d = win.d[sl];
        fix_row<T, KIND>(j, jl, first, a, b, c, d);
        if (j + W < M) {
            load_row(in, lo, win.a[sl], win.b[sl], win.c[sl], win.d[sl]);
            // (a slot passed over reads the row of the next slot)
            lo = opaque(lo + ((KIND != kPad || j + W + 1 <= jl) && have(j + W) ? rs : 0));
        }
    };
    T a, b, c, dd;
    // Stage A: row 0 normalised and set aside
    take(0, a, b, c, dd);
    T piv = b;
    bad |= dev::bad_pivot(piv);
    T g = dev::recip(piv);
    const T a0 = a * g, c0 = c * g, d0 = dd * g;
    // row 1: the first interior row (x_0 is a parameter)
    take(1, a, b, c, dd);
    piv = b;
    bad |= dev::bad_pivot(piv);
    g = dev::recip(piv);
    al[1] = a * g;
    ga[1] = c * g;
    de[1] = dd * g;
    T dh = de[1], ah = al[1], ch = ga[1];
    // first-row spike: x_1 = dt1 - at1 x_0 - ct1 x_{M-1} with running
    // products pi_1 = 1, pi_{j+1} = -c^_j pi_j
    T pi = T(1), dt1 = dh, at1 = ah;
#pragma unroll
    for (int j = 2; j < M; ++j) {
        take(j, a, b, c, dd);
        piv = b - a * ch;
        bad |= have(j) && dev::bad_pivot(piv);
        g = dev::recip(piv);
        const T alj = a * g, gaj = c * g, dej = dd * g;
        if (maybe(j)) {
            const bool h = have(j);
            const T npi = -ch * pi, ndh = dej - alj * dh, nah = -alj * ah;
            dh = h ? ndh : dh;
            ah = h ? nah : ah;
            pi = h ? npi : pi;
            ch = h ? gaj : ch;
            dt1 = h ? dt1 + pi * dh : dt1;
            at1 = h ? at1 + pi * ah : at1;
            al[j] = alj;
            ga[j] = gaj;
            de[j] = dej;
        } else {
            dh = dej - alj * dh;
            ah = -alj * ah;
            pi = -ch * pi;
            ch = gaj;
            if (j <= M - 2) {
                al[j] = alj;
                ga[j] = gaj;
                de[j] = dej;
                dt1 += pi * dh;
                at1 += pi * ah;
            }
        }
        if ((j & 3) == 3) __builtin_amdgcn_sched_barrier(0);
    }
    Iface f;
    {
        const double ct1 = -(double)pi;
        const double den = 1.0 - (double)c0 * (double)at1;
        bad |= dev::bad_pivot(den);
        const double rho = dev::recip(den);
        f.fa = rho * (double)a0;
        f.fc = -rho * (double)c0 * ct1;
        f.fd = rho * ((double)d0 - (double)c0 * (double)dt1);
        f.la = (double)ah;
        f.lc = (double)ch;
        f.ld = (double)dh;
    }
    // the window is free: the next tile's first rows
    load_window<T, W, KIND>(in, no, jl, rs, win);

    // Stage B
    double xfd, xld;
    iface_stage_b<PQ>(XC, S, s, p, P, P_log2, f, xfd, xld, bad);

    // Stage C, forward: e_j in place of delta_j
    const T xf = (T)xfd;
    T e = xf;
#pragma unroll
    for (int j = 1; j <= M - 2; ++j) {
        const T ne = de[j] - al[j] * e;
        e = have(j) ? ne : e;
        de[j] = e;
    }
    // backward: x_j, stored at once (rows j <= jl)
    int64_t xo = o0 + (int64_t)((KIND == kUneven ? cnt : M) - 1) * rs;
    T xn = (T)xld;
    if (store && (KIND != kPad || M - 1 <= jl)) __builtin_nontemporal_store(xn, x + xo);
#pragma unroll
    for (int j = M - 2; j >= 1; --j) {
        T xj = de[j] - ga[j] * xn;
        if (maybe(j)) xj = have(j) ? xj : xn;
        xj = opaque(xj);
        xo = opaque(xo - (have(j) ? rs : 0));
        if (store && have(j) && (KIND != kPad || j <= jl)) __builtin_nontemporal_store(xj, x + xo);
        xn = xj;
        if ((j & 3) == 1) __builtin_amdgcn_sched_barrier(0);
    }
    if (store && (KIND != kPad || 0 <= jl)) __builtin_nontemporal_store(xf, x + o0);
}

// Resident workgroups walk the tiles t0, t0 + G, ...; a lane past the last
// system solves a copy of system 0's rows and stores nothing.  Tile rows
// narrower than a 128-byte line start XCD-aware (t0 from dev::xcd_tile), so
// that the tiles sharing a line run under one L2 (44,544 lines of 1500 rows,
// 8 systems per tile: 1246 -> 912 us).
// MT: lanes of the largest workgroup (the registers per lane follow from it).
template <typename T, int M, int W, int KIND, int MT, int PQ>
__global__ void __launch_bounds__(MT)
k_perrow_stream(SysMap map, Coef coef, const T *d, T *x, int S_log2, int P_log2, int32_t ntiles,
                int *err) {
    extern __shared__ double lds[];
    const int tid = threadIdx.x;
    const int S = 1 << S_log2, P = 1 << P_log2;
    const int s = tid & (S - 1);
    const int p = tid >> S_log2;
    const int64_t n = map.n, rs = map.row_stride;
    // the lane's first row, and its rows
    const int nq = (int)n >> P_log2, nr = (int)n & (P - 1);
    const int r0 = KIND == kUneven ? p * nq + (p < nr ? p : nr) : p * M;
    const int cnt = KIND == kUneven ? nq + (p < nr ? 1 : 0) : M;
    const int32_t nsys0 = (int32_t)map.nsys0;
    const int32_t nsys = (int32_t)map.nsys;
    // the slot of the system's last row counted from the lane's first (>= M:
    // in another lane; kPad: < 0 when none of the lane's rows is inside)
    const int jl = KIND == kUneven ? (p == P - 1 ? M - 1 : M) : (int)(n - 1 - r0);
    RowArrays<T> in;
    in.a = (const T *)coef.a;
    in.b = (const T *)coef.b;
    in.c = (const T *)coef.c;
    in.d = d;
    const int32_t step = (int32_t)gridDim.x << S_log2;
    int32_t t = (int32_t)(S * (int)sizeof(T) < 128 ? dev::xcd_tile(blockIdx.x, gridDim.x) : blockIdx.x);
    Walk w;
    w.init(nsys0, (t << S_log2) + s, step);
    auto origin = [&](const Walk &ww, bool ok) {
        return (ok ? (int64_t)ww.s0 * map.sys_stride0 + (int64_t)ww.s1 * map.sys_stride1 : 0) +
               (int64_t)r0 * rs;
    };
    bool ok = w.k < nsys;
    int64_t o0 = origin(w, ok);
    bool bad = false;
    Window<T, W> win;
    load_window<T, W, KIND>(in, o0, jl, rs, win);
    for (;;) {
        w.advance(nsys0, step);
        const bool nok = w.k < nsys;
        const int64_t no = origin(w, nok);
        bool bad_t = false;
        perrow_solve<T, M, W, KIND, PQ>(lds, S, s, p, P, P_log2, jl, cnt, rs, in, win, o0, no, x, ok, bad_t);
        bad |= bad_t && ok;
        t += gridDim.x;
        if (t >= ntiles) break;
        o0 = no;
        ok = nok;
    }
    if (bad) atomicOr(err, 1);
}

template <typename T, int M, int W, int KIND, int MT, int PQ>
hipError_t launch_prq(const SysMap &map, const Coef &coef, const TileShape &sh, const void *d, void *x,
                      int *err, hipStream_t st) {
    const int S = 1 << sh.S_log2;
    const int P_log2 = __builtin_ctz((unsigned)sh.P);
    const size_t lds = perrow_lds_bytes(sh);
    const int64_t ntiles = (map.nsys + S - 1) / S;
    if (ntiles == 0) return hipSuccess;
    int dev = 0, cus = 0, per_cu = 0;
    hipError_t e = hipGetDevice(&dev);
    if (e == hipSuccess) e = hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev);
    if (e == hipSuccess)
        e = hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, k_perrow_stream<T, M, W, KIND, MT, PQ>,
                                                         sh.threads(), lds);
    if (e != hipSuccess) return e;
    if (per_cu < 1) return hipErrorInvalidConfiguration;
    const int64_t resident = (int64_t)cus * per_cu;
    const int64_t grid = ntiles < resident ? ntiles : resident;
    hipLaunchKernelGGL((k_perrow_stream<T, M, W, KIND, MT, PQ>), dim3((unsigned)grid), dim3(sh.threads()), lds,
                       st, map, coef, (const T *)d, (T *)x, sh.S_log2, P_log2, (int32_t)ntiles, err);
    return hipGetLastError();
}

// Stage B in its wavefront-shuffle form: the DPP form's extra registers cost
// this kernel more in spills than its shorter interface solve saves (1024^3
// per-row lines: 12.0 against 10.8 ms).
template <typename T, int M, int W, int KIND, int MT>
hipError_t launch_pr(const SysMap &map, const Coef &coef, const TileShape &sh, const void *d, void *x,
                     int *err, hipStream_t st) {
    return launch_prq<T, M, W, KIND, MT, 0>(map, coef, sh, d, x, err, st);
}

template <typename T, int M, int W, int MT = perrow_max_threads<T, M>()>
hipError_t launch_pr_kind(const SysMap &map, const Coef &coef, const TileShape &sh, const void *d,
                          void *x, int *err, hipStream_t st) {
    if ((int64_t)sh.P * M == map.n) return launch_pr<T, M, W, kFull, MT>(map, coef, sh, d, x, err, st);
    if (perrow_uneven(map.n, sh)) return launch_pr<T, M, W, kUneven, MT>(map, coef, sh, d, x, err, st);
    if constexpr (M == 16 || M == 32) return launch_pr<T, M, W, kPad, MT>(map, coef, sh, d, x, err, st);
    return hipErrorInvalidValue;
}

}  // namespace

size_t perrow_lds_bytes(const TileShape &sh) {
    return (size_t)3 * ((size_t)1 << sh.S_log2) * (2 * sh.P + 1) * sizeof(double);
}

// Whether partitions of floor(n/P) and floor(n/P) + 1 rows fit M slots with
// at most kSlack to spare.
bool perrow_uneven(int64_t n, const TileShape &sh) {
    return n <= (int64_t)sh.P * sh.M && n / sh.P >= sh.M - kSlack;
}

// Kernel 5: M = 16, 20, 24, 28 or 32 rows per lane (20, 24 and 28 for lengths
// that fill or nearly fill them: callers check perrow_uneven), P a power of
// two 2..64, 1024 lanes (512 above 16 rows in FP64), strided uniform layouts
// whose walk stays in 32-bit system indices.
bool perrow_supported(int dtype, const TileShape &sh) {
    if (sh.kernel != 5 || sh.contig || sh.pdd) return false;
    if (dtype != TDMA_F64 && dtype != TDMA_F32) return false;
    if (sh.M < 16 || sh.M > 32 || sh.M % 4 != 0) return false;
    if (sh.P < 2 || sh.P > 64 || (sh.P & (sh.P - 1)) != 0) return false;
    const int maxt = sh.M > 16 && dtype == TDMA_F64 ? 512 : 1024;
    if (sh.S_log2 < 0 || sh.threads() > maxt) return false;
    return perrow_lds_bytes(sh) <= 160 * 1024;
}

bool perrow_layout_ok(const SysMap &m, const TileShape &sh) {
    if (m.offsets || m.sys_list || m.count || m.row_stride == 1) return false;
    const int64_t S = (int64_t)1 << sh.S_log2;
    const int64_t ntiles = (m.nsys + S - 1) / S;
    return 3 * (ntiles + 1) * S < ((int64_t)1 << 31);
}

hipError_t launch_perrow(int dtype, const SysMap &map, const Coef &coef, const TileShape &sh,
                         const void *d, void *x, int *err, hipStream_t st) {
    if (!perrow_supported(dtype, sh) || !perrow_layout_ok(map, sh) || coef.mode != TDMA_COEF_LIKE_D ||
        coef.shift != nullptr)
        return hipErrorInvalidValue;
    if (dtype == TDMA_F64) {
        switch (sh.M) {
            case 16: return launch_pr_kind<double, 16, 2>(map, coef, sh, d, x, err, st);
            case 20: return launch_pr_kind<double, 20, 4>(map, coef, sh, d, x, err, st);
            case 24: return launch_pr_kind<double, 24, 4>(map, coef, sh, d, x, err, st);
            case 28: return launch_pr_kind<double, 28, 3>(map, coef, sh, d, x, err, st);
            case 32: return launch_pr_kind<double, 32, 2>(map, coef, sh, d, x, err, st);
        }
        return hipErrorInvalidValue;
    }
    // FP32 above 20 rows: up to 512 lanes a window of four rows, beyond (the
    // 128 registers of 1024 lanes) of two
    const bool wide = sh.threads() > 512;
    switch (sh.M) {
        case 16: return launch_pr_kind<float, 16, 4>(map, coef, sh, d, x, err, st);
        case 20: return launch_pr_kind<float, 20, 4>(map, coef, sh, d, x, err, st);
        case 24: return wide ? launch_pr_kind<float, 24, 2>(map, coef, sh, d, x, err, st)
                             : launch_pr_kind<float, 24, 4, 512>(map, coef, sh, d, x, err, st);
        case 28: return wide ? launch_pr_kind<float, 28, 2>(map, coef, sh, d, x, err, st)
                             : launch_pr_kind<float, 28, 4, 512>(map, coef, sh, d, x, err, st);
        case 32: return wide ? launch_pr_kind<float, 32, 2>(map, coef, sh, d, x, err, st)
                             : launch_pr_kind<float, 32, 4, 512>(map, coef, sh, d, x, err, st);
    }
    return hipErrorInvalidValue;
}

}  // namespace tdma
