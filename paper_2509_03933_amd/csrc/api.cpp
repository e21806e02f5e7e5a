// Host side of the C ABI: argument validation, per-device state, planning of
// tile shapes, dispatch, and the sticky device error flag.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cstdarg>
#include <cstdio>
#include <cstring>
#include <map>
#include <memory>
#include <mutex>
#include <string>
#include <vector>

#include "api_internal.h"

namespace tdma {

// ---------------------------------------------------------------------------
// error state

static thread_local std::string g_last_error;

int fail(int status, const char *fmt, ...) {
    char buf[512];
    va_list ap;
    va_start(ap, fmt);
    vsnprintf(buf, sizeof buf, fmt, ap);
    va_end(ap);
    g_last_error = std::string(tdma_status_string(status)) + ": " + buf;
    return status;
}

int hip_fail(hipError_t e, const char *what) {
    return fail(TDMA_EHIP, "%s: %s", what, hipGetErrorString(e));
}

void clear_error() { g_last_error.clear(); }

// ---------------------------------------------------------------------------
// per-device state

static std::mutex g_mutex;
static std::map<int, std::unique_ptr<DeviceCtx>> g_ctx;

DeviceCtx::~DeviceCtx() { release(); }

void DeviceCtx::release() {
    int cur = -1;
    (void)hipGetDevice(&cur);
    (void)hipSetDevice(dev);
    (void)hipDeviceSynchronize();   // nothing issued may still use what is freed
    for (auto &kv : ragged_cache) free_ragged_plan(&kv.second);
    ragged_cache.clear();
    for (auto &w : workspaces) (void)hipFree(w.ptr);
    workspaces.clear();
    for (auto e : events) (void)hipEventDestroy(e);
    events.clear();
    if (staged_done) (void)hipEventDestroy(staged_done);
    staged_done = nullptr;
    for (auto s : streams) (void)hipStreamDestroy(s);
    streams.clear();
    if (d_err) (void)hipFree(d_err);
    d_err = nullptr;
    if (cur >= 0) (void)hipSetDevice(cur);
}

int get_ctx(DeviceCtx **out) {
    int dev = 0;
    hipError_t e = hipGetDevice(&dev);
    if (e != hipSuccess) return hip_fail(e, "hipGetDevice");
    std::lock_guard<std::mutex> g(g_mutex);
    auto it = g_ctx.find(dev);
    if (it == g_ctx.end()) {
        auto c = std::make_unique<DeviceCtx>();
        c->dev = dev;
        e = hipMalloc(&c->d_err, 4 * sizeof(int));
        if (e != hipSuccess) return fail(TDMA_ENOMEM, "device error flag: %s", hipGetErrorString(e));
        e = hipMemset(c->d_err, 0, 4 * sizeof(int));
        if (e != hipSuccess) return hip_fail(e, "hipMemset");
        hipDeviceProp_t prop;
        if (hipGetDeviceProperties(&prop, dev) == hipSuccess) c->num_cus = prop.multiProcessorCount;
        it = g_ctx.emplace(dev, std::move(c)).first;
    }
    *out = it->second.get();
    return TDMA_OK;
}

// Device workspace of at least `bytes`, tagged by `slot` (kept across calls).
int DeviceCtx::workspace(int slot, size_t bytes, void **out) {
    for (auto &w : workspaces) {
        if (w.slot == slot) {
            if (w.bytes >= bytes) { *out = w.ptr; return TDMA_OK; }
            hipError_t e = hipDeviceSynchronize();
            if (e != hipSuccess) return hip_fail(e, "hipDeviceSynchronize");
            (void)hipFree(w.ptr);
            w.ptr = nullptr;
            w.bytes = 0;
            e = hipMalloc(&w.ptr, bytes);
            if (e != hipSuccess) return fail(TDMA_ENOMEM, "workspace of %zu bytes", bytes);
            w.bytes = bytes;
            *out = w.ptr;
            return TDMA_OK;
        }
    }
    Workspace w;
    w.slot = slot;
    hipError_t e = hipMalloc(&w.ptr, bytes);
    if (e != hipSuccess) return fail(TDMA_ENOMEM, "workspace of %zu bytes", bytes);
    w.bytes = bytes;
    workspaces.push_back(w);
    *out = w.ptr;
    return TDMA_OK;
}

int DeviceCtx::get_streams(int count, hipStream_t **out) {
    while ((int)streams.size() < count) {
        hipStream_t s;
        hipError_t e = hipStreamCreateWithFlags(&s, hipStreamNonBlocking);
        if (e != hipSuccess) return hip_fail(e, "hipStreamCreate");
        streams.push_back(s);
    }
    *out = streams.data();
    return TDMA_OK;
}

int DeviceCtx::get_events(int count, hipEvent_t **out) {
    while ((int)events.size() < count) {
        hipEvent_t ev;
        hipError_t e = hipEventCreateWithFlags(&ev, hipEventDisableTiming);
        if (e != hipSuccess) return hip_fail(e, "hipEventCreate");
        events.push_back(ev);
    }
    *out = events.data();
    return TDMA_OK;
}

// ---------------------------------------------------------------------------
// validation

int validate(const tdma_layout *L, const tdma_coeffs *C, int dtype, const void *d, const void *x) {
    if (!L) return fail(TDMA_EINVAL, "layout is NULL");
    if (!C) return fail(TDMA_EINVAL, "coeffs is NULL");
    if (dtype != TDMA_F64 && dtype != TDMA_F32) return fail(TDMA_EINVAL, "unknown dtype %d", dtype);
    if (!d || !x) return fail(TDMA_EINVAL, "d and x must be non-NULL");
    if (!C->a || !C->b || !C->c) return fail(TDMA_EINVAL, "a, b and c must be non-NULL");
    if (C->mode != TDMA_COEF_LIKE_D && C->mode != TDMA_COEF_SHARED)
        return fail(TDMA_EINVAL, "unknown coefficient mode %d", C->mode);
    if (x == C->a || x == C->b || x == C->c || (C->b_shift && x == C->b_shift))
        return fail(TDMA_EINVAL, "x must not alias the coefficients");
    if (L->nsys0 < 0 || L->nsys1 < 0) return fail(TDMA_EINVAL, "negative system count");
    if (L->nsys1 > 0 && L->nsys0 > INT64_MAX / L->nsys1) return fail(TDMA_EINVAL, "nsys overflows");
    // one workgroup at most per system and 32-bit system indices in the
    // streaming kernels: a call takes fewer than 2^31 systems
    if (L->nsys0 * L->nsys1 > (int64_t)0x7fffffff)
        return fail(TDMA_EUNSUPPORTED, "%lld systems in one call (at most 2^31 - 1; split the batch)",
                    (long long)(L->nsys0 * L->nsys1));
    if (L->offsets) {
        if (L->nsys1 != 1) return fail(TDMA_EINVAL, "ragged layout needs nsys1 == 1");
        if (C->mode != TDMA_COEF_LIKE_D)
            return fail(TDMA_EINVAL, "ragged layout needs per-row (LIKE_D) coefficients");
        for (int64_t k = 0; k < L->nsys0; ++k) {
            const int64_t len = L->offsets[k + 1] - L->offsets[k];
            if (len < 2) return fail(TDMA_EINVAL, "ragged system %lld has %lld rows (< 2)",
                                     (long long)k, (long long)len);
            if (len > kMaxRaggedRows)
                return fail(TDMA_EUNSUPPORTED, "ragged system %lld has %lld rows (> %lld)",
                            (long long)k, (long long)len, (long long)kMaxRaggedRows);
        }
        if (L->offsets[0] < 0) return fail(TDMA_EINVAL, "negative offset");
        return TDMA_OK;
    }
    if (L->nsys0 * L->nsys1 == 0) return TDMA_OK;
    if (L->n < 2) return fail(TDMA_EINVAL, "n = %lld (< 2)", (long long)L->n);
    if (L->row_stride == 0 && L->n > 1) return fail(TDMA_EINVAL, "row_stride is 0");
    if (L->row_stride < 0 || L->sys_stride0 < 0 || L->sys_stride1 < 0)
        return fail(TDMA_EINVAL, "negative stride");
    // the last element any system reaches, in 128-bit arithmetic: device
    // index math is 64-bit, so the layout must span fewer than 2^62 elements
    const __int128 last = (__int128)(L->n - 1) * L->row_stride +
                          (__int128)(L->nsys0 - 1) * L->sys_stride0 +
                          (__int128)(L->nsys1 - 1) * L->sys_stride1;
    if (last >= ((__int128)1 << 62))
        return fail(TDMA_EINVAL, "the layout spans more than 2^62 elements");
    return TDMA_OK;
}

// ---------------------------------------------------------------------------
// planning of the fused path

static int ilog2_floor(int64_t v) {
    int r = 0;
    while ((int64_t)1 << (r + 1) <= v) ++r;
    return r;
}

// Contiguous per-row lines: systems per block (up to 192 lanes) such that the
// fewest lanes of its wavefronts idle, the smaller block on ties (one
// wavefront where that loses nothing: its barriers cost nothing).  Lines of one
// partition take 64 systems (FP32, 2^26 unknowns in lines of 8 rows: 242 us, with 32
// 410).
static int contig_perrow_s_log2(int64_t P) {
    int best = 0;
    double best_use = 0.0;
    for (int s = 0; s <= 6; ++s) {
        const int64_t lanes = P << s;
        if (lanes > 192 && s > 0) break;
        const double use = (double)lanes / (double)((lanes + 63) / 64 * 64);
        if (use > best_use + 1e-9) {
            best = s;
            best_use = use;
        }
    }
    return best;
}

// Built-in tile rule for uniform layouts (the autotune cache overrides it).
// Strided systems: S consecutive systems per tile so that each row load is a
// full 128-byte line (S = 16 in FP64, 32 in FP32); P partitions of M rows so
// that P*M covers n.  Contiguous rows: the tile is staged through LDS.
// Small problems (fewer than 2^20 unknowns; contiguous FP64 lines that take 8
// rows per lane 2^19) are latency-bound: short partitions (M = 4 first) and one system per
// tile, so the solve spreads over as many CUs as it can and each lane's
// serial chain is short.  (A block has 16 lanes at least: shifted x-lines of 2
// rows, 2^19 unknowns, blocks of one lane 60 us, of 16 16.)
// Contiguous per-row FP64 lines beyond that: 8 rows per lane up to 2,048
// rows.  A lane holds all four inputs of its rows, so 8 rows take half the
// registers of 16 and twice the blocks run per CU, one's loads beside the
// other's arithmetic: 120,000 x 720 rows 785 -> 695 us (M = 16, S = 4 against
// M = 8, S = 2), 120,000 x 250 255 -> 228, 16,384 x 1000 161 -> 135, 40,000 x
// 1500 552 -> 511.  Around the line, 2^24 unknowns, 8 rows against 16: 2000 rows
// 136 and 147, 2300 208 and 198, 3000 188 and 166.  In FP32, 16 rows
// take those registers already and 8 measured slower (436 against 515 us).
// Systems per block: contig_perrow_s_log2 (41,856 x 400: S = 1, 50 lanes, 136
// us, S = 2 149; 27,904 x 600: S = 2, 150 lanes, 157, S = 1 176).
// Contiguous lines of a shared operator past the streaming kernel's lengths:
// 8 rows per lane in FP64 and about 512 lanes (16,384 x 2048 315 -> 256 us,
// 11,136 x 3000 529 -> 365; FP32, 16 rows, 11,136 x 3000 331 -> 220), fewer where
// that leaves less than half a block per CU (FP32, 215 x 6000: S = 1 26 us, 2 34).
bool default_shape(int dtype, int64_t n, int64_t nsys, bool contig, bool like_d, bool shift,
                   TileShape *out) {
    const int esz = dtype == TDMA_F64 ? 8 : 4;
    const bool lines = contig && like_d, long_shared = contig && !like_d && !shift;
    const bool rows8 = dtype == TDMA_F64 && ((lines && n <= 2048) || long_shared);
    const bool small = n * nsys < ((int64_t)1 << (rows8 ? 19 : 20));
    const int Ms_rows8[] = {8, 16, 4};
    const int Ms_f64[] = {16, 8, 4};
    const int Ms_f32[] = {16, 32, 8, 4};
    const int Ms_small[] = {4, 8, 16};
    const int *Ms = small ? Ms_small : (rows8 ? Ms_rows8 : (dtype == TDMA_F64 ? Ms_f64 : Ms_f32));
    const int nM = small ? 3 : (dtype == TDMA_F64 ? 3 : 4);
    for (int mi = 0; mi < nM; ++mi) {
        const int M = Ms[mi];
        const int64_t P = (n + M - 1) / M;
        if (P > 1024) continue;
        TileShape sh;
        sh.M = M;
        sh.P = (int)P;
        sh.contig = contig;
        int S_log2 = contig ? ilog2_floor(std::max<int64_t>(1, 256 / P)) : ilog2_floor(128 / esz);
        // short strided lines: a wavefront's worth of lanes (n = 4: 1283 -> 557 us)
        while (!contig && S_log2 < 6 && P << S_log2 < 64) ++S_log2;
        if (lines) S_log2 = contig_perrow_s_log2(P);
        if (long_shared) {
            S_log2 = ilog2_floor(std::max<int64_t>(1, std::min<int64_t>(16 / esz, 768 / P)));
            while (S_log2 > 0 && nsys < ((int64_t)128 << S_log2)) --S_log2;
        }
        const int maxt = fused_max_threads(dtype, M);
        while (S_log2 > 0 && ((int64_t)1 << S_log2) * P > maxt) --S_log2;
        // a tile larger than the number of systems only wastes lanes
        while (S_log2 > 0 && ((int64_t)1 << (S_log2 - 1)) >= nsys) --S_log2;
        if (small) {
            S_log2 = 0;
            while (P << S_log2 < 16) ++S_log2;
        }
        sh.S_log2 = S_log2;
        if (((int64_t)1 << S_log2) * P > maxt) continue;
        if (contig && fused_lds_bytes(dtype, sh) > 96 * 1024) continue;
        *out = sh;
        return true;
    }
    return false;
}

bool default_shared_shape(int dtype, int64_t n, int64_t nsys, bool contig, TileShape *out, bool allow_roll);

// Batches too small to give every CU a tile or two of the walking kernels
// (shared operator; strided rows also with a shift or per-row coefficients):
// the generic kernel with small blocks.  The walking kernels' long unrolled
// bodies and per-block tables pay over many tiles; on a few, each block runs
// its code once, cold, and most CUs have none.  16 rows per lane for strided
// rows (the walking kernels have 8 to 32), 8 for contiguous ones;
// blocks of 128 lanes below 2^19 unknowns, 256 (contiguous 512) above, and
// most of a wavefront at least: short lines take up to 64 systems per block
// (500,000 unknowns in z-lines of 2 rows, FP32 per-row: 118 us in blocks of one
// lane, 7.5 in blocks of 64; walking 36).  The block has its lanes whatever the
// system count: those past the last system load operator rows too.  Walking
// against generic kernel, us per call in a
// captured stream, FP64, lines of n rows x systems: shared z-lines 128 x 64
// 9.7 / 5.1, 1000 x 64 23.1 / 8.7, 1000 x 1024 22.7 / 11.1, 1000 x 2500 28.5 /
// 18.7, 1000 x 4096 26.1 / 26.6; shifted z-lines 250 x 256 8.5 / 5.7, 1000 x
// 1024 20.7 / 11.2, 1000 x 2500 27.8 / 19.1, 1000 x 4096 25.4 / 26.9; shared
// x-lines 250 x 256 18.2 / 8.3, 1000 x 1024 21.1 / 13.7, 777 x 2500 28.9 / 29.0;
// per-row z-lines 250 x 256 15.6 / 6.1, 1000 x 1024 34.7 / 14.6, 512 x 4096
// 17.1 / 19.0.  small_limit draws the line from these.  Contiguous lines that no
// streaming shape holds keep default_shape's tiles, those of fewer than 16 rows
// the streaming kernel (2 rows, 262,144 unknowns: 8.3 / 9.6).  FP32 per-row lines
// of 28 to 128 rows stay with the walking kernel (4.5 against 5.1 us), and so do
// fewer than 16 per-row lines that fill 32 or 64 partitions of 32 rows (8 x 1024,
// FP32, 7.4 against 9.1).  FP32 batches of a
// shared operator keep the shared-operator kernel, whose factors are formed in
// FP64, with small tiles of short partitions (one tile per block on strided
// rows): z-lines 250 x 64 11.6 -> 8.0 us, 1000 x 1024 16.9 -> 13.2, x-lines 250 x
// 64 17.3 -> 8.6, 1000 x 1024 25.1 -> 12.9.
//
// small_limit: the unknowns from which the walking kernels (past 2,048 rows
// default_shape's wider tiles) are the faster ones: 3 x 2^20, and 3 x 2^19 for
// contiguous rows and per-row coefficients.  Earlier where the generic kernel's
// blocks hold few systems or the walking tiles are the best filled, walking
// against generic kernel: shared lines of up to 48 rows 2^20 (40 rows, 2^21.4
// unknowns: 15.0 / 16.9), of more than 1,024 rows 2^21 (2000 rows in y, 2^21.3: 27.6 /
// 38.6; 2^20.9: 27.1 / 24.7), shifted FP64 ones 2^20 (2000 rows in y, 2^21.2: 21.6 /
// 39.5) and 2^21 where they fill 64 partitions (2048 rows, 2^20.8: 35.3 / 25.8), per-row
// lines of 512 rows, which fill 16 partitions, 2^20 (in y, 2^20.2: 15.2 / 24.4).
// FP32 shared ones against their small tiles: 2^20 from 129 to 256 rows (250 rows in
// y, 2^20.3: 1.10 of the walking time), 3 x 2^19 up to 128 rows (2^20.3: 0.86) and
// where the streaming kernel has 12 or 24 rows per lane (640 rows, 2^21.4: 17 / 27;
// 512 rows 13.6 / 11.4).  Past 2,048 rows 2^20 for per-row lines and shifted FP32 ones (4096
// rows, 2^19.3: 29 / 24; 2500 rows, 2^20.3: 27 / 46), none for the others (614 FP64
// lines of 4096 rows: 37 / 50).
static int64_t small_limit(int dtype, int64_t n, int64_t nsys, bool contig, bool like_d, bool shared_op) {
    const int64_t k19 = (int64_t)1 << 19;
    if (contig) return 3 * k19;
    if (n > 2048) return like_d || (dtype == TDMA_F32 && !shared_op) ? 2 * k19 : 0;
    if (like_d) return n == 16 * 32 ? 2 * k19 : 3 * k19;
    if (shared_op) {
        if (n <= 48 || (dtype == TDMA_F32 && n > 128 && n <= 256)) return 2 * k19;
        TileShape w;
        if (dtype == TDMA_F32 &&
            (n <= 128 ||
             (default_shared_shape(dtype, n, nsys, false, &w, true) && (w.M == 12 || w.M == 24))))
            return 3 * k19;
    }
    if (n > 1024 && dtype == TDMA_F64) return shared_op || n == 64 * 32 ? 4 * k19 : 2 * k19;
    return 6 * k19;
}

static bool small_shape(int dtype, int64_t n, int64_t nsys, bool contig, bool like_d, bool shared_op,
                        TileShape *out) {
    if (n > 16384 || (contig && n < 16)) return false;
    if (like_d && dtype == TDMA_F32 && n >= 28 && n <= 128) return false;
    if (like_d && nsys < 16 && (n == 32 * 32 || n == 64 * 32)) return false;
    const int64_t total = n * nsys;
    if (total >= small_limit(dtype, n, nsys, contig, like_d, shared_op)) return false;
    if (shared_op && dtype == TDMA_F32) {
        TileShape sh;
        sh.kernel = contig ? 2 : 1;
        sh.M = n <= 256 ? 8 : (n <= 1024 ? 16 : (n <= 1536 ? 24 : 32));
        if (n > 64 * (int64_t)sh.M) return false;
        sh.P = 1;
        while ((int64_t)sh.P * sh.M < n) sh.P <<= 1;
        sh.contig = contig;
        const int lanes = total >= ((int64_t)1 << 19) ? 512 : (sh.P > 32 ? 256 : 128);
        sh.S_log2 = 4;
        while (sh.S_log2 > 0 && sh.P << sh.S_log2 > lanes) --sh.S_log2;
        while (sh.P << sh.S_log2 < 48) ++sh.S_log2;
        if (!shared_supported(dtype, sh)) return false;
        *out = sh;
        return true;
    }
    for (int M : {contig ? 8 : 16, 16}) {
        const int64_t P = (n + M - 1) / M;
        const int maxt = fused_max_threads(dtype, M);
        if (P > maxt) continue;
        const int64_t lanes = total < ((int64_t)1 << 19) ? 128 : (contig ? 512 : 256);
        TileShape sh;
        sh.kernel = 0;
        sh.M = M;
        sh.P = (int)P;
        sh.contig = contig;
        sh.S_log2 = 4;
        while (sh.S_log2 > 0 && P << sh.S_log2 > lanes) --sh.S_log2;
        while (P << sh.S_log2 < 48) ++sh.S_log2;
        // (per-row lines have no operator rows to load: no lanes past the last system)
        while (like_d && sh.S_log2 > 0 && ((int64_t)1 << (sh.S_log2 - 1)) >= nsys) --sh.S_log2;
        if (!fused_supported(dtype, sh) || (contig && fused_lds_bytes(dtype, sh) > 96 * 1024)) continue;
        *out = sh;
        return true;
    }
    return false;
}

// Shared-operator kernel, streaming form: P a power of two <= 64 (one
// system's interface rows fit one wavefront), M rows per lane from
// {16, 32, 8, 12, 24}, the one that pads the system least (P*M - n; 12 and
// 24 fit the 3*2^k lengths exactly, measured 5-16% faster than padding them
// to 16 or 32); on ties, for strided layouts the one with at most 16
// partitions (whose interface exchange is DPP row shifts; y-lines of
// n = 512: 32 rows x 16 partitions 1.84 ms, 16 x 32 1.97-1.99 ms), then the
// earlier in that order, for contiguous rows the larger M (fewer
// partitions), in FP64 only up to 24 (the streaming blocks of 32 rows hold
// 256 lanes) and only where that takes the partitions below 64 or 32 and not
// below 8 (300,000 x 96: 12 x 8 partitions 92 us, 24 x 4 101).  Strided layouts take
// S = 32 systems per tile (measured best on the 256^3 ADI sweep in FP64 and
// FP32), contiguous rows S = 16 and at least 256 lanes (FP64 at 16 rows and
// 16 partitions or more: S = 8, where two blocks fit a CU's LDS; FP64 at most 32,
// one partition of more than 16 rows 64); both as far as the lanes and LDS
// allow.  Lines of one short partition want the whole block: 33.5 M lines of 2
// rows (FP64) 412 us with 256 systems, 635 with 32, FP32 20 rows 128 with 256, 208
// with 32; but FP64 31 rows 440 with 256, 310 with 64.  Contiguous x-lines of n = 768 (FP64): 24 rows x 32
// partitions x 16 systems 1.94 ms, 12 x 64 x 8 2.26 ms, 24 x 32 x 8 2.68 ms;
// n = 384: 24 x 16 x 16 0.248 ms, 12 x 32 x 8 0.279 ms; 167,680 x 200: 16 x 16 x 8
// 0.118, 16 x 16 x 16 0.130; 480,000 x 250: 0.393, 0.383, 32 x 8 x 32 0.495; 100,000 x 512: 16 x 32 x 8 0.182, 16 x 32 x 16
// 0.195, 32 x 16 x 16 0.225; 62,500 x 1000: 16 x 64 x 8 0.246, 32 x 32 x 8 0.287.
// A streaming
// block holds its CU's LDS for the whole launch, so the whole 160 KB is
// available to it.  allow_roll admits the rolling form (kernel 6) below; the
// streamed copy keeps the two-set shape, whose lane bound its kernel shares.
bool default_shared_shape(int dtype, int64_t n, int64_t nsys, bool contig, TileShape *out,
                          bool allow_roll) {
    const int Ms[] = {16, 32, 8, 12, 24};
    bool found = false;
    TileShape best;
    for (int M : Ms) {
        int64_t P = 1;
        while (P * M < n) P <<= 1;
        if (P > 64) continue;
        TileShape sh;
        sh.kernel = 2;
        sh.M = M;
        sh.P = (int)P;
        sh.contig = contig;
        int64_t S_want = contig ? std::max<int64_t>(16, 256 / P) : 32;
        if (contig && dtype == TDMA_F64 && (P > 1 || M > 16)) S_want = std::min<int64_t>(S_want, P > 1 ? 32 : 64);
        if (contig && dtype == TDMA_F64 && M == 16 && P >= 16) S_want = 8;
        int S_log2 = ilog2_floor(S_want);
        const int maxt = shared_max_threads(dtype, M, sh.kernel, contig);
        while (S_log2 > 0 && ((int64_t)1 << S_log2) * P > maxt) --S_log2;
        while (S_log2 > 0 && ((int64_t)1 << (S_log2 - 1)) >= nsys) --S_log2;
        sh.S_log2 = S_log2;
        while (sh.S_log2 > 0 && shared_lds_bytes(dtype, sh) > 160 * 1024) --sh.S_log2;
        if (!shared_supported(dtype, sh)) continue;
        const int64_t pad = (int64_t)sh.P * sh.M, best_pad = found ? (int64_t)best.P * best.M : 0;
        const bool tie_wins = contig ? sh.M > best.M && (dtype == TDMA_F32 || (sh.M < 32 && best.P > 8))
                                     : (sh.P <= 16 && best.P > 16);
        if (!found || pad < best_pad || (pad == best_pad && tie_wins)) {
            best = sh;
            found = true;
        }
    }
    // Strided rows whose two-set streaming tile is narrower than a 128-byte
    // line (its lanes are capped where M rows fill 192 bytes: the 1536-row
    // z-lines of the large sweeps take 8 systems), with partitions that cover
    // n exactly: the rolling form holds one register set and fits the full
    // 128-byte width (z-lines of 1536 rows: 3.24 -> 2.44 ms).
    const int esz = dtype == TDMA_F64 ? 8 : 4;
    if (found && allow_roll && !contig && (int64_t)best.P * best.M == n &&
        ((int64_t)esz << best.S_log2) < 128) {
        TileShape r = best;
        r.kernel = 6;
        r.S_log2 = ilog2_floor(128 / esz);
        const int maxt = shared_max_threads(dtype, r.M, 6, false);
        while (r.S_log2 > 0 && ((int64_t)1 << r.S_log2) * r.P > maxt) --r.S_log2;
        while (r.S_log2 > 0 && ((int64_t)1 << (r.S_log2 - 1)) >= nsys) --r.S_log2;
        while (r.S_log2 > 0 && shared_lds_bytes(dtype, r) > 160 * 1024) --r.S_log2;
        if (r.S_log2 > best.S_log2 && shared_supported(dtype, r)) best = r;
    }
    if (found) *out = best;
    return found;
}

// Shared operator with a per-system shift on a strided layout (the
// FFT-Poisson lines).  FP64 above 256 rows: the walk that recomputes its pivots
// (kernel 7), P the fewest partitions (16, 32 or 64) of at most 32 rows, the
// rows spread evenly over them in M = 20, 24, 28 or 32 slots, and S = 32
// consecutive systems (256-byte rows; 16 with 64 partitions).  Above 896 rows,
// where the tiles are few (2.5 per CU; 0.75 where the slots stay a quarter empty in
// kernel 3) and the rows lie less than 32 KB apart: kernel 3, whose shorter chain
// per tile and half as wide tiles fill the chip sooner (y-lines of 256 systems,
// 2^22 unknowns, 2000 rows: 22.5 against 38; 2^24.5: 0.87 of kernel 3's time in
// kernel 7; z-lines of 1000 rows, 2^22.3: kernel 7 0.78).  Up to 256 rows:
// lengths that fill partitions of 32 rows take the rolling walk that keeps
// its pivots (kernel 3) with S = 32, others the generic kernel (false).  FP32:
// kernel 3, M = 32 rows per lane (else 16, 8), P a power of two <= 64, S = 32.
// Measured on 2^27 unknowns in lines along z (FP64, us): n = 1024 kernel 7 509,
// kernel 3 with 16 x 32 x 32 538, 16 x 64 x 16 675; n = 300 kernel 7 480, kernel 3
// with identity rows past the end 729, 640 495 and 797, 1000 540 and 629, 2048
// 665 and 1043; n = 64 kernel 3
// 453 (S = 16 498, kernel 7 472), 256 458 (538, 494); n = 40 generic 498, kernel
// 3 with identity rows 1158, 100 464 and 624, 200 488 and 647.
static bool default_shift_shape(int dtype, int64_t n, int64_t nsys, int64_t row_stride, TileShape *out) {
    TileShape sh;
    sh.contig = false;
    if (dtype == TDMA_F64) {
        int64_t P = 1;
        while (P * 32 < n) P <<= 1;
        if (P > 64) return false;
        sh.P = (int)P;
        if (n <= 256) {
            if (P * 32 != n) return false;
            sh.kernel = 3;
            sh.M = 32;
        } else {
            sh.kernel = 7;
            sh.M = (int)(((n + P - 1) / P + 3) / 4 * 4);
        }
        sh.S_log2 = P > 32 ? 4 : 5;
        const int64_t tiles_min = 4 * n < 3 * 32 * P ? 192 : 640;
        if (sh.kernel == 7 && n > 896 && (P > 32 || n < 32 * P) && row_stride < 4096 &&
            nsys < tiles_min << sh.S_log2) {
            sh.kernel = 3;
            sh.M = 32;
            --sh.S_log2;
        }
        while (sh.S_log2 > 0 && ((int64_t)1 << (sh.S_log2 - 1)) >= nsys) --sh.S_log2;
        if (!shift_uneven(n, sh) && !shift_supported(dtype, sh)) return false;
        *out = sh;
        return true;
    }
    for (int M : {32, 16, 8}) {
        int64_t P = 1;
        while (P * M < n) P <<= 1;
        if (P > 64) continue;
        sh.kernel = 3;
        sh.M = M;
        sh.P = (int)P;
        int S_log2 = 5;
        while (S_log2 > 0 && ((int64_t)1 << S_log2) * P > 1024) --S_log2;
        while (S_log2 > 0 && ((int64_t)1 << (S_log2 - 1)) >= nsys) --S_log2;
        sh.S_log2 = S_log2;
        if (!shift_supported(dtype, sh)) continue;
        *out = sh;
        return true;
    }
    return false;
}

// Per-row coefficients on strided layouts: the walking kernel.  P the fewest
// partitions (a power of two) of at most 32 rows, the rows spread evenly over
// them; M the slots that hold ceil(n/P) rows (16, 20, 24, 28 or 32).  S
// systems so that a tile fills 512 lanes (FP32 1024 from 16 partitions on,
// 512 there for M above 24 unless n fills it), halved to no less than a
// 128-byte tile row while the tiles are fewer than two per CU (FP32 to 64 bytes,
// 32 with 64 partitions, while they are fewer than 128: 2048 rows, 2^20.7
// unknowns in y, 8 systems 24 us, 16 37; 1024 rows, 2^21, 16 systems 27, 32 33).
// FP32 lines of 64 and 128 rows below 2^19 unknowns take 16 rows per lane (64 x
// 1024 5.7 us, 32 rows 7.1).  Measured on
// 2^26 unknowns in lines along z, us, against the best of 16 and 32 rows per
// lane with identity rows past the end and 64- or 128-byte tile rows: FP64 n =
// 100 490, 16 x 8 x 32 545; 500 558, 730; 512 555, 643; 768 603, 914; 1000 640,
// 829; 1024 711, 711; 1500 912; FP32 300 297, 457; 768 315, 699; 1024 391, 712.
// FP32 lines that leave M = 32 partly empty go to the generic kernel (1000
// rows 400 against 414, 1800 507 against 617), and so do lines of fewer than
// 28 rows (FP64 n = 20: 524 against 819).
static bool default_perrow_shape(int dtype, int64_t n, int64_t nsys, TileShape *out) {
    if (n < 28) return false;   // no 16-row slots that two partitions nearly fill
    int64_t P = 2;
    while (P * 32 < n) P <<= 1;
    if (P > 64) return false;
    TileShape sh;
    sh.kernel = 5;
    // FP32 below 2^19 unknowns: 16 rows where they fill exactly
    if (dtype == TDMA_F32 && n <= 128 && n == 32 * P && n * nsys < ((int64_t)1 << 19)) P *= 2;
    sh.M = (int)std::max<int64_t>(16, ((n + P - 1) / P + 3) / 4 * 4);
    sh.P = (int)P;
    sh.contig = false;
    const bool full = P * sh.M == n;
    if (dtype == TDMA_F32 && sh.M == 32 && !full && P >= 32) return false;
    const bool wide = dtype == TDMA_F32 && P >= 16 && (P > 16 || sh.M <= 24 || full);
    const int64_t S_min = 128 / (dtype == TDMA_F64 ? 8 : 4);
    int64_t S = std::min<int64_t>(128, (wide ? 1024 : 512) / P);
    while (S > S_min && nsys < S * 512) S >>= 1;
    while (dtype == TDMA_F32 && S > (P > 32 ? 8 : 16) && nsys < S * 128) S >>= 1;
    while (S > 1 && S / 2 >= nsys) S >>= 1;
    sh.S_log2 = ilog2_floor(S);
    if (!perrow_supported(dtype, sh)) return false;
    *out = sh;
    return true;
}

// Ragged layout: systems are bucketed by the power-of-two partition count
// they need; one launch per non-empty bucket (contiguous rows, LDS-staged).
// build_ragged_plan allocates the plan's device tables and uploads them
// synchronously; the caller owns them (free_ragged_plan).
// Bucket of a ragged system of len rows: 16 rows per lane, P the power of two
// that covers len / 16.  With the four per-row arrays loaded at once and staged
// without bank conflicts, 16 rows per lane measured faster than 8 on the
// longest systems (FP64, 6,144 rows: 118 against 143 us for 1,245 systems), and
// in FP32 than 32 (10,000 systems of 32 to 8,192 rows 133 against 120 us).
static void ragged_bucket(int64_t len, int *M_out, int *P_out) {
    const int64_t P = (len + 15) / 16;
    int64_t Pb = 1;
    while (Pb < P) Pb <<= 1;
    *M_out = 16;
    *P_out = (int)std::min<int64_t>(Pb, 1 << 30);
}

// min_block, the smallest block of the per-row tile list (lanes): on the
// 10,000 systems of 32..8192 rows (FP64) alone, blocks of 512 lanes
// throughout 248 us, 256 and 512 227 us, 128, 256 and 512 242 us (each block
// size is a launch of its own); beside the 768x512x1536 sweeps in a graph
// the 256-lane blocks take CUs from the sweeps (graph 6.79 -> 6.86 ms), so
// graphs build their plans with 512-lane blocks (FP32 systems of more than
// 8,192 rows 1024; 1024 for all of them slowed 50,000 FP32 systems of 500 to 1,000
// rows from 323 to 350 us).
int build_ragged_plan(const tdma_layout *L, int dtype, RaggedPlan *out, int min_block) {
    const int64_t nsys = L->nsys0;
    std::map<std::pair<int, int>, std::vector<int32_t>> buckets;   // (M, P) -> systems
    for (int64_t k = 0; k < nsys; ++k) {
        const int64_t len = L->offsets[k + 1] - L->offsets[k];
        int M, P;
        ragged_bucket(len, &M, &P);
        buckets[{M, P}].push_back((int32_t)k);
    }
    for (auto &kv : buckets)
        if (kv.first.second > fused_max_threads(dtype, kv.first.first))
            return fail(TDMA_EUNSUPPORTED, "a ragged system needs %d partitions of %d rows (max %d)",
                        kv.first.second, kv.first.first, fused_max_threads(dtype, kv.first.first));
    RaggedPlan rp;
    rp.nsys = nsys;
    rp.dtype = dtype;
    rp.offsets.assign(L->offsets, L->offsets + nsys + 1);
    std::vector<int32_t> all;
    for (auto &kv : buckets) {
        const int M = kv.first.first, P = kv.first.second;
        RaggedBucket b;
        b.shape.M = M;
        b.shape.P = P;
        b.shape.contig = true;
        int S_log2 = ilog2_floor(std::max(1, 256 / P));
        while (S_log2 > 0 && (P << S_log2) > fused_max_threads(dtype, M)) --S_log2;
        b.shape.S_log2 = S_log2;
        b.first = (int64_t)all.size();
        b.count = (int64_t)kv.second.size();
        all.insert(all.end(), kv.second.begin(), kv.second.end());
        rp.buckets.push_back(b);
    }
    // the tile-list form: per rows-per-lane class, tiles of every bucket
    // (longest systems first) whose S*P lanes fill a block of
    // max(min_block, P) lanes: smaller blocks let two run on a CU at once,
    // one block's loads beside the other's arithmetic (one launch per block
    // size)
    std::vector<RaggedTile> tiles;
    auto block_of = [&](int M, int P) {
        const int maxt = fused_max_threads(dtype, M);
        return std::min(maxt, std::max(min_block, P));
    };
    std::vector<std::pair<int, int>> classes;   // (M, block lanes), largest blocks first
    for (const RaggedBucket &b : rp.buckets) {
        const std::pair<int, int> c{b.shape.M, block_of(b.shape.M, b.shape.P)};
        if (std::find(classes.begin(), classes.end(), c) == classes.end()) classes.push_back(c);
    }
    std::sort(classes.begin(), classes.end(),
              [](const std::pair<int, int> &x, const std::pair<int, int> &y) {
                  return x.first != y.first ? x.first < y.first : x.second > y.second;
              });
    bool groups_ok = true;
    for (const auto &cl : classes) {
        const int M = cl.first;
        if (!fused_tiles_supported(dtype, M)) { groups_ok = false; break; }
        RaggedGroup g;
        g.M = M;
        g.threads = cl.second;
        g.first_tile = (int64_t)tiles.size();
        std::vector<const RaggedBucket *> bs;
        for (const RaggedBucket &b : rp.buckets)
            if (b.shape.M == M && block_of(M, b.shape.P) == cl.second) bs.push_back(&b);
        if (bs.empty()) continue;
        std::sort(bs.begin(), bs.end(),
                  [](const RaggedBucket *x, const RaggedBucket *y) { return x->shape.P > y->shape.P; });
        for (const RaggedBucket *b : bs) {
            const int P = b->shape.P;
            if (P > g.threads) { groups_ok = false; break; }
            const int S = g.threads / P;
            TileShape sh;
            sh.M = M;
            sh.P = P;
            sh.S_log2 = ilog2_floor(S);
            sh.contig = true;
            g.lds = std::max(g.lds, fused_lds_bytes(dtype, sh));
            for (int64_t k = 0; k < b->count; k += S) {
                RaggedTile t;
                t.first = (int32_t)(b->first + k);
                t.count = (int32_t)std::min<int64_t>(S, b->count - k);
                t.P_log2 = ilog2_floor(P);
                t.S_log2 = sh.S_log2;
                tiles.push_back(t);
            }
        }
        g.ntiles = (int64_t)tiles.size() - g.first_tile;
        if (g.lds > 160 * 1024) groups_ok = false;
        if (!groups_ok) break;
        rp.groups.push_back(g);
    }
    if (!groups_ok || tiles.size() > (size_t)INT32_MAX) {
        rp.groups.clear();
        tiles.clear();
    }
    hipError_t e = hipMalloc(&rp.d_offsets, (nsys + 1) * sizeof(int64_t));
    if (e != hipSuccess) return fail(TDMA_ENOMEM, "ragged offsets");
    e = hipMalloc(&rp.d_list, std::max<size_t>(1, all.size()) * sizeof(int32_t));
    if (e != hipSuccess) { (void)hipFree(rp.d_offsets); return fail(TDMA_ENOMEM, "ragged list"); }
    if (!tiles.empty()) {
        e = hipMalloc(&rp.d_tiles, tiles.size() * sizeof(RaggedTile));
        if (e != hipSuccess) {
            rp.d_tiles = nullptr;
            free_ragged_plan(&rp);
            return fail(TDMA_ENOMEM, "ragged tiles");
        }
    }
    e = hipMemcpy(rp.d_offsets, L->offsets, (nsys + 1) * sizeof(int64_t), hipMemcpyHostToDevice);
    if (e == hipSuccess && !all.empty())
        e = hipMemcpy(rp.d_list, all.data(), all.size() * sizeof(int32_t), hipMemcpyHostToDevice);
    if (e == hipSuccess && !tiles.empty())
        e = hipMemcpy(rp.d_tiles, tiles.data(), tiles.size() * sizeof(RaggedTile), hipMemcpyHostToDevice);
    if (e != hipSuccess) {
        free_ragged_plan(&rp);
        return hip_fail(e, "upload ragged plan");
    }
    *out = rp;
    return TDMA_OK;
}

void free_ragged_plan(RaggedPlan *rp) {
    if (rp->d_offsets) (void)hipFree(rp->d_offsets);
    if (rp->d_list) (void)hipFree(rp->d_list);
    if (rp->d_tiles) (void)hipFree(rp->d_tiles);
    rp->d_tiles = nullptr;
    rp->d_offsets = nullptr;
    rp->d_list = nullptr;
}

// Plans of recently seen ragged layouts, keyed by a hash of the offsets and
// confirmed by comparing the offsets and dtype in full.
int plan_ragged(DeviceCtx *ctx, const tdma_layout *L, int dtype, const RaggedPlan **out) {
    const int64_t nsys = L->nsys0;
    uint64_t h = 1469598103934665603ull;
    for (int64_t k = 0; k <= nsys; ++k) {
        h ^= (uint64_t)L->offsets[k];
        h *= 1099511628211ull;
    }
    h ^= (uint64_t)dtype * 0x9E3779B97F4A7C15ull;
    auto it = ctx->ragged_cache.find(h);
    if (it != ctx->ragged_cache.end() && it->second.nsys == nsys && it->second.dtype == dtype &&
        std::equal(it->second.offsets.begin(), it->second.offsets.end(), L->offsets)) {
        *out = &it->second;
        return TDMA_OK;
    }
    RaggedPlan rp;
    int rc = build_ragged_plan(L, dtype, &rp);
    if (rc != TDMA_OK) return rc;
    if (ctx->ragged_cache.size() >= 8 || it != ctx->ragged_cache.end()) {
        // full (or a hash collision): drop the cached plans (the stream
        // order keeps launches already issued from them valid: their device
        // tables are freed only after a device synchronisation)
        (void)hipDeviceSynchronize();
        for (auto &kv : ctx->ragged_cache) free_ragged_plan(&kv.second);
        ctx->ragged_cache.clear();
    }
    auto res = ctx->ragged_cache.emplace(h, std::move(rp));
    *out = &res.first->second;
    return TDMA_OK;
}

SysMap make_map(const tdma_layout *L) {
    SysMap m;
    m.n = L->n;
    m.nsys = L->nsys0 * L->nsys1;
    m.nsys0 = std::max<int64_t>(1, L->nsys0);
    m.row_stride = L->row_stride;
    m.sys_stride0 = L->sys_stride0;
    m.sys_stride1 = L->sys_stride1;
    m.offsets = nullptr;
    m.sys_list = nullptr;
    m.count = nullptr;
    return m;
}

Coef make_coef(const tdma_coeffs *C) {
    Coef c;
    c.mode = C->mode;
    c.a = C->a;
    c.b = C->b;
    c.c = C->c;
    c.shift = C->b_shift;
    return c;
}

// Per-row coefficients without a shift: one launch per rows-per-lane class
// of the plan's tile list.  Otherwise one launch per bucket.
int launch_ragged(const RaggedPlan &rp, const tdma_layout *L, const tdma_coeffs *C, int dtype,
                  const void *d, void *x, int *err, hipStream_t st, const hipStream_t *aux,
                  int naux, const hipEvent_t *ev) {
    const Coef coef = make_coef(C);
    if (C->mode == TDMA_COEF_LIKE_D && C->b_shift == nullptr && !rp.groups.empty()) {
        for (const RaggedGroup &g : rp.groups) {
            SysMap m = make_map(L);
            m.offsets = rp.d_offsets;
            m.sys_list = rp.d_list;
            const hipError_t e = launch_fused_tiles(dtype, g.M, m, coef, d, x, rp.d_tiles + g.first_tile,
                                                    g.ntiles, g.threads, g.lds, err, st);
            if (e != hipSuccess) return hip_fail(e, "fused launch (ragged tiles)");
        }
        return TDMA_OK;
    }
    const int nb = (int)rp.buckets.size();
    // a stream for every two buckets: forking one more and joining it costs more
    // than a small bucket's launch (2,000 shifted FP32 systems of 8 to 64 rows,
    // three buckets: 63 us on two streams, 73 on three)
    const int nuse = std::max(0, std::min(naux, nb / 2));
    hipError_t e = hipSuccess;
    if (nuse > 0) {
        e = hipEventRecord(ev[0], st);
        for (int i = 0; i < nuse && e == hipSuccess; ++i) e = hipStreamWaitEvent(aux[i], ev[0], 0);
        if (e != hipSuccess) return hip_fail(e, "ragged fork");
    }
    for (int k = 0; k < nb; ++k) {
        const RaggedBucket &b = rp.buckets[k];
        const int lane = k % (nuse + 1);
        SysMap m = make_map(L);
        m.n = (int64_t)b.shape.P * b.shape.M;
        m.nsys = b.count;
        m.offsets = rp.d_offsets;
        m.sys_list = rp.d_list + b.first;
        e = launch_fused(dtype, m, coef, b.shape, d, x, err, lane == 0 ? st : aux[lane - 1]);
        if (e != hipSuccess) return hip_fail(e, "fused launch (ragged)");
    }
    for (int i = 0; i < nuse && e == hipSuccess; ++i) {
        e = hipEventRecord(ev[1 + i], aux[i]);
        if (e == hipSuccess) e = hipStreamWaitEvent(st, ev[1 + i], 0);
    }
    if (e != hipSuccess) return hip_fail(e, "ragged join");
    return TDMA_OK;
}

// Kernels 3, 4 and 7 on systems of n rows: kernel 7 on partitions that cover n
// exactly or (FP64) leave few of their slots empty.
static bool shift_shape_ok(int dtype, int64_t n, const TileShape &sh) {
    if (shift_supported(dtype, sh)) return sh.kernel != 7 || (int64_t)sh.P * sh.M == n || shift_uneven(n, sh);
    if (dtype != TDMA_F64 || sh.P < 1 || !shift_uneven(n, sh)) return false;
    TileShape widest = sh;
    widest.M = 32;
    return shift_supported(dtype, widest);
}

// Whether a tile shape can run a uniform layout with these coefficients.
bool shape_fits(int dtype, const tdma_layout *L, bool shared_op, const TileShape &sh,
                bool shifted_op, bool perrow_op) {
    if ((int64_t)sh.P * sh.M < L->n) return false;
    if (sh.kernel == 3 || sh.kernel == 4 || sh.kernel == 7)
        return shifted_op && shift_shape_ok(dtype, L->n, sh) && shift_layout_ok(make_map(L), sh);
    if (sh.kernel == 5) {
        if (!perrow_op || !perrow_supported(dtype, sh) || !perrow_layout_ok(make_map(L), sh)) return false;
        return sh.M == 16 || sh.M == 32 || perrow_uneven(L->n, sh);
    }
    if (sh.kernel == 1 || sh.kernel == 2) return shared_op && shared_supported(dtype, sh);
    if (sh.kernel == 6) return shared_op && shared_supported(dtype, sh) && shared_roll_ok(make_map(L), sh);
    if (sh.kernel != 0 || !fused_supported(dtype, sh)) return false;
    return !(sh.contig && fused_lds_bytes(dtype, sh) > 160 * 1024);
}

// The built-in rules (shared-operator kernel first where it applies); false: n is
// too long for the fused path.
bool builtin_shape(const tdma_layout *L, const tdma_coeffs *C, int dtype, TileShape *out) {
    const int64_t nsys = L->nsys0 * L->nsys1;
    const bool contig = L->row_stride == 1;
    const bool shared_op = C->mode == TDMA_COEF_SHARED && C->b_shift == nullptr;
    const bool shifted_op = C->mode == TDMA_COEF_SHARED && C->b_shift != nullptr;
    const bool perrow_op = C->mode == TDMA_COEF_LIKE_D && C->b_shift == nullptr;
    TileShape ssh;
    if ((contig ? shared_op && default_shared_shape(dtype, L->n, nsys, true, &ssh, true)
                : shared_op || shifted_op || perrow_op) &&
        small_shape(dtype, L->n, nsys, contig, perrow_op, shared_op, &ssh)) {
        *out = ssh;
        return true;
    }
    if ((shifted_op && !contig && default_shift_shape(dtype, L->n, nsys, L->row_stride, &ssh) &&
         shift_layout_ok(make_map(L), ssh)) ||
        (perrow_op && !contig && default_perrow_shape(dtype, L->n, nsys, &ssh) &&
         perrow_layout_ok(make_map(L), ssh))) {
        *out = ssh;
        return true;
    }
    if (shared_op && default_shared_shape(dtype, L->n, nsys, contig, &ssh, true)) {
        if (ssh.kernel == 6 && !shared_roll_ok(make_map(L), ssh))
            default_shared_shape(dtype, L->n, nsys, contig, &ssh, false);
        *out = ssh;
        return true;
    }
    return default_shape(dtype, L->n, nsys, contig, C->mode == TDMA_COEF_LIKE_D, C->b_shift != nullptr, out);
}

// Tile shape of a uniform layout: the forced shape, else the autotune cache
// (an entry that no longer fits, e.g. from an edited cache file, is
// ignored), else the built-in rules.
int plan_uniform(DeviceCtx *ctx, const tdma_layout *L, const tdma_coeffs *C, int dtype,
                 const TileShape *force, TileShape *out) {
    TileShape sh;
    const bool contig = L->row_stride == 1;
    const bool shared_op = C->mode == TDMA_COEF_SHARED && C->b_shift == nullptr;
    const bool shifted_op = C->mode == TDMA_COEF_SHARED && C->b_shift != nullptr;
    const bool perrow_op = C->mode == TDMA_COEF_LIKE_D && C->b_shift == nullptr;
    if (force) {
        sh = *force;
        if ((int64_t)sh.P * sh.M < L->n)
            return fail(TDMA_EINVAL, "tile shape M=%d P=%d S=%d does not cover n=%lld", sh.M, sh.P,
                        1 << sh.S_log2, (long long)L->n);
        if ((sh.kernel == 1 || sh.kernel == 2 || sh.kernel == 6) && !shared_op)
            return fail(TDMA_EINVAL, "the shared-operator kernel needs shared coefficients without "
                        "a shift (M=%d P=%d S=%d)", sh.M, sh.P, 1 << sh.S_log2);
        if ((sh.kernel == 3 || sh.kernel == 4 || sh.kernel == 7) && !shifted_op)
            return fail(TDMA_EINVAL, "the shifted-operator kernel needs shared coefficients with "
                        "a shift (M=%d P=%d S=%d)", sh.M, sh.P, 1 << sh.S_log2);
        if (sh.kernel == 5 && !perrow_op)
            return fail(TDMA_EINVAL, "the per-row kernel needs per-row coefficients without a "
                        "shift (M=%d P=%d S=%d)", sh.M, sh.P, 1 << sh.S_log2);
        if (!shape_fits(dtype, L, shared_op, sh, shifted_op, perrow_op))
            return fail(TDMA_EINVAL, "unsupported tile shape M=%d P=%d S=%d (kernel %d)", sh.M, sh.P,
                        1 << sh.S_log2, sh.kernel);
    } else if (!(lookup_tuned(ctx->dev, L, C, dtype, &sh) && sh.contig == contig &&
                 shape_fits(dtype, L, shared_op, sh, shifted_op, perrow_op))) {
        if (!builtin_shape(L, C, dtype, &sh))
            return fail(TDMA_EUNSUPPORTED, "n = %lld is too long for the fused path (use "
                        "tdma_solve_partitioned)", (long long)L->n);
    }
    *out = sh;
    return TDMA_OK;
}

int launch_uniform(const TileShape &sh, const tdma_layout *L, const tdma_coeffs *C, int dtype,
                   const void *d, void *x, int *err, hipStream_t st) {
    const SysMap m = make_map(L);
    if (m.nsys == 0) return TDMA_OK;
    const Coef coef = make_coef(C);
    hipError_t e;
    if (sh.kernel == 3 || sh.kernel == 4 || sh.kernel == 7)
        e = launch_shift(dtype, m, coef, sh, d, x, err, st);
    else if (sh.kernel == 5)
        e = launch_perrow(dtype, m, coef, sh, d, x, err, st);
    else if (sh.kernel != 0)
        e = launch_shared(dtype, m, coef, sh, d, x, err, st);
    else
        e = launch_fused(dtype, m, coef, sh, d, x, err, st);
    if (e != hipSuccess) return hip_fail(e, "fused launch");
    return TDMA_OK;
}

int run_fused(DeviceCtx *ctx, const tdma_layout *L, const tdma_coeffs *C, int dtype, const void *d,
              void *x, hipStream_t st, const TileShape *force) {
    if (L->offsets) {
        // A ragged call builds (or finds in the library's cache) a plan whose
        // device tables it allocates and uploads synchronously, and a cache
        // entry can later be freed: neither may happen inside, or be recorded
        // by, a capture the caller started.  Graphs of ragged solves are made
        // by tdma_graph_create, which gives them tables of their own.
        hipStreamCaptureStatus cs = hipStreamCaptureStatusNone;
        const hipError_t ce = hipStreamIsCapturing(st, &cs);
        if (ce != hipSuccess) return hip_fail(ce, "hipStreamIsCapturing");
        if (cs != hipStreamCaptureStatusNone)
            return fail(TDMA_EUNSUPPORTED, "a ragged layout cannot be solved on a stream that is being "
                        "captured (use tdma_graph_create)");
        const RaggedPlan *rp = nullptr;
        int rc = plan_ragged(ctx, L, dtype, &rp);
        if (rc != TDMA_OK) return rc;
        // buckets on the caller's stream and kRaggedAux library streams at once
        hipStream_t *aux = nullptr;
        hipEvent_t *ev = nullptr;
        rc = ctx->get_streams(kRaggedAux, &aux);
        if (rc == TDMA_OK) rc = ctx->get_events(kRaggedAux + 1, &ev);
        if (rc != TDMA_OK) return rc;
        return launch_ragged(*rp, L, C, dtype, d, x, ctx->d_err, st, aux, kRaggedAux, ev);
    }
    if (L->nsys0 * L->nsys1 == 0) return TDMA_OK;
    TileShape sh;
    int rc = plan_uniform(ctx, L, C, dtype, force, &sh);
    if (rc != TDMA_OK) return rc;
    return launch_uniform(sh, L, C, dtype, d, x, ctx->d_err, st);
}

}  // namespace tdma

using namespace tdma;

extern "C" {

const char *tdma_status_string(int status) {
    switch (status) {
        case TDMA_OK: return "TDMA_OK";
        case TDMA_EINVAL: return "TDMA_EINVAL (invalid argument)";
        case TDMA_ENOMEM: return "TDMA_ENOMEM (allocation failed)";
        case TDMA_EHIP: return "TDMA_EHIP (HIP runtime error)";
        case TDMA_ESINGULAR: return "TDMA_ESINGULAR (zero or non-finite pivot)";
        case TDMA_ENOCONV: return "TDMA_ENOCONV (refinement did not converge)";
        case TDMA_EUNSUPPORTED: return "TDMA_EUNSUPPORTED (unsupported combination)";
        default: return "unknown tdma status";
    }
}

const char *tdma_last_error(void) { return g_last_error.c_str(); }

int tdma_solve_batched(const tdma_layout *layout, const tdma_coeffs *coeffs, int dtype,
                       const void *d, void *x, void *stream) {
    clear_error();
    int rc = validate(layout, coeffs, dtype, d, x);
    if (rc != TDMA_OK) return rc;
    DeviceCtx *ctx = nullptr;
    rc = get_ctx(&ctx);
    if (rc != TDMA_OK) return rc;
    std::lock_guard<std::mutex> lk(ctx->mu);
    return run_fused(ctx, layout, coeffs, dtype, d, x, (hipStream_t)stream, nullptr);
}

int tdma_solve_batched_tiled(const tdma_layout *layout, const tdma_coeffs *coeffs, int dtype,
                             const void *d, void *x, const tdma_tile *tile, void *stream) {
    clear_error();
    int rc = validate(layout, coeffs, dtype, d, x);
    if (rc != TDMA_OK) return rc;
    if (!tile) return fail(TDMA_EINVAL, "tile is NULL");
    if (layout->offsets) return fail(TDMA_EINVAL, "explicit tiles need a uniform layout");
    const int S = tile->systems_per_tile;
    if (S < 1 || (S & (S - 1)) != 0) return fail(TDMA_EINVAL, "systems_per_tile must be a power of two");
    TileShape sh;
    sh.M = tile->rows_per_lane;
    sh.P = tile->partitions;
    sh.S_log2 = 0;
    while ((1 << sh.S_log2) < S) ++sh.S_log2;
    sh.contig = layout->row_stride == 1;
    sh.kernel = tile->kernel;
    if (sh.kernel < 0 || sh.kernel > 7) return fail(TDMA_EINVAL, "unknown kernel %d", sh.kernel);
    if (sh.kernel == 0 && !fused_supported(dtype, sh))
        return fail(TDMA_EINVAL, "unsupported tile M=%d S=%d P=%d", sh.M, S, sh.P);
    if ((sh.kernel == 3 || sh.kernel == 4 || sh.kernel == 7) && !shift_supported(dtype, sh))
        return fail(TDMA_EINVAL, "unsupported shifted-operator tile M=%d S=%d P=%d", sh.M, S, sh.P);
    if (sh.kernel == 5 && (!perrow_supported(dtype, sh) || (sh.M != 16 && sh.M != 32) ||
                           (sh.M == 32 && sh.threads() > 512)))
        return fail(TDMA_EINVAL, "unsupported per-row tile M=%d S=%d P=%d", sh.M, S, sh.P);
    if ((sh.kernel == 1 || sh.kernel == 2 || sh.kernel == 6) && !shared_supported(dtype, sh))
        return fail(TDMA_EINVAL, "unsupported shared-operator tile M=%d S=%d P=%d", sh.M, S, sh.P);
    if (sh.kernel == 7 && (int64_t)sh.M * sh.P != layout->n)
        return fail(TDMA_EINVAL, "kernel 7 needs partitions that cover n exactly (M=%d P=%d, n = %lld)",
                    sh.M, sh.P, (long long)layout->n);
    if (sh.kernel == 6 && !shared_roll_ok(make_map(layout), sh))
        return fail(TDMA_EINVAL, "kernel 6 needs strided rows and partitions that cover n exactly "
                    "(M=%d P=%d, n = %lld)", sh.M, sh.P, (long long)layout->n);
    if ((int64_t)sh.M * sh.P < layout->n) return fail(TDMA_EINVAL, "tile covers %lld rows < n = %lld",
                                                      (long long)sh.M * sh.P, (long long)layout->n);
    if (sh.kernel == 0 && sh.contig && fused_lds_bytes(dtype, sh) > 160 * 1024)
        return fail(TDMA_EINVAL, "tile needs %zu bytes of LDS", fused_lds_bytes(dtype, sh));
    DeviceCtx *ctx = nullptr;
    rc = get_ctx(&ctx);
    if (rc != TDMA_OK) return rc;
    std::lock_guard<std::mutex> lk(ctx->mu);
    return run_fused(ctx, layout, coeffs, dtype, d, x, (hipStream_t)stream, &sh);
}

int tdma_copy_streamed(const tdma_layout *layout, int dtype, const void *src, void *dst,
                       void *stream) {
    clear_error();
    if (src == dst && src) return fail(TDMA_EINVAL, "src and dst must differ");
    tdma_coeffs none{};   // validation only, never read
    none.a = none.b = none.c = src;
    none.mode = TDMA_COEF_SHARED;
    int rc = validate(layout, &none, dtype, src, dst);
    if (rc != TDMA_OK) return rc;
    if (layout->offsets) return fail(TDMA_EUNSUPPORTED, "the streamed copy takes uniform layouts");
    if (layout->row_stride == 1)
        return fail(TDMA_EUNSUPPORTED, "the streamed copy follows the strided solve (row_stride != 1)");
    const int64_t nsys = layout->nsys0 * layout->nsys1;
    if (nsys == 0) return TDMA_OK;
    TileShape sh;
    if (!default_shared_shape(dtype, layout->n, nsys, false, &sh, false))
        return fail(TDMA_EUNSUPPORTED, "n = %lld has no streaming shape", (long long)layout->n);
    const SysMap map = make_map(layout);
    if (!copy_streamed_supported(map, sh))
        return fail(TDMA_EUNSUPPORTED, "layout beyond the streaming walk's 32-bit indices");
    DeviceCtx *ctx = nullptr;
    rc = get_ctx(&ctx);
    if (rc != TDMA_OK) return rc;
    std::lock_guard<std::mutex> lk(ctx->mu);
    const hipError_t e = launch_copy_streamed(dtype, map, sh, src, dst, (hipStream_t)stream);
    if (e != hipSuccess) return hip_fail(e, "streamed copy launch");
    return TDMA_OK;
}

int tdma_solve_pdd(const tdma_layout *layout, const tdma_coeffs *coeffs, int dtype,
                   int rows_per_partition, const void *d, void *x, void *stream) {
    clear_error();
    int rc = validate(layout, coeffs, dtype, d, x);
    if (rc != TDMA_OK) return rc;
    if (layout->offsets) return fail(TDMA_EINVAL, "the PDD solve takes uniform layouts");
    const int m = rows_per_partition;
    TileShape sh;
    sh.kernel = 0;
    sh.M = m;
    sh.pdd = true;
    sh.contig = layout->row_stride == 1;
    sh.S_log2 = 0;
    sh.P = 1;
    if (!fused_supported(dtype, sh))
        return fail(TDMA_EINVAL, "rows_per_partition = %d (4, 8 or 16; 32 too in FP32)", m);
    const int64_t nsys = layout->nsys0 * layout->nsys1;
    if (nsys == 0) return TDMA_OK;
    const int64_t P = (layout->n + m - 1) / m;
    const int maxt = fused_max_threads(dtype, m);
    if (P > maxt)
        return fail(TDMA_EUNSUPPORTED, "n = %lld needs %lld partitions of %d rows (at most %d)",
                    (long long)layout->n, (long long)P, m, maxt);
    sh.P = (int)P;
    const int esz = dtype == TDMA_F64 ? 8 : 4;
    int S_log2 = sh.contig ? ilog2_floor(std::max<int64_t>(1, 256 / P)) : ilog2_floor(128 / esz);
    while (S_log2 > 0 && ((int64_t)1 << S_log2) * P > maxt) --S_log2;
    while (S_log2 > 0 && ((int64_t)1 << (S_log2 - 1)) >= nsys) --S_log2;
    sh.S_log2 = S_log2;
    while (sh.contig && sh.S_log2 > 0 && fused_lds_bytes(dtype, sh) > 96 * 1024) --sh.S_log2;
    if (sh.contig && fused_lds_bytes(dtype, sh) > 160 * 1024)
        return fail(TDMA_EUNSUPPORTED, "a tile of n = %lld contiguous rows exceeds the LDS",
                    (long long)layout->n);
    DeviceCtx *ctx = nullptr;
    rc = get_ctx(&ctx);
    if (rc != TDMA_OK) return rc;
    std::lock_guard<std::mutex> lk(ctx->mu);
    return launch_uniform(sh, layout, coeffs, dtype, d, x, ctx->d_err, (hipStream_t)stream);
}

int tdma_solve_multi(const tdma_layout *layout, const tdma_coeffs *coeffs, int dtype, int nrhs,
                     int64_t rhs_stride, const void *d, void *x, void *stream) {
    clear_error();
    int rc = validate(layout, coeffs, dtype, d, x);
    if (rc != TDMA_OK) return rc;
    if (layout->offsets) return fail(TDMA_EINVAL, "several right-hand sides need a uniform layout");
    if (coeffs->mode != TDMA_COEF_SHARED)
        return fail(TDMA_EUNSUPPORTED, "several right-hand sides share one operator "
                                       "(mode TDMA_COEF_SHARED)");
    if (nrhs < 1) return fail(TDMA_EINVAL, "nrhs = %d (< 1)", nrhs);
    if (rhs_stride < 0) return fail(TDMA_EINVAL, "negative rhs_stride");
    if (nrhs > 1 && rhs_stride == 0) return fail(TDMA_EINVAL, "rhs_stride is 0 with nrhs = %d", nrhs);
    const int64_t nsys = layout->nsys0 * layout->nsys1;
    if (nsys == 0) return TDMA_OK;
    const __int128 last = (__int128)(layout->n - 1) * layout->row_stride +
                          (__int128)(layout->nsys0 - 1) * layout->sys_stride0 +
                          (__int128)(layout->nsys1 - 1) * layout->sys_stride1 +
                          (__int128)(nrhs - 1) * rhs_stride;
    if (last >= ((__int128)1 << 62))
        return fail(TDMA_EINVAL, "the layout and its right-hand sides span more than 2^62 elements");
    MultiShape sh;
    if (!multi_shape(dtype, layout->n, nsys, &sh))
        return fail(TDMA_EUNSUPPORTED, "n = %lld is longer than the %d rows the multi-right-hand-side "
                    "kernel holds", (long long)layout->n, dtype == TDMA_F64 ? 1024 : 2048);
    const size_t esz = dtype == TDMA_F64 ? 8 : 4;
    const auto even = [](int64_t v) { return (v & 1) == 0; };
    const bool vec = nrhs >= 2 && rhs_stride == 1 && even(layout->row_stride) &&
                     (layout->nsys0 == 1 || even(layout->sys_stride0)) &&
                     (layout->nsys1 == 1 || even(layout->sys_stride1)) &&
                     (uintptr_t)d % (2 * esz) == 0 && (uintptr_t)x % (2 * esz) == 0;
    DeviceCtx *ctx = nullptr;
    rc = get_ctx(&ctx);
    if (rc != TDMA_OK) return rc;
    std::lock_guard<std::mutex> lk(ctx->mu);
    const hipError_t e = launch_multi(dtype, make_map(layout), make_coef(coeffs), sh, nrhs,
                                      rhs_stride, vec, d, x, ctx->d_err, (hipStream_t)stream);
    if (e != hipSuccess) return hip_fail(e, "multi-right-hand-side launch");
    return TDMA_OK;
}

int tdma_check(void *stream) {
    clear_error();
    DeviceCtx *ctx = nullptr;
    int rc = get_ctx(&ctx);
    if (rc != TDMA_OK) return rc;
    hipError_t e = hipStreamSynchronize((hipStream_t)stream);
    if (e != hipSuccess) return hip_fail(e, "hipStreamSynchronize");
    std::lock_guard<std::mutex> lk(ctx->mu);
    int flag[4] = {0, 0, 0, 0};
    e = hipMemcpy(flag, ctx->d_err, sizeof flag, hipMemcpyDeviceToHost);
    if (e != hipSuccess) return hip_fail(e, "read error flag");
    if (flag[0]) {
        e = hipMemset(ctx->d_err, 0, 4 * sizeof(int));
        if (e != hipSuccess) return hip_fail(e, "clear error flag");
        return fail(TDMA_ESINGULAR, "a kernel met a zero or non-finite pivot");
    }
    return TDMA_OK;
}

void tdma_shutdown(void) {
    std::lock_guard<std::mutex> g(g_mutex);
    g_ctx.clear();
    clear_tuned();
}

}  // extern "C"
