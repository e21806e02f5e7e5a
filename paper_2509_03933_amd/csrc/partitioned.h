// Launchers of the staged (split) path, partitioned.hip.
#pragma once
#include "tdma_internal.h"

namespace tdma {

// Workspace of one batch: the recurrence states Stage A keeps for Stage C
// (nseg per partition; keep_rows: of every row), the reduced rows, the
// interface solution and the scratch of the sequential Stage B.
struct StageWs {
    void *ws_d = nullptr, *ws_a = nullptr, *ws_c = nullptr;
    double *red = nullptr, *X = nullptr, *scratch = nullptr;
    int nseg = 0;
    bool keep_rows = false;
};

// Bytes of the workspace for `batch` of the map's systems in P partitions;
// with mem, `out` points into it (mem null: the size alone).
size_t stage_ws(int dtype, const SysMap &map, const Coef &coef, int64_t batch, int P, void *mem,
                StageWs *out);

hipError_t launch_stage_a(int dtype, const SysMap &map, const Coef &coef, const void *d,
                          const StageWs &w, int64_t k_begin, int64_t nb, int P, int *err,
                          hipStream_t st);
hipError_t launch_stage_b(const StageWs &w, int64_t nb, int P, int *err, hipStream_t st);
hipError_t launch_stage_c(int dtype, const SysMap &map, const Coef &coef, const void *d, void *x,
                          const StageWs &w, int64_t k_begin, int64_t nb, int P, hipStream_t st);

}  // namespace tdma
