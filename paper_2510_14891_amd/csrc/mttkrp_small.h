// One-launch MTTKRP for tensors whose calls are bound by launches and latency (see small.hip).  Internal to
// the library: mttkrp.hip decides when it runs and fills in the problem.
#ifndef MTTKRP_SMALL_H
#define MTTKRP_SMALL_H

#include <hip/hip_runtime.h>

#include <stdint.h>

#include "../../include/mttkrp.h"

constexpr int kSmallModes = MTTKRP_MAX_NDIM - 1;   // column modes at most (d - 1 for k = 0)
constexpr int kSmallWaves = 16;                    // wavefronts per workgroup at most

// How a call is cut up: see mttkrp_small_plan in small.hip.
struct SmallPlan {
    int JB = 1, n_jchunk = 1;        // 16-column blocks of the output per workgroup, workgroups along them
    int RB = 1;                      // 16-row blocks per wavefront
    int waves = 1;                   // wavefronts per workgroup
    int n_tiles = 1;                 // row tiles of 16 RB rows (k != 0: all in one workgroup)
    int n_ranges = 1;                // pieces of the column space (wavefronts of a workgroup take (tile, piece) pairs)
    int cols_per_range = 4;          // multiple of 4
    int n_groups = 1;                // workgroups that share the columns of an output row (1: no partial sums)
    int cols_per_group = 4;
    int64_t blocks = 1;              // workgroups per chunk of output columns and group
};

template <typename T> struct SmallArgs {
    const T* X;
    const T* A0;                     // factor of mode 0 (k != 0)
    const T* A[kSmallModes];         // factors of the column modes, lowest mode first
    T* out;                          // M, or the groups' partial sums (group_stride values apart)
    const T* lambda;
    double beta;
    int32_t dim[kSmallModes], ld[kSmallModes], sx[kSmallModes];   // extents, row strides, strides in X
    uint32_t magic[kSmallModes], shift[kSmallModes];              // q / dim = mulhi(q, magic) >> shift for q < 2^31
    int32_t n;                       // column modes
    int32_t I0, R, C, ld0, ld_out;
    int32_t sx_batch;                // stride of mode k in X
    int32_t n_tiles, n_ranges, cols_per_range, cols_per_group;
    int64_t group_stride, row_stride;  // of the partial sums: group, output row
};

// The launch returns an mttkrp_status.
__attribute__((visibility("hidden"))) SmallPlan mttkrp_small_plan(int ndim, const int64_t* dims, int R, int k, int sbytes, int groups);
// magic and shift for divisions by d >= 2 of numbers below 2^31
__attribute__((visibility("hidden"))) void mttkrp_small_divisor(uint32_t d, uint32_t& magic, uint32_t& shift);
template <typename T>
__attribute__((visibility("hidden"))) int mttkrp_small_launch(const SmallPlan& pl, const SmallArgs<T>& a, bool first_mode, hipStream_t st);

#endif
