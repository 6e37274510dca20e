// Contraction over the leading index through LDS (see contract.hip).  Internal to the library.
#ifndef MTTKRP_CONTRACT_H
#define MTTKRP_CONTRACT_H

#include <hip/hip_runtime.h>

#include <stdint.h>

#include "../../include/mttkrp.h"

#define MTTKRP_INTERNAL __attribute__((visibility("hidden")))

struct ContractPlan {
    bool ok = false;             // the kernel takes this shape
    int JB = 1;                  // 16-column blocks of the output
    int CW = 4;                  // wavefronts along the tensor columns, 16 each
    int64_t n_ctile = 1;         // tiles of 16 CW tensor columns
    int n_rsplit = 1;
    int64_t rows_per_split = 0;  // a stage's rows at least (the last split takes what is left)
    int chain = 0;               // fp32: stages that are added in fp32 before they go into fp64 sums (0: all of a split)
    int64_t n_items = 1;
    int grid = 1;                // persistent workgroups
};

template <typename T> struct ContractArgs {
    const T* X;                  // P x Q, first index fastest
    const T* K;                  // P x R, row-major, leading dimension ldK
    T* out;                      // row c, split s at out + (c n_rsplit + s) ld_out
    int64_t P, Q, ldK, ld_out;
    int64_t rows_per_split, n_items;
    int32_t R, n_rsplit, n_ctile, chain;
};

// max_splits: row splits at most; target_items > 0: row splits until that many work items exist; max_rows > 0: rows per
// split at most; fp32: max_chain > 0: rows that are added in fp32 at most (else those of a split, at most 4096)
MTTKRP_INTERNAL ContractPlan mttkrp_contract_plan(int64_t P, int64_t Q, int R, int sbytes, int64_t max_splits, int64_t target_items,
                                                  int64_t max_rows, int64_t max_chain);
template <typename T>
MTTKRP_INTERNAL int mttkrp_contract_launch(const ContractPlan& pl, const ContractArgs<T>& a, hipStream_t st);

// What the shared sweep calls.  compact: with plans of little workspace for sweeps that take too much of it otherwise (no
// workgroups that share a small tensor's columns, any chosen streaming plan, the kernel through LDS wherever it can run).
MTTKRP_INTERNAL size_t mttkrp_dense_bytes(int ndim, const int64_t* dims, int R, int k, int sbytes, bool compact);
MTTKRP_INTERNAL size_t mttkrp_leading_bytes(int64_t P, int64_t Q, int R, int sbytes, bool compact);
template <typename T>
MTTKRP_INTERNAL int mttkrp_dense_run(int ndim, const int64_t* dims, const T* X, const T* const* factors, int R, int k, T* M,
                                     void* workspace, size_t workspace_bytes, void* stream, bool compact);
template <typename T>
MTTKRP_INTERNAL int mttkrp_leading_run(int64_t P, int64_t Q, const T* X, const T* K, int R, T* out, void* workspace,
                                       size_t workspace_bytes, void* stream, bool compact);

// A mode's result from the contraction over mode 0, S(q, s, j) (see mttkrp_modesum_kernel).
template <typename T, typename TP> struct ModeSumArgs {
    const T* S;                  // [q][n_split][R]
    TP* part;                    // [i_t][segment][R]
    const T* A[MTTKRP_MAX_NDIM]; // factors of the modes of q (entry t is not read)
    int64_t ld[MTTKRP_MAX_NDIM];
    int32_t dim[MTTKRP_MAX_NDIM];
    int64_t ld_part;             // row stride of part
    int32_t n, t, R;
    uint32_t n_split, n_pairs, per_seg;      // pairs (o, s) in all, and per segment
};
template <typename T, typename TP>
MTTKRP_INTERNAL int mttkrp_modesum_launch(const ModeSumArgs<T, TP>& a, int64_t I_t, int n_seg, hipStream_t st);

#endif
