// Minimal CP-ALS driver and all-modes sweep on top of the dense MTTKRP.
// C ABI, the iteration and its conventions: include/mttkrp_cpals.h.  Everything
// but the MTTKRP itself is small (R x R or I_k x R) and runs in plain fp64 HIP
// kernels with fixed-order reductions.
#include <hip/hip_runtime.h>

#include <math.h>
#include <stdint.h>
#include <string.h>

#include <chrono>
#include <type_traits>

#include "../../include/mttkrp.h"
#include "../../include/mttkrp_cpals.h"
#include "mttkrp_contract.h"

namespace {

constexpr int kSmallRank = 64;     // up to here the R x R matrices are handled in one workgroup's LDS
constexpr int kNormBlocks = 4096;  // partial sums of ||X||^2
constexpr int kGramBlocks = 128;   // workgroups of an update (ranks up to 64) at most
constexpr int kScaleBlocks = 256;  // ... of its second launch
constexpr int kFitChunks = 256;    // row chunks of the fit's inner product (ranks above 64)
constexpr int kFailed = 1, kStopped = 2;       // values of the flag: a pivot that is not positive; the fit has settled

__host__ __device__ inline int64_t ceil_div(int64_t a, int64_t b) { return (a + b - 1) / b; }

// Sum of 256 per-thread values in a fixed tree order; result in every thread.
__device__ __forceinline__ double block_sum_256(double v, double* lds)
{
    lds[threadIdx.x] = v;
    __syncthreads();
    for (int s = 128; s > 0; s >>= 1) {
        if ((int)threadIdx.x < s)
            lds[threadIdx.x] += lds[threadIdx.x + s];
        __syncthreads();
    }
    const double r = lds[0];
    __syncthreads();
    return r;
}

// partial[b] = sum of squares of block b's share of X (fixed assignment and order).  One read of X at
// what a plain stream reaches: four 16-byte non-temporal loads in flight per lane, blocks interleaved
// (8 GB: 1.41 ms with one 8-byte load in flight, contiguous shares; 1.20 ms so).  X is 8-byte aligned;
// an odd first value and a last one are added by block 0.
typedef double double2_t __attribute__((ext_vector_type(2)));
typedef double double4_t __attribute__((ext_vector_type(4)));
__global__ void __launch_bounds__(256) sumsq_partial(const double* __restrict__ X, int64_t N, double* partial)
{
    __shared__ double lds[256];
    const int64_t head = ((uintptr_t)X & 15u) != 0 ? 1 : 0;
    const double2_t* const x2 = (const double2_t*)(X + head);
    const int64_t n2 = (N - head) >> 1;
    const int64_t stride = (int64_t)gridDim.x * 256;
    int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
    double s = 0.0;
    for (; i + 3 * stride < n2; i += 4 * stride) {
        double2_t v[4];
#pragma unroll
        for (int u = 0; u < 4; ++u)
            v[u] = __builtin_nontemporal_load(x2 + i + u * stride);
#pragma unroll
        for (int u = 0; u < 4; ++u)
            s += v[u].x * v[u].x + v[u].y * v[u].y;
    }
    for (; i < n2; i += stride) {
        const double2_t v = x2[i];
        s += v.x * v.x + v.y * v.y;
    }
    if (blockIdx.x == 0 && threadIdx.x == 0) {
        if (head)
            s += X[0] * X[0];
        if (head + 2 * n2 < N)
            s += X[N - 1] * X[N - 1];
    }
    s = block_sum_256(s, lds);
    if (threadIdx.x == 0)
        partial[blockIdx.x] = s;
}

// Sum of v[b * stride] for b = first, first + by, ... below n, eight requested before the first is added, in order.
__device__ __forceinline__ double sum_strided(const double* __restrict__ v, int first, int by, int n, int64_t stride)
{
    double s = 0.0;
    for (int b = first; b < n; b += 8 * by) {
        double t[8];
#pragma unroll
        for (int u = 0; u < 8; ++u)
            t[u] = v[(int64_t)min(b + u * by, n - 1) * stride];
#pragma unroll
        for (int u = 0; u < 8; ++u)
            s += b + u * by < n ? t[u] : 0.0;
    }
    return s;
}

// The Gram matrices of the factors a call starts from (ranks up to 64): workgroups [first[m], first[m + 1]) take the rows of mode m, a
// wavefront 16 at a time, and leave partial matrices ws[workgroup][R * R]; gram_reduce adds a mode's.
struct GramSet {
    const double* A[MTTKRP_MAX_NDIM];
    int64_t I[MTTKRP_MAX_NDIM];
    int32_t first[MTTKRP_MAX_NDIM + 1];
};
// workgroups for a mode: 1 to 4 MB of partial matrices at most
int gram_blocks(int64_t I, int R)
{
    const int64_t n = ceil_div(I, 64), most = R <= 16 ? 512 : (R <= 32 ? 256 : 128);
    return (int)(n < most ? n : most);
}
// The accumulators of the pairs of column blocks (p, q), p >= q: += Y^T Y of 16 rows, of which lane (n16, kq) holds y[u][s] = (4 s + kq, 16 u + n16).
template <int NB> __device__ __forceinline__ void gram_rows(double4_t (&acc)[NB * (NB + 1) / 2], const double (&y)[NB][4])
{
#pragma unroll
    for (int p = 0; p < NB; ++p)
#pragma unroll
        for (int q = 0; q <= p; ++q)
#pragma unroll
            for (int s = 0; s < 4; ++s)
                acc[p * (p + 1) / 2 + q] = __builtin_amdgcn_mfma_f64_16x16x4f64(y[p][s], y[q][s], acc[p * (p + 1) / 2 + q], 0, 0, 0);
}
template <int NB> __global__ void __launch_bounds__(256) gram_partial(const GramSet g, int ndim, int R, double* __restrict__ ws)
{
    constexpr int PAIRS = NB * (NB + 1) / 2;
    __shared__ double red[3][PAIRS][256];
    int m = 0;
    while (m + 1 < ndim && (int)blockIdx.x >= g.first[m + 1])
        ++m;
    const int tid = (int)threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6), n16 = lane & 15, kq = lane >> 4;
    const double* const A = g.A[m];
    const int64_t I = g.I[m], n_tiles = ceil_div(I, 16), step = 4 * (g.first[m + 1] - g.first[m]);
    double4_t acc[PAIRS];
#pragma unroll
    for (int i = 0; i < PAIRS; ++i)
        acc[i] = {0.0, 0.0, 0.0, 0.0};
    for (int64_t t = 4 * ((int)blockIdx.x - g.first[m]) + wave; t < n_tiles; t += step) {
        double y[NB][4];
#pragma unroll
        for (int s = 0; s < 4; ++s) {
            const int64_t r = 16 * t + 4 * s + kq;
#pragma unroll
            for (int u = 0; u < NB; ++u) {
                const double v = A[(r < I ? r : I - 1) * R + min(16 * u + n16, R - 1)];
                y[u][s] = r < I && 16 * u + n16 < R ? v : 0.0;
            }
        }
        gram_rows<NB>(acc, y);
    }
    if (wave > 0) {
#pragma unroll
        for (int i = 0; i < PAIRS; ++i)
#pragma unroll
            for (int q = 0; q < 4; ++q)
                red[wave - 1][i][64 * q + lane] = acc[i][q];
    }
    __syncthreads();
    if (wave > 0)
        return;
    double* const out = ws + (int64_t)blockIdx.x * R * R;
#pragma unroll
    for (int p = 0; p < NB; ++p)
#pragma unroll
        for (int q = 0; q <= p; ++q)
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                const int i = p * (p + 1) / 2 + q, r = 16 * p + 4 * e + kq, c = 16 * q + n16;
                const double v = ((acc[i][e] + red[0][i][64 * e + lane]) + red[1][i][64 * e + lane]) + red[2][i][64 * e + lane];
                if (r < R && c < R) {
                    out[r * R + c] = v;
                    if (p != q)
                        out[c * R + r] = v;
                }
            }
}

// G[m] = sum of mode m's partial matrices, 64 entries a workgroup, a wavefront for an eighth of the matrices; and where blockIdx.y is
// ndim, norm2[0] = ||X||^2 from its n_norm partial sums and the flag cleared.  Fixed orders.
__global__ void __launch_bounds__(512) gram_reduce(const GramSet g, const double* __restrict__ ws, int ndim, int RR, double* G,
                                                   const double* __restrict__ norm_part, int n_norm, double* norm2, int* flag)
{
    __shared__ double red[512];
    const int tid = (int)threadIdx.x, lane = tid & 63, wave = tid >> 6, m = (int)blockIdx.y;
    if (m == ndim) {
        if (blockIdx.x > 0)
            return;
        red[tid] = sum_strided(norm_part, tid, 512, n_norm, 1);
        __syncthreads();
        for (int s = 256; s > 0; s >>= 1) {
            if (tid < s)
                red[tid] += red[tid + s];
            __syncthreads();
        }
        if (tid == 0) {
            norm2[0] = red[0];
            flag[0] = 0;
        }
        return;
    }
    const int e = min((int)blockIdx.x * 64 + lane, RR - 1);
    red[tid] = sum_strided(ws + (int64_t)g.first[m] * RR + e, wave, 8, g.first[m + 1] - g.first[m], RR);
    __syncthreads();
    if (wave == 0 && (int)blockIdx.x * 64 + lane < RR) {
        double v = 0.0;
        for (int q = 0; q < 8; ++q)
            v += red[64 * q + lane];
        G[(int64_t)m * RR + e] = v;
    }
}

// The power of two whose square brings a diagonal entry of V to [1, 4).  V is factorised as S V S and the rows of M and A
// are multiplied by S: products with powers of two are exact, and the pivots and their reciprocals stay normal
// numbers for start factors of any scale.
__device__ __forceinline__ double unit_scale(double d) { return d > 0.0 && d < INFINITY ? ldexp(1.0, -(ilogb(d) >> 1)) : 1.0; }

// S V S with V = Hadamard product of the Gram matrices of all modes but `skip`, and the diagonal of S.  L (ldL x ldL) gets zeros
// in its rows and columns from R on.
__global__ void __launch_bounds__(256) hadamard_grams(const double* __restrict__ G, int ndim, int R, int skip, double* V, double* S,
                                                      double* L, int ldL)
{
    const int e = blockIdx.x * 256 + threadIdx.x, RR = R * R;
    if (e >= RR) {
        const int pad = ldL - R, t = e - RR;         // columns R .. of all rows, then rows R .. of the others
        if (t < ldL * pad)
            L[(int64_t)(t / pad) * ldL + R + t % pad] = 0.0;
        else if (t < ldL * pad + pad * R)
            L[(int64_t)R * ldL + (int64_t)((t - ldL * pad) / R) * ldL + (t - ldL * pad) % R] = 0.0;
        return;
    }
    const int a = e / R, c = e - a * R;
    double v = 1.0, da = 1.0, dc = 1.0;
    for (int m = 0; m < ndim; ++m)
        if (m != skip) {
            v *= G[(int64_t)m * RR + e];
            da *= G[(int64_t)m * RR + (int64_t)a * R + a];
            dc *= G[(int64_t)m * RR + (int64_t)c * R + c];
        }
    da = unit_scale(da);
    V[e] = v * da * unit_scale(dc);
    if (a == c)
        S[a] = da;
}

// ---------------------------------------------------------------------------
// Update of one factor: A_k = M V^{-1} with V = L D L^T (unit lower L; the pivots are those of the
// Cholesky factorisation, squared), then the columns' 2-norms, the normalised columns and their Gram
// matrix.  These steps are short chains, bound by launches and by latency, not by arithmetic.
// ---------------------------------------------------------------------------

// The failure flag, read once for a whole workgroup.  In the kernels that factorise V, workgroup 0 may set it while others
// are still starting: read by each wavefront for itself, some of a workgroup could leave and the rest go on with
// columns in LDS that nobody wrote.  (Every workgroup finds the same bad pivot, so it does not matter which value it sees.)
__device__ __forceinline__ bool failed_before(const int* flag) { return __syncthreads_or(flag[0]) != 0; }

// 1 / d for a pivot of the scaled V: the hardware estimate and two Newton steps (an IEEE division is
// three times as long a chain, and a step of the factorisation waits for it).  Against a Cholesky factor with
// divisions and square roots the factors of one sweep are 0.95 times as far from extended precision (384 calls, R = 3 to 97).
__device__ __forceinline__ double reciprocal(double d)
{
    double r = __builtin_amdgcn_rcp(d);
    r = fma(fma(-d, r, 1.0), r, r);
    r = fma(fma(-d, r, 1.0), r, r);
    return r;
}

// The value of lane n of each 16 lanes in all of them, and acc += that value of a times b in one instruction (the compiler makes
// a copy, a wait and a move of it; the two wait states are those between a register's write and its use by DPP).
template <int n> __device__ __forceinline__ double row_value(double v) { return __builtin_amdgcn_update_dpp(0.0, v, 0x150 + n, 0xf, 0xf, true); }
template <int n> __device__ __forceinline__ void row_fma(double& acc, double a, double b)
{
    asm("s_nop 1\n\tv_fmac_f64_dpp %0, %1, %2 row_newbcast:%3 row_mask:0xf bank_mask:0xf" : "+v"(acc) : "v"(a), "v"(b), "n"(n));
}
// Steps 0 .. N - 1, with the step as a constant.
template <int N, int n = 0, typename Step> __device__ __forceinline__ void steps(Step step)
{
    if constexpr (n < N) {
        step(std::integral_constant<int, n>());
        steps<N, n + 1>(step);
    }
}

// Column j of the factorisation below: a[i] += (a[i] of lane j) * t * r for i = j + 1 .. 15, t being minus the pivot row where it is still to
// be used and r the reciprocal of the pivot; and the next pivot d and its reciprocal (as reciprocal() has it), whose chain of
// dependent instructions lies between the row operations: those of a column after it took 165 cycles a column.  One block, so that nothing
// comes between its instructions: a register is read by DPP two wait states after it was written, and the estimate of the reciprocal one.
template <int j> __device__ __forceinline__ void pivot_column(double (&a)[16], double t, double& d, double& r)
{
    double w, e, dn, rn;
#define PC_ROW(i) ".if " #i " > %c21\n\tv_fmac_f64_dpp %" #i ", %" #i ", %16 row_newbcast:%c21 row_mask:0xf bank_mask:0xf\n\t.endif\n\t"
#define PC_AT(i, k, op) ".if " #i " == %c21 + " #k "\n\t" op "\n\t.endif\n\t"
#define PC_PIVOT(i) "v_mov_b64_dpp %18, %" #i " row_newbcast:" #i " row_mask:0xf bank_mask:0xf"
#define PC_RCP "v_rcp_f64 %19, %18"
#define PC_E "v_fma_f64 %17, -%18, %19, 1.0"
#define PC_R "v_fma_f64 %19, %17, %19, %19"
// (i: the row; p: the row three before it, the next pivot's where i == j + 4)
#define PC_STEP(i, p) PC_AT(i, 4, PC_PIVOT(p)) PC_AT(i, 5, PC_RCP) PC_AT(i, 7, PC_E) PC_AT(i, 8, PC_R) PC_AT(i, 9, PC_E) PC_AT(i, 10, PC_R) PC_ROW(i)
// (what the rows left have no place for)
#define PC_LAST(k, op) ".if %c21 + " #k " > 15\n\ts_nop 1\n\t" op "\n\t.endif\n\t"
#define PC_LAST_PIVOT(i) ".if " #i " == %c21 + 1 && %c21 + 4 > 15\n\ts_nop 1\n\t" PC_PIVOT(i) "\n\t.endif\n\t"
    asm("s_nop 1\n\tv_mul_f64 %16, %20, %22\n\t" PC_ROW(1) PC_ROW(2) PC_ROW(3) PC_STEP(4, 1) PC_STEP(5, 2) PC_STEP(6, 3) PC_STEP(7, 4) PC_STEP(8, 5)
            PC_STEP(9, 6) PC_STEP(10, 7) PC_STEP(11, 8) PC_STEP(12, 9) PC_STEP(13, 10) PC_STEP(14, 11) PC_STEP(15, 12)
                PC_LAST_PIVOT(13) PC_LAST_PIVOT(14) PC_LAST_PIVOT(15) PC_LAST(5, PC_RCP) PC_LAST(7, PC_E) PC_LAST(8, PC_R) PC_LAST(9, PC_E) PC_LAST(10, PC_R)
        : "+v"(a[0]), "+v"(a[1]), "+v"(a[2]), "+v"(a[3]), "+v"(a[4]), "+v"(a[5]), "+v"(a[6]), "+v"(a[7]), "+v"(a[8]), "+v"(a[9]),
          "+v"(a[10]), "+v"(a[11]), "+v"(a[12]), "+v"(a[13]), "+v"(a[14]), "+v"(a[15]), "=&v"(w), "=&v"(e), "=&v"(dn), "=&v"(rn)
        : "v"(t), "n"(j), "v"(r));
#undef PC_LAST_PIVOT
#undef PC_LAST
#undef PC_STEP
#undef PC_R
#undef PC_E
#undef PC_RCP
#undef PC_PIVOT
#undef PC_AT
#undef PC_ROW
    d = dn;
    r = rn;
}

// L D L^T of a 16 x 16 block by one wavefront without barriers: lane c of each 16 lanes (all four hold the same) has column c in
// a[0 .. 15], the whole symmetric block, so that the pivot row is a register and the pivot column a lane's registers.
// Afterwards a[i] = L(i, c) D(c) for i > c; dinv[0 .. 15] (LDS) = 1 / D.  False when a pivot is not positive.
__device__ __forceinline__ bool factorise16(double (&a)[16], double* dinv)
{
    const int c = (int)threadIdx.x & 15;
    double d = row_value<0>(a[0]), r = reciprocal(d);
    bool ok = d > 0.0;
    dinv[0] = r;
    steps<15>([&](auto J) {
        constexpr int j = decltype(J)::value;
        pivot_column<j>(a, c > j ? -a[j] : 0.0, d, r);
        ok = ok && d > 0.0;
        dinv[j + 1] = r;
    });
    return ok;
}

// v / n with 1 / n at hand: the product and one correction, which leaves it within the rounding of a division (n from about 1e-162 to
// 1e154, as norms are).
__device__ __forceinline__ double quotient(double v, double n, double inverse)
{
    const double q = v * inverse;
    return fma(fma(-n, q, v), inverse, q);
}

// The end of a sweep on the device: fit = 1 - sqrt(max(||X||^2 + ||X^||^2 - 2 <X, X^>, 0)) / ||X|| into the sweep's record, and
// the flag that ends the updates (kStopped) when it has changed by less than tol.  The host reads the records of many sweeps
// at once: a wait for the GPU and the launches after it cost 40 us, as much as a sweep over a small tensor.
constexpr int kRecords = 16;                   // sweeps between two reads at most
constexpr double kWaitUs = 40.0, kAheadUs = 2000.0;
struct SweepRecord { double fit; int64_t status; };      // status: 0 go on, kStopped this was the last sweep, -1 not run, kFailed
__device__ void end_sweep(double* scalars, int* flag, SweepRecord* record, double inner, double model2, double tol, bool first)
{
    if (flag[0] != 0) {
        record->status = flag[0] == kFailed ? kFailed : -1;
        return;
    }
    const double norm2 = scalars[0], norm = sqrt(norm2);
    double resid2 = norm2 + model2 - 2.0 * inner;
    // What is left below the rounding of the three terms is none: an exact model's fit is 1 in every sweep, not 1 or 1 - 2e-8 by how the
    // last sums were rounded (which of the two depends on the order of the MTTKRP's sums).
    if (resid2 < 8.0 * 0x1p-52 * norm2)
        resid2 = 0.0;
    const double fit = norm > 0.0 ? 1.0 - sqrt(resid2) / norm : 1.0;
    const bool settled = !first && fabs(fit - scalars[1]) < tol;
    scalars[1] = fit;
    record->fit = fit;
    record->status = settled ? kStopped : 0;
    if (settled)
        flag[0] = kStopped;
}
// ... and where a sweep's last update leaves it (record == nullptr: not the last one)
struct SweepEnd {
    double* scalars;
    SweepRecord* record;
    double tol;
    bool first;
};

// y[t] += (y[t] of lane a of each 16 lanes) * f[a] for a = 0 .. 15 in order (FORWARD) or 15 .. 0: the substitution with a unit triangular 16 x 16
// block, for 16 rows of which a lane has column lane % 16 of four.  One block of instructions: four rows take turns, so that a
// register is read by DPP three instructions after it was written; the waits in front and behind are those of matrix
// instructions beside it, which the compiler does not see through the block.
template <bool FORWARD> __device__ __forceinline__ void substitute16(double (&y)[4], const double (&f)[16])
{
#define SUB_ROW(t, a, fa) "v_fmac_f64_dpp %" #t ", %" #t ", %" #fa " row_newbcast:" #a " row_mask:0xf bank_mask:0xf\n\t"
#define SUB_STEP(a, fa) SUB_ROW(0, a, fa) SUB_ROW(1, a, fa) SUB_ROW(2, a, fa) SUB_ROW(3, a, fa)
#define SUB_OPERANDS : "+&v"(y[0]), "+&v"(y[1]), "+&v"(y[2]), "+&v"(y[3]) \
        : "v"(f[0]), "v"(f[1]), "v"(f[2]), "v"(f[3]), "v"(f[4]), "v"(f[5]), "v"(f[6]), "v"(f[7]), "v"(f[8]), "v"(f[9]), "v"(f[10]), \
          "v"(f[11]), "v"(f[12]), "v"(f[13]), "v"(f[14]), "v"(f[15])
    if constexpr (FORWARD)
        asm("s_nop 15\n\ts_nop 7\n\t" SUB_STEP(0, 4) SUB_STEP(1, 5) SUB_STEP(2, 6) SUB_STEP(3, 7) SUB_STEP(4, 8) SUB_STEP(5, 9) SUB_STEP(6, 10)
                SUB_STEP(7, 11) SUB_STEP(8, 12) SUB_STEP(9, 13) SUB_STEP(10, 14) SUB_STEP(11, 15) SUB_STEP(12, 16) SUB_STEP(13, 17)
                    SUB_STEP(14, 18) "s_nop 3" SUB_OPERANDS);
    else
        asm("s_nop 15\n\ts_nop 7\n\t" SUB_STEP(15, 19) SUB_STEP(14, 18) SUB_STEP(13, 17) SUB_STEP(12, 16) SUB_STEP(11, 15) SUB_STEP(10, 14)
                SUB_STEP(9, 13) SUB_STEP(8, 12) SUB_STEP(7, 11) SUB_STEP(6, 10) SUB_STEP(5, 9) SUB_STEP(4, 8) SUB_STEP(3, 7)
                    SUB_STEP(2, 6) SUB_STEP(1, 5) "s_nop 3" SUB_OPERANDS);
#undef SUB_OPERANDS
#undef SUB_STEP
#undef SUB_ROW
}

// What als_update keeps in LDS: V = L D L^T (then -L), one step's rows of L D, tiles of 16 rows of the factor.  Rows of four doubles
// more than the columns: both operand layouts of the matrix cores then meet each bank twice.
constexpr int update_ld(int nb) { return 16 * nb + 4; }
constexpr int update_sums(int nb) { return nb == 1 ? 7 * 256 : (nb == 2 ? 9 * 256 : 0); }       // blocks of the Gram matrix from several wavefronts
constexpr int update_lds_doubles(int nb, int tiles) { return 16 * nb * update_ld(nb) + 16 * (nb - 1) * 20 + update_sums(nb) + tiles * 16 * update_ld(nb); }
// tiles of a factor that fit the 160 KB beside V and 6 KB of smaller arrays
constexpr int update_most_tiles(int nb) { return (154 * 1024 / 8 - update_lds_doubles(nb, 0)) / (16 * update_ld(nb)); }

// Up to rank 64, NB blocks of 16 columns.  V is formed (Hadamard product of the Gram matrices of the other modes) and factorised
// by every workgroup for itself, 16 columns at a time: the first wavefront factorises the diagonal block, one wavefront for 16 rows solves
// the rows below against it, and the pieces to the right are updated on the matrix cores while the first wavefront goes on.  Then a
// wavefront takes 16 rows of M at a time through both substitutions in the matrix cores' own accumulator layout: 16 unknowns by
// DPP (substitute16), the columns that follow by matrix instructions.  The Gram matrix of the new rows, by pairs of column
// blocks, also holds the columns' squared norms.
//   WHOLE (one workgroup, all rows stay in LDS): the norms, the normalised rows, the Gram matrix and after a sweep's last mode its
//   record follow in the same launch.  Otherwise every workgroup leaves its Gram matrix in gram_ws and als_normalise does the rest.
// Bound by the chain of the pivots, by latency and by instruction fetches.  A row a quad of lanes, V in the threads' registers, four columns
// a barrier and all of it unrolled (67 KB of code at R = 49 to 64, where the cache holds 64) took, against this: 293 rows at R = 62 59 us
// and 12 in the second launch -> 26 and 10; 62 rows 59 and 12 -> 20; 96 rows at R = 48 40 and 12 -> 17; 32 rows at R = 24 22 -> 12; 145071 rows at R = 10
// 91 and 40 -> 26 and 11; 100 rows at R = 10, in a kernel for up to 16 columns, 7.7 -> 6.6.
template <int NB, int WAVES, bool WHOLE>
__global__ void __launch_bounds__(64 * WAVES)
als_update(double* G, int ndim, int k, int R, const double* __restrict__ M, double* A, int64_t I, int64_t n_tiles,
           double* gram_ws, double* lambda, double* inner, int* flag, SweepEnd end)
{
    constexpr int THREADS = 64 * WAVES, LD = update_ld(NB), RP = 16 * NB, TILE = 16 * LD;
    constexpr int PAIRS = NB * (NB + 1) / 2;                                 // blocks (p, q), p >= q, of a symmetric matrix
    constexpr int KS = NB == 1 ? 8 : (NB == 2 ? 4 : 1);                      // wavefronts that share a block of the Gram matrix
    constexpr int UNITS = PAIRS * KS, PER = (UNITS + WAVES - 1) / WAVES;
    extern __shared__ double lds[];
    double* const P = lds;                       // [RP][LD]
    double* const W = P + RP * LD;               // [NB - 1][16][20]
    double* const Sums = W + 16 * (NB - 1) * 20;
    double* const T = Sums + update_sums(NB);    // tiles
    __shared__ double dinv[RP], nrm[RP], inverse[RP], weight[RP], scale[RP], red[2 * WAVES];
    __shared__ int bad;
    const int tid = (int)threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int n16 = lane & 15, kq = lane >> 4;
    const int64_t RR = (int64_t)R * R;
    auto block_row = [](int b) { return b < 1 ? 0 : (b < 3 ? 1 : (b < 6 ? 2 : 3)); };
    auto block_col = [&](int b) { const int p = block_row(b); return b - p * (p + 1) / 2; };
    // rows of tile t in the accumulator layout: entry (4 q + kq, 16 u + n16)
    auto load_rows = [&](int64_t t, double (&m)[NB][4]) {
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            const int64_t r = 16 * t + 4 * q + kq;
            const double* const row = M + (r < I ? r : I - 1) * R;
#pragma unroll
            for (int u = 0; u < NB; ++u)
                m[u][q] = row[min(16 * u + n16, R - 1)];
        }
    };
    // (every lane loads, from the last row or column where its own does not exist: behind branches each load is waited for)
    const int stop = flag[0];
    // this thread's entries (r, c) of the blocks on and below the diagonal
    constexpr int NV = (PAIRS * 256 + THREADS - 1) / THREADS;
    auto own_entry = [&](int i, auto take) {
        const int b = (tid >> 8) + i * (THREADS / 256);
        if (b < PAIRS)
            take(16 * block_row(b) + ((tid >> 4) & 15), 16 * block_col(b) + (tid & 15), block_row(b) != block_col(b));
    };
    double v[NV];                    // of V before it is scaled
    {
        double d = 1.0;
#pragma unroll
        for (int i = 0; i < NV; ++i)
            v[i] = 1.0;
        const int others = ndim - 1;
        for (int m0 = 0; m0 < others; m0 += 2) {
            double g[2][NV + 1];
#pragma unroll
            for (int h = 0; h < 2; ++h) {
                const int o = min(m0 + h, others - 1);
                const double* const Gm = G + (int64_t)(o + (o >= k ? 1 : 0)) * RR;
#pragma unroll
                for (int i = 0; i < NV; ++i) {
                    const int b = min((tid >> 8) + i * (THREADS / 256), PAIRS - 1);
                    const int r = 16 * block_row(b) + ((tid >> 4) & 15), c = 16 * block_col(b) + (tid & 15);
                    g[h][i] = Gm[min(r, R - 1) * R + min(c, R - 1)];
                }
                const int j = min(tid, R - 1);
                g[h][NV] = Gm[(int64_t)j * R + j];
            }
#pragma unroll
            for (int h = 0; h < 2; ++h)
                if (m0 + h < others) {
#pragma unroll
                    for (int i = 0; i < NV; ++i)
                        v[i] *= g[h][i];
                    d *= g[h][NV];
                }
        }
        if (__syncthreads_or(stop) != 0) {      // an earlier update failed or the fit has settled: every factor stays as it is
            if (WHOLE && end.record && tid == 0)
                end_sweep(end.scalars, flag, end.record, 0.0, 0.0, end.tol, end.first);
            return;
        }
        if (tid < RP)
            scale[tid] = tid < R ? unit_scale(d) : 1.0;
        if (tid == 0)
            bad = 0;
        __syncthreads();
#pragma unroll
        for (int i = 0; i < NV; ++i)
            own_entry(i, [&](int r, int c, bool) { P[r * LD + c] = r < R && c < R ? v[i] * scale[r] * scale[c] : (r == c ? 1.0 : 0.0); });
    }
    double m[NB][4];                 // the first tile's rows: on their way while V is factorised
    load_rows((int64_t)blockIdx.x * WAVES + wave, m);
    __syncthreads();
    // piece (t, u) of V minus the product of what the columns of step g - 1 have become: (-L)(t, g - 1) times (L D)(u, g - 1)^T
    auto update_piece = [&](int t, int u, int g) {
        double4_t acc;
#pragma unroll
        for (int q = 0; q < 4; ++q)
            acc[q] = P[(16 * t + 4 * q + kq) * LD + 16 * u + n16];
#pragma unroll
        for (int s = 0; s < 4; ++s)
            acc = __builtin_amdgcn_mfma_f64_16x16x4f64(P[(16 * t + n16) * LD + 16 * (g - 1) + 4 * s + kq], W[((u - 1) * 16 + n16) * 20 + 4 * s + kq], acc, 0, 0, 0);
#pragma unroll
        for (int q = 0; q < 4; ++q)
            P[(16 * t + 4 * q + kq) * LD + 16 * u + n16] = acc[q];
    };
    for (int g = 0; g < NB; ++g) {
        if (wave == 0) {
            if (g > 0)
                update_piece(g, g, g);
            __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
            double a[16];
#pragma unroll
            for (int i = 0; i < 16; ++i)
                a[i] = P[(16 * g + (i > n16 ? i : n16)) * LD + 16 * g + (i > n16 ? n16 : i)];
            const bool ok = factorise16(a, dinv + 16 * g);
            if (!ok && lane == 0)
                bad = 1;
            const double rd = dinv[16 * g + n16];
            if (kq == 0) {
#pragma unroll
                for (int i = 0; i < 16; ++i)
                    P[(16 * g + i) * LD + 16 * g + n16] = i > n16 ? -a[i] * rd : 0.0;
            }
        } else if (g > 0) {
            int n = 1;
            for (int t = g + 1; t < NB; ++t)
                for (int u = g; u <= t; ++u, ++n)
                    if (n == wave)
                        update_piece(t, u, g);
        }
        __syncthreads();
        if (wave < NB - 1 - g) {
            const int t = g + 1 + wave;
            double y[4], f[16];
#pragma unroll
            for (int q = 0; q < 4; ++q)
                y[q] = P[(16 * t + 4 * q + kq) * LD + 16 * g + n16];
#pragma unroll
            for (int a = 0; a < 16; ++a)
                f[a] = P[(16 * g + n16) * LD + 16 * g + a];
            substitute16<true>(y, f);
            const double rd = dinv[16 * g + n16];
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                W[((t - 1) * 16 + 4 * q + kq) * 20 + n16] = y[q];
                P[(16 * t + 4 * q + kq) * LD + 16 * g + n16] = -y[q] * rd;
            }
        }
        __syncthreads();
    }
    if (bad) {
        if (blockIdx.x == 0 && tid == 0) {
            flag[0] = kFailed;
            if (WHOLE && end.record)
                end_sweep(end.scalars, flag, end.record, 0.0, 0.0, end.tol, end.first);
        }
        return;
    }
    double sc[NB], dv[NB];
#pragma unroll
    for (int u = 0; u < NB; ++u) {
        sc[u] = scale[16 * u + n16];
        dv[u] = 16 * u + n16 < R ? dinv[16 * u + n16] : 0.0;
    }
    double4_t acc[2][PER];
#pragma unroll
    for (int i = 0; i < PER; ++i)
        acc[0][i] = acc[1][i] = {0.0, 0.0, 0.0, 0.0};
    // this wavefront's blocks of Y^T Y over the tiles in LDS
    auto gram_of = [&](int tiles) {
        int p[PER], q[PER];
#pragma unroll
        for (int i = 0; i < PER; ++i) {
            const int b = min(wave + i * WAVES, UNITS - 1) / KS;
            p[i] = 16 * block_row(b) + n16;
            q[i] = 16 * block_col(b) + n16;
        }
        if (wave >= UNITS)
            return;
        const int mine = wave + WAVES < UNITS ? PER : 1;         // blocks of this wavefront
        auto operands = [&](int t, double (&x)[PER][4], double (&z)[PER][4]) {
            const double* const Y = T + min(t, tiles - 1) * TILE;
#pragma unroll
            for (int i = 0; i < PER; ++i)
#pragma unroll
                for (int s = 0; s < 4; ++s) {
                    x[i][s] = Y[(4 * s + kq) * LD + p[i]];
                    z[i][s] = Y[(4 * s + kq) * LD + q[i]];
                }
        };
        if constexpr (!WHOLE && NB % 2 == 0) {                   // (short of registers: a tile and a block after the other)
#pragma unroll
            for (int i = 0; i < PER; ++i)
                if (i < mine)
                    for (int t = wave % KS; t < tiles; t += KS)
#pragma unroll
                        for (int s = 0; s < 4; ++s) {
                            const double* const row = T + t * TILE + (4 * s + kq) * LD;
                            acc[0][i] = __builtin_amdgcn_mfma_f64_16x16x4f64(row[p[i]], row[q[i]], acc[0][i], 0, 0, 0);
                        }
        } else {
            double x[PER][4], z[PER][4];
            auto add = [&](const double (&x)[PER][4], const double (&z)[PER][4], double4_t (&to)[PER]) {
#pragma unroll
                for (int i = 0; i < PER; ++i)
                    if (i < mine)
#pragma unroll
                        for (int s = 0; s < 4; ++s)
                            to[i] = __builtin_amdgcn_mfma_f64_16x16x4f64(x[i][s], z[i][s], to[i], 0, 0, 0);
            };
            // (every other tile goes into sums of its own: shorter chains of roundings)
            operands(wave % KS, x, z);
            for (int t = wave % KS; t < tiles; t += 2 * KS) {
                double x1[PER][4], z1[PER][4];
                operands(t + KS, x1, z1);                        // (under the matrix instructions)
                add(x, z, acc[0]);
                operands(t + 2 * KS, x, z);
                if (t + KS < tiles)
                    add(x1, z1, acc[1]);
            }
        }
    };
    const int64_t step = (int64_t)gridDim.x * WAVES;
    for (int64_t t0 = (int64_t)blockIdx.x * WAVES; t0 < n_tiles; t0 += step) {
        const int64_t tile = t0 + wave;
        double* const Y = T + (WHOLE ? (tile < n_tiles ? (int)tile : 0) : wave) * TILE;
        if (!WHOLE || tile < n_tiles) {
            double y[NB][4];
#pragma unroll
            for (int u = 0; u < NB; ++u)
#pragma unroll
                for (int q = 0; q < 4; ++q)
                    y[u][q] = 16 * tile + 4 * q + kq < I && 16 * u + n16 < R ? m[u][q] * sc[u] : 0.0;
            if (t0 + step < n_tiles)
                load_rows(tile + step, m);
            asm volatile("" ::: "memory");          // (or the operands of all tiles are read once, into more registers than there are)
            double a[4], f[16];
            // (the tile's place in LDS takes a block's unknowns from the accumulator layout to that of a left operand)
            auto turn = [&](int g) {
#pragma unroll
                for (int q = 0; q < 4; ++q)
                    Y[(4 * q + kq) * LD + 16 * g + n16] = y[g][q];
                __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
#pragma unroll
                for (int s = 0; s < 4; ++s)
                    a[s] = Y[n16 * LD + 16 * g + 4 * s + kq];
            };
            auto take = [&](int u, const double (&l)[4]) {
                double4_t c = {y[u][0], y[u][1], y[u][2], y[u][3]};
#pragma unroll
                for (int s = 0; s < 4; ++s)
                    c = __builtin_amdgcn_mfma_f64_16x16x4f64(a[s], l[s], c, 0, 0, 0);
#pragma unroll
                for (int q = 0; q < 4; ++q)
                    y[u][q] = c[q];
            };
#pragma unroll
            for (int g = 0; g < NB; ++g) {
#pragma unroll
                for (int i = 0; i < 16; ++i)
                    f[i] = P[(16 * g + n16) * LD + 16 * g + i];
                substitute16<true>(y[g], f);
                if (g + 1 < NB)
                    turn(g);
#pragma unroll
                for (int u = g + 1; u < NB; ++u) {
                    double l[4];
#pragma unroll
                    for (int s = 0; s < 4; ++s)
                        l[s] = P[(16 * u + n16) * LD + 16 * g + 4 * s + kq];
                    take(u, l);
                }
            }
#pragma unroll
            for (int u = 0; u < NB; ++u)
#pragma unroll
                for (int q = 0; q < 4; ++q)
                    y[u][q] *= dv[u];
#pragma unroll
            for (int g = NB - 1; g >= 0; --g) {
#pragma unroll
                for (int i = 0; i < 16; ++i)
                    f[i] = P[(16 * g + i) * LD + 16 * g + n16];
                substitute16<false>(y[g], f);
                if (g > 0)
                    turn(g);
#pragma unroll
                for (int u = 0; u < g; ++u) {
                    double l[4];
#pragma unroll
                    for (int s = 0; s < 4; ++s)
                        l[s] = P[(16 * g + 4 * s + kq) * LD + 16 * u + n16];
                    take(u, l);
                }
            }
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                const int64_t r = 16 * tile + 4 * q + kq;
#pragma unroll
                for (int u = 0; u < NB; ++u) {
                    const double v = y[u][q] * sc[u];
                    Y[(4 * q + kq) * LD + 16 * u + n16] = v;
                    if (!WHOLE && r < I && 16 * u + n16 < R)
                        A[r * R + 16 * u + n16] = v;
                }
            }
        }
        if (!WHOLE) {
            __syncthreads();
            gram_of(WAVES);
            __syncthreads();
        }
    }
    if (WHOLE) {
        __syncthreads();
        gram_of((int)n_tiles);
    }
#pragma unroll
    for (int i = 0; i < PER; ++i)
        acc[0][i] += acc[1][i];
    const bool owner = wave % KS == 0;
    if (KS > 1) {          // a block's sums in the order of their wavefronts
        double* const mine = Sums + (wave / KS * (KS - 1) + wave % KS - 1) * 256 + lane;
        if (!owner && wave < UNITS) {
#pragma unroll
            for (int q = 0; q < 4; ++q)
                mine[64 * q] = acc[0][0][q];
        }
        __syncthreads();
        if (owner && wave < UNITS) {
            for (int i = 0; i < KS - 1; ++i)
#pragma unroll
                for (int q = 0; q < 4; ++q)
                    acc[0][0][q] += Sums[(wave / KS * (KS - 1) + i) * 256 + 64 * q + lane];
        }
    }
    // entry q of this lane's part of a block, (r, c), of the blocks whose sums this wavefront has
    auto entries = [&](auto take) {
#pragma unroll
        for (int i = 0; i < PER; ++i) {
            const int unit = wave + i * WAVES;
            if (unit < UNITS && owner) {
                const int b = unit / KS, p = block_row(b), q = block_col(b);
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    const int r = 16 * p + 4 * e + kq, c = 16 * q + n16;
                    if (r < R && c < R)
                        take(r, c, acc[0][i][e], p != q);
                }
            }
        }
    };
    if (!WHOLE) {
        double* const o = gram_ws + (int64_t)blockIdx.x * RR;
        double* const diag = gram_ws + (int64_t)gridDim.x * RR + (int64_t)blockIdx.x * R;
        entries([&](int r, int c, double v, bool off) {
            o[r * R + c] = v;
            if (off)
                o[c * R + r] = v;
            if (r == c)
                diag[r] = v;
        });
        return;
    }
    entries([&](int r, int c, double v, bool) { P[r * LD + c] = v; });       // (V is no longer needed)
    __syncthreads();
    if (tid < R) {
        const double l = sqrt(P[tid * LD + tid]), n = l > 0.0 ? l : 1.0;       // a zero column is left alone
        nrm[tid] = n;
        inverse[tid] = 1.0 / n;
        weight[tid] = l;
        lambda[tid] = l;
    }
    __syncthreads();
    double model2 = 0.0, with_m = 0.0;       // this thread's shares of ||X^||^2 and <X, X^> (a sweep's last update)
#pragma unroll
    for (int i = 0; i < NV; ++i)
        own_entry(i, [&](int r, int c, bool off) {
            if (r < R && c < R) {
                const double gk = quotient(quotient(P[r * LD + c], nrm[r], inverse[r]), nrm[c], inverse[c]);
                G[k * RR + r * R + c] = gk;
                if (off)
                    G[k * RR + c * R + r] = gk;
                model2 += (off ? 2.0 : 1.0) * weight[r] * weight[c] * gk * v[i];
            }
        });
    constexpr int J = NB == 3 ? 64 : RP;     // threads of a row
    const int j = tid % J;
    if (j < R) {
        const double n = nrm[j], in = inverse[j];
        constexpr int STEP = THREADS / J;
        for (int i = tid / J; i < (int)I; i += 4 * STEP) {
            double y[4], f[4] = {0.0, 0.0, 0.0, 0.0};
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                const int r = min(i + u * STEP, (int)I - 1);
                y[u] = T[(r >> 4) * TILE + (r & 15) * LD + j];
                if (end.record)
                    f[u] = M[(int64_t)r * R + j];
            }
#pragma unroll
            for (int u = 0; u < 4; ++u)
                if (i + u * STEP < (int)I) {
                    const double a = quotient(y[u], n, in);
                    A[(int64_t)(i + u * STEP) * R + j] = a;
                    with_m += f[u] * a;
                }
        }
        with_m *= weight[j];
    }
    if (!end.record)
        return;
#pragma unroll
    for (int d = 1; d < 64; d <<= 1) {
        model2 += __shfl_xor(model2, d);
        with_m += __shfl_xor(with_m, d);
    }
    if (lane == 0) {
        red[2 * wave] = model2;
        red[2 * wave + 1] = with_m;
    }
    __syncthreads();
    if (tid == 0) {
        double fit = 0.0, m2 = 0.0;
#pragma unroll
        for (int q = 0; q < WAVES; ++q) {
            m2 += red[2 * q];
            fit += red[2 * q + 1];
        }
        end_sweep(end.scalars, flag, end.record, fit, m2, end.tol, end.first);
    }
}

// Second launch of the update for longer factors: every workgroup adds up the columns' squared norms (n_gram
// partial diagonals), normalises its rows and its share of the Gram matrix (64 entries at a time, a wavefront for an eighth of
// the partial matrices), and after a sweep's last mode (inner != nullptr) leaves its column sums of M * A in inner[block][R].
// Bound by latency: eight requests in flight a thread.
template <int RP>
__global__ void __launch_bounds__(512)
als_normalise(const double* __restrict__ gram_ws, int n_gram, int R, double* A, const double* __restrict__ M, int64_t I,
              int64_t rows_per_block, double* Gk, double* lambda, double* inner, const int* flag)
{
    __shared__ double red[512], nrm[RP], inverse[RP];
    if (flag[0])
        return;
    const int tid = (int)threadIdx.x, j = tid % RP, lane = tid & 63, wave = tid >> 6;
    const int RR = R * R;
    red[tid] = j < R ? sum_strided(gram_ws + (int64_t)n_gram * RR + j, tid / RP, 512 / RP, n_gram, R) : 0.0;
    __syncthreads();
    if (tid < RP) {
        double v = 0.0;
        for (int q = tid; q < 512; q += RP)
            v += red[q];
        const double n = sqrt(v);
        nrm[tid] = n > 0.0 ? n : 1.0;       // a zero column is left alone
        inverse[tid] = 1.0 / nrm[tid];
        if (blockIdx.x == 0 && tid < R)
            lambda[tid] = n;
    }
    __syncthreads();
    for (int e0 = (int)blockIdx.x * 64; e0 < RR; e0 += (int)gridDim.x * 64) {
        const int e = min(e0 + lane, RR - 1);
        red[tid] = sum_strided(gram_ws + e, wave, 8, n_gram, RR);
        __syncthreads();
        if (wave == 0 && e0 + lane < RR) {
            double v = 0.0;
            for (int q = 0; q < 8; ++q)
                v += red[64 * q + lane];
            const int r = e / R, c = e - r * R;
            Gk[e] = quotient(quotient(v, nrm[r], inverse[r]), nrm[c], inverse[c]);
        }
        __syncthreads();
    }
    const int64_t r0 = (int64_t)blockIdx.x * rows_per_block, r1 = I < r0 + rows_per_block ? I : r0 + rows_per_block;
    constexpr int64_t STEP = 512 / RP;
    double s = 0.0;
    if (j < R)
        for (int64_t i = r0 + tid / RP; i < r1; i += 4 * STEP) {
            double a[4], m[4] = {0.0, 0.0, 0.0, 0.0};
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                const int64_t e = (i + u * STEP < r1 ? i + u * STEP : r1 - 1) * R + j;
                a[u] = A[e];
                if (inner)
                    m[u] = M[e];
            }
#pragma unroll
            for (int u = 0; u < 4; ++u)
                if (i + u * STEP < r1) {
                    const double v = quotient(a[u], nrm[j], inverse[j]);
                    A[(i + u * STEP) * R + j] = v;
                    s += m[u] * v;
                }
        }
    if (!inner)
        return;
    red[tid] = s;
    __syncthreads();
    if (tid < R) {
        double v = 0.0;
        for (int q = tid; q < 512; q += RP)
            v += red[q];
        inner[(int64_t)blockIdx.x * R + tid] = v;
    }
}

// Fit terms up to rank 64, one workgroup: sum_j lambda_j (sum over the blocks of inner[b][j]) = <X, X^> and
// lambda^T (Hadamard product of all Gram matrices) lambda = ||X^||^2, then the sweep's record.
__global__ void __launch_bounds__(256) fit_terms_small(const double* __restrict__ G, int ndim, int R, const double* __restrict__ lambda,
                                                        const double* __restrict__ inner, int n_inner, double* scalars, int* flag,
                                                        SweepRecord* record, double tol, bool first)
{
    __shared__ double lds[256];
    double s = 0.0, t = 0.0;
    const int per = 256 / R, j = (int)threadIdx.x % R;          // threads of a column
    if ((int)threadIdx.x < per * R)
        s = sum_strided(inner + j, (int)threadIdx.x / R, per, n_inner, R) * lambda[j];
    for (int e = threadIdx.x; e < R * R; e += 256) {
        double v = lambda[e / R] * lambda[e % R];
        for (int m = 0; m < ndim; ++m)
            v *= G[(int64_t)m * R * R + e];
        t += v;
    }
    s = block_sum_256(s, lds);
    t = block_sum_256(t, lds);
    if (threadIdx.x == 0)
        end_sweep(scalars, flag, record, s, t, tol, first);
}

// ---------------------------------------------------------------------------
// Ranks above 64: Gram matrices, the factorisation and the triangular solves run blocked, 32 columns
// at a time, every sum still in a fixed order.
// ---------------------------------------------------------------------------
constexpr int kNB = 32;

// G = A^T A: a 16 x 16 block of G (on or below the diagonal) per workgroup, a wavefront for every eighth 16 rows of A, on the matrix cores;
// the wavefronts' sums are added in their order.  G(p, q) and G(q, p) are one value.  Bound by latency: two tiles requested before the first
// is used (129 rows at R = 500 in chunks of 16 through LDS with two barriers each: 11 us -> 5).
__global__ void __launch_bounds__(512) gram_tiled(const double* __restrict__ A, int64_t I, int R, double* G)
{
    __shared__ double red[8][256];
    if (blockIdx.x > blockIdx.y)
        return;
    const int tid = (int)threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6), n16 = lane & 15, kq = lane >> 4;
    const int p = (int)blockIdx.y * 16 + n16, q = (int)blockIdx.x * 16 + n16;
    const int64_t n_tiles = ceil_div(I, 16);
    double4_t acc = {0.0, 0.0, 0.0, 0.0};
    for (int64_t t = wave; t < n_tiles; t += 16) {
        double x[2][4], y[2][4];
#pragma unroll
        for (int h = 0; h < 2; ++h)
#pragma unroll
            for (int s = 0; s < 4; ++s) {
                const int64_t r = 16 * (t + 8 * h) + 4 * s + kq;
                const double* const row = A + (r < I ? r : I - 1) * R;
                x[h][s] = row[min(p, R - 1)];
                y[h][s] = row[min(q, R - 1)];
            }
#pragma unroll
        for (int h = 0; h < 2; ++h)
#pragma unroll
            for (int s = 0; s < 4; ++s) {
                const bool real = 16 * (t + 8 * h) + 4 * s + kq < I;
                acc = __builtin_amdgcn_mfma_f64_16x16x4f64(real ? x[h][s] : 0.0, real ? y[h][s] : 0.0, acc, 0, 0, 0);
            }
    }
#pragma unroll
    for (int e = 0; e < 4; ++e)
        red[wave][64 * e + lane] = acc[e];
    __syncthreads();
    if (tid >= 256)
        return;
    double v = 0.0;
#pragma unroll
    for (int w = 0; w < 8; ++w)
        v += red[w][tid];
    const int r = (int)blockIdx.y * 16 + 4 * (tid >> 6) + kq, c = q;
    if (r < R && c < R) {
        G[(int64_t)r * R + c] = v;
        G[(int64_t)c * R + r] = v;
    }
}

// One launch per 64 columns of V = L D L^T, V holding what is still to be factorised.  Workgroup (tj, ti),
// ti >= tj, owns the 64 x 64 tile (ti, tj) of the trailing lower triangle.  It takes 192 rows of the block column through LDS, the diagonal
// block and the 64 rows of its tile's rows and of its columns, 16 columns at a time: the first wavefront factorises the
// 16 x 16 diagonal block, the rows below are solved against it (a wavefront for 16 rows) and subtracted from the
// columns that follow on the matrix cores, the next diagonal block first, which the first wavefront then factorises
// while the others go on.  At the end the tile's rows and columns are multiplied and subtracted from the tile: no workgroup waits for
// another, and a step is one launch.  The chain of the columns bounds it (16 columns
// take 2.6 us: 1.2 for their reciprocals and row operations, the rest for the exchanges): 22.3 us a launch, eight at R = 500 (25.3 with the reciprocals
// behind the row operations and a row a quad of lanes in the solves).
// The block column of V is only read; the tiles on the diagonal write their rows of -L (which is what the solves add) and the same
// above the diagonal, transposed, so that both solves read whole lines; workgroup (0, 0) the block's own rows and dinv = 1 / D.
constexpr int kPB = 64;
constexpr int kPanelLds = 3 * kPB * (kPB + 1) * (int)sizeof(double);
__global__ void __launch_bounds__(512)
factorise_panel(double* V, int R, int j0, double* L, int ldL, double* dinv_out, int* flag)
{
    extern __shared__ double P[];               // [3 kPB][LD]: L D of the diagonal block, of the tile's rows and of its columns
    __shared__ double Lg[2][16 * 17], dinv[kPB];
    __shared__ int bad;
    constexpr int LD = kPB + 1, WAVES = 8;
    if (blockIdx.x > blockIdx.y)
        return;
    const int tid = (int)threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int n16 = lane & 15, kq = lane >> 4;
    const int nb = R - j0 < kPB ? R - j0 : kPB, j1 = j0 + nb;
    const int ng = (nb + 15) / 16;
    const bool trailing = j1 < R;               // then nb == 64
    auto v_row = [&](int r) { return r < kPB ? j0 + r : j1 + kPB * (int)(r < 2 * kPB ? blockIdx.y : blockIdx.x) + (r & (kPB - 1)); };
    {
        // (every lane loads, from the last row or column where its own does not exist: behind branches each load would be waited for)
        double x[192 / WAVES];
        const int c = lane, cl = c < nb ? c : nb - 1;
#pragma unroll
        for (int i = 0; i < 192 / WAVES; ++i) {
            const int vi = v_row(wave + WAVES * i);
            x[i] = V[(int64_t)(vi < R ? vi : R - 1) * R + j0 + cl];
        }
#pragma unroll
        for (int i = 0; i < 192 / WAVES; ++i) {
            const int r = wave + WAVES * i;
            P[r * LD + c] = c < nb && v_row(r) < R && (r >= kPB || (r >= c && r < nb)) ? x[i] : 0.0;
        }
    }
    // this wavefront's 16 x 16 pieces of the tile: row wave / 4 + WAVES / 4 t, column wave % 4 (none above the diagonal)
    constexpr int NT = 16 / WAVES;
    double4_t v[NT];
    int vr[NT];
    const int vc = j1 + kPB * (int)blockIdx.x + 16 * (wave & 3);
    bool has[NT];
#pragma unroll
    for (int t = 0; t < NT; ++t) {
        vr[t] = j1 + kPB * (int)blockIdx.y + 16 * ((wave >> 2) + WAVES / 4 * t);
        has[t] = trailing && vr[t] >= vc && vr[t] < R;
#pragma unroll
        for (int q = 0; q < 4; ++q)
            v[t][q] = V[(int64_t)min(vr[t] + 4 * q + kq, R - 1) * R + min(vc + n16, R - 1)];       // (what does not exist is not stored)
    }
    if (tid == 0)
        bad = 0;
    if (failed_before(flag))      // (behind the loads, so that it does not delay them)
        return;
    // rows [r0, r0 + 16) of P solved against the diagonal block of columns 16 g ..
    auto solve = [&](int r0, int g) {
        double y[4], f[16];
        double* const at = P + (r0 + kq) * LD + 16 * g + n16;
#pragma unroll
        for (int q = 0; q < 4; ++q)
            y[q] = at[4 * q * LD];
#pragma unroll
        for (int a = 0; a < 16; ++a)
            f[a] = Lg[g & 1][a * 17 + n16];
        substitute16<true>(y, f);
#pragma unroll
        for (int q = 0; q < 4; ++q)
            at[4 * q * LD] = y[q];
    };
    // piece (rows r0 .., columns 16 u ..) of P minus the product of its rows' and the column rows' solved columns 16 g ..
    auto update = [&](int r0, int u, int g) {
        double4_t acc;
#pragma unroll
        for (int q = 0; q < 4; ++q)
            acc[q] = P[(r0 + 4 * q + kq) * LD + 16 * u + n16];
#pragma unroll
        for (int k = 16 * g; k < 16 * g + 16; k += 4)
            acc = __builtin_amdgcn_mfma_f64_16x16x4f64(-P[(r0 + n16) * LD + k + kq], P[(16 * u + n16) * LD + k + kq] * dinv[k + kq], acc, 0, 0, 0);
#pragma unroll
        for (int q = 0; q < 4; ++q)
            P[(r0 + 4 * q + kq) * LD + 16 * u + n16] = acc[q];
    };
    auto factor = [&](int g) {            // by the first wavefront; columns from R on as those of the identity
        double a[16];
#pragma unroll
        for (int i = 0; i < 16; ++i) {
            const double p = P[(16 * g + (i > n16 ? i : n16)) * LD + 16 * g + (i > n16 ? n16 : i)];
            a[i] = i == n16 && 16 * g + i >= nb ? 1.0 : p;
        }
        if (!factorise16(a, dinv + 16 * g) && lane == 0)
            bad = 1;
        const double rd = dinv[16 * g + n16];
        if (kq == 0) {
#pragma unroll
            for (int i = 0; i < 16; ++i) {
                Lg[g & 1][n16 * 17 + i] = i > n16 ? -a[i] * rd : 0.0;
                if (i > n16)
                    P[(16 * g + i) * LD + 16 * g + n16] = a[i];
            }
        }
    };
    // (one copy of each step's code: what runs once or twice waits for its instructions)
    for (int g = 0; g <= ng; ++g) {
        if (wave == 0) {
            if (g < ng) {
                if (g > 0)
                    update(16 * g, g, g - 1);
                factor(g);
            }
        } else if (g > 0) {
            // columns 16 (g - 1) .. are solved for the diagonal block's rows: what they take from its other pieces, and the
            // tile's rows and columns (8 pieces of 16 rows, two of them for one wavefront)
            int n = 0;
            for (int t = g + 1; t < ng; ++t)
                for (int u = g; u <= t; ++u)
                    if (n++ % (WAVES - 1) == wave - 1)
                        update(16 * t, u, g - 1);
            if (trailing)
                for (int t = wave; t < 9; t += WAVES - 1) {
                    solve(kPB + 16 * (t - 1), g - 1);
                    for (int u = g; u < 4; ++u)
                        update(kPB + 16 * (t - 1), u, g - 1);
                }
        }
        __syncthreads();
        if (wave < ng - 1 - g)
            solve(16 * (g + 1 + wave), g);
        __syncthreads();
    }
    if (bad) {
        if (blockIdx.x == 0 && blockIdx.y == 0 && tid == 0)
            flag[0] = 1;
        return;
    }
    if (blockIdx.x == 0 && blockIdx.y == 0) {
        for (int r = wave; r < nb; r += WAVES)
            if (lane != r && lane < nb)
                L[(int64_t)(j0 + r) * ldL + j0 + lane] = lane < r ? -P[r * LD + lane] * dinv[lane] : -P[lane * LD + r] * dinv[r];
        if (tid < nb)
            dinv_out[j0 + tid] = dinv[tid];
    }
    if (!trailing)
        return;
    if (blockIdx.x == blockIdx.y) {
        const int row0 = v_row(2 * kPB);
        for (int r = wave; r < kPB; r += WAVES) {
            if (row0 + r < R)
                L[(int64_t)(row0 + r) * ldL + j0 + lane] = -P[(2 * kPB + r) * LD + lane] * dinv[lane];
            if (row0 + lane < R)
                L[(int64_t)(j0 + r) * ldL + row0 + lane] = -P[(2 * kPB + lane) * LD + r] * dinv[r];
        }
    }
    const double* const wb = P + (2 * kPB + 16 * (wave & 3) + n16) * LD + kq;
#pragma unroll
    for (int t = 0; t < NT; ++t)
        if (has[t]) {
            const double* const wa = P + (kPB + 16 * ((wave >> 2) + WAVES / 4 * t) + n16) * LD + kq;
#pragma unroll
            for (int k = 0; k < kPB; k += 4)
                v[t] = __builtin_amdgcn_mfma_f64_16x16x4f64(-wa[k], wb[k] * dinv[k + kq], v[t], 0, 0, 0);
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                const int vi = vr[t] + 4 * q + kq;
                if (vi < R && vc + n16 <= vi)
                    V[(int64_t)vi * R + vc + n16] = v[t][q];
            }
        }
}

// The whole factorisation up to rank 128 in one workgroup: V = S (Hadamard product of the Gram matrices of all modes but `skip`) S lies in LDS, 16
// columns at a time as in als_update: the first wavefront factorises the diagonal block, one wavefront for 16 rows solves those below
// against it, the others take the products off the pieces to the right while the first goes on with the next block.  Leaves what
// hadamard_grams and factorise_panel leave: -L, symmetric with zeros in rows and columns from R on, dinv = 1 / D and the scales S.
// Bound by the chain of the blocks, 2.5 us each.
constexpr int kLdsRank = 128;
constexpr int lds_factor_bytes(int nb) { return (16 * nb * (16 * nb + 4) + 16 * (nb - 1) * 20) * (int)sizeof(double); }
__global__ void __launch_bounds__(1024)
factorise_lds(const double* __restrict__ G, int ndim, int R, int skip, double* L, int ldL, double* dinv_out, double* S, int* flag)
{
    extern __shared__ double P[];                // [16 nb][16 nb + 4], then one step's rows of L D, [nb - 1][16][20]
    __shared__ double dinv[kLdsRank], scale[kLdsRank];
    __shared__ int bad;
    const int tid = (int)threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int n16 = lane & 15, kq = lane >> 4, nb = (R + 15) / 16, LD = 16 * nb + 4;
    const int64_t RR = (int64_t)R * R;
    double* const W = P + 16 * nb * LD;
    if (failed_before(flag))
        return;
    if (tid < kLdsRank) {
        double d = 1.0;
        for (int m = 0; m < ndim; ++m)
            if (m != skip)
                d *= G[m * RR + (int64_t)min(tid, R - 1) * (R + 1)];
        scale[tid] = tid < R ? unit_scale(d) : 1.0;
    }
    if (tid == 0)
        bad = 0;
    __syncthreads();
    // a wavefront takes rows r0 + 16 u, up to the end of their diagonal block
    for (int r0 = wave; r0 < 16 * nb; r0 += 64) {
        double v[4][2];
#pragma unroll
        for (int u = 0; u < 4; ++u)
            v[u][0] = v[u][1] = 1.0;
        for (int m = 0; m < ndim; ++m) {
            if (m == skip)
                continue;
            double x[4][2];
#pragma unroll
            for (int u = 0; u < 4; ++u)
#pragma unroll
                for (int h = 0; h < 2; ++h)
                    x[u][h] = G[m * RR + (int64_t)min(r0 + 16 * u, R - 1) * R + min(lane + 64 * h, R - 1)];
#pragma unroll
            for (int u = 0; u < 4; ++u)
#pragma unroll
                for (int h = 0; h < 2; ++h)
                    v[u][h] *= x[u][h];
        }
#pragma unroll
        for (int u = 0; u < 4; ++u)
#pragma unroll
            for (int h = 0; h < 2; ++h) {
                const int r = r0 + 16 * u, c = lane + 64 * h;
                if (r < 16 * nb && c < (r | 15) + 1)
                    P[r * LD + c] = r < R && c < R ? v[u][h] * scale[r] * scale[c] : (r == c ? 1.0 : 0.0);
            }
    }
    __syncthreads();
    // piece (t, u) of V minus the product of what the columns of step g - 1 have become: (-L)(t, g - 1) times (L D)(u, g - 1)^T
    auto update_piece = [&](int t, int u, int g) {
        double4_t acc;
#pragma unroll
        for (int q = 0; q < 4; ++q)
            acc[q] = P[(16 * t + 4 * q + kq) * LD + 16 * u + n16];
#pragma unroll
        for (int s = 0; s < 4; ++s)
            acc = __builtin_amdgcn_mfma_f64_16x16x4f64(P[(16 * t + n16) * LD + 16 * (g - 1) + 4 * s + kq], W[((u - 1) * 16 + n16) * 20 + 4 * s + kq], acc, 0, 0, 0);
#pragma unroll
        for (int q = 0; q < 4; ++q)
            P[(16 * t + 4 * q + kq) * LD + 16 * u + n16] = acc[q];
    };
    for (int g = 0; g < nb; ++g) {
        if (wave == 0) {
            if (g > 0)
                update_piece(g, g, g);
            __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
            double a[16];
#pragma unroll
            for (int i = 0; i < 16; ++i)
                a[i] = P[(16 * g + (i > n16 ? i : n16)) * LD + 16 * g + (i > n16 ? n16 : i)];
            if (!factorise16(a, dinv + 16 * g) && lane == 0)
                bad = 1;
            const double rd = dinv[16 * g + n16];
            if (kq == 0) {
#pragma unroll
                for (int i = 0; i < 16; ++i)
                    P[(16 * g + i) * LD + 16 * g + n16] = i > n16 ? -a[i] * rd : 0.0;
            }
        } else if (g > 0) {
            int n = 1;
            for (int t = g + 1; t < nb; ++t)
                for (int u = g; u <= t; ++u) {
                    if (n == wave)
                        update_piece(t, u, g);
                    n = n == 15 ? 1 : n + 1;
                }
        }
        __syncthreads();
        if (wave < nb - 1 - g) {
            const int t = g + 1 + wave;
            double y[4], f[16];
#pragma unroll
            for (int q = 0; q < 4; ++q)
                y[q] = P[(16 * t + 4 * q + kq) * LD + 16 * g + n16];
#pragma unroll
            for (int a = 0; a < 16; ++a)
                f[a] = P[(16 * g + n16) * LD + 16 * g + a];
            substitute16<true>(y, f);
            const double rd = dinv[16 * g + n16];
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                W[((t - 1) * 16 + 4 * q + kq) * 20 + n16] = y[q];
                P[(16 * t + 4 * q + kq) * LD + 16 * g + n16] = -y[q] * rd;
            }
        }
        __syncthreads();
    }
    if (bad) {
        if (tid == 0)
            flag[0] = kFailed;
        return;
    }
    for (int r = wave; r < ldL; r += 16)
        for (int c = lane; c < ldL; c += 64)
            L[(int64_t)r * ldL + c] = r < R && c < R && r != c ? P[max(r, c) * LD + min(r, c)] : 0.0;
    if (tid < R) {
        dinv_out[tid] = dinv[tid];
        S[tid] = scale[tid];
    }
}

// Rows of A = M V^{-1} = M S (L D L^T)^{-1} S.  A workgroup owns 16 rows and takes them through the whole forward and
// backward solve, a block of 32 unknowns at a time.  Four wavefronts solve four rows each against the diagonal block (16
// lanes hold a row's unknowns, and one that is final goes to them by DPP) while the others wait: an fp64 MFMA keeps its SIMD for 64
// cycles, and every step of the chain would wait for one.  Then all subtract the block's multiples from the columns
// that follow, 16 at a time on the matrix cores.  The 16 x R slab lies in LDS (LDSY, R <= 1024) or in A itself.
// Bound by the chain of 2 R / 32 blocks, 0.55 us for the solve and about 2 for the operands and MFMAs on few compute units: 129 rows at
// R = 500 137 -> 106 us.
template <int WAVES, bool LDSY>
__global__ void __launch_bounds__(64 * WAVES)
solve_rows_blocked(const double* __restrict__ L, int ldL, const double* __restrict__ dinv, const double* __restrict__ S, int R,
                   const double* __restrict__ M, double* A, int64_t I, const int* flag)
{
    extern __shared__ double slab[];
    __shared__ double Ld[2][kNB * (kNB + 1)];
    constexpr int THREADS = 64 * WAVES;
    if (flag[0])
        return;
    const int tid = (int)threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int n16 = lane & 15, kq = lane >> 4;
    const int64_t r0 = (int64_t)blockIdx.x * 16;
    const int rows = (int)(I - r0 < 16 ? I - r0 : 16);
    const int nblk = (R + kNB - 1) / kNB;
    const int ldy = nblk * kNB + 1;
    auto get = [&](int r, int c) -> double {
        if (LDSY)
            return slab[r * ldy + c];
        return r < rows && c < R ? A[(r0 + r) * R + c] : 0.0;
    };
    auto put = [&](int r, int c, double v) {
        if (LDSY)
            slab[r * ldy + c] = v;
        else if (r < rows && c < R)
            A[(r0 + r) * R + c] = v;
    };
    for (int r = wave; r < 16; r += WAVES)
        for (int c = lane; c < nblk * kNB; c += 64)
            put(r, c, r < rows && c < R ? M[(r0 + r) * R + c] * S[c] : 0.0);
    // entry t = 32 c + a of the diagonal block b, -L(c, a) for c > a, and where it lies in Ld
    auto diag_entry = [&](int b, int t) {
        const int a = t & (kNB - 1), c = t / kNB, j0 = b * kNB;
        const double l = L[(int64_t)(j0 + c) * ldL + j0 + a];
        return c > a ? l : 0.0;
    };
    auto diag_at = [](int t) { return (t & (kNB - 1)) * (kNB + 1) + t / kNB; };
    const int ncol = (R + 15) / 16;
    auto sweep = [&](auto forward) {
        constexpr bool F = decltype(forward)::value;
        const int step = F ? 1 : -1, first = F ? 0 : nblk - 1;
        // A wavefront takes a block's unknowns to the pieces of 16 columns first_piece(b) + i WAVES.  Their operands, entry (32 b + 8 kq + s,
        // 16 ct + n) of the symmetric -L, are requested a block ahead for the first two; always, since behind a branch they would be
        // waited for at once: past the last piece all lanes read one value, which costs next to nothing.
        constexpr int kAhead = 2;
        auto first_piece = [&](int b) { return (F ? 2 * (b + 1) : 0) + wave; };
        auto end_piece = [&](int b) { return F ? ncol : 2 * b; };
        // (from a base in scalar registers: address arithmetic of the lanes would wait for the other wavefronts' MFMAs)
        const uint32_t lane_off = (uint32_t)(8 * kq * ldL + n16) * (uint32_t)sizeof(double);
        auto load = [&](int b, int ct, double (&bt)[8]) {
            const bool some = ct < end_piece(b);
            const char* const src = (const char*)(L + (some ? (int64_t)b * kNB * ldL + 16 * ct : 0));
            const uint32_t off = some ? lane_off : 0u;
#pragma unroll
            for (int s = 0; s < 8; ++s)
                bt[s] = *(const double*)(src + (int64_t)s * ldL * (int64_t)sizeof(double) + off);
        };
        auto update = [&](int b, int ct, const double (&bt)[8]) {
            double4_t acc;
#pragma unroll
            for (int q = 0; q < 4; ++q)
                acc[q] = get(4 * q + kq, 16 * ct + n16);
#pragma unroll
            for (int s = 0; s < 8; ++s)
                acc = __builtin_amdgcn_mfma_f64_16x16x4f64(get(n16, b * kNB + 8 * kq + s), bt[s], acc, 0, 0, 0);
#pragma unroll
            for (int q = 0; q < 4; ++q)
                put(4 * q + kq, 16 * ct + n16, acc[q]);
        };
        double bt[kAhead][8], diag[kNB * kNB / THREADS];       // ... and the diagonal block after the next one
#pragma unroll
        for (int i = 0; i < kNB * kNB / THREADS; ++i)
            diag[i] = diag_entry(F ? min(1, nblk - 1) : max(nblk - 2, 0), tid + i * THREADS);
#pragma unroll
        for (int i = 0; i < kAhead; ++i)
            load(first, first_piece(first) + i * WAVES, bt[i]);
        for (int b = first; b >= 0 && b < nblk; b += step) {
            if (wave < 4) {
                double y[2];
#pragma unroll
                for (int t = 0; t < 2; ++t)
                    y[t] = get(4 * wave + kq, kNB * b + 16 * t + n16);
                const double* const Lb = Ld[b & 1];
                if (F) {
                    steps<16>([&](auto A) {
                        constexpr int a = decltype(A)::value;
                        row_fma<a>(y[1], y[0], Lb[a * (kNB + 1) + 16 + n16]);
                        row_fma<a>(y[0], y[0], Lb[a * (kNB + 1) + n16]);
                    });
                    steps<16>([&](auto A) {
                        constexpr int a = decltype(A)::value;
                        row_fma<a>(y[1], y[1], Lb[(16 + a) * (kNB + 1) + 16 + n16]);
                    });
                } else {
                    steps<16>([&](auto A) {
                        constexpr int a = 15 - decltype(A)::value;
                        row_fma<a>(y[0], y[1], Lb[n16 * (kNB + 1) + 16 + a]);
                        row_fma<a>(y[1], y[1], Lb[(16 + n16) * (kNB + 1) + 16 + a]);
                    });
                    steps<16>([&](auto A) {
                        constexpr int a = 15 - decltype(A)::value;
                        row_fma<a>(y[0], y[0], Lb[n16 * (kNB + 1) + a]);
                    });
                }
#pragma unroll
                for (int t = 0; t < 2; ++t)
                    put(4 * wave + kq, kNB * b + 16 * t + n16, y[t]);
            }
            __syncthreads();
            const int follow = F ? min(b + 1, nblk - 1) : max(b - 1, 0), after = F ? min(b + 2, nblk - 1) : max(b - 2, 0);
            if (follow != b) {
#pragma unroll
                for (int i = 0; i < kNB * kNB / THREADS; ++i)
                    Ld[follow & 1][diag_at(tid + i * THREADS)] = diag[i];
            }
#pragma unroll
            for (int i = 0; i < kNB * kNB / THREADS; ++i)
                diag[i] = diag_entry(after, tid + i * THREADS);
#pragma unroll
            for (int i = 0; i < kAhead; ++i) {
                if (first_piece(b) + i * WAVES < end_piece(b))
                    update(b, first_piece(b) + i * WAVES, bt[i]);
                load(follow, first_piece(follow) + i * WAVES, bt[i]);
            }
            for (int ct = first_piece(b) + kAhead * WAVES; ct < end_piece(b); ct += 2 * WAVES) {
                double rest[2][8];
                load(b, ct, rest[0]);
                load(b, ct + WAVES, rest[1]);
                update(b, ct, rest[0]);
                if (ct + WAVES < end_piece(b))
                    update(b, ct + WAVES, rest[1]);
            }
            __syncthreads();
        }
    };
    for (int t = tid; t < kNB * kNB; t += THREADS)
        Ld[0][diag_at(t)] = diag_entry(0, t);
    __syncthreads();
    sweep(std::true_type());
    for (int r = wave; r < 16; r += WAVES)
        for (int c = lane; c < R; c += 64)
            put(r, c, get(r, c) * dinv[c]);
    __syncthreads();
    sweep(std::false_type());          // Ld[b & 1] holds block b: the last one is still there
    for (int r = wave; r < rows; r += WAVES)
        for (int c = lane; c < R; c += 64)
            A[(r0 + r) * R + c] = get(r, c) * S[c];
}

// The same for ranks up to 32 WAVES: a wavefront keeps the 16 rows' unknowns of two blocks of 16 (wave and wave + WAVES) in the accumulators of the
// matrix cores.  A block that is final goes to the others through LDS; the wavefront that has the next one updates and solves it
// (substitute16) before its other block, so a step of the chain is four matrix instructions, a substitution and a barrier.  -L is symmetric
// as it lies in memory, so both sweeps read the same lines, two steps ahead.
// Bound by that chain, 2 R / 16 steps (0.7 us each with four wavefronts, 1.4 with sixteen), and by the matrix instructions of few compute
// units.  With the unknowns in LDS and blocks of 32, solve_rows_blocked, against this: 129 rows at R = 500 106 -> 100 us, 300 rows at
// R = 200 37 -> 30, 240 rows at R = 82 17.8 -> 15.4, 4736 at R = 87 21.9 -> 19.2.
template <int WAVES>
__global__ void __launch_bounds__(64 * WAVES)
solve_rows(const double* __restrict__ L, int ldL, const double* __restrict__ dinv, const double* __restrict__ S, int R,
           const double* __restrict__ M, double* A, int64_t I, const int* flag)
{
    extern __shared__ double diag[];             // [block][16][17]: row a of the diagonal blocks of -L
    __shared__ double Yb[2][16 * 20];            // a final block, rows of four doubles more than the columns
    if (flag[0])
        return;
    const int lane = (int)threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
    const int n16 = lane & 15, kq = lane >> 4;
    const int64_t r0 = (int64_t)blockIdx.x * 16;
    const int nb = (R + 15) / 16;
    // rows 16 b + 4 s + kq of -L, columns of this wavefront's blocks (from bases in scalar registers)
    const uint32_t lane_off = (uint32_t)(kq * ldL + n16) * (uint32_t)sizeof(double);
    auto load = [&](int b, double (&l)[2][4]) {
#pragma unroll
        for (int i = 0; i < 2; ++i)
#pragma unroll
            for (int s = 0; s < 4; ++s) {
                const char* const src = (const char*)(L + (16 * b + 4 * s) * ldL + 16 * min(wave + WAVES * i, nb - 1));
                l[i][s] = *(const double*)(src + lane_off);
            }
    };
    double y[2][4], l[3][2][4];
    load(0, l[0]);
    load(min(1, nb - 1), l[1]);
    for (int t = (int)threadIdx.x; t < 256 * nb; t += 64 * WAVES) {
        const int b = t >> 8, r = (t >> 4) & 15, c = t & 15;
        diag[(b * 16 + r) * 17 + c] = r != c ? L[(int64_t)(16 * b + r) * ldL + 16 * b + c] : 0.0;
    }
#pragma unroll
    for (int i = 0; i < 2; ++i) {
        const int c = 16 * (wave + WAVES * i) + n16;
        const double sc = c < R ? S[c] : 0.0;
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            const int64_t r = r0 + 4 * q + kq;
            const double m = M[(r < I ? r : I - 1) * R + min(c, R - 1)];
            y[i][q] = r < I && c < R ? m * sc : 0.0;
        }
    }
    auto sweep = [&](auto forward) {
        constexpr bool F = decltype(forward)::value;
        double f[16];
        auto entries = [&](int b) {                  // of block b's own part of -L
#pragma unroll
            for (int a = 0; a < 16; ++a) {
                const double t = diag[(b * 16 + a) * 17 + n16];
                f[a] = (F ? n16 > a : n16 < a) ? t : 0.0;
            }
        };
        // block i of this wavefront is final but for itself: solve it and pass it on
        auto finish = [&](auto I_) {
            constexpr int i = decltype(I_)::value;
            const int b = wave + WAVES * i;
            if (WAVES == 16)                         // (no registers for them before)
                entries(b);
            substitute16<F>(y[i], f);
#pragma unroll
            for (int q = 0; q < 4; ++q)
                Yb[b & 1][(4 * q + kq) * 20 + n16] = y[i][q];
        };
        auto with = [&](int i, auto take) {      // (the block as a constant)
            if (i == 0)
                take(std::integral_constant<int, 0>());
            else
                take(std::integral_constant<int, 1>());
        };
        auto step = [&](int b, const double (&now)[2][4], double (&ahead)[2][4]) {
            __syncthreads();
            double a[4];
#pragma unroll
            for (int s = 0; s < 4; ++s)
                a[s] = Yb[b & 1][n16 * 20 + 4 * s + kq];
            load(F ? min(b + 2, nb - 1) : max(b - 2, 0), ahead);     // (always: behind a branch all loads would be waited for)
            const int next = F ? b + 1 : b - 1;
            const int mine = next >= 0 && next < nb && next % WAVES == wave ? next / WAVES : -1;     // which of its blocks comes next
            auto update = [&](auto I_) {
                constexpr int i = decltype(I_)::value;
                double4_t c = {y[i][0], y[i][1], y[i][2], y[i][3]};
#pragma unroll
                for (int s = 0; s < 4; ++s)
                    c = __builtin_amdgcn_mfma_f64_16x16x4f64(a[s], now[i][s], c, 0, 0, 0);
#pragma unroll
                for (int q = 0; q < 4; ++q)
                    y[i][q] = c[q];
            };
            if (mine >= 0) {
                __builtin_amdgcn_s_setprio(3);       // (the others wait for this)
                with(mine, update);
                with(mine, finish);
                __builtin_amdgcn_s_setprio(0);
            }
#pragma unroll
            for (int i = 0; i < 2; ++i) {
                const int u = wave + WAVES * i;
                if (i != mine && u < nb && (F ? u > b : u < b))
                    with(i, update);
            }
            const int soon = F ? b + 2 : b - 2;
            if (WAVES < 16 && soon >= 0 && soon < nb && soon % WAVES == wave)
                entries(soon);
        };
        const int first = F ? 0 : nb - 1, second = F ? min(1, nb - 1) : max(nb - 2, 0);
        if (first % WAVES == wave) {
            entries(first);
            with(first / WAVES, finish);
        }
        if (WAVES < 16 && second != first && second % WAVES == wave)
            entries(second);
        for (int n = 0; n < nb; n += 3) {
            step(F ? n : nb - 1 - n, l[0], l[2]);
            if (n + 1 < nb)
                step(F ? n + 1 : nb - 2 - n, l[1], l[0]);
            if (n + 2 < nb)
                step(F ? n + 2 : nb - 3 - n, l[2], l[1]);
        }
    };
    __syncthreads();                             // (the diagonal blocks)
    sweep(std::true_type());
    __syncthreads();
    load(nb - 1, l[0]);
    load(max(nb - 2, 0), l[1]);
#pragma unroll
    for (int i = 0; i < 2; ++i) {
        const int c = 16 * (wave + WAVES * i) + n16;
        const double d = c < R ? dinv[c] : 0.0;
#pragma unroll
        for (int q = 0; q < 4; ++q)
            y[i][q] *= d;
    }
    sweep(std::false_type());
#pragma unroll
    for (int i = 0; i < 2; ++i) {
        const int c = 16 * (wave + WAVES * i) + n16;
        const double sc = c < R ? S[c] : 0.0;
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            const int64_t r = r0 + 4 * q + kq;
            if (r < I && c < R)
                A[r * R + c] = y[i][q] * sc;
        }
    }
}

// Columns of A (n entries) divided by their norms = the roots of the diagonal of the Gram matrix S, and the
// normalised Gram matrix.  One thread per entry of A, then of S.
__global__ void __launch_bounds__(256)
scale_by_gram(const double* __restrict__ S, int R, double* A, int64_t n, double* Gk, double* lambda, const int* flag)
{
    if (flag[0])
        return;
    const int64_t RR = (int64_t)R * R;
    for (int64_t e = (int64_t)blockIdx.x * 256 + threadIdx.x; e < n + RR; e += (int64_t)gridDim.x * 256) {
        if (e < n) {
            const int j = (int)(e % R);
            const double nrm = sqrt(S[(int64_t)j * R + j]);
            if (nrm > 0.0)
                A[e] /= nrm;
            if (e < R)
                lambda[j] = nrm;
        } else {
            const int64_t t = e - n;
            const int a = (int)(t / R), c = (int)(t - (int64_t)a * R);
            const double na = sqrt(S[(int64_t)a * R + a]), nc = sqrt(S[(int64_t)c * R + c]);
            Gk[t] = S[t] / ((na > 0.0 ? na : 1.0) * (nc > 0.0 ? nc : 1.0));
        }
    }
}

// Fit terms, partial sums: blocks [0, n_chunks) add lambda_j M(i, j) A(i, j) over their rows, blocks n_chunks + a
// lambda_a V(a, c) lambda_c over c, with V the Hadamard product of all Gram matrices.
__global__ void __launch_bounds__(256)
fit_terms_partial(const double* __restrict__ G, int ndim, int R, const double* __restrict__ lambda, const double* __restrict__ M,
                  const double* __restrict__ A, int64_t I, int n_chunks, int64_t rows_per_chunk, double* part)
{
    __shared__ double lds[256];
    double s = 0.0;
    if ((int)blockIdx.x < n_chunks) {
        const int64_t i0 = (int64_t)blockIdx.x * rows_per_chunk;
        const int64_t i1 = i0 + rows_per_chunk < I ? i0 + rows_per_chunk : I;
        for (int j = threadIdx.x; j < R; j += 256) {
            double t = 0.0;
            for (int64_t i = i0; i < i1; ++i)
                t += M[i * R + j] * A[i * R + j];
            s += lambda[j] * t;
        }
    } else {
        const int a = (int)blockIdx.x - n_chunks;
        for (int c = threadIdx.x; c < R; c += 256) {
            double v = lambda[a] * lambda[c];
            for (int m = 0; m < ndim; ++m)
                v *= G[((int64_t)m * R + a) * R + c];
            s += v;
        }
    }
    s = block_sum_256(s, lds);
    if (threadIdx.x == 0)
        part[blockIdx.x] = s;
}

// The two fit terms from their partial sums, one workgroup, fixed order, then the sweep's record.
__global__ void __launch_bounds__(256) fit_terms_sum(const double* __restrict__ part, int n_chunks, int R, double* scalars, int* flag,
                                                      SweepRecord* record, double tol, bool first)
{
    __shared__ double lds[256];
    double s = 0.0, t = 0.0;
    for (int i = threadIdx.x; i < n_chunks; i += 256)
        s += part[i];
    for (int i = n_chunks + threadIdx.x; i < n_chunks + R; i += 256)
        t += part[i];
    s = block_sum_256(s, lds);
    t = block_sum_256(t, lds);
    if (threadIdx.x == 0)
        end_sweep(scalars, flag, record, s, t, tol, first);
}

// The driver's device memory: one allocation, cut up by cpals_run.
struct Buffers {
    char* base = nullptr;
    double* M = nullptr;        // max_n I_n x R
    double* G = nullptr;        // d x R x R Gram matrices
    double* V = nullptr;        // R x R (ranks above 64)
    double* L = nullptr;        // R x R padded to whole blocks, then R values 1 / D and the R scales (ranks above 64)
    double* gram_ws = nullptr;  // partial Gram matrices, or the fit's partial sums
    double* inner = nullptr;    // column sums of M * A (ranks up to 64)
    double* partial = nullptr;  // kNormBlocks values
    double* scalars = nullptr;  // ||X||^2, the fit of the sweep before, then the flag
    int* flag = nullptr;
    SweepRecord* records = nullptr;     // kRecords of them
    void* shared_ws = nullptr;  // intermediates of the sweeps that share partial contractions
    ~Buffers() { (void)hipFree(base); }
};

void gram_big(const double* A, int64_t I, int R, double* G, hipStream_t st)
{
    const unsigned nt = (unsigned)ceil_div(R, 16);
    hipLaunchKernelGGL(gram_tiled, dim3(nt, nt), dim3(512), 0, st, A, I, R, G);
}

// The update of a factor up to rank 64: one workgroup where its rows fit the workgroup's LDS (then a second launch would take
// longer than its further tiles), else two launches.  Returns the number of blocks that left column sums of M * A in b.inner.
// The update that ends a sweep also leaves its record where it can: `end` then has none any more.
int update_small(const Buffers& b, int ndim, int k, int R, double* A, int64_t I, double* lambda, SweepEnd& end, hipStream_t st)
{
    double* const Gk = b.G + (int64_t)k * R * R;
    const SweepEnd now = k == ndim - 1 ? end : SweepEnd{nullptr, nullptr, 0.0, false};
    auto go = [&](auto nb, auto waves, auto rp) {
        constexpr int NB = decltype(nb)::value, WAVES = decltype(waves)::value, RP = decltype(rp)::value;
        const int64_t tiles = ceil_div(I, 16);
        if (tiles <= update_most_tiles(NB)) {
            const int lds = update_lds_doubles(NB, (int)tiles) * (int)sizeof(double);
            (void)hipFuncSetAttribute((const void*)als_update<NB, WAVES, true>, hipFuncAttributeMaxDynamicSharedMemorySize, lds);
            hipLaunchKernelGGL((als_update<NB, WAVES, true>), dim3(1), dim3(64 * WAVES), lds, st, b.G, ndim, k, R, b.M, A, I, tiles,
                               b.gram_ws, lambda, b.inner, b.flag, now);
            if (k == ndim - 1)
                end.record = nullptr;
            return 1;
        }
        const int64_t groups = ceil_div(tiles, WAVES);
        const int n_gram = (int)(groups < kGramBlocks ? groups : kGramBlocks);
        const int64_t want = ceil_div(I * R, 2048);
        const int64_t rows = ceil_div(I, want < kScaleBlocks ? want : kScaleBlocks);
        const int n_scale = (int)ceil_div(I, rows);
        const int lds = update_lds_doubles(NB, WAVES) * (int)sizeof(double);
        (void)hipFuncSetAttribute((const void*)als_update<NB, WAVES, false>, hipFuncAttributeMaxDynamicSharedMemorySize, lds);
        hipLaunchKernelGGL((als_update<NB, WAVES, false>), dim3((unsigned)n_gram), dim3(64 * WAVES), lds, st, b.G, ndim, k, R, b.M, A, I,
                           tiles, b.gram_ws, lambda, b.inner, b.flag, SweepEnd{nullptr, nullptr, 0.0, false});
        hipLaunchKernelGGL((als_normalise<RP>), dim3((unsigned)n_scale), dim3(512), 0, st, b.gram_ws, n_gram, R, A, b.M, I,
                           rows, Gk, lambda, k == ndim - 1 ? b.inner : nullptr, b.flag);
        return n_scale;
    };
    using std::integral_constant;
    if (R <= 16)
        return I <= 128 ? go(integral_constant<int, 1>(), integral_constant<int, 8>(), integral_constant<int, 16>())
                        : go(integral_constant<int, 1>(), integral_constant<int, 16>(), integral_constant<int, 16>());
    if (R <= 32)
        return go(integral_constant<int, 2>(), integral_constant<int, 16>(), integral_constant<int, 32>());
    if (R <= 48)
        return go(integral_constant<int, 3>(), integral_constant<int, 8>(), integral_constant<int, 64>());
    return go(integral_constant<int, 4>(), integral_constant<int, 8>(), integral_constant<int, 64>());
}

// -L, 1 / D and the scales of V for the update of factor k above rank 64.  Up to rank 128 in one workgroup: 24 us at R = 82, 29 at 99 and 34 at 128,
// where the product and two panels in launches of their own took 36, 37 and 49.
void factor_big(const Buffers& b, int ndim, int k, int R, int ldL, hipStream_t st)
{
    double* const dinv = b.L + (size_t)ldL * ldL;
    if (R <= kLdsRank) {
        const int lds = lds_factor_bytes((int)ceil_div(R, 16));
        (void)hipFuncSetAttribute((const void*)factorise_lds, hipFuncAttributeMaxDynamicSharedMemorySize, lds);
        hipLaunchKernelGGL(factorise_lds, dim3(1), dim3(1024), lds, st, b.G, ndim, R, k, b.L, ldL, dinv, dinv + R, b.flag);
        return;
    }
    hipLaunchKernelGGL(hadamard_grams, dim3((unsigned)ceil_div(ldL * ldL, 256)), dim3(256), 0, st, b.G, ndim, R, k, b.V, dinv + R, b.L, ldL);
    (void)hipFuncSetAttribute((const void*)factorise_panel, hipFuncAttributeMaxDynamicSharedMemorySize, kPanelLds);
    for (int j0 = 0; j0 < R; j0 += kPB) {
        const unsigned nt = R - j0 > kPB ? (unsigned)ceil_div(R - j0 - kPB, kPB) : 1u;
        hipLaunchKernelGGL(factorise_panel, dim3(nt, nt), dim3(512), kPanelLds, st, b.V, R, j0, b.L, ldL, dinv, b.flag);
    }
}

// Rows of A = M V^{-1} above rank 64.  Up to rank 512 the unknowns stay in registers; not where eight and sixteen wavefronts, one workgroup a
// compute unit, would take a second round that two to four of the other kernel's four wavefronts do not need (20000 rows at R = 130 101
// against 69 us, 300 297 and 201; 500, where its slab leaves one of them too, 531 and 607).  Beyond, few rows: sixteen wavefronts share a
// workgroup's columns; many rows: four.  Above rank 1024 the slab does not fit the 160 KB of LDS.
void solve_big(const double* L, int ldL, const double* dinv, const double* S, int R, const double* M, double* A, int64_t I, const int* flag, hipStream_t st)
{
    const unsigned grid = (unsigned)ceil_div(I, 16);
    const size_t lds = (size_t)16 * (ceil_div(R, kNB) * kNB + 1) * sizeof(double);
    if (R <= 128 || (R <= 512 && (grid <= 256 || R > 448))) {
        const int diag = (int)ceil_div(R, 16) * 16 * 17 * (int)sizeof(double);
        auto go = [&](auto waves) {
            constexpr int W = decltype(waves)::value;
            (void)hipFuncSetAttribute((const void*)solve_rows<W>, hipFuncAttributeMaxDynamicSharedMemorySize, diag);
            hipLaunchKernelGGL((solve_rows<W>), dim3(grid), dim3(64 * W), diag, st, L, ldL, dinv, S, R, M, A, I, flag);
        };
        R <= 128 ? go(std::integral_constant<int, 4>()) : R <= 256 ? go(std::integral_constant<int, 8>()) : go(std::integral_constant<int, 16>());
    } else if (R > 1024) {
        hipLaunchKernelGGL((solve_rows_blocked<16, false>), dim3(grid), dim3(1024), 0, st, L, ldL, dinv, S, R, M, A, I, flag);
    } else if (grid <= 512) {
        (void)hipFuncSetAttribute((const void*)solve_rows_blocked<16, true>, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
        hipLaunchKernelGGL((solve_rows_blocked<16, true>), dim3(grid), dim3(1024), lds, st, L, ldL, dinv, S, R, M, A, I, flag);
    } else {
        (void)hipFuncSetAttribute((const void*)solve_rows_blocked<4, true>, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
        hipLaunchKernelGGL((solve_rows_blocked<4, true>), dim3(grid), dim3(256), lds, st, L, ldL, dinv, S, R, M, A, I, flag);
    }
}


// ---------------------------------------------------------------------------
// Sweep that shares partial contractions between the modes (two passes over X).
// ---------------------------------------------------------------------------

// K(r, j) = prod over the modes m of A_m(r_m, j), r decomposed with the lowest mode fastest;
// row-major with leading dimension R.  One thread per entry.
template <typename T> struct ModeSet {
    const T* A[MTTKRP_MAX_NDIM];
    int64_t ld[MTTKRP_MAX_NDIM];
    int32_t dim[MTTKRP_MAX_NDIM];
    int32_t n;
};
template <typename T>
__global__ void __launch_bounds__(256) khatri_rao_rows(const ModeSet<T> p, int64_t n_entries, int R, T* __restrict__ K)
{
    const int64_t e = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (e >= n_entries)
        return;
    int64_t r = e / R;
    const int j = (int)(e - r * R);
    T v = (T)1;
    for (int m = 0; m < p.n; ++m) {
        const int64_t rn = r / p.dim[m];
        v *= p.A[m][(r - rn * p.dim[m]) * p.ld[m] + j];
        r = rn;
    }
    K[e] = v;
}

// M(i, j) = sum over the segments, in order.  One thread per entry.
template <typename T>
__global__ void __launch_bounds__(256)
sum_segments(const double* __restrict__ part, int64_t n_entries, int R, int n_seg, T* __restrict__ M, int64_t ldM)
{
    const int64_t e = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (e >= n_entries)
        return;
    const int64_t i = e / R;
    const int j = (int)(e - i * R);
    double v = 0.0;
    const double* src = part + i * n_seg * R + j;
    int q = 0;
    for (; q + 8 <= n_seg; q += 8) {         // eight requested before the first is added
        double t[8];
#pragma unroll
        for (int u = 0; u < 8; ++u)
            t[u] = src[(int64_t)(q + u) * R];
#pragma unroll
        for (int u = 0; u < 8; ++u)
            v += t[u];
    }
    for (; q < n_seg; ++q)
        v += src[(int64_t)q * R];
    M[i * ldM + j] = (T)v;
}

// The same for more segments than sixteen: 64 threads share an entry's, eight requested before the first is added, and their sums are added
// in order.  16 entries of 1024 segments 20.5 -> 3.9 us, 32 of 2048 37.8 -> 4.0.
template <typename T>
__global__ void __launch_bounds__(1024)
sum_many_segments(const double* __restrict__ part, int64_t n_entries, int R, int n_seg, T* __restrict__ M, int64_t ldM)
{
    __shared__ double red[64][17], four[16][17];
    const int n = (int)threadIdx.x & 15, g = (int)threadIdx.x >> 4;
    const int64_t own = (int64_t)blockIdx.x * 16 + n, e = own < n_entries ? own : n_entries - 1;
    const int64_t i = e / R;
    const int j = (int)(e - i * R);
    const double* const src = part + i * n_seg * R + j;
    const int per = (n_seg + 63) / 64, q1 = min(n_seg, (g + 1) * per);
    double v = 0.0;
    for (int q = g * per; q < q1; q += 8) {
        double t[8];
#pragma unroll
        for (int u = 0; u < 8; ++u)
            t[u] = src[(int64_t)min(q + u, q1 - 1) * R];
#pragma unroll
        for (int u = 0; u < 8; ++u)
            v += q + u < q1 ? t[u] : 0.0;
    }
    red[g][n] = v;
    __syncthreads();
    if (g < 16)
        four[g][n] = (red[4 * g][n] + red[4 * g + 1][n]) + (red[4 * g + 2][n] + red[4 * g + 3][n]);
    __syncthreads();
    if (g == 0 && own < n_entries) {
        v = 0.0;
#pragma unroll
        for (int u = 0; u < 16; ++u)
            v += four[u][n];
        M[i * ldM + j] = (T)v;
    }
}

// Where the modes are cut into a leading set (modes 0 .. s-1, P_L entries) and a trailing
// set (modes s .. d-1, P_R entries), and what lies where in the caller's buffer.
struct SharedPlan {
    int s = 0;
    int64_t PL = 1, PR = 1;
    int max_seg = 1;
    size_t off_TR = 0, off_KL = 0, off_TL = 0, off_part = 0, off_lead = 0, lead_bytes = 0, total = 0;
    // the first pass is a first-mode core call on (P_L, I_s, ..., I_{d-1}); its workspace
    int nd_first = 0;
    int64_t dims_first[MTTKRP_MAX_NDIM];
    size_t off_first = 0, first_bytes = 0;
    bool compact = false;       // both passes over X with the plans of least workspace
};

size_t align256(size_t n) { return (n + 255) / 256 * 256; }

// segments of the other indices for one mode: enough workgroups to fill the chip, but one, without a launch to add them, where a
// workgroup has its indices in a few rounds of requests (CP-ALS 7 x 8 x 10 x 10 x 9 x 9 at R = 8, four sweeps, 545 -> 504 us, 17 x 11 x 17 x 17 x 16 at
// R = 16 527 -> 505; 1024 x 1024 x 512 at R = 32 level)
constexpr int64_t kOneSegment = 512;
int segments(int64_t I_t, int64_t n_others)
{
    if (n_others <= kOneSegment)
        return 1;
    int64_t n = ceil_div(4096, I_t);
    const int64_t most = ceil_div(n_others, 64);
    if (n > most)
        n = most;
    return (int)(n < 1 ? 1 : n);
}

int plan_shared(int ndim, const int64_t* dims, int R, int sbytes, SharedPlan& sp)
{
    if (!dims || ndim < 2 || R < 1 || (sbytes != 4 && sbytes != 8))
        return MTTKRP_ERR_INVALID_ARG;
    if (ndim > MTTKRP_MAX_NDIM)
        return MTTKRP_ERR_UNSUPPORTED;
    int64_t N = 1;
    for (int m = 0; m < ndim; ++m) {
        if (dims[m] < 1)
            return MTTKRP_ERR_INVALID_ARG;
        if (N > ((int64_t)1 << 57) / dims[m])
            return MTTKRP_ERR_INVALID_ARG;
        N *= dims[m];
    }
    // the cut with the smallest intermediates
    int best = 0;
    int64_t best_sum = 0, PL = 1;
    for (int s = 1; s < ndim; ++s) {
        PL *= dims[s - 1];
        const int64_t PR = N / PL;
        if (PL >= ((int64_t)1 << 31) - 64 || PR >= ((int64_t)1 << 31) - 64)
            continue;
        if (best == 0 || PL + PR < best_sum) {
            best = s;
            best_sum = PL + PR;
        }
    }
    if (best == 0)
        return MTTKRP_ERR_UNSUPPORTED;
    sp.s = best;
    sp.PL = 1;
    for (int m = 0; m < best; ++m)
        sp.PL *= dims[m];
    sp.PR = N / sp.PL;
    const size_t row = (size_t)R * (size_t)sbytes;
    size_t off = 0;
    if (sp.s > 1) {
        sp.off_TR = off;  off += align256((size_t)sp.PL * row);
        sp.off_KL = off;  off += align256((size_t)sp.PL * row);
    }
    if (ndim - sp.s > 1) {
        sp.off_TL = off;  off += align256((size_t)sp.PR * row);
    }
    // segment totals of mttkrp_modesum_kernel (fp64), the largest over the modes that use it
    size_t part = 0;
    sp.max_seg = 1;
    for (int k = 0; k < ndim; ++k) {
        const bool left = k < sp.s;
        if ((left && sp.s == 1) || (!left && ndim - sp.s == 1))
            continue;
        const int n_seg = segments(dims[k], (left ? sp.PL : sp.PR) / dims[k]);
        const size_t b = (size_t)dims[k] * (size_t)n_seg * (size_t)R * sizeof(double);
        if (b > part)
            part = b;
        if (n_seg > sp.max_seg)
            sp.max_seg = n_seg;
    }
    sp.off_part = off;  off += align256(part);
    sp.nd_first = 1 + ndim - sp.s;
    sp.dims_first[0] = sp.PL;
    for (int m = sp.s; m < ndim; ++m)
        sp.dims_first[1 + m - sp.s] = dims[m];
    // the intermediates must stay small beside the tensor: an eighth of it, or 64 MiB
    double limit = 0.125 * (double)N * sbytes;
    if (limit < 64.0 * 1048576.0)
        limit = 64.0 * 1048576.0;
    for (int compact = 0; compact < 2; ++compact) {
        sp.lead_bytes = mttkrp_leading_bytes(sp.PL, sp.PR, R, sbytes, compact != 0);
        sp.first_bytes = mttkrp_dense_bytes(sp.nd_first, sp.dims_first, R, 0, sbytes, compact != 0);
        if (sp.lead_bytes == (size_t)-1 || sp.first_bytes == (size_t)-1)
            return MTTKRP_ERR_UNSUPPORTED;
        sp.compact = compact != 0;
        sp.off_lead = off;
        sp.off_first = off + align256(sp.lead_bytes);
        sp.total = sp.off_first + align256(sp.first_bytes);
        if (sp.total == 0)
            sp.total = 256;
        if ((double)sp.total <= limit)
            return MTTKRP_OK;
    }
    return MTTKRP_ERR_UNSUPPORTED;
}

template <typename T>
int mode_from_partial(const T* Tp, int n, const int64_t* dims, const T* const* factors, int t, int R, T* M,
                      double* part, hipStream_t st)
{
    // Tp (P x R, row-major, leading dimension R) holds, for every multi-index of the set's modes (lowest fastest), the sum
    // of Eq. (elem) over the other modes; mode t gets the sum over its own set's other indices, weighted with their factors
    int64_t P = 1;
    for (int m = 0; m < n; ++m)
        P *= dims[m];
    const int64_t n_others = P / dims[t];
    const int n_seg = segments(dims[t], n_others);
    if (dims[t] >= ((int64_t)1 << 31) || P >= ((int64_t)1 << 31) || n_seg > 65535 || ceil_div(R, 32) > 65535)
        return MTTKRP_ERR_UNSUPPORTED;
    auto run = [&](auto* out) {
        ModeSumArgs<T, std::remove_pointer_t<decltype(out)>> ms;
        memset(&ms, 0, sizeof(ms));
        ms.S = Tp;
        ms.part = out;
        ms.n = n;
        ms.t = t;
        ms.R = R;
        ms.ld_part = R;
        ms.n_split = 1;
        for (int m = 0; m < n; ++m) {
            ms.A[m] = m == t ? nullptr : factors[m];
            ms.ld[m] = R;
            ms.dim[m] = (int32_t)dims[m];
        }
        ms.n_pairs = (uint32_t)n_others;
        ms.per_seg = (uint32_t)ceil_div(n_others, n_seg);
        return mttkrp_modesum_launch(ms, dims[t], n_seg, st);
    };
    if (n_seg == 1)             // no segments to add
        return run(M);
    const int rc = run(part);
    if (rc != MTTKRP_OK)
        return rc;
    const int64_t n_entries = dims[t] * (int64_t)R;
    if (n_seg > 16)
        hipLaunchKernelGGL((sum_many_segments<T>), dim3((unsigned)ceil_div(n_entries, 16)), dim3(1024), 0, st,
                           part, n_entries, R, n_seg, M, (int64_t)R);
    else
        hipLaunchKernelGGL((sum_segments<T>), dim3((unsigned)ceil_div(n_entries, 256)), dim3(256), 0, st,
                           part, n_entries, R, n_seg, M, (int64_t)R);
    return hipGetLastError() == hipSuccess ? MTTKRP_OK : MTTKRP_ERR_DEVICE;
}

// The sweep: M_out[k] for k = 0 .. d-1 in this order; after(k) runs right after M_out[k] has
// been enqueued (CP-ALS updates factors[k] there: later modes then read the new factor, as in
// d separate calls).  Two passes over X: one contracts the trailing modes (every leading
// mode's result follows from it), one the leading modes.
template <typename T, typename After>
int shared_sweep(int ndim, const int64_t* dims, const T* X, const T* const* factors, int R, T* const* M_out,
                 void* workspace, size_t workspace_bytes, void* stream, After after)
{
    if (!X || !factors || !M_out)
        return MTTKRP_ERR_INVALID_ARG;
    SharedPlan sp;
    int rc = plan_shared(ndim, dims, R, (int)sizeof(T), sp);
    if (rc != MTTKRP_OK)
        return rc;
    if (!workspace || workspace_bytes < sp.total)
        return MTTKRP_ERR_WORKSPACE;
    for (int m = 0; m < ndim; ++m)
        if (!factors[m] || !M_out[m])
            return MTTKRP_ERR_INVALID_ARG;
    hipStream_t st = (hipStream_t)stream;
    char* const ws = (char*)workspace;
    double* const part = (double*)(ws + sp.off_part);
    const int s = sp.s, nr = ndim - s;
    // pass 1: contraction over the trailing modes
    if (s == 1) {
        rc = mttkrp_dense_run<T>(ndim, dims, X, factors, R, 0, M_out[0], ws + sp.off_first, sp.first_bytes, stream, sp.compact);
        if (rc != MTTKRP_OK)
            return rc;
        rc = after(0);
        if (rc != MTTKRP_OK)
            return rc;
    } else {
        const T* f2[MTTKRP_MAX_NDIM];
        f2[0] = nullptr;
        for (int m = 0; m < nr; ++m)
            f2[1 + m] = factors[s + m];
        T* const TR = (T*)(ws + sp.off_TR);
        rc = mttkrp_dense_run<T>(sp.nd_first, sp.dims_first, X, f2, R, 0, TR, ws + sp.off_first, sp.first_bytes, stream, sp.compact);
        if (rc != MTTKRP_OK)
            return rc;
        for (int k = 0; k < s; ++k) {
            rc = mode_from_partial<T>(TR, s, dims, factors, k, R, M_out[k], part, st);
            if (rc != MTTKRP_OK)
                return rc;
            rc = after(k);
            if (rc != MTTKRP_OK)
                return rc;
        }
    }
    // pass 2: contraction over the leading modes, whose factors are final now
    const T* K = factors[0];
    if (s > 1) {
        ModeSet<T> ms;
        ms.n = s;
        for (int m = 0; m < s; ++m) {
            ms.A[m] = factors[m];
            ms.ld[m] = R;
            ms.dim[m] = (int32_t)dims[m];
        }
        T* const KL = (T*)(ws + sp.off_KL);
        const int64_t n_entries = sp.PL * (int64_t)R;
        hipLaunchKernelGGL((khatri_rao_rows<T>), dim3((unsigned)ceil_div(n_entries, 256)), dim3(256), 0, st,
                           ms, n_entries, R, KL);
        K = KL;
    }
    T* const TL = nr == 1 ? M_out[ndim - 1] : (T*)(ws + sp.off_TL);
    rc = mttkrp_leading_run<T>(sp.PL, sp.PR, X, K, R, TL, ws + sp.off_lead, sp.lead_bytes, stream, sp.compact);
    if (rc != MTTKRP_OK)
        return rc;
    if (nr == 1)
        return after(ndim - 1);
    for (int k = s; k < ndim; ++k) {
        rc = mode_from_partial<T>(TL, nr, dims + s, factors + s, k - s, R, M_out[k], part, st);
        if (rc != MTTKRP_OK)
            return rc;
        rc = after(k);
        if (rc != MTTKRP_OK)
            return rc;
    }
    return MTTKRP_OK;
}

}  // namespace

extern "C" {

int mttkrp_dense_all_modes_f64(int ndim, const int64_t* dims, const double* X, const double* const* factors,
                               int R, double* const* M_out, void* stream)
{
    if (!M_out || ndim < 2 || ndim > MTTKRP_MAX_NDIM)
        return !M_out || ndim < 2 ? MTTKRP_ERR_INVALID_ARG : MTTKRP_ERR_UNSUPPORTED;
    for (int k = 0; k < ndim; ++k) {
        const int rc = mttkrp_dense_f64(ndim, dims, X, factors, R, k, M_out[k], stream);
        if (rc != MTTKRP_OK)
            return rc;
    }
    return MTTKRP_OK;
}

int mttkrp_dense_all_modes_f32(int ndim, const int64_t* dims, const float* X, const float* const* factors,
                               int R, float* const* M_out, void* stream)
{
    if (!M_out || ndim < 2 || ndim > MTTKRP_MAX_NDIM)
        return !M_out || ndim < 2 ? MTTKRP_ERR_INVALID_ARG : MTTKRP_ERR_UNSUPPORTED;
    for (int k = 0; k < ndim; ++k) {
        const int rc = mttkrp_dense_f32(ndim, dims, X, factors, R, k, M_out[k], stream);
        if (rc != MTTKRP_OK)
            return rc;
    }
    return MTTKRP_OK;
}

size_t mttkrp_dense_all_modes_shared_bytes(int ndim, const int64_t* dims, int R, int dtype_bytes)
{
    SharedPlan sp;
    if (plan_shared(ndim, dims, R, dtype_bytes, sp) != MTTKRP_OK)
        return 0;
    return sp.total;
}

int mttkrp_dense_all_modes_shared_f64(int ndim, const int64_t* dims, const double* X, const double* const* factors,
                                      int R, double* const* M_out, void* workspace, size_t workspace_bytes,
                                      void* stream)
{
    return shared_sweep<double>(ndim, dims, X, factors, R, M_out, workspace, workspace_bytes, stream,
                                [](int) { return (int)MTTKRP_OK; });
}

int mttkrp_dense_all_modes_shared_f32(int ndim, const int64_t* dims, const float* X, const float* const* factors,
                                      int R, float* const* M_out, void* workspace, size_t workspace_bytes,
                                      void* stream)
{
    return shared_sweep<float>(ndim, dims, X, factors, R, M_out, workspace, workspace_bytes, stream,
                               [](int) { return (int)MTTKRP_OK; });
}

}  // extern "C"

namespace {

// How many sweeps to enqueue before the host reads their records, after `done` sweeps with the last fits f[0], f[1], f[2], when a
// sweep takes about `us`.  Without a tolerance every sweep is wanted: as many as take 2 ms (a factorisation that fails is
// reported so much later).  With one, those behind the last sweep would run their MTTKRPs for nothing, so only as many go
// ahead as will not settle if the fit's changes shrink as they did from the last sweep but one to the last, by a margin
// of two; and what is lost when that prediction fails stays below what a wait for each of the sweeps so far costs.  60 CP-ALS
// runs of 5 to 200 sweeps (numpy), against a wait a sweep: 0.84 times as long in the mean at 60 us a sweep and a tolerance of 1e-4, 0.93 at 150,
// 0.98 at 350, at worst 1.08 (half as many as have run, whatever the fits: 0.92, 1.03, 1.06, at worst 1.24).
int sweeps_ahead(int done, const double (&f)[3], double tol, double us)
{
    const int most = us > kAheadUs ? 1 : (kAheadUs / us < kRecords ? (int)(kAheadUs / us) : kRecords);
    if (tol == 0.0)
        return most;
    if (done < 3)
        return 1;
    const double before = fabs(f[1] - f[0]), last = fabs(f[2] - f[1]);
    const double shrinks = last < 0.95 * before ? last / before : 0.95;
    const int affordable = 1 + (int)(kWaitUs * done / us < kRecords ? kWaitUs * done / us : kRecords);
    int n = 1;
    for (double change = last * shrinks; n < most && n < affordable && change > 2.0 * tol; change *= shrinks)
        ++n;
    return n;
}

int cpals_run(int ndim, const int64_t* dims, const double* X, double* const* factors, double* lambda,
              int R, int max_iters, double tol, int* iters, double* fits, void* stream, bool shared)
{
    if (!dims || !X || !factors || !lambda || !iters || ndim < 2 || R < 1 || max_iters < 1 || !(tol >= 0.0))
        return MTTKRP_ERR_INVALID_ARG;
    if (ndim > MTTKRP_MAX_NDIM || R > MTTKRP_CPALS_MAX_RANK)
        return MTTKRP_ERR_UNSUPPORTED;
    const bool big = R > kSmallRank;
    int64_t N = 1, max_I = 1;
    for (int m = 0; m < ndim; ++m) {
        if (dims[m] < 1 || !factors[m])
            return MTTKRP_ERR_INVALID_ARG;
        if (dims[m] >= ((int64_t)1 << 31))
            return MTTKRP_ERR_UNSUPPORTED;
        if (N > ((int64_t)1 << 57) / dims[m])
            return MTTKRP_ERR_INVALID_ARG;
        N *= dims[m];
        if (dims[m] > max_I)
            max_I = dims[m];
    }
    if (big && max_I > (int64_t)65535 * 16)
        return MTTKRP_ERR_UNSUPPORTED;     // the limit the header states
    *iters = 0;
    hipStream_t st = (hipStream_t)stream;
    const int RR = R * R;
    const int ldL = (int)ceil_div(R, kNB) * kNB;      // L in whole blocks (ranks above 64)
    // shared sweeps: the intermediates' buffer; without a cut that fits, d separate passes
    SharedPlan sp;
    if (shared && plan_shared(ndim, dims, R, (int)sizeof(double), sp) != MTTKRP_OK)
        shared = false;
    // One allocation: an allocation and a free each cost about as much as a sweep over a small tensor.
    Buffers b;
    GramSet gs;
    memset(&gs, 0, sizeof(gs));
    {
        size_t off = 0;
        auto take = [&](size_t values) {
            const size_t at = off;
            off += align256(values * sizeof(double));
            return at;
        };
        int64_t chunks = 0;      // partial Gram matrices of the initial factors
        if (!big)
            for (int m = 0; m < ndim; ++m) {
                gs.first[m] = (int32_t)chunks;
                gs.A[m] = factors[m];
                gs.I[m] = dims[m];
                chunks += gram_blocks(dims[m], R);
                gs.first[m + 1] = (int32_t)chunks;
            }
        const size_t o_M = take((size_t)max_I * R), o_G = take((size_t)ndim * RR), o_V = take(big ? RR : 0),
                     o_L = take(big ? (size_t)ldL * ldL + 2 * R : 0),
                     o_ws = take(big ? (size_t)kFitChunks + R : (size_t)(chunks > kGramBlocks ? chunks : kGramBlocks) * (RR + R)),
                     o_in = take(big ? 0 : (size_t)kScaleBlocks * R), o_part = take(kNormBlocks), o_sc = take(4), o_rec = take(kRecords * sizeof(SweepRecord) / sizeof(double));
        const size_t o_shared = off;
        if (hipMalloc(&b.base, off + (shared ? sp.total : 0)) != hipSuccess) {
            (void)hipGetLastError();
            b.base = nullptr;
            return MTTKRP_ERR_DEVICE;
        }
        b.M = (double*)(b.base + o_M);
        b.G = (double*)(b.base + o_G);
        b.V = (double*)(b.base + o_V);
        b.L = (double*)(b.base + o_L);
        b.gram_ws = (double*)(b.base + o_ws);
        b.inner = (double*)(b.base + o_in);
        b.partial = (double*)(b.base + o_part);
        b.scalars = (double*)(b.base + o_sc);
        b.flag = (int*)(b.scalars + 3);
        b.records = (SweepRecord*)(b.base + o_rec);
        b.shared_ws = b.base + o_shared;
    }

    // ||X||^2 once, Gram matrices of the initial factors, and the flag cleared
    const int64_t want_nb = ceil_div(N, 2048);
    const int nb = (int)(want_nb < kNormBlocks ? want_nb : kNormBlocks);
    hipLaunchKernelGGL(sumsq_partial, dim3(nb), dim3(256), 0, st, X, N, b.partial);
    if (big) {
        for (int m = 0; m < ndim; ++m)
            gram_big(factors[m], dims[m], R, b.G + (int64_t)m * RR, st);
    } else {
        const dim3 grid((unsigned)gs.first[ndim]);
        if (R <= 16)
            hipLaunchKernelGGL((gram_partial<1>), grid, dim3(256), 0, st, gs, ndim, R, b.gram_ws);
        else if (R <= 32)
            hipLaunchKernelGGL((gram_partial<2>), grid, dim3(256), 0, st, gs, ndim, R, b.gram_ws);
        else if (R <= 48)
            hipLaunchKernelGGL((gram_partial<3>), grid, dim3(256), 0, st, gs, ndim, R, b.gram_ws);
        else
            hipLaunchKernelGGL((gram_partial<4>), grid, dim3(256), 0, st, gs, ndim, R, b.gram_ws);
    }
    hipLaunchKernelGGL(gram_reduce, dim3(big ? 1u : (unsigned)ceil_div(RR, 64), big ? 1u : (unsigned)(ndim + 1)), dim3(512), 0, st, gs, b.gram_ws,
                       big ? 0 : ndim, RR, b.G, b.partial, nb, b.scalars, b.flag);

    const double* cf[MTTKRP_MAX_NDIM];
    double* mo[MTTKRP_MAX_NDIM];
    for (int m = 0; m < ndim; ++m) {
        cf[m] = factors[m];
        mo[m] = b.M;
    }
    int n_inner = 1;            // blocks that left column sums of M * A at the last update
    SweepEnd end = {nullptr, nullptr, 0.0, false};
    // the update of factor k from its MTTKRP in b.M
    auto update = [&](int k) {
        double* const Gk = b.G + (int64_t)k * RR;
        const int64_t I = dims[k];
        if (!big) {
            n_inner = update_small(b, ndim, k, R, factors[k], I, lambda, end, st);
        } else {
            double* const dinv = b.L + (size_t)ldL * ldL;
            factor_big(b, ndim, k, R, ldL, st);
            solve_big(b.L, ldL, dinv, dinv + R, R, b.M, factors[k], I, b.flag, st);
            gram_big(factors[k], I, R, b.V, st);
            const int64_t want = ceil_div(I * R + RR, 1024);
            hipLaunchKernelGGL(scale_by_gram, dim3((unsigned)(want < 4096 ? want : 4096)), dim3(256), 0, st, b.V, R, factors[k],
                               I * (int64_t)R, Gk, lambda, b.flag);
        }
        return (int)MTTKRP_OK;
    };
    // A sweep's time, estimated and then measured (the fastest group so far): MTTKRPs, launches, above rank 64 the chains of the
    // factorisation and the solves (0.6 us a column: 300 us a mode at R = 500) and their products.
    double us = 60.0 + 1e6 * ndim * (double)N * (2.0 * R / 6e13 > 8.0 / 6e12 ? 2.0 * R / 6e13 : 8.0 / 6e12);
    if (big)
        for (int m = 0; m < ndim; ++m)
            us += 0.6 * R + 1e6 * (double)RR * (4.0 * (double)dims[m] + R) / 3e13;
    // Sweeps are enqueued ahead of the records that say whether they were needed (those behind the last one change nothing but
    // b.M and V).
    SweepRecord rec[kRecords];
    double last_fits[3] = {0.0, 0.0, 0.0};
    for (int done = 0; done < max_iters;) {
        int ahead = sweeps_ahead(done, last_fits, tol, us);
        if (ahead > max_iters - done)
            ahead = max_iters - done;
        const auto start = std::chrono::steady_clock::now();
        for (int n = 0; n < ahead; ++n) {
            const bool first = done + n == 0;
            end = {b.scalars, b.records + n, tol, first};
            if (shared) {
                const int rc = shared_sweep<double>(ndim, dims, X, cf, R, mo, b.shared_ws, sp.total, stream, update);
                if (rc != MTTKRP_OK)
                    return rc;
            } else {
                for (int k = 0; k < ndim; ++k) {
                    const int rc = mttkrp_dense_f64(ndim, dims, X, cf, R, k, b.M, stream);
                    if (rc != MTTKRP_OK)
                        return rc;
                    update(k);
                }
            }
            // fit terms, unless the last update has left them: b.M still holds the last mode's MTTKRP
            if (!end.record)
                continue;
            if (big) {
                const int64_t I = dims[ndim - 1];
                const int64_t per = ceil_div(I, kFitChunks) > 16 ? ceil_div(I, kFitChunks) : 16;
                const int chunks = (int)ceil_div(I, per);
                hipLaunchKernelGGL(fit_terms_partial, dim3((unsigned)(chunks + R)), dim3(256), 0, st, b.G, ndim, R, lambda, b.M,
                                   factors[ndim - 1], I, chunks, per, b.gram_ws);
                hipLaunchKernelGGL(fit_terms_sum, dim3(1), dim3(256), 0, st, b.gram_ws, chunks, R, b.scalars, b.flag,
                                   b.records + n, tol, first);
            } else {
                hipLaunchKernelGGL(fit_terms_small, dim3(1), dim3(256), 0, st, b.G, ndim, R, lambda, b.inner, n_inner, b.scalars,
                                   b.flag, b.records + n, tol, first);
            }
        }
        if (hipMemcpyAsync(rec, b.records, (size_t)ahead * sizeof(SweepRecord), hipMemcpyDeviceToHost, st) != hipSuccess ||
            hipStreamSynchronize(st) != hipSuccess)
            return MTTKRP_ERR_DEVICE;
        const double took = std::chrono::duration<double, std::micro>(std::chrono::steady_clock::now() - start).count() / ahead;
        us = done == 0 || took < us ? took : us;
        for (int n = 0; n < ahead; ++n) {
            if (rec[n].status == kFailed)
                return MTTKRP_ERR_NUMERICAL;   // a Gram Hadamard product was not positive definite
            if (fits)
                fits[done] = rec[n].fit;
            last_fits[0] = last_fits[1];
            last_fits[1] = last_fits[2];
            last_fits[2] = rec[n].fit;
            *iters = ++done;
            if (rec[n].status == kStopped)
                return hipGetLastError() == hipSuccess ? MTTKRP_OK : MTTKRP_ERR_DEVICE;
        }
    }
    return hipGetLastError() == hipSuccess ? MTTKRP_OK : MTTKRP_ERR_DEVICE;
}

}  // namespace

extern "C" {

int mttkrp_cpals_f64(int ndim, const int64_t* dims, const double* X, double* const* factors, double* lambda,
                     int R, int max_iters, double tol, int* iters, double* fits, void* stream)
{
    return cpals_run(ndim, dims, X, factors, lambda, R, max_iters, tol, iters, fits, stream, false);
}

int mttkrp_cpals_shared_f64(int ndim, const int64_t* dims, const double* X, double* const* factors, double* lambda,
                            int R, int max_iters, double tol, int* iters, double* fits, void* stream)
{
    return cpals_run(ndim, dims, X, factors, lambda, R, max_iters, tol, iters, fits, stream, true);
}

}  // extern "C"
