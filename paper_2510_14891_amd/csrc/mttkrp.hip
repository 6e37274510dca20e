// Matrix-free dense mode-k MTTKRP for gfx950 (MI355X): kernels and C ABI.
//
// Computes M(n,j) = sum_{i: i_k=n} X(i) prod_{m!=k} A_m(i_m,j)  (paper Sec. II-B,
// Eq. (elem), lambda = 1) in one streaming pass over X.
//
// How the sum is organised (our own schedule; the paper's ELEM/SUB/TILE
// schedules of Sec. III recompute the whole product per element):
//
//   rows    = mode 0 (contiguous in memory, so loads along it coalesce)
//   batch   = mode k when k != 0 (one output row per batch value)
//   columns = every other mode; the lowest suitable one is the "inner" mode,
//             the rest are "outer" modes walked by a wave-uniform odometer
//
//   T(r, j)  = sum_c X(r, c) * P_c(j),   P_c(j) = prod_{column modes} A_m(c_m, j)
//   k == 0:  M(r, j) = T(r, j)
//   k != 0:  M(i_k, j) = sum_r A_0(r, j) * T(r, j)        (epilogue, once per item)
//
// The first line is a dense (rows x columns) * (columns x R) contraction with
// the right operand generated on the fly: a wavefront owns 16*RB rows, walks
// its columns four at a time and issues RB*JB 16x16x4 MFMAs per step, the A
// operand being X exactly as it lies in memory and the B operand being four
// freshly built partial Khatri-Rao rows.  Wavefronts never synchronise; each
// one writes a partial tile which a small second kernel sums in a fixed order
// (deterministic, no atomics; Sec. III-D's atomics are what this replaces).
#include <hip/hip_runtime.h>

#include <stdint.h>
#include <stdio.h>
#include <string.h>

#include <mutex>
#include <new>

#include "../../include/mttkrp.h"
#include "mttkrp_contract.h"
#include "mttkrp_small.h"

// Scratch memory of mttkrp_dense_f64_noalloc, the entry point for callers that cannot allocate:
// a fixed array in the library's code object, so each GPU the library runs on holds one copy at
// its own address until the process ends.  Host code never uses this name as an address; it
// asks the runtime for the device address once per device (scratch_address below).
#define MTTKRP_NOALLOC_SCRATCH_BYTES (64u << 20)
static __device__ __align__(256) unsigned char scratch[MTTKRP_NOALLOC_SCRATCH_BYTES];

// All-zero array that padding lanes of the streaming kernel load their operands from (never
// written; one copy per GPU, address looked up per device like `scratch`).
#define MTTKRP_ZERO_PAD_BYTES 4096
static __device__ __align__(256) unsigned char zero_pad[MTTKRP_ZERO_PAD_BYTES];

namespace {

constexpr int kMaxOuter = MTTKRP_MAX_NDIM - 2;
constexpr int kWaves = 4;           // independent wavefronts per workgroup
constexpr int kBlockThreads = 64 * kWaves;
constexpr int kMaxDevices = 16;
constexpr int kMaxBatchSteps = 4;   // steps of loads a batch keeps in flight at most

typedef double double4_t __attribute__((ext_vector_type(4)));
typedef float float4_t __attribute__((ext_vector_type(4)));

// 16x16x4 MFMA of each data type.  Operand A: lane l holds A[l%16][l/16];
// operand B: lane l holds B[l/16][l%16]; result: lane l, register q holds
// D[row(l,q)][l%16].
template <typename T> struct Mfma;
template <> struct Mfma<double> {
    typedef double4_t acc_t;
    static __device__ __forceinline__ acc_t run(double a, double b, acc_t c) {
        return __builtin_amdgcn_mfma_f64_16x16x4f64(a, b, c, 0, 0, 0);
    }
    static __device__ __forceinline__ int row(int lane, int q) { return 4 * q + (lane >> 4); }
};
template <> struct Mfma<float> {
    typedef float4_t acc_t;
    static __device__ __forceinline__ acc_t run(float a, float b, acc_t c) {
        return __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, 0, 0, 0);
    }
    static __device__ __forceinline__ int row(int lane, int q) { return 4 * (lane >> 4) + q; }
};


// ---------------------------------------------------------------------------
// Software-pipelined runs, one per instantiation (Pipe<T, RB, JB>, generated by
// gen_pipe.py).  The compiler places its waits for outstanding loads
// conservatively around control flow, which keeps a wavefront from overlapping
// its own loads with its own MFMAs; the hand-scheduled loop keeps several steps
// of loads in flight while the MFMAs of an earlier one run.  It covers any run of
// at least that many consecutive unmasked steps of one sweep: the bases of X and of
// the inner factor advance by constant strides (in scalar registers, lanes keep
// constant 32-bit offsets from them, or in lanes), one weight Q per column block.
// Temporaries live in fixed registers (declared as clobbers); the loads of step
// t go to operand set t modulo the ring size; every wait names how many later
// loads may still be outstanding (memory operations return in issue order).
#include "mttkrp_pipe.inc"

template <typename T> struct StreamArgs {
    const T* X;
    const T* A_row;              // factor of mode 0; epilogue weight when k != 0
    const T* A_in;               // factor of the inner column mode, null if none
    const T* A_out[kMaxOuter];   // factors of the outer column modes
    T* out;                      // M itself or the partial-sum workspace
    int64_t sx_in;               // stride of the inner mode in X (elements)
    int64_t sx_batch;            // stride of mode k in X (0 when k == 0)
    int64_t sx_out[kMaxOuter];
    int64_t o_total;             // outer iterations in all
    int64_t o_per_item;          // outer iterations per work item
    int32_t dim_out[kMaxOuter];
    int32_t n_out;
    int32_t I0, I_in, R;
    int32_t ld_in, ld_row, ld_dst;   // row strides (values) of the inner factor, of A_0, of the destination
    int32_t ld_out[kMaxOuter];      // ... of the outer modes' factors
    int32_t first_mode;          // 1 when k == 0
    int32_t n_rowblk, n_jchunk, n_batch, n_isplit;
    int32_t cols_per_isplit;     // inner columns per inner split (multiple of 4)
    int32_t n_items;
    int32_t n_slots;             // partial slots per output row (k != 0)
    int32_t n_splits;            // column-space splits (outer splits x inner splits)
    int32_t xcd_remap;
    int32_t group4;              // first mode: 1 = four wavefronts per partial tile (LDS sum)
    int32_t no_inner;            // 1: no column mode at all; A_in is only a readable dummy
    const void* zeros;           // kZeroPadBytes of zeros (operands of padding lanes)
    int32_t linear;              // 1: split s takes steps [s T / n_splits ...) of all T = o_total * steps of a sweep,
                                 //    wherever in a sweep they begin and end (n_isplit = 1, o_per_item unused)
    int32_t seg;                 // > 0: the rows are the pairs (i_0, i_1) of modes 0 and 1, I0 = seg * I_1 of them, and
                                 //    one of the two is the output mode: row r belongs to output row r / seg with weight
                                 //    A_0(r % seg, :) (A_row = A_0), or, with seg_first, to output row r % seg with
                                 //    weight A_1(r / seg, :) (A_row = A_1)
    int32_t seg_first;           // 2: the same, but the weighted tile is stored as it is (see the epilogue)
    int32_t seg_nblk;            // seg_first = 0: row tiles that can overlap one output row (slots per split)
};


// How the N 16-wide MFMA blocks of a wavefront tile map to rows (or output
// columns).  A lane feeds MFMA index m of every block, so giving it N consecutive
// rows lets one wide load instruction fetch its entries for all N blocks: block b
// holds rows N*m + b.  A load instruction carries at most 16 bytes per lane, so
// more than 16 bytes are split into two chunks of n0 and n1 blocks; chunk 0 covers
// the first 16*n0 rows, chunk 1 the next 16*n1, and within each chunk every
// 16-lane group still reads one contiguous piece of memory.
template <typename T, int N> struct Lay {
    static constexpr int G = 16 / (int)sizeof(T);
    static constexpr int n0 = N < G ? N : G;
    static constexpr int n1 = N - n0;
    static_assert(n1 <= G, "at most two chunks");
    // offset of block b's entry for MFMA index m from the tile's first row (column)
    static __device__ __forceinline__ int off(int b, int m)
    {
        return b < n0 ? n0 * m + b : 16 * n0 + n1 * m + (b - n0);
    }
};

// Load of a tensor entry.  When every 16-row segment a load instruction reads is
// a whole, aligned 128-byte line (fp64, I_0 a multiple of 16, aligned X), the line
// is never needed again and a non-temporal load keeps it from displacing the
// factor rows in L2.  Otherwise neighbouring load instructions share lines
// (fp32 segments are half lines, unaligned segments straddle two), and the
// line has to stay cacheable until its other half has been read.
template <bool NT, typename T> __device__ __forceinline__ T stream_load(const T* p)
{
    if (NT)
        return __builtin_nontemporal_load(p);
    return *p;
}

// n consecutive values; the compiler merges them into one wide load instruction
template <bool NT, int N, typename T> __device__ __forceinline__ void load_vec(const T* p, T* out)
{
#pragma unroll
    for (int i = 0; i < N; ++i)
        out[i] = stream_load<NT>(p + i);
}
// Rows use the same scheme in fp32 and for three fp64 row blocks.  With two or
// four fp64 row blocks every row block keeps a load instruction of its own (block
// b holds rows 16*b + m, 8 bytes per lane): measured on 1024- and 16384-row
// tensors, 16-byte non-temporal tensor loads cost 3 to 15 % of the bandwidth there.
template <typename T, int N> struct LayRows : Lay<T, N> {};
template <> struct LayRows<double, 2> {
    static constexpr int n0 = 1;
    static constexpr int n1 = 0;
    static __device__ __forceinline__ int off(int b, int m) { return 16 * b + m; }
};
template <> struct LayRows<double, 4> : LayRows<double, 2> {};

// the entries of one lane for all N row blocks; d1 = lane offset of chunk 1
template <bool NT, int N, typename T>
__device__ __forceinline__ void load_blocks(const T* p, int d1, T* out)
{
    typedef LayRows<T, N> L;
    if constexpr (L::n0 == 1 && L::n1 == 0 && N > 1) {
#pragma unroll
        for (int b = 0; b < N; ++b)
            out[b] = stream_load<NT>(p + 16 * b);
    } else {
        load_vec<NT, L::n0>(p, out);
        if constexpr (L::n1 > 0)
            load_vec<NT, L::n1>(p + d1, out + L::n0);
    }
}

__device__ __forceinline__ int uni(int v) { return __builtin_amdgcn_readfirstlane(v); }
__device__ __forceinline__ int64_t uni64(int64_t v)
{
    const uint32_t lo = (uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)v);
    const uint32_t hi = (uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)((uint64_t)v >> 32));
    return (int64_t)(((uint64_t)hi << 32) | lo);
}

// Register budget of one instantiation (fitted to what the compiler allocates):
// accumulators take RB*JB*4 values, every step of a batch RB + 2*JB values (X,
// factor entries, weights), and the rest is about 22 + 20*JB registers in fp64,
// 26 + 11*JB in fp32.  Aim for four wavefronts per SIMD (128 registers) when four
// steps per batch still fit, else three (168 registers) with at least two
// steps, else two (256 registers).
template <typename T, int RB, int JB> struct Budget {
    static constexpr int w = (int)sizeof(T) / 4;                 // registers per value
    static constexpr int acc = RB * JB * 4 * w;
    static constexpr int fixed = w == 2 ? 22 + 20 * JB : 26 + 11 * JB;
    static constexpr int per_step = (RB + 2 * JB) * w;
    static constexpr int fit(int regs) { return (regs - fixed - acc) / per_step; }
    static constexpr int waves = fit(128 + 8) >= 4 ? 4 : (fit(168 + 8) >= 2 ? 3 : 2);
    static constexpr int raw = waves == 4 ? fit(128 + 8) : (waves == 3 ? fit(168 + 8) : fit(256));
    static constexpr int steps = raw > kMaxBatchSteps ? kMaxBatchSteps : (raw < 2 ? 2 : raw);
};

// Runs of these tiles keep X's addresses in pointers of the lanes (gen_pipe.py: lane_pointers).
__host__ __device__ constexpr bool run_of_lane_pointers(int sbytes, int RB, int JB)
{
    return sbytes == 8 ? RB == 3 && JB == 2 : JB == 1 || RB * JB <= 2;
}
// The others take offsets of a step's four columns from the first one's start in 32 bits: an inner mode's stride (values) below 1.4 GB.
__host__ __device__ inline bool lane_offsets_fit(int64_t sx_in, int64_t sbytes) { return (3 * sx_in + 64) * sbytes < ((int64_t)1 << 32); }

// One wavefront = one work item = (row block, column-block chunk, batch value,
// inner split, outer split).  No LDS, no barriers.
//
// Outer column modes: the first one ("mid") is walked by a plain counter; the
// others ("far") only change when mid wraps, and are then re-derived from the
// linear outer index by division (rare).
//
// DEEP selects between two builds of the same kernel: with the hand-scheduled
// pipelined run (few wavefronts, many steps in flight each: best for long work
// items) or with batches only (more wavefronts: best when items are so short that
// their prologue and epilogue dominate).
template <typename T, int RB, int JB, bool NT, bool DEEP>
__global__ void __launch_bounds__(kBlockThreads, (DEEP && Pipe<T, RB, JB>::value ? Pipe<T, RB, JB>::waves : Budget<T, RB, JB>::waves))
mttkrp_stream_kernel(const StreamArgs<T> p)
{
    constexpr bool kPipe = DEEP && Pipe<T, RB, JB>::value;
    // steps per batch = steps of loads in flight; where the hand-scheduled run takes the bulk
    // of the steps, short batches leave the registers to it
    constexpr int U = kPipe ? 2 : Budget<T, RB, JB>::steps;
    typedef Mfma<T> MF;
    typedef typename MF::acc_t acc_t;

    const int lane = threadIdx.x & 63;
    const int wave = uni((int)(threadIdx.x >> 6));
    uint32_t blk = blockIdx.x;
    if (p.xcd_remap)   // workgroups go round-robin over the 8 XCDs: give each XCD a contiguous range
        blk = (blk & 7u) * (gridDim.x >> 3) + (blk >> 3);
    // Item decode.  First mode: the four wavefronts of a workgroup share (row
    // block, column chunk) and take four consecutive column-space splits, so that
    // their tiles can be summed in LDS; a whole workgroup is in range or not.
    // Other modes: one independent item per wavefront.
    const bool grouped = p.first_mode && p.group4;   // four wavefronts sum their tiles in LDS
    uint32_t it = grouped ? blk : blk * kWaves + wave;
    if (it >= (uint32_t)(grouped ? p.n_items / kWaves : p.n_items))
        return;
    // chunks of output columns first: the items that read the same piece of X are neighbours (the
    // wavefronts of one workgroup, or neighbouring workgroups), so the later ones hit in cache
    const int jchunk = uni((int)(it % (uint32_t)p.n_jchunk));  it /= (uint32_t)p.n_jchunk;
    const int rowblk = uni((int)(it % (uint32_t)p.n_rowblk));  it /= (uint32_t)p.n_rowblk;
    const int batch = uni((int)(it % (uint32_t)p.n_batch));    it /= (uint32_t)p.n_batch;
    const int group = uni((int)it);                             // first mode: split group (or split)
    const uint32_t sp = grouped ? it * kWaves + wave : it;        // column-space split
    const bool empty = sp >= (uint32_t)p.n_splits;              // padding of the last split group
    const int osp = empty ? 0 : uni((int)(sp / (uint32_t)p.n_isplit));
    const int isp = empty ? 0 : uni((int)(sp - (uint32_t)osp * (uint32_t)p.n_isplit));

    typedef LayRows<T, RB> LR;  // rows of the RB row blocks
    typedef Lay<T, JB> LC;      // output columns of the JB column blocks
    const int il = lane & 15;   // MFMA index of this lane: row index for operand A, column index for B and D
    const int kk = lane >> 4;   // which of the step's four columns this lane feeds
    const int R = p.R;

    // Rows: the last row block is shifted down to end at I0 so that every load
    // stays inside the tensor; rows it shares with the previous block are
    // dropped in the epilogue.  With fewer than 16 rows lanes clamp instead.
    const int first_row = rowblk * (16 * RB);
    int row_base = first_row;
    if (row_base + 16 * RB > p.I0)
        row_base = p.I0 > 16 * RB ? p.I0 - 16 * RB : 0;
    const int lrow = min(LR::n0 * il, p.I0 - LR::n0 - row_base);        // this lane's first row in the tile (chunk 0)
    const int xd1 = 16 * LR::n0 + (LR::n1 - LR::n0) * il;              // from there to its first row of chunk 1

    // Columns of the output (j).  A lane holds LC::n0 consecutive columns (and LC::n1 more of
    // chunk 1).  Where such a group would cross R it is moved back to end at R, so that every
    // load stays inside the factor rows; the columns it then shares with a lower lane are
    // computed twice and stored by their owner only.
    const int j_first = jchunk * (16 * JB);
    const int jt0 = j_first + LC::n0 * il;
    const int jt1 = j_first + 16 * LC::n0 + LC::n1 * il;
    const int js0 = min(jt0, R - LC::n0);
    const int js1 = LC::n1 > 0 ? min(jt1, R - LC::n1) : 0;
    int jc[JB];          // column of block jb in this lane
    bool jown[JB];       // and whether this lane stores it
#pragma unroll
    for (int jb = 0; jb < JB; ++jb) {
        jc[jb] = jb < LC::n0 ? js0 + jb : js1 + (jb - LC::n0);
        jown[jb] = jb < LC::n0 ? jc[jb] >= jt0 : jc[jb] >= jt1;
    }
    auto load_cols = [&](const T* row, T (&out)[JB]) {     // entries of a factor row at this lane's columns
        load_vec<false, LC::n0>(row + js0, out);
        if constexpr (LC::n1 > 0)
            load_vec<false, LC::n1>(row + js1, out + LC::n0);
    };
    // The same for a row that is the same for the whole wavefront: the row pointer is pinned to
    // scalar registers, so the address is formed at the load (scalar base + 32-bit lane offset)
    // and no per-lane 64-bit pointer per factor stays live across the streaming loop.
    const uint32_t joff0 = (uint32_t)js0 * (uint32_t)sizeof(T), joff1 = (uint32_t)js1 * (uint32_t)sizeof(T);
    auto load_cols_uniform = [&](const T* row, T (&out)[JB]) {
        const char* const r = (const char*)(uintptr_t)uni64((int64_t)(uintptr_t)row);
        load_vec<false, LC::n0>((const T*)(r + joff0), out);
        if constexpr (LC::n1 > 0)
            load_vec<false, LC::n1>((const T*)(r + joff1), out + LC::n0);
    };

    // Range of this item in the (outer iteration, inner column) space.
    const int ia_begin = isp * p.cols_per_isplit;
    const int ia_end = min(p.I_in, ia_begin + p.cols_per_isplit);
    const int steps_in = (ia_end - ia_begin + 3) >> 2;
    // Linear splits: the item's steps are a range of the whole (outer iteration, step) sequence,
    // balanced to within one step; it may begin and end inside a sweep.
    int64_t o_begin = (int64_t)osp * p.o_per_item;
    int o_count = empty ? 0 : uni((int)min(p.o_per_item, p.o_total - o_begin));
    int s_first = 0;                    // step of its sweep the item begins at
    int n_linear = 0;
    if (p.linear) {
        const int64_t total = p.o_total * (int64_t)steps_in;
        const int64_t q = total / p.n_splits, r = total - q * p.n_splits;
        const int64_t l0 = (int64_t)sp * q + min((int64_t)sp, r);
        n_linear = empty ? 0 : uni((int)(q + ((int64_t)sp < r ? 1 : 0)));
        o_begin = uni64(l0 / steps_in);
        s_first = uni((int)(l0 - o_begin * steps_in));
        o_count = 0;
    }

    // X is addressed from a wave-uniform base (the tile's first row at the step's first column) and a lane's constant offset, or
    // (kLane) by a pointer of each lane that holds both.  Without the run, in fp32 and with one row block, the sum of the two costs more
    // than the pointer: 45 calls with one row block 1.016 times as long, up to 1.08 (fp32 5 x 12 x 63878 x 7 at R = 6, third
    // mode 149 against 160 us), fp32 with more 1.002; fp64 with two and more row blocks is even (four by two 0.95, 4 calls).
    constexpr bool kLane = kPipe ? Pipe<T, RB, JB>::lane : RB == 1 || sizeof(T) == 4;
    static_assert(!kPipe || Pipe<T, RB, JB>::lane == run_of_lane_pointers(sizeof(T), RB, JB), "gen_pipe.py: lane_pointers");
    const int64_t xlane = lrow + (int64_t)kk * p.sx_in;
    const T* const xtile = p.X + (int64_t)batch * p.sx_batch + row_base + (kLane ? xlane : 0);
    const int64_t xl = kLane ? 0 : xlane;
    const int64_t x_step = 4 * p.sx_in;
    const bool no_inner = p.no_inner != 0;   // then A_in is a readable dummy and b = 1
    const int dim_mid = p.dim_out[0];        // 1 when there is no outer mode
    const int64_t sx_mid = p.sx_out[0];
    const bool has_mid = p.n_out > 0;
    const T* const A_mid = has_mid ? p.A_out[0] : p.A_in;   // dummy when unused

    // Last step of a sweep: lanes whose column lies beyond the inner range are padding (they
    // load zeros, see issue()).  Which lanes those are depends only on the item, not on the step.
    const bool lane_ok = kk <= ((ia_end - ia_begin - 1) & 3);

    // State of the outer walk (all wave-uniform except the factor values).
    int i_mid = 0;
    int i_far[kMaxOuter];         // i_far[m] for outer modes m >= 1
    int64_t xoff_far = 0;         // X offset of the far modes
    T Qfar[JB];                   // product of the far modes' factor entries
    T Q[JB];                      // ... times the mid mode's entry: weight of the sweep being issued
    auto load_far = [&]() {       // Qfar from the current far indices (rare)
#pragma unroll
        for (int jb = 0; jb < JB; ++jb)
            Qfar[jb] = (T)1;
#pragma unroll
        for (int m = 1; m < kMaxOuter; ++m) {
            if (m < p.n_out) {
                T a[JB];
                load_cols_uniform(p.A_out[m] + (int64_t)i_far[m] * p.ld_out[m], a);
#pragma unroll
                for (int jb = 0; jb < JB; ++jb)
                    Qfar[jb] *= a[jb];
            }
        }
    };
    auto load_Q = [&]() {         // Q of the sweep the cursor enters
        T a[JB];
        load_cols_uniform(A_mid + (int64_t)(has_mid ? i_mid : 0) * p.ld_out[0], a);
#pragma unroll
        for (int jb = 0; jb < JB; ++jb)
            Q[jb] = has_mid ? Qfar[jb] * a[jb] : Qfar[jb];
    };
#pragma unroll
    for (int m = 0; m < kMaxOuter; ++m)
        i_far[m] = 0;
    if (o_begin > 0) {   // decode the first outer index of this item (the only divisions of the walk)
        int64_t t = uni64(o_begin / dim_mid);
        i_mid = uni((int)(o_begin - t * dim_mid));
#pragma unroll
        for (int m = 1; m < kMaxOuter; ++m) {
            i_far[m] = 0;
            if (m < p.n_out) {
                const int64_t tn = uni64(t / p.dim_out[m]);
                i_far[m] = uni((int)(t - tn * p.dim_out[m]));
                t = tn;
                xoff_far += (int64_t)i_far[m] * p.sx_out[m];
            }
        }
    }
    load_far();
    load_Q();

    // Cursor of the issue side: it points at the next step to issue.
    int s_in = s_first;                 // step inside the current sweep
    const T* xp = xtile + xoff_far + (int64_t)i_mid * sx_mid + (int64_t)(ia_begin + 4 * s_first) * p.sx_in;
    const T* bbase = p.A_in + (int64_t)(ia_begin + 4 * s_first) * p.ld_in;   // wave-uniform: factor row of the step's first column
    // per-lane byte offsets of (column kk, first output column of chunk 0 / chunk 1)
    const uint32_t boff0 = ((uint32_t)kk * (uint32_t)p.ld_in + (uint32_t)js0) * (uint32_t)sizeof(T);
    const uint32_t boff1 = ((uint32_t)kk * (uint32_t)p.ld_in + (uint32_t)js1) * (uint32_t)sizeof(T);
    auto load_b = [&](const char* row, T (&out)[JB]) {      // factor entries of one step
        load_vec<false, LC::n0>((const T*)(row + boff0), out);
        if constexpr (LC::n1 > 0)
            load_vec<false, LC::n1>((const T*)(row + boff1), out + LC::n0);
    };
    const int n_steps = p.linear ? n_linear : o_count * steps_in;   // < 2^30, checked on the host
    int remaining = n_steps;        // steps not yet issued, the cursor's included
    bool parked = false;                // all steps issued: the cursor stays on the last one, weight 0
    // Steps that need no lane masking: all of a sweep when its length is a multiple of four
    // columns, else all but the last.
    const int steps_plain = ((ia_end - ia_begin) & 3) == 0 ? steps_in : steps_in - 1;

    auto next_sweep = [&]() {           // wave-uniform, once per inner sweep
        s_in = 0;
        bbase = p.A_in + (int64_t)ia_begin * p.ld_in;
        i_mid += 1;
        if (i_mid >= dim_mid) {         // mid wraps: carry into the far modes
            i_mid = 0;
            bool carry = true;
#pragma unroll
            for (int m = 1; m < kMaxOuter; ++m) {
                if (m < p.n_out && carry) {
                    i_far[m] += 1;
                    xoff_far += p.sx_out[m];
                    if (i_far[m] < p.dim_out[m]) {
                        carry = false;
                    } else {
                        xoff_far -= (int64_t)i_far[m] * p.sx_out[m];
                        i_far[m] = 0;
                    }
                }
            }
            load_far();
        }
        load_Q();
        xp = xtile + xoff_far + (int64_t)i_mid * sx_mid + (int64_t)ia_begin * p.sx_in;
    };
    // Generic single step: issue the loads of the cursor's step into one operand set ...
    // A lane whose part of the step is padding (a column past the inner range, or a step past the
    // item's last) loads both operands from a small all-zero array instead, so that the padding
    // adds exact zeros whatever the tensor and the factors hold (a non-finite value times a zero
    // weight would be a NaN).
    auto issue = [&](T (&xn)[RB], T (&bn)[JB], T (&qn)[JB]) {
        const bool last = s_in == steps_in - 1;           // wave-uniform
        const bool pad = parked || (last && !lane_ok);
        const T* const zero = reinterpret_cast<const T*>(p.zeros);
        const T* xe = pad ? zero : xp + xl;
        const char* be = pad ? (const char*)zero - boff0 : (const char*)bbase;   // (load_b adds boff0 / boff1 again)
        load_blocks<NT, RB>(xe, xd1, xn);
        load_b(be, bn);
        if (no_inner) {
#pragma unroll
            for (int jb = 0; jb < JB; ++jb)
                bn[jb] = (T)1;
        }
#pragma unroll
        for (int jb = 0; jb < JB; ++jb)
            qn[jb] = Q[jb];
    };
    // ... and move the cursor one step on.
    auto advance = [&]() {
        remaining -= 1;
        if (remaining <= 0) {
            parked = true;
            return;
        }
        s_in += 1;
        if (s_in < steps_in) {
            xp += x_step;
            bbase += 4 * (int64_t)p.ld_in;
        } else {
            next_sweep();
        }
    };

    acc_t acc[RB][JB];
#pragma unroll
    for (int r = 0; r < RB; ++r)
#pragma unroll
        for (int jb = 0; jb < JB; ++jb)
            acc[r][jb] = (acc_t)(0);

    // Steps are taken in batches of U: first all loads of the batch are issued
    // (U steps of X and factor rows in flight per wavefront), then the MFMAs of
    // the U steps run in issue order, each waiting only for its own operands.
    // Other wavefronts of the SIMD fill the gaps between batches.
    //   plain batch:   U unmasked steps of one sweep: one weight Q, constant strides
    //   generic batch: any steps (sweep boundaries, masked last step, parked padding)
    // the pipelined run takes a lane's offsets as 32-bit numbers (of X only without lane pointers)
    const bool pipe_ok = kPipe && (int64_t)p.I_in * p.ld_in * (int64_t)sizeof(T) < ((int64_t)1 << 31) &&
                         (kLane || lane_offsets_fit(p.sx_in, sizeof(T)));
    int done = 0;
    while (done < n_steps) {
        if constexpr (kPipe) {
            const int avail = parked || !pipe_ok || no_inner ? 0 : min(remaining, steps_plain - s_in);
            if (avail >= Pipe<T, RB, JB>::depth) {
                const int n_run = avail;
                const uint32_t b_step = 4u * (uint32_t)p.ld_in * (uint32_t)sizeof(T);
                if constexpr (kLane) {
                    Pipe<T, RB, JB>::template run<NT>(acc, xp, xp + xd1, x_step * (int64_t)sizeof(T), bbase, boff0, boff1, b_step, Q,
                                                      avail - Pipe<T, RB, JB>::depth);
                } else {
                    Pipe<T, RB, JB>::template run<NT>(acc, (const T*)(uintptr_t)uni64((int64_t)(uintptr_t)xp),
                                                      (uint32_t)xl * (uint32_t)sizeof(T), (uint32_t)(xl + xd1) * (uint32_t)sizeof(T),
                                                      x_step * (int64_t)sizeof(T), bbase, boff0, boff1, b_step, Q,
                                                      avail - Pipe<T, RB, JB>::depth);
                    xp += n_run * x_step;
                }
                bbase += (int64_t)n_run * 4 * p.ld_in;
                s_in += n_run;
                remaining -= n_run;
                done += n_run;
                if (remaining <= 0) {   // park on the run's last step
                    parked = true;
                    s_in -= 1;
                    xp -= x_step;
                    bbase -= 4 * (int64_t)p.ld_in;
                } else if (s_in >= steps_in) {
                    next_sweep();
                }
                continue;
            }
        }
        T xs[U][RB], bs[U][JB], qs[U][JB];
        done += U;
        if (!parked && remaining >= U && s_in + U <= steps_plain) {
            const T* xu = xp + xl;
            const char* bu = (const char*)bbase;
#pragma unroll
            for (int u = 0; u < U; ++u) {
                load_blocks<NT, RB>(xu, xd1, xs[u]);
                load_b(bu, bs[u]);
#pragma unroll
                for (int jb = 0; jb < JB; ++jb)
                    qs[u][jb] = Q[jb];
                xu += x_step;
                bu += 4 * (int64_t)p.ld_in * (int64_t)sizeof(T);
            }
            remaining -= U;
            if (remaining <= 0) {       // park on the batch's last step
                parked = true;
                s_in += U - 1;
                xp += (U - 1) * x_step;
                bbase += (U - 1) * 4 * (int64_t)p.ld_in;
            } else {
                s_in += U;
                xp += U * x_step;
                bbase += U * 4 * (int64_t)p.ld_in;
                if (s_in >= steps_in)
                    next_sweep();
            }
        } else {
#pragma unroll
            for (int u = 0; u < U; ++u) {
                issue(xs[u], bs[u], qs[u]);
                advance();
            }
        }
#pragma unroll
        for (int u = 0; u < U; ++u) {
            T bc[JB];
#pragma unroll
            for (int jb = 0; jb < JB; ++jb)
                bc[jb] = bs[u][jb] * qs[u][jb];
#pragma unroll
            for (int r = 0; r < RB; ++r)
#pragma unroll
                for (int jb = 0; jb < JB; ++jb)
                    acc[r][jb] = MF::run(xs[u][r], bc[jb], acc[r][jb]);
        }
    }

    // Epilogue.
    if (p.first_mode && !grouped) {
        T* o = p.out + (int64_t)group * ((int64_t)p.I0 * p.ld_dst);
#pragma unroll
        for (int r = 0; r < RB; ++r)
#pragma unroll
            for (int jb = 0; jb < JB; ++jb)
#pragma unroll
                for (int q = 0; q < 4; ++q) {
                    const int row = row_base + LR::off(r, MF::row(lane, q));
                    if (row >= first_row && row < p.I0 && jown[jb])
                        o[(int64_t)row * p.ld_dst + jc[jb]] = acc[r][jb][q];
                }
    } else if (p.first_mode) {
        // Sum the four wavefronts' tiles in LDS in a fixed order, (w0 + w2) + (w1 + w3);
        // all hold the same (row, column) entries in the same registers.
        extern __shared__ unsigned char lds_raw[];
        T* lds = reinterpret_cast<T*>(lds_raw);
        constexpr int kTile = RB * JB * 4 * 64;          // values per wavefront tile
        if (wave >= 2) {
            T* dst = lds + (wave - 2) * kTile + lane;
#pragma unroll
            for (int r = 0; r < RB; ++r)
#pragma unroll
                for (int jb = 0; jb < JB; ++jb)
#pragma unroll
                    for (int q = 0; q < 4; ++q)
                        dst[((r * JB + jb) * 4 + q) * 64] = acc[r][jb][q];
        }
        __syncthreads();
        if (wave < 2) {
            const T* src = lds + wave * kTile + lane;
#pragma unroll
            for (int r = 0; r < RB; ++r)
#pragma unroll
                for (int jb = 0; jb < JB; ++jb)
#pragma unroll
                    for (int q = 0; q < 4; ++q)
                        acc[r][jb][q] += src[((r * JB + jb) * 4 + q) * 64];
        }
        __syncthreads();
        if (wave == 1) {
            T* dst = lds + lane;
#pragma unroll
            for (int r = 0; r < RB; ++r)
#pragma unroll
                for (int jb = 0; jb < JB; ++jb)
#pragma unroll
                    for (int q = 0; q < 4; ++q)
                        dst[((r * JB + jb) * 4 + q) * 64] = acc[r][jb][q];
        }
        __syncthreads();
        if (wave == 0) {
            const T* src = lds + lane;
            T* o = p.out + (int64_t)group * ((int64_t)p.I0 * p.ld_dst);
#pragma unroll
            for (int r = 0; r < RB; ++r)
#pragma unroll
                for (int jb = 0; jb < JB; ++jb)
#pragma unroll
                    for (int q = 0; q < 4; ++q) {
                        const T v = acc[r][jb][q] + src[((r * JB + jb) * 4 + q) * 64];
                        const int row = row_base + LR::off(r, MF::row(lane, q));
                        if (row >= first_row && row < p.I0 && jown[jb])
                            o[(int64_t)row * p.ld_dst + jc[jb]] = v;
                    }
        }
    } else if (p.seg > 0) {
        // Rows are pairs (i_0, i_1) of modes 0 and 1, and one of the two is the output mode (Eq. 2
        // with the sum over the other taken last): row r belongs to output row r / seg and takes the
        // weight A_0(r mod seg, :) (second mode), or belongs to output row r mod seg and takes the
        // weight A_1(r / seg, :) (first mode, seg_first).  The weights go into the accumulators in
        // place (rows the tile does not own become 0), then the tile's rows are summed per output row.
        constexpr int RG = 64 / (4 * JB * (int)(sizeof(T) / 4)) < 1 ? 1 : 64 / (4 * JB * (int)(sizeof(T) / 4));
        constexpr int kTileRows = 16 * RB;
#pragma unroll
        for (int r0 = 0; r0 < RB; r0 += RG) {
            T w[RG][4][JB];
#pragma unroll
            for (int rr = 0; rr < RG; ++rr)
#pragma unroll
                for (int q = 0; q < 4; ++q)
                    if (r0 + rr < RB) {
                        const int row = min(row_base + LR::off(r0 + rr, MF::row(lane, q)), p.I0 - 1);
                        const int hi = row / p.seg;
                        load_cols(p.A_row + (int64_t)(p.seg_first ? hi : row - hi * p.seg) * p.ld_row, w[rr][q]);
                    }
#pragma unroll
            for (int rr = 0; rr < RG; ++rr)
#pragma unroll
                for (int q = 0; q < 4; ++q)
#pragma unroll
                    for (int jb = 0; jb < JB; ++jb)
                        if (r0 + rr < RB)
                            asm volatile("" : "+v"(w[rr][q][jb]));   // keeps the loads unconditional and ahead of the products
#pragma unroll
            for (int rr = 0; rr < RG; ++rr)
#pragma unroll
                for (int q = 0; q < 4; ++q)
                    if (r0 + rr < RB) {
                        const int row = row_base + LR::off(r0 + rr, MF::row(lane, q));
                        const bool ok = row >= first_row && row < p.I0;
#pragma unroll
                        for (int jb = 0; jb < JB; ++jb) {
                            const double t = (double)acc[r0 + rr][jb][q] * (double)w[rr][q][jb];
                            acc[r0 + rr][jb][q] = ok ? (T)t : (T)0;
                        }
                    }
        }
        if (p.seg_first == 2) {
            // Long first mode: a tile's rows are (nearly) all different output rows, so nothing can be
            // summed here.  The weighted tile goes to the split's own copy of all I_0 I_1 rows,
            // [split][row][R]; row i_0 + I_0 i_1 of it is slot (split, i_1) of output row i_0 for the
            // combine kernel.  Every row of every copy is written by the one tile that owns it.
            T* const o = p.out + (int64_t)sp * p.I0 * p.ld_dst;
#pragma unroll
            for (int r = 0; r < RB; ++r)
#pragma unroll
                for (int q = 0; q < 4; ++q) {
                    const int row = row_base + LR::off(r, MF::row(lane, q));
                    if (row >= first_row && row < p.I0) {
#pragma unroll
                        for (int jb = 0; jb < JB; ++jb)
                            if (jown[jb])
                                o[(int64_t)row * p.ld_dst + jc[jb]] = acc[r][jb][q];
                    }
                }
        } else if (!p.seg_first) {
            // Output rows first_row / seg .. (last row of the tile) / seg.  Each owns seg_nblk slots per
            // split, one per row tile that can overlap its seg rows: this tile is number rowblk -
            // (first tile that overlaps them).  Slots that no tile writes are zero-filled before the launch.
            const int row_end = min(first_row + kTileRows, p.I0);
            const int o_first = uni(first_row / p.seg), o_last = uni((row_end - 1) / p.seg);
            for (int io = o_first; io <= o_last; ++io) {
                const int lo = io * p.seg, hi = lo + p.seg;
                double v[JB];
#pragma unroll
                for (int jb = 0; jb < JB; ++jb)
                    v[jb] = 0.0;
#pragma unroll
                for (int r = 0; r < RB; ++r)
#pragma unroll
                    for (int q = 0; q < 4; ++q) {
                        const int row = row_base + LR::off(r, MF::row(lane, q));
                        const bool in = row >= lo && row < hi;
#pragma unroll
                        for (int jb = 0; jb < JB; ++jb)
                            v[jb] += in ? (double)acc[r][jb][q] : 0.0;
                    }
                T* o = p.out + ((int64_t)io * p.n_slots + (int64_t)sp * p.seg_nblk + (rowblk - lo / kTileRows)) * p.ld_dst;
#pragma unroll
                for (int jb = 0; jb < JB; ++jb) {
                    double t = v[jb];
                    t += __shfl_xor(t, 16);
                    t += __shfl_xor(t, 32);
                    if (kk == 0 && jown[jb])
                        o[jc[jb]] = (T)t;
                }
            }
        } else {
            // Every output row i_0 < seg gets one slot per (split, row tile), written by every tile
            // (0 where the tile holds no row of that i_0).
            int rem[RB][4];          // row mod seg
#pragma unroll
            for (int r = 0; r < RB; ++r)
#pragma unroll
                for (int q = 0; q < 4; ++q) {
                    const int row = row_base + LR::off(r, MF::row(lane, q));
                    rem[r][q] = row - (row / p.seg) * p.seg;
                }
            const int64_t slot = (int64_t)sp * p.n_rowblk + rowblk;
            for (int io = 0; io < p.seg; ++io) {
                double v[JB];
#pragma unroll
                for (int jb = 0; jb < JB; ++jb)
                    v[jb] = 0.0;
#pragma unroll
                for (int r = 0; r < RB; ++r)
#pragma unroll
                    for (int q = 0; q < 4; ++q)
#pragma unroll
                        for (int jb = 0; jb < JB; ++jb)
                            v[jb] += rem[r][q] == io ? (double)acc[r][jb][q] : 0.0;
                T* o = p.out + ((int64_t)io * p.n_slots + slot) * p.ld_dst;
#pragma unroll
                for (int jb = 0; jb < JB; ++jb) {
                    double t = v[jb];
                    t += __shfl_xor(t, 16);
                    t += __shfl_xor(t, 32);
                    if (kk == 0 && jown[jb])
                        o[jc[jb]] = (T)t;
                }
            }
        }
    } else {
        const int64_t slot = (int64_t)sp * p.n_rowblk + rowblk;
        T* o = p.out + ((int64_t)batch * p.n_slots + slot) * p.ld_dst;
        // Weighted sum over the tile's rows: M(i_k, j) += sum_r A_0(r, j) T(r, j).  The weights
        // of a group of row blocks are all loaded before any is used (one round trip to L2 per
        // group); rows this item does not own (overlap of the shifted last block) get weight 0.
        constexpr int RG = 64 / (4 * JB * (int)(sizeof(T) / 4)) < 1 ? 1 : 64 / (4 * JB * (int)(sizeof(T) / 4));
        double v[JB];
#pragma unroll
        for (int jb = 0; jb < JB; ++jb)
            v[jb] = 0.0;
#pragma unroll
        for (int r0 = 0; r0 < RB; r0 += RG) {
            T w[RG][4][JB];
#pragma unroll
            for (int rr = 0; rr < RG; ++rr)
#pragma unroll
                for (int q = 0; q < 4; ++q)
                    if (r0 + rr < RB) {
                        const int row = row_base + LR::off(r0 + rr, MF::row(lane, q));
                        load_cols(p.A_row + (int64_t)min(row, p.I0 - 1) * p.ld_row, w[rr][q]);
                    }
#pragma unroll
            for (int rr = 0; rr < RG; ++rr)
#pragma unroll
                for (int q = 0; q < 4; ++q)
#pragma unroll
                    for (int jb = 0; jb < JB; ++jb)
                        if (r0 + rr < RB)
                            asm volatile("" : "+v"(w[rr][q][jb]));   // keeps the loads unconditional and ahead of the sums
#pragma unroll
            for (int rr = 0; rr < RG; ++rr)
#pragma unroll
                for (int q = 0; q < 4; ++q)
                    if (r0 + rr < RB) {
                        const int row = row_base + LR::off(r0 + rr, MF::row(lane, q));
                        const bool ok = row >= first_row && row < p.I0;
#pragma unroll
                        for (int jb = 0; jb < JB; ++jb) {
                            const double t = (double)acc[r0 + rr][jb][q] * (double)w[rr][q][jb];
                            v[jb] += ok ? t : 0.0;
                        }
                    }
        }
#pragma unroll
        for (int jb = 0; jb < JB; ++jb) {
            double t = v[jb];
            t += __shfl_xor(t, 16);
            t += __shfl_xor(t, 32);
            if (kk == 0 && jown[jb])
                o[jc[jb]] = (T)t;
        }
    }
}

// What a streaming launch needs beforehand, in one launch (three separate ones cost about 4 us each):
//   the product matrices of up to two fused pairs of modes, F(i_a + I_a i_b, j) = A_a(i_a, j) A_b(i_b, j),
//   row-major with leading dimension R, one thread per entry;
//   zeros in n_words 32-bit words of the partial sums (grid-stride over the remaining blocks).
template <typename T> struct PrepareArgs {
    const T* Aa[2];
    const T* Ab[2];
    T* F[2];
    int64_t lda[2], ldb[2];
    uint32_t Ia[2], n_entries[2], blocks[2];     // n_entries < 2^31: product matrices are at most 32 MiB
    uint32_t* zero;
    int64_t n_words;
    uint32_t zero_blocks;
    int32_t R;
};
template <typename T>
__global__ void __launch_bounds__(256)
mttkrp_prepare_kernel(const PrepareArgs<T> p)
{
    uint32_t b = blockIdx.x;
#pragma unroll
    for (int f = 0; f < 2; ++f) {
        if (b < p.blocks[f]) {
            const uint32_t e = b * 256 + threadIdx.x;
            if (e < p.n_entries[f]) {
                const uint32_t row = e / (uint32_t)p.R, j = e - row * (uint32_t)p.R;
                const uint32_t ib = row / p.Ia[f], ia = row - ib * p.Ia[f];
                p.F[f][e] = p.Aa[f][ia * p.lda[f] + j] * p.Ab[f][ib * p.ldb[f] + j];
            }
            return;
        }
        b -= p.blocks[f];
    }
    for (int64_t e = (int64_t)b * 256 + threadIdx.x; e < p.n_words; e += (int64_t)p.zero_blocks * 256)
        p.zero[e] = 0u;
}

// M(n, j) = sum of the partial sums of all slots, in fp64 and in a fixed order:
// SL threads share one output entry, thread q adds slots q, q + SL, ... in
// increasing order, then the SL subtotals are added in order of q.  A block
// covers 16 consecutive entries, so each slot is read in contiguous pieces.
// SL = 16, or 64 when the output is small and the slots are many (few blocks
// would otherwise each walk a long chain of dependent loads); which one runs
// depends on the sizes only, so results are reproducible.
template <typename T, int SL>
__global__ void __launch_bounds__(16 * SL)
mttkrp_combine_kernel(const T* __restrict__ ws, T* __restrict__ M, int64_t n_elems, int R,
                      int n_slots, int64_t stride_row, int64_t stride_slot,
                      const T* __restrict__ lambda, double beta, int64_t ldM)
{
    __shared__ double part[SL][17];
    const int el = threadIdx.x & 15;
    const int sl = threadIdx.x >> 4;
    const int64_t e = (int64_t)blockIdx.x * 16 + el;
    double s = 0.0;
    if (e < n_elems) {
        const int64_t n = e / R;
        const int j = (int)(e - n * R);
        const T* src = ws + n * stride_row + j;
        int t = sl;
        for (; t + 3 * SL < n_slots; t += 4 * SL) {
            const double v0 = (double)src[(int64_t)t * stride_slot];
            const double v1 = (double)src[(int64_t)(t + SL) * stride_slot];
            const double v2 = (double)src[(int64_t)(t + 2 * SL) * stride_slot];
            const double v3 = (double)src[(int64_t)(t + 3 * SL) * stride_slot];
            s += v0;
            s += v1;
            s += v2;
            s += v3;
        }
        for (; t < n_slots; t += SL)
            s += (double)src[(int64_t)t * stride_slot];
    }
    part[sl][el] = s;
    __syncthreads();
    if (sl == 0 && e < n_elems) {
        double v = 0.0;
#pragma unroll
        for (int q = 0; q < SL; ++q)
            v += part[q][el];
        const int64_t n = e / R;
        const int64_t dst = n * ldM + (e - n * R);
        if (lambda)                      // Eq. (krp): ... diag(lambda)
            v *= (double)lambda[e % R];
        if (beta != 0.0)                 // M is read only when it is accumulated into
            v += beta * (double)M[dst];
        M[dst] = (T)v;
    }
}

// The same sums, bit for bit those of SL = 16, by one thread an entry: subtotal q of slots q, q + 16, ... in a register of its own, Q
// slots requested before the first is added.  With at most Q = 4 or 16 slots the kernel above keeps 16 threads, 16 LDS
// entries and a barrier for as many values, and with large outputs there are threads enough without them: 145071 x 10
// entries of one slot in fp64 47 -> 9.3 us, 10 x 132904 x 10 x 10 fp32 at R = 32, all modes, 907 -> 798; small outputs are level.
template <typename T, int Q>
__global__ void __launch_bounds__(256)
mttkrp_combine_entries_kernel(const T* __restrict__ ws, T* M, int64_t n_elems, int R, int n_slots, int64_t stride_row,
                              int64_t stride_slot, const T* __restrict__ lambda, double beta, int64_t ldM)
{
    const int64_t e = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (e >= n_elems)
        return;
    const int64_t n = n_elems <= 0xffffffffll ? (int64_t)((uint32_t)e / (uint32_t)R) : e / R;
    const int j = (int)(e - n * R);
    const T* const src = ws + n * stride_row + j;
    T* const dst = M + n * ldM + j;
    const double before = beta != 0.0 ? (double)*dst : 0.0;      // M is read only when it is accumulated into
    const double weight = lambda ? (double)lambda[j] : 1.0;
    double part[Q];
#pragma unroll
    for (int q = 0; q < Q; ++q)
        part[q] = 0.0;
    for (int t = 0; t < n_slots; t += Q) {
        T v[Q];
#pragma unroll
        for (int q = 0; q < Q; ++q)
            v[q] = src[(int64_t)min(t + q, n_slots - 1) * stride_slot];
#pragma unroll
        for (int q = 0; q < Q; ++q)
            part[q] += t + q < n_slots ? (double)v[q] : 0.0;
    }
    double v = 0.0;
#pragma unroll
    for (int q = 0; q < Q; ++q)
        v += part[q];
    if (lambda)
        v *= weight;
    if (beta != 0.0)
        v += beta * before;
    *dst = (T)v;
}

// First of two passes when the output is small and the slots are very many (the combine kernel
// alone would run on a handful of compute units): block (x, g) adds the slots of group g, chunk
// consecutive ones, for 16 entries as the combine kernel does, and leaves the sum in the group's
// first slot.  A block reads all it needs of that slot before it writes it, and no other block
// touches the slots of group g for these entries.
template <typename T>
__global__ void __launch_bounds__(1024)
mttkrp_fold_kernel(T* __restrict__ ws, int64_t n_elems, int R, int n_slots, int chunk,
                   int64_t stride_row, int64_t stride_slot)
{
    constexpr int SL = 64;
    __shared__ double part[SL][17];
    const int el = threadIdx.x & 15;
    const int sl = threadIdx.x >> 4;
    const int64_t e = (int64_t)blockIdx.x * 16 + el;
    const int t_first = (int)blockIdx.y * chunk;
    const int t_end = min(n_slots, t_first + chunk);
    double s = 0.0;
    T* src = nullptr;
    if (e < n_elems) {
        const int64_t n = e / R;
        src = ws + n * stride_row + (e - n * R);
        for (int t = t_first + sl; t < t_end; t += SL)
            s += (double)src[(int64_t)t * stride_slot];
    }
    part[sl][el] = s;
    __syncthreads();
    if (sl == 0 && e < n_elems) {
        double v = 0.0;
#pragma unroll
        for (int q = 0; q < SL; ++q)
            v += part[q][el];
        src[(int64_t)t_first * stride_slot] = (T)v;
    }
}

template <typename T>
void launch_combine(T* ws, T* M, int64_t n_elems, int R, int n_slots, int64_t stride_row, int64_t stride_slot,
                    const T* lambda, double beta, int64_t ldM, hipStream_t st)
{
    const dim3 grid((unsigned)((n_elems + 15) / 16));
    if (grid.x < 64 && n_slots >= 2048) {
        // (10^8 entries, 10 x 8 outputs, 10 000 slots: 29 us on five compute units)
        int groups = (int)((256 + grid.x - 1) / grid.x);
        if (groups > n_slots / 64)
            groups = n_slots / 64;
        const int chunk = (n_slots + groups - 1) / groups;
        groups = (n_slots + chunk - 1) / chunk;
        hipLaunchKernelGGL((mttkrp_fold_kernel<T>), dim3(grid.x, (unsigned)groups), dim3(1024), 0, st, ws, n_elems, R,
                           n_slots, chunk, stride_row, stride_slot);
        n_slots = groups;
        stride_slot *= chunk;
    }
    // (few entries: a workgroup of one wavefront each, on more compute units)
    const dim3 threads(n_elems < 65536 ? 64 : 256), entries((unsigned)((n_elems + threads.x - 1) / threads.x));
    if (n_slots <= 4)
        hipLaunchKernelGGL((mttkrp_combine_entries_kernel<T, 4>), entries, threads, 0, st, ws, M, n_elems, R, n_slots,
                           stride_row, stride_slot, lambda, beta, ldM);
    else if (n_slots <= 16 || (n_elems >= 131072 && n_slots < 256))
        hipLaunchKernelGGL((mttkrp_combine_entries_kernel<T, 16>), entries, threads, 0, st, ws, M, n_elems, R, n_slots,
                           stride_row, stride_slot, lambda, beta, ldM);
    else if (n_elems <= 65536 && n_slots >= 256)
        hipLaunchKernelGGL((mttkrp_combine_kernel<T, 64>), grid, dim3(1024), 0, st, ws, M, n_elems, R, n_slots,
                           stride_row, stride_slot, lambda, beta, ldM);
    else
        hipLaunchKernelGGL((mttkrp_combine_kernel<T, 16>), grid, dim3(256), 0, st, ws, M, n_elems, R, n_slots,
                           stride_row, stride_slot, lambda, beta, ldM);
}

// ---------------------------------------------------------------------------
// Second schedule, for k != 0 when the column space (all modes other than 0 and
// k) is short and mode 0 is long: the streaming kernel above would cut the work
// into very many items of a few steps each, every one paying its prologue and
// its epilogue.  Here the MFMA contraction runs over mode 0 instead:
//
//   S(c, j)   = sum_r X(r, i_k, c) * A_0(r, j)            K dimension = rows
//   M(i_k, j) = sum_c W(c, j) * S(c, j),   W(c, j) = prod_{column modes} A_m(c_m, j)
//
// which is Eq. (elem) with the sums taken in another order.  W (C x R, C small)
// is formed by a small kernel first.  A wavefront owns 16*CB columns c of one
// i_k and 16*JB output columns j, and walks a range of rows 16 at a time: lane
// (il, kq) holds the four rows 4 kq .. 4 kq + 3 of column c = il, MFMA t of the step
// takes row t of every lane, and the B operand holds the matching rows of A_0.  In
// the pipelined run the fp64 tensor loads read whole 128-byte lines (the two lanes of
// an even/odd column pair load and exchange halves, see gen_rows_pipe.py).  Loads of U steps are kept in flight
// in a ring of operand sets.  The epilogue weights the tile with W, sums it over c
// and writes one partial row of M per item (slot = row split x column chunk),
// which the combine kernel adds up.
constexpr int kRowSumMaxSets = 4;   // operand sets in the plain loop's ring at most
template <typename T> struct RowSumArgs {
    const T* X;
    const T* A0;                 // factor of mode 0, leading dimension ld0
    const T* W;                  // weights of the column space, C x R, leading dimension R
    T* out;                      // M itself (one slot) or the partial-sum workspace
    int64_t sx_batch;            // stride of mode k in X (elements)
    int64_t sx_lo, sx_hi;        // strides of the column indices below and above k
    int32_t C_lo, C;             // columns below k; columns in all (c = c_lo + C_lo * c_hi)
    int32_t I0, R, ld0, ld_dst;
    int32_t n_cchunk, n_jchunk, n_batch, n_rsplit;
    int32_t rows_per_split;      // multiple of 16
    int32_t n_items, n_slots;
    int32_t store_s;             // 1: write S(c, j) itself (one output row per column c), no weights
};

// Software-pipelined runs of this kernel's loop (RowsPipe<T, CB, JB>, generated by
// gen_rows_pipe.py): any number >= depth of full 16-row steps, D steps of loads in flight.
#include "mttkrp_rows_pipe.inc"

template <typename T, int CB, int JB> struct RowSumBudget {
    static constexpr int w = (int)sizeof(T) / 4;
    static constexpr int acc = CB * JB * 4 * w;
    static constexpr int per_step = (CB + JB) * 4 * w;
    static constexpr int fixed = 56;
    // operand sets in the ring: as many as fit next to the accumulators, at most kRowSumMaxSets
    static constexpr int fitU = (244 - acc - fixed) / per_step;
    static constexpr bool piped = RowsPipe<T, CB, JB>::value;
    // with a pipelined run the plain loop only takes items shorter than the run's depth: two sets
    static constexpr int U = piped || fitU < 2 ? 2 : (fitU > kRowSumMaxSets ? kRowSumMaxSets : fitU);
    static constexpr int regs = acc + U * per_step + fixed;
    static constexpr int waves = piped ? RowsPipe<T, CB, JB>::waves : (regs <= 128 ? 4 : (regs <= 168 ? 3 : 2));
};

template <typename T, int CB, int JB>
__global__ void __launch_bounds__(kBlockThreads, (RowSumBudget<T, CB, JB>::waves))
mttkrp_rowsum_kernel(const RowSumArgs<T> p)
{
    constexpr int U = RowSumBudget<T, CB, JB>::U;
    typedef Mfma<T> MF;
    typedef typename MF::acc_t acc_t;

    const int lane = threadIdx.x & 63;
    const int wave = uni((int)(threadIdx.x >> 6));
    uint32_t it = blockIdx.x * kWaves + wave;
    if (it >= (uint32_t)p.n_items)
        return;
    // items that share tensor data are neighbours: column-block chunks of j first
    const int jchunk = uni((int)(it % (uint32_t)p.n_jchunk));  it /= (uint32_t)p.n_jchunk;
    const int cchunk = uni((int)(it % (uint32_t)p.n_cchunk));  it /= (uint32_t)p.n_cchunk;
    const int batch = uni((int)(it % (uint32_t)p.n_batch));    it /= (uint32_t)p.n_batch;
    const int rsplit = uni((int)it);
    const int il = lane & 15;   // operand A: column c of the tile; operand B and result: output column j
    const int kq = lane >> 4;   // which four rows of a 16-row step this lane feeds
    // Rows of a step fed by this lane: 4 kq + t for MFMA t = 0..3.
    constexpr int kLaneRows = 4;
    constexpr int kHalf = 2;
    auto t_row = [](int t) { return t; };
    const int lane_row = kLaneRows * kq;

    const int r_begin = rsplit * p.rows_per_split;
    const int n_rows = min(p.I0 - r_begin, p.rows_per_split);     // >= 1
    const int n_full = n_rows >> 4;
    const int ld0 = p.ld0;

    // Columns beyond C read column C - 1 and get weight 0 in the epilogue.
    const int c_first = cchunk * (16 * CB);
    const T* xcol[CB];          // this lane's first row (r_begin + 4 kq) of its column of block cb
#pragma unroll
    for (int cb = 0; cb < CB; ++cb) {
        const int c = min(c_first + 16 * cb + il, p.C - 1);
        const int c_hi = c / p.C_lo;
        const int c_lo = c - c_hi * p.C_lo;
        xcol[cb] = p.X + (int64_t)batch * p.sx_batch + (int64_t)c_lo * p.sx_lo + (int64_t)c_hi * p.sx_hi +
                   (r_begin + lane_row);
    }
    // Output columns as in the streaming kernel, for up to eight column blocks: the JB blocks are
    // taken in chunks of G (what one 16-byte load holds); in chunk ch a lane holds n consecutive
    // columns, so that one wide load fetches its entries of a row of A_0 or W for the chunk's
    // blocks.  A group that would cross R is moved back to end at R and stores only the columns
    // it owns.
    constexpr int G = 16 / (int)sizeof(T);
    constexpr int NCH = (JB + G - 1) / G;
    const int j_first = jchunk * (16 * JB);
    int js[NCH];         // first column this lane loads in chunk ch
    int jc[JB];          // column of block jb in this lane
    bool jown[JB];       // and whether this lane stores it
#pragma unroll
    for (int ch = 0; ch < NCH; ++ch) {
        const int n = JB - G * ch < G ? JB - G * ch : G;
        const int jt = j_first + 16 * G * ch + n * il;
        js[ch] = min(jt, p.R - n);
#pragma unroll
        for (int e = 0; e < n; ++e) {
            jc[G * ch + e] = js[ch] + e;
            jown[G * ch + e] = js[ch] + e >= jt;
        }
    }
    auto load_cols = [&](const T* row, T (&out)[JB]) {
#pragma unroll
        for (int ch = 0; ch < NCH; ++ch) {
            constexpr int kLast = JB - G * (NCH - 1);
            if (ch < NCH - 1)
                load_vec<false, G>(row + js[ch], out + G * ch);
            else
                load_vec<false, kLast>(row + js[ch], out + G * ch);
        }
    };
    const T* const bp = p.A0 + (int64_t)(r_begin + lane_row) * ld0;   // this lane's first row of A_0

    acc_t acc[CB][JB];
#pragma unroll
    for (int cb = 0; cb < CB; ++cb)
#pragma unroll
        for (int jb = 0; jb < JB; ++jb)
            acc[cb][jb] = (acc_t)(0);

    auto load_step = [&](int s, T (&x)[CB][4], T (&b)[4][JB]) {     // s: wave-uniform step, all 16 rows exist
#pragma unroll
        for (int cb = 0; cb < CB; ++cb) {
            load_vec<false, 2>(xcol[cb] + 16 * (int64_t)s, x[cb]);
            load_vec<false, 2>(xcol[cb] + 16 * (int64_t)s + kHalf, x[cb] + 2);
        }
        const T* br = bp + (int64_t)s * 16 * ld0;
#pragma unroll
        for (int t = 0; t < 4; ++t)
            load_cols(br + (int64_t)t_row(t) * ld0, b[t]);
    };
    auto compute = [&](const T (&x)[CB][4], const T (&b)[4][JB]) {
#pragma unroll
        for (int t = 0; t < 4; ++t)
#pragma unroll
            for (int cb = 0; cb < CB; ++cb)
#pragma unroll
                for (int jb = 0; jb < JB; ++jb)
                    acc[cb][jb] = MF::run(x[cb][t], b[t][jb], acc[cb][jb]);
    };

    bool piped = false;
    if constexpr (RowsPipe<T, CB, JB>::value) {
        // the run addresses A_0 with 32-bit byte offsets from the item's first row
        const bool pipe_ok = ((int64_t)p.rows_per_split + 16) * ld0 * (int64_t)sizeof(T) < ((int64_t)1 << 31);
        if (pipe_ok && n_full >= RowsPipe<T, CB, JB>::depth) {
            // Tensor pointers of the run.  fp32: this lane's column, rows 4 kq ...  fp64: the two
            // columns of the lane's even/odd pair, 16-byte piece 2 kq + e of their lines (e = il & 1):
            // the run's loads then read whole 128-byte lines and the pair exchanges halves.
            constexpr int XP = RowsPipe<T, CB, JB>::xptrs;
            const T* xq[XP];
            if constexpr (XP == CB) {
#pragma unroll
                for (int cb = 0; cb < CB; ++cb)
                    xq[cb] = xcol[cb];
            } else {
#pragma unroll
                for (int cb = 0; cb < CB; ++cb)
#pragma unroll
                    for (int h = 0; h < 2; ++h) {
                        const int c = min(c_first + 16 * cb + ((il & ~1) | h), p.C - 1);
                        const int c_hi = c / p.C_lo;
                        const int c_lo = c - c_hi * p.C_lo;
                        xq[2 * cb + h] = p.X + (int64_t)batch * p.sx_batch + (int64_t)c_lo * p.sx_lo +
                                         (int64_t)c_hi * p.sx_hi + (r_begin + 2 * (2 * kq + (il & 1)));
                    }
            }
            const T* const row0 = p.A0 + (int64_t)r_begin * ld0;
            const T* const bb[4] = {row0, row0 + ld0, row0 + (int64_t)t_row(2) * ld0, row0 + (int64_t)t_row(3) * ld0};
            uint32_t bo[NCH];       // byte offsets of this lane's entries of a row of A_0, one per chunk
#pragma unroll
            for (int ch = 0; ch < NCH; ++ch)
                bo[ch] = ((uint32_t)lane_row * (uint32_t)ld0 + (uint32_t)js[ch]) * (uint32_t)sizeof(T);
            RowsPipe<T, CB, JB>::run(acc, xq, (int64_t)(16 * sizeof(T)), bb, bo,
                                     16u * (uint32_t)ld0 * (uint32_t)sizeof(T), n_full - RowsPipe<T, CB, JB>::depth);
            piped = true;
        }
    }
    if (n_full > 0 && !piped) {
        // Ring of U operand sets: set u holds step s + u when the pass over s begins; the load
        // issued in sub-step u refills the set that was consumed in the sub-step before.  Steps
        // past the last one re-read the last one (never consumed).
        T xs[U][CB][4], bs[U][4][JB];
        const int last = n_full - 1;
#pragma unroll
        for (int u = 0; u < U - 1; ++u)
            load_step(min(u, last), xs[u], bs[u]);
        const int n_main = n_full - n_full % U;
        for (int s = 0; s < n_main; s += U) {
#pragma unroll
            for (int u = 0; u < U; ++u) {
                load_step(min(s + u + U - 1, last), xs[(u + U - 1) % U], bs[(u + U - 1) % U]);
                compute(xs[u], bs[u]);
            }
        }
        const int rem = n_full - n_main;       // < U steps left, already in sets 0 .. rem - 1
#pragma unroll
        for (int u = 0; u < U - 1; ++u)
            if (u < rem)
                compute(xs[u], bs[u]);
    }
    if (n_rows & 15) {
        // Last, partial step: rows past the end read the item's last row and enter as zeros.
        T x[CB][4], b[4][JB];
#pragma unroll
        for (int t = 0; t < 4; ++t) {
            const int r = 16 * n_full + lane_row + t_row(t);  // relative to r_begin
            const bool ok = r < n_rows;
            const int d = (ok ? r : n_rows - 1) - lane_row;   // relative to this lane's first row
#pragma unroll
            for (int cb = 0; cb < CB; ++cb) {
                const T v = xcol[cb][d];
                x[cb][t] = ok ? v : (T)0;
            }
            load_cols(bp + (int64_t)d * ld0, b[t]);
#pragma unroll
            for (int jb = 0; jb < JB; ++jb)
                b[t][jb] = ok ? b[t][jb] : (T)0;
        }
        compute(x, b);
    }

    if (p.store_s) {
        // Partial contraction over mode 0 only: S(c, j) is the result, row c of the output (one
        // slot per row split).  Every lane holds four rows c of each accumulator tile.
#pragma unroll
        for (int cb = 0; cb < CB; ++cb)
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                const int c = c_first + 16 * cb + MF::row(lane, q);
                if (c < p.C) {
                    T* const o = p.out + ((int64_t)c * p.n_slots + rsplit) * p.ld_dst;
#pragma unroll
                    for (int jb = 0; jb < JB; ++jb)
                        if (jown[jb])
                            o[jc[jb]] = acc[cb][jb][q];
                }
            }
        return;
    }
    // Epilogue: M(i_k, j) += sum_c W(c, j) S(c, j) over the tile's columns, in fp64.
    const int slot = rsplit * p.n_cchunk + cchunk;
    T* o = p.out + ((int64_t)batch * p.n_slots + slot) * p.ld_dst;
    double v[JB];
#pragma unroll
    for (int jb = 0; jb < JB; ++jb)
        v[jb] = 0.0;
#pragma unroll
    for (int cb = 0; cb < CB; ++cb) {
        T w[4][JB];
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            const int c = c_first + 16 * cb + MF::row(lane, q);
            load_cols(p.W + (int64_t)min(c, p.C - 1) * p.R, w[q]);
        }
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            const int c = c_first + 16 * cb + MF::row(lane, q);
#pragma unroll
            for (int jb = 0; jb < JB; ++jb) {
                const double t = (double)acc[cb][jb][q] * (double)w[q][jb];
                v[jb] += c < p.C ? t : 0.0;
            }
        }
    }
#pragma unroll
    for (int jb = 0; jb < JB; ++jb) {
        double t = v[jb];
        t += __shfl_xor(t, 16);
        t += __shfl_xor(t, 32);
        if (kq == 0 && jown[jb])
            o[jc[jb]] = (T)t;
    }
}

// W(c, j) = prod over the column modes of A_m(c_m, j), c decomposed with the lowest
// mode fastest; row-major with leading dimension R.  One thread per entry.
template <typename T> struct ColWeightArgs {
    const T* A[MTTKRP_MAX_NDIM - 1];
    int64_t ld[MTTKRP_MAX_NDIM - 1];
    int32_t dim[MTTKRP_MAX_NDIM - 1];
    int32_t n;                   // column modes (0: W is all ones)
};
template <typename T>
__global__ void __launch_bounds__(256)
mttkrp_colweights_kernel(const ColWeightArgs<T> p, int64_t n_entries, int R, T* __restrict__ W)
{
    const int64_t e = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (e >= n_entries)
        return;
    int64_t c = e / R;
    const int j = (int)(e - c * R);
    T v = (T)1;
    for (int m = 0; m < p.n; ++m) {
        const int64_t cn = c / p.dim[m];
        v *= p.A[m][(c - cn * p.dim[m]) * p.ld[m] + j];
        c = cn;
    }
    W[e] = v;
}

// ---------------------------------------------------------------------------
// Host side: plan, launch, C ABI
// ---------------------------------------------------------------------------

// What a plan may take beyond the one it replaces: the array of mttkrp_dense_f64_noalloc, so that no call is refused there
// for a faster plan.
constexpr double kNoallocBytes = 67108864.0;

struct Tuning {
    int64_t row_blocks = 0;
    int64_t target_items = 0;
    int64_t max_steps = 0;
    int64_t xcd_remap = 0;
    int64_t ws_percent = 0;
    int64_t max_col_blocks = 0;
    int64_t first_group = 0;
    int64_t waves_per_simd = 0;
    int64_t nt_loads = 0;
    int64_t deep = 0;
    int64_t fuse_bytes = 0;
    int64_t inner_splits = 0;
    int64_t contract_rows = 0;
    int64_t rows_col_blocks = 0;
    int64_t linear = 0;
    int64_t pair_rows = 0;
    int64_t fuse_rows = 0;
    int64_t lead_last = 0;
    int64_t small_route = 0;
    int64_t small_groups = 0;
    int64_t lds_contract = 0;
};
Tuning g_tune;
std::mutex g_mutex;

// The keys as they are now.  Taken once per call: what is planned in pieces is planned with the same keys throughout.
Tuning tuning()
{
    std::lock_guard<std::mutex> lock(g_mutex);
    return g_tune;
}
// ... for a contraction over the leading index with little workspace
Tuning tuning_for(bool compact)
{
    Tuning tn = tuning();
    if (compact && tn.lds_contract == 0)
        tn.lds_contract = 1;
    return tn;
}

// The keys, and what the library itself asks of one plan among others (choose_plan).
struct Wanted : Tuning {
    Wanted() = default;
    Wanted(const Tuning& keys) : Tuning(keys) {}
    bool plain_rows = false;    // row blocks of wide fp64 tiles by the general costs
    int waves = 0;              // wavefronts a SIMD that whole rounds are counted with (0: those that run)
};

struct LeadingPlan {
    int JB = 1, n_jchunk = 1, CB = 1, n_cchunk = 1, n_rsplit = 1, rows_per_split = 16;
    int64_t n_items = 0;
    size_t ws_bytes = 0;        // partial sums of the row splits (0: the kernel writes T itself)
    int plain_rsplit = 1;       // row splits of mttkrp_rowsum_kernel
    ContractPlan cp;            // ok: the kernel through LDS (contract.hip) runs, with its own row splits (copied above)
};

struct Plan {
    int ndim = 0, R = 0, k = 0, sbytes = 0;
    int64_t dims[MTTKRP_MAX_NDIM];
    int64_t strides[MTTKRP_MAX_NDIM];
    int64_t N = 0;
    int RB = 1, JB = 1, n_jchunk = 1;
    int inner = -1;
    int n_out = 0;
    int out_modes[kMaxOuter];
    int64_t I_in = 1;
    int n_rowblk = 1, n_batch = 1, n_isplit = 1, cols_per_isplit = 4;
    int64_t o_total = 1, o_per_item = 1, n_osplit = 1;
    int64_t n_items = 0;
    int64_t n_slots = 1;       // partial sums per output entry
    int64_t n_splits = 1;      // column-space splits
    int64_t steps_per_item = 0;
    size_t part_bytes = 0;     // partial sums (0: the streaming kernel writes M itself)
    size_t fused_bytes = 0;    // product matrices of fused modes, in all
    size_t ws_bytes = 0;       // workspace in all
    int fuse_a = -1;           // index (in the problem the kernels see) of the fused column mode, or -1
    // Fused pairs of adjacent modes: the kernels see mode `red` of I_a * I_b entries in place of
    // the caller's modes a and a + 1; its factor is formed at `offset` bytes into the fused area.
    struct Fusion { int red = 0, a = 0; int64_t Ia = 0, Ib = 0; size_t offset = 0; };
    int n_fuse = 0;
    Fusion fus[2];
    int orig[MTTKRP_MAX_NDIM]; // caller's mode (the first one, for a fused pair) of every mode the kernels see
    // Second schedule (contraction over mode 0, see mttkrp_rowsum_kernel)
    bool contract_rows = false;
    int CB = 1, n_cchunk = 1, n_rsplit = 1, rows_per_split = 16;
    int64_t C = 1, C_lo = 1;
    // ... or, for k != 0 as well, S(q, j) for every combination q of the modes above 0 (contract.hip), then a weighted sum
    ContractPlan cp;
    int cp_segs = 1;           // workgroups per output row of that sum
    bool xcd_remap = true;
    int group = 4;             // first mode: wavefronts per partial tile
    int wave_cap = 0;          // > 0: resident wavefronts per SIMD are capped (by reserving LDS)
    bool nt_off = false;       // never use non-temporal tensor loads
    bool deep = true;          // kernel build with the pipelined run (long items) or with batches only
    bool linear = false;       // column-space splits are balanced ranges of steps (may cut sweeps)
    // k = 0 or 1 with the rows taken as the pairs (i_0, i_1): the kernels see I_0 * I_1 rows and an
    // output mode of one entry; seg = I_0 (0: not taken), out_rows = I_k, seg_nblk = slots per split
    // Last mode as a contraction over all other modes at once (see maybe_lead_route)
    bool lead_route = false;
    LeadingPlan lead;
    int64_t lead_P = 0, lead_Q = 0;
    int64_t seg = 0, out_rows = 0;
    bool seg_first = false;    // the output mode is mode 0 (else mode 1)
    bool seg_store = false;    // ... and the weighted tiles are stored whole (I_0 > 32)
    // The call runs on the small kernel instead (small.hip); everything else here still describes the general
    // decomposition, whose workspace a caller provides in any case.
    bool small = false;
    SmallPlan sp;
    size_t small_bytes = 0;    // its partial sums
    int seg_nblk = 0;
};

int64_t ceil_div(int64_t a, int64_t b) { return (a + b - 1) / b; }

int plan_leading(int64_t P, int64_t Q, int R, int sbytes, const Tuning& tn, LeadingPlan& pl)
{
    if (P < 1 || Q < 1 || R < 1 || (sbytes != 4 && sbytes != 8))
        return MTTKRP_ERR_INVALID_ARG;
    if (P > ((int64_t)1 << 57) / Q)
        return MTTKRP_ERR_INVALID_ARG;
    if (P >= ((int64_t)1 << 31) - 64 || Q >= ((int64_t)1 << 31) - 64 || R >= (1 << 27))
        return MTTKRP_ERR_UNSUPPORTED;
    // tiles as in the second schedule: at most eight accumulator tiles per wavefront
    const int jb_total = (int)ceil_div(R, 16);
    const int jb_max = tn.max_col_blocks >= 1 && tn.max_col_blocks <= 8 ? (int)tn.max_col_blocks
                     : (jb_total > 4 && sbytes == 4 ? 8 : 4);
    pl.n_jchunk = (int)ceil_div(jb_total, jb_max);
    pl.JB = (int)ceil_div(jb_total, pl.n_jchunk);
    const int64_t cb_total = ceil_div(Q, 16);
    int cb_max = pl.JB <= 2 ? 4 : (pl.JB <= 4 ? 2 : 1);
    if (tn.rows_col_blocks >= 1 && tn.rows_col_blocks < cb_max)
        cb_max = (int)tn.rows_col_blocks;
    const int64_t n_cchunk = ceil_div(cb_total, cb_max);
    pl.CB = (int)ceil_div(cb_total, n_cchunk);
    const int64_t base_items = n_cchunk * pl.n_jchunk;
    // rows are split only when the columns alone give too few items to fill the chip once
    const int64_t target = tn.target_items > 0 ? tn.target_items : (base_items >= 2048 ? 1 : 4096);
    const int64_t F = ceil_div(target, base_items);
    int64_t rows = ceil_div(ceil_div(P, F), 16) * 16;
    if (rows < 256)
        rows = 256;
    if (sbytes == 4 && rows > 4096)
        rows = 4096;           // fp32: accumulation chains of at most 4096 terms
    if (tn.max_steps > 0 && rows > 16 * tn.max_steps)
        rows = 16 * tn.max_steps;
    pl.rows_per_split = (int)rows;
    const int64_t n_rsplit = ceil_div(P, rows);
    pl.n_items = base_items * n_rsplit;
    if (pl.n_items >= ((int64_t)1 << 31) - 64 || n_cchunk >= ((int64_t)1 << 31) || n_rsplit >= (1 << 20))
        return MTTKRP_ERR_UNSUPPORTED;
    pl.n_cchunk = (int)n_cchunk;
    pl.n_rsplit = pl.plain_rsplit = (int)n_rsplit;
    // The kernel through LDS wherever it takes the shape (its tiles are not the ones the two keys choose among)
    if (tn.rows_col_blocks == 0 && tn.max_col_blocks == 0 && tn.lds_contract != 2)
        // (fp32: chains of fp32 sums no longer than the other kernel's, whose row splits are added in fp64)
        pl.cp = mttkrp_contract_plan(P, Q, R, sbytes, n_rsplit, tn.target_items, 16 * tn.max_steps, rows);
    // ... unless its wider tiles (64 or 128 columns against 16 to 64) hold over 1.2 times the columns: up to there 3486 fp64 calls
    // are 0.80 times as long in the mean and 1.6 % of them more than 5 % slower, the 500 beyond 1.10 times and up to 1.93
    // (260971 rows x 4 columns at R = 2: 11.4 against 22.0 us).
    if (pl.cp.ok && tn.lds_contract != 1 && (double)pl.cp.n_ctile * pl.cp.CW > 1.2 * (double)(n_cchunk * pl.CB))
        pl.cp = ContractPlan();
    if (pl.cp.ok) {
        pl.n_rsplit = pl.cp.n_rsplit;
        pl.rows_per_split = (int)pl.cp.rows_per_split;
        pl.n_items = pl.cp.n_items * pl.cp.CW;
        pl.ws_bytes = pl.n_rsplit > 1 ? (size_t)Q * (size_t)pl.n_rsplit * (size_t)R * (size_t)sbytes : 0;
        return MTTKRP_OK;
    }
    pl.ws_bytes = n_rsplit > 1 ? (size_t)Q * (size_t)n_rsplit * (size_t)R * (size_t)sbytes : 0;
    return MTTKRP_OK;
}


// Resident wavefronts per SIMD of the streaming kernel's build with the pipelined run
// (what its __launch_bounds__ asks for), for the planner's count of wavefront slots.
template <typename T, int RB> int stream_waves_jb(int JB)
{
    switch (JB) {
    case 1: return Pipe<T, RB, 1>::value ? Pipe<T, RB, 1>::waves : Budget<T, RB, 1>::waves;
    case 2: return Pipe<T, RB, 2>::value ? Pipe<T, RB, 2>::waves : Budget<T, RB, 2>::waves;
    case 3: return Pipe<T, RB, 3>::value ? Pipe<T, RB, 3>::waves : Budget<T, RB, 3>::waves;
    default: return Pipe<T, RB, 4>::value ? Pipe<T, RB, 4>::waves : Budget<T, RB, 4>::waves;
    }
}
template <typename T> int stream_waves_rb(int RB, int JB)
{
    switch (RB) {
    case 1: return stream_waves_jb<T, 1>(JB);
    case 2: return stream_waves_jb<T, 2>(JB);
    case 3: return stream_waves_jb<T, 3>(JB);
    default: return stream_waves_jb<T, 4>(JB);
    }
}
// ... and its steps of loads in flight
template <typename T, int RB> int stream_depth_jb(int JB)
{
    switch (JB) {
    case 1: return Pipe<T, RB, 1>::value ? Pipe<T, RB, 1>::depth : 3;
    case 2: return Pipe<T, RB, 2>::value ? Pipe<T, RB, 2>::depth : 3;
    case 3: return Pipe<T, RB, 3>::value ? Pipe<T, RB, 3>::depth : 3;
    default: return Pipe<T, RB, 4>::value ? Pipe<T, RB, 4>::depth : 3;
    }
}
template <typename T> int stream_depth_rb(int RB, int JB)
{
    switch (RB) {
    case 1: return stream_depth_jb<T, 1>(JB);
    case 2: return stream_depth_jb<T, 2>(JB);
    case 3: return stream_depth_jb<T, 3>(JB);
    default: return stream_depth_jb<T, 4>(JB);
    }
}
int stream_depth(int sbytes, int RB, int JB)
{
    return sbytes == 8 ? stream_depth_rb<double>(RB, JB) : stream_depth_rb<float>(RB, JB);
}
int stream_waves(int sbytes, int RB, int JB)
{
    return sbytes == 8 ? stream_waves_rb<double>(RB, JB) : stream_waves_rb<float>(RB, JB);
}

int validate(int ndim, const int64_t* dims, int R, int k, int sbytes)
{
    if (!dims || ndim < 2 || R < 1 || k < 0 || k >= ndim || (sbytes != 4 && sbytes != 8))
        return MTTKRP_ERR_INVALID_ARG;
    int64_t n = 1;
    for (int m = 0; m < ndim && m < 64; ++m) {
        if (dims[m] < 1)
            return MTTKRP_ERR_INVALID_ARG;
        if (n > (INT64_MAX / 16) / dims[m])   // N * 8 bytes must fit int64 with headroom
            return MTTKRP_ERR_INVALID_ARG;
        n *= dims[m];
    }
    if (ndim > MTTKRP_MAX_NDIM)
        return MTTKRP_ERR_UNSUPPORTED;
    for (int m = 0; m < ndim; ++m)
        if (dims[m] >= (int64_t)1 << 31)
            return MTTKRP_ERR_UNSUPPORTED;
    if ((int64_t)R >= ((int64_t)1 << 27))
        return MTTKRP_ERR_UNSUPPORTED;
    return MTTKRP_OK;
}

// Row blocks per wavefront for a row extent: the RB (<= 4, and no more rows than the tensor has)
// with the lowest cost = rows of all tiles (the last tile is shifted back to end at the last row,
// what it shares with the tile before is computed twice) x a per-row factor that falls with RB (a
// wavefront with RB blocks uses every Khatri-Rao row it forms for 16 RB rows).  The factors are
// fitted to launches on 3.7 to 3.9 GB 4-way tensors (ms at RB = 1 / 2 / 3 / 4, fp64, R = 32, first
// mode): 80 rows 0.91 / 0.94 / 0.80 / 0.98; 100 rows 1.15 / 0.94 / 0.93 / 0.78; 160 rows 0.90 /
// 0.76 / 0.80 / 0.78; 200 rows 1.03 / 0.87 / 0.86 / 0.79; 272 rows 0.89 / 0.79 / 0.72 / 0.77; 400
// rows 0.92 / 0.80 / 0.78 / 0.70; 129 rows (7.7 GB) 2.50 / 2.00 / 1.61 / 2.23.  eff[rb] receives
// the share of the tiles' rows that are rows of the tensor.
const double per_row[5] = {0.0, 1.5, 1.2, 1.06, 1.0};
// With four blocks of output columns in fp64 a wavefront is bound by its MFMAs and two row blocks are nearly as good as
// three: 3 to 5 % a row in the first mode, 5 to 6 % elsewhere (eleven shapes at R = 64 to 1000: 245 rows at R = 208
// 1.81 -> 1.69 ms, 401 rows at R = 1000, first mode, 17.2 -> 16.1).
const double per_row_wide[4] = {0.0, 1.31, 1.12, 1.06};
const double per_row_wide_first[4] = {0.0, 1.31, 1.095, 1.06};
int choose_row_blocks(int64_t rows, int R, int sbytes, double (&eff)[5], int& rb_max, bool plain, bool first = false)
{
    // fp64 accumulators of more than 12 MFMA tiles do not fit the register file next to the operands
    const int jb_all = (int)ceil_div(ceil_div(R, 16), ceil_div(ceil_div(R, 16), 4));
    const int rb_cap = sbytes == 8 && jb_all == 4 ? 3 : 4;
    rb_max = rows >= 16 ? (int)(rows / 16 < rb_cap ? rows / 16 : rb_cap) : 1;
    int best = 1;
    double best_cost = 0.0;
    for (int rb = 0; rb < 5; ++rb)
        eff[rb] = 0.0;
    for (int rb = 1; rb <= rb_max; ++rb) {
        const double tiles = (double)(ceil_div(rows, 16 * rb) * 16 * rb);
        eff[rb] = (double)rows / tiles;
        const double cost = tiles * (rb_cap == 4 || plain ? per_row : (first ? per_row_wide_first : per_row_wide))[rb];
        if (rb == 1 || cost < best_cost - 1e-9) {     // equal cost: the fewer rows
            best = rb;
            best_cost = cost;
        }
    }
    return best;
}

int make_plan_for(int ndim, const int64_t* dims, int R, int k, int sbytes, const Wanted& tn, Plan& pl, bool prefer_rows,
                  bool no_pair_first = false)
{
    const int64_t* const dims_in = dims;
    const int k_in = k, ndim_in = ndim;
    int rc = validate(ndim, dims, R, k, sbytes);
    if (rc != MTTKRP_OK)
        return rc;
    // Fusing two adjacent modes: they are treated as one mode of I_a * I_b entries whose factor
    // is the row-wise product of the two factors, (I_a I_b) x R, formed in the workspace by a
    // small kernel at every call.  X needs no change: adjacent modes of a first-index-fastest
    // tensor are one index already.  Only done while a product matrix stays small (default
    // 8 MiB each), so extra memory remains bounded by a constant.  Two uses:
    //   columns: when the lowest column mode is short (its sweeps would be a few steps) and the
    //            next mode is a column mode too; the fused mode becomes the inner mode;
    //   rows:    modes 0 and 1 (k >= 2), when I_0 is not near a multiple of the 16-row MFMA
    //            blocks a wavefront holds, so that padded rows would waste MFMA work.
    // For k = 1 the same padding is avoided without a product matrix: the rows become the pairs
    // (i_0, i_1), and the epilogue sums each tile's rows per value of i_1 (see StreamArgs::seg).
    int64_t red_dims[MTTKRP_MAX_NDIM];
    pl.fuse_a = -1;
    pl.fused_bytes = 0;
    pl.n_fuse = 0;
    for (int m = 0; m < ndim; ++m) {
        pl.orig[m] = m;
        red_dims[m] = dims[m];
    }
    // Short column space, long mode 0: contract over mode 0 instead (second schedule).
    if (k != 0) {
        int64_t C = 1, C_lo = 1;
        for (int m = 1; m < ndim && C <= 4096; ++m)
            if (m != k) {
                C *= dims[m];
                if (m < k)
                    C_lo *= dims[m];
            }
        const bool can = C <= 1024;
        // When it pays (measured against the streaming kernel's short items, mode 2 of 16384 x I_1 x 64):
        // with at most 16 column entries always (20 to 65 % on 16384 x 2048 x 16, 16384 x 8192 x 7 in
        // fp32, 4096 x 8 x 16384, 2048 x 4 x 4 x 16384); with up to 127 from R = 32 on in fp64 and
        // R = 64 in fp32 (I_1 = 2040: 15 % at R = 32, 42 % at R = 64, 52 % at R = 128, 31 % in fp32 at
        // R = 64; slower at R = 16).  When the columns lie a large power of two apart (I_1 = 2048:
        // 2^28 bytes) all columns of a load share one cache set; the fp64 run reads whole lines and
        // is only about 5 % slower there, but the many same-set lines in flight still cost enough that
        // the schedule wins from R = 64 on only (fp64); the fp32 run reads half lines per step and
        // loses more.
        int64_t col_stride = sbytes;                 // smallest stride between two columns, bytes
        for (int m = 0; m < ndim; ++m) {
            if (m >= 1 && m != k && dims[m] > 1)
                break;
            col_stride *= dims[m];
        }
        // (measured: multiples of 2^24 bytes and more conflict, 255 * 2^20 does not)
        const bool conflicts = col_stride % ((int64_t)1 << 22) == 0;
        const int r_min = conflicts ? (sbytes == 8 ? 48 : (1 << 30)) : (sbytes == 8 ? 16 : 32);
        // (from 128 column entries on the streaming kernel's items are 32 steps and longer and it wins:
        // 5000 x 300 x 200 at R = 32: 0.45 against 0.57 ms)
        // (up to 32 column entries the streaming kernel's items are eight steps or fewer and lose at any
        // rank unless the strides conflict: 10^6 x 20 x 20 at R = 8: 0.78 against 0.61 ms, fp32 at R = 32:
        // 1.66 against 0.91 ms; 10^6 x 30 x 30 fp32 at R = 16: 0.81 against 0.74 ms; at 100 entries and
        // R = 8 the streaming kernel wins, 1.22 against 1.28 ms)
        const bool pays = dims[0] >= 8 * C && dims[0] >= 256 &&
                          (C <= 16 || (C <= 32 && !conflicts) || (C < 128 && R > r_min));
        const bool want = tn.contract_rows == 1 ? can
                        : (tn.contract_rows == 2 ? false : (can && (pays || prefer_rows)));
        if (want) {
            pl.contract_rows = true;
            pl.ndim = ndim; pl.R = R; pl.k = k; pl.sbytes = sbytes;
            int64_t st = 1;
            for (int m = 0; m < ndim; ++m) {
                pl.dims[m] = dims[m];
                pl.strides[m] = st;
                st *= dims[m];
            }
            pl.N = st;
            pl.C = C;
            pl.C_lo = C_lo;
            // At most eight accumulator tiles per wavefront: 2 or 4 column blocks of c times up to 4
            // of j, or one block of c times up to 8 of j, so that 128 output columns take one pass over
            // X (every further chunk of j re-reads it).  The latter keeps only one step of loads in
            // flight and reads more of A_0 per MFMA; measured at R = 128 on 16384 x 2040 x 64 it is
            // faster in fp32 (5.28 against 5.99 ms) and slower in fp64 (9.7 against 9.1 ms).
            const int jb_total = (int)ceil_div(R, 16);
            const int jb_max = tn.max_col_blocks >= 1 && tn.max_col_blocks <= 8 ? (int)tn.max_col_blocks
                             : (jb_total > 4 && sbytes == 4 ? 8 : 4);
            pl.n_jchunk = (int)ceil_div(jb_total, jb_max);
            pl.JB = (int)ceil_div(jb_total, pl.n_jchunk);
            const int cb_total = (int)ceil_div(C, 16);
            int cb_max = pl.JB <= 2 ? 4 : (pl.JB <= 4 ? 2 : 1);
            if (tn.rows_col_blocks >= 1 && tn.rows_col_blocks < cb_max)
                cb_max = (int)tn.rows_col_blocks;
            pl.n_cchunk = (int)ceil_div(cb_total, cb_max);
            pl.CB = (int)ceil_div(cb_total, pl.n_cchunk);
            pl.n_batch = (int)dims[k];
            const int64_t base_items = (int64_t)pl.n_batch * pl.n_cchunk * pl.n_jchunk;
            const int64_t target = tn.target_items > 0 ? tn.target_items : 12288;
            const int64_t F = ceil_div(target, base_items);
            int64_t rows = ceil_div(ceil_div(dims[0], F), 16) * 16;
            if (rows < 256)
                rows = 256;            // at least 16 steps per item
            if (sbytes == 4 && rows > 4096)
                rows = 4096;           // fp32: accumulation chains of at most 4096 terms, as in the streaming kernel
            if (tn.max_steps > 0 && rows > 16 * tn.max_steps)
                rows = 16 * tn.max_steps;
            pl.rows_per_split = (int)(rows < ((int64_t)1 << 30) ? rows : (int64_t)1 << 30);
            pl.n_rsplit = (int)ceil_div(dims[0], pl.rows_per_split);
            pl.n_splits = pl.n_rsplit;
            pl.n_slots = (int64_t)pl.n_rsplit * pl.n_cchunk;
            pl.n_items = base_items * pl.n_rsplit;
            pl.steps_per_item = pl.rows_per_split / 16;
            if (pl.n_items >= ((int64_t)1 << 31) - 64 || pl.n_slots >= ((int64_t)1 << 31))
                return MTTKRP_ERR_UNSUPPORTED;
            pl.part_bytes = pl.n_slots > 1
                ? (size_t)pl.n_slots * (size_t)dims[k] * (size_t)R * (size_t)sbytes : 0;
            pl.fused_bytes = ((size_t)C * (size_t)R * (size_t)sbytes + 255) / 256 * 256;     // W
            pl.ws_bytes = (pl.part_bytes + 255) / 256 * 256 + pl.fused_bytes;
            pl.xcd_remap = false;
            // All column indices at once, whatever mode they belong to: no tile is padded at the end of a batch (20 column
            // entries in tiles of 32: 10^6 x 20 x 20, fp32, R = 32 0.50 -> 0.40 ms), and the kernel through LDS can run.
            // Its intermediate is written and read once: taken while that stays below 2 % of the tensor's bytes, from 8 MB on, and
            // where its tiles hold fewer columns than those of the batches, at most 0.9 (fp32 0.75) times as many: 1300 such calls
            // are 0.67 times as long in the mean and 5 % of them more than 5 % slower, the others 1.08 times and up to 2.06
            // (1634685 x 2 x 7 fp32 at R = 4, second mode: 33 against 69 us).  "lds_contract" = 1 keeps the limits on memory alone.
            const Tuning none;
            Tuning rest = tn;
            rest.small_route = rest.small_groups = rest.lds_contract = 0;
            const int64_t Q = pl.N / dims[0];
            if (tn.lds_contract != 2 && memcmp(&rest, &none, sizeof(rest)) == 0 && dims[0] < ((int64_t)1 << 31) && Q < ((int64_t)1 << 31) - 256) {
                // (fp32: accumulation chains no longer than the other kernel's)
                const ContractPlan cp = mttkrp_contract_plan(dims[0], Q, R, sbytes, 4096, 0, sbytes == 4 ? pl.rows_per_split : 0, 0);
                const double s_bytes = (double)Q * cp.n_rsplit * R * sbytes;
                const int64_t pairs = C * cp.n_rsplit;
                int64_t segs = ceil_div(2048, dims[k] * ceil_div(R, 32));
                if (segs > ceil_div(pairs, 64))
                    segs = ceil_div(pairs, 64);
                if (segs < 1)
                    segs = 1;
                const double bytes = s_bytes + 512.0 + (segs > 1 ? (double)dims[k] * (double)segs * R * sbytes : 0.0);
                // (and never beyond what mttkrp_dense_f64_noalloc has)
                const bool pays_lds = s_bytes <= 0.02 * (double)pl.N * sbytes && pl.N * sbytes >= ((int64_t)1 << 23) &&
                                      (double)cp.n_ctile * cp.CW <= (sbytes == 8 ? 0.9 : 0.75) * (double)dims[k] * pl.n_cchunk * pl.CB;
                if (cp.ok && (pays_lds || tn.lds_contract == 1) && pairs < ((int64_t)1 << 31) &&
                    (bytes <= kNoallocBytes || bytes <= (double)pl.ws_bytes)) {
                    pl.cp = cp;
                    pl.cp_segs = (int)segs;
                    pl.n_rsplit = cp.n_rsplit;
                    pl.n_splits = cp.n_rsplit;
                    pl.n_items = cp.n_items * cp.CW;
                    pl.rows_per_split = (int)(cp.rows_per_split < ((int64_t)1 << 30) ? cp.rows_per_split : (int64_t)1 << 30);
                    pl.steps_per_item = cp.rows_per_split / 16;
                    pl.CB = 1;
                    pl.JB = cp.JB;
                    pl.n_jchunk = 1;
                    pl.n_cchunk = (int)cp.n_ctile;
                    pl.n_slots = pl.cp_segs;
                    pl.part_bytes = pl.cp_segs > 1 ? (size_t)dims[k] * (size_t)pl.cp_segs * (size_t)R * (size_t)sbytes : 0;
                    pl.fused_bytes = ((size_t)s_bytes + 255) / 256 * 256;       // S
                    pl.ws_bytes = (pl.part_bytes + 255) / 256 * 256 + pl.fused_bytes;
                }
            }
            return MTTKRP_OK;
        }
    }
    {
        const int64_t cap = tn.fuse_bytes > 0 ? tn.fuse_bytes : (int64_t)8 << 20;
        auto small_enough = [&](int64_t a, int64_t b) {
            return a > 1 && b > 1 && a * b < ((int64_t)1 << 31) / R && a * b * (int64_t)R * sbytes <= cap;
        };
        // the column pair of a problem (nd, d, kk): index of its first mode, or -1
        auto column_pair = [&](int nd, const int64_t* d, int kk) {
            const int c0 = kk == 1 ? 2 : 1;                 // lowest column mode
            // the lowest column mode and the next one, or, when mode k sits between them, the
            // two modes above k
            const int fa = c0 + 1 < nd && c0 + 1 != kk ? c0 : (c0 + 1 == kk && kk + 2 < nd ? kk + 1 : -1);
            if (fa >= 0 && c0 < nd && d[c0] < 256 && small_enough(d[fa], d[fa + 1]))
                return fa;
            return -1;
        };
        // entries of the inner mode that column_pair / the inner-mode rule below would give
        auto inner_entries = [&](int nd, const int64_t* d, int kk, int fa) {
            if (fa >= 0)
                return d[fa] * d[fa + 1];
            int64_t best = 1;
            for (int m = 1; m < nd; ++m)
                if (m != kk) {
                    if (d[m] >= 32)
                        return d[m];
                    if (d[m] > best)
                        best = d[m];
                }
            return best;
        };
        auto fuse_at = [&](int i) {        // merge modes i and i + 1 of the current problem
            Plan::Fusion& f = pl.fus[pl.n_fuse++];
            f.red = i;
            f.a = pl.orig[i];
            f.Ia = red_dims[i];
            f.Ib = red_dims[i + 1];
            f.offset = pl.fused_bytes;
            pl.fused_bytes += (size_t)(((f.Ia * f.Ib * (int64_t)R * sbytes) + 255) / 256 * 256);
            red_dims[i] = f.Ia * f.Ib;
            for (int m = i + 1; m < ndim - 1; ++m) {
                red_dims[m] = red_dims[m + 1];
                pl.orig[m] = pl.orig[m + 1];
            }
            if (k > i)
                k -= 1;
            ndim -= 1;
        };
        // Rows first: worth it when I_0 alone fills its tiles badly (rows_gain below)
        // and the sweeps that remain stay long (at least 64 steps, or no shorter than without).
        // (the rows' product matrix is only read in the epilogue, one row per accumulator entry:
        // it may be four times as large as one that is read in the streaming loop)
        auto small_rows = [&](int64_t a, int64_t b) {
            return a > 1 && b > 1 && a * b < ((int64_t)1 << 31) / R && a * b * (int64_t)R * sbytes <= 4 * cap;
        };
        // What the choice of row blocks below makes of a row extent: blocks per wavefront, and the
        // share of the tiles' rows that are rows of the tensor.
        auto tile_rows = [&](int64_t rows, int& rb_out) {
            double eff[5];
            int rb_max = 1;
            rb_out = choose_row_blocks(rows, R, sbytes, eff, rb_max, tn.plain_rows);
            if (tn.row_blocks >= 1 && tn.row_blocks <= rb_max)
                rb_out = (int)tn.row_blocks;
            return eff[rb_out];
        };
        // Rows of two modes taken as one pay when I_0 alone leaves more than 1 % of the tiles' rows
        // empty, or allows only one or two row blocks per wavefront where the pair allows more.
        // Measured on 4-way fp64 tensors of 3.7 to 3.9 GB at R = 32 (ms, I_0 alone -> paired or fused):
        // I_0 = 80: 0.89 -> 0.62 (k = 1), 0.86 -> 0.65 (k = 2); 400: 0.66 -> 0.63, 0.68 -> 0.63;
        // 1000: 0.71 -> 0.63, 0.68 -> 0.64; 250 and 500 (k = 2): 0.69 -> 0.65; exact multiples of the
        // tile lose 2 to 5 % (48, 96, 144 rows; 1024: 0.68 -> 0.69).
        auto rows_gain = [&](int64_t alone, int64_t both) {
            int rb_a = 1, rb_b = 1;
            const double e_a = tile_rows(alone, rb_a), e_b = tile_rows(both, rb_b);
            return e_a < 0.99 * e_b || (rb_a <= 2 && rb_b > rb_a);
        };
        // A first mode of more than 32 entries stores its weighted tiles whole (one copy of all rows
        // per split, written once and read once by the combine kernel): that pays only against tiles
        // of fewer than four row blocks or with more than 15 % of their rows empty (129 rows at
        // R = 32: 1.62 -> 1.52 ms; 401 rows, 64-row tiles 89 % full, in one round of long items:
        // 0.759 -> 0.748 ms at R = 32, 0.694 -> 0.718 ms at R = 10).
        auto poor_tiles = [&](int64_t rows) {
            int rb = 1;
            const double e = tile_rows(rows, rb);
            return rb < 4 || e < 0.85;
        };
        // k = 1, or k = 0 with a short first mode (the epilogue then walks over all I_0 output rows):
        // the pairs (i_0, i_1) are the rows and the output mode has one entry for the kernel
        // (row arithmetic in the kernel is 32-bit: first row of a tile + 64 must not overflow)
        if (k <= 1 && ndim >= 3 && dims[1] > 1 && dims[0] * dims[1] < ((int64_t)1 << 31) - 128 &&
            (k == 1 || !no_pair_first) && tn.pair_rows != 2 &&
            (tn.pair_rows == 1 || (rows_gain(dims[0], dims[0] * dims[1]) && (k == 1 || dims[0] <= 32 || poor_tiles(dims[0]))))) {
            pl.seg = dims[0];
            pl.seg_first = k == 0;
            pl.seg_store = k == 0 && dims[0] > 32;
            pl.out_rows = dims[k];
            red_dims[0] = dims[0] * dims[1];
            red_dims[1] = 1;
            k = 1;
        }
        // Shorter sweeps are still worth it when I_0 alone wastes most of its tiles: cost per entry =
        // the row tiles' cost (choose_row_blocks) x (steps + 20) / steps for the sweeps (3 x 1000 x
        // 1000 x 100, third mode: sweeps of 25 steps on full tiles against 250 steps on tiles with 3
        // rows of 16, 1.8 ms).
        auto much_cheaper = [&](int64_t rows_both, int64_t with_entries, int64_t without_entries) {
            int rb_a = 1, rb_b = 1;
            const double e_a = tile_rows(dims[0], rb_a), e_b = tile_rows(rows_both, rb_b);
            const double st_w = (double)ceil_div(with_entries, 4), st_wo = (double)ceil_div(without_entries, 4);
            const double c_with = per_row[rb_b] / e_b * (st_w + 20.0) / st_w;
            const double c_without = per_row[rb_a] / e_a * (st_wo + 20.0) / st_wo;
            return with_entries >= 32 && c_with < 0.7 * c_without;
        };
        if (k >= 2 && small_rows(dims[0], dims[1])) {
            int64_t rd[MTTKRP_MAX_NDIM];
            rd[0] = dims[0] * dims[1];
            for (int m = 1; m < ndim - 1; ++m)
                rd[m] = dims[m + 1];
            const int64_t with = inner_entries(ndim - 1, rd, k - 1, column_pair(ndim - 1, rd, k - 1));
            const int64_t without = inner_entries(ndim, dims, k, column_pair(ndim, dims, k));
            if (tn.fuse_rows != 2 &&
                (tn.fuse_rows == 1 || (rows_gain(dims[0], rd[0]) && (with >= 256 || with >= without || much_cheaper(rd[0], with, without)))))
                fuse_at(0);
        }
        const int fa = column_pair(ndim, red_dims, k);
        if (fa >= 0) {
            fuse_at(fa);
            pl.fuse_a = fa;
        }
        dims = red_dims;
    }
    pl.ndim = ndim; pl.R = R; pl.k = k; pl.sbytes = sbytes;
    int64_t s = 1;
    for (int m = 0; m < ndim; ++m) {
        pl.dims[m] = dims[m];
        pl.strides[m] = s;
        s *= dims[m];
    }
    pl.N = s;
    const int64_t I0 = dims[0];

    // Row blocks per wavefront (see choose_row_blocks).
    {
        double eff[5];
        int rb_max = 1;
        int best = choose_row_blocks(I0, R, sbytes, eff, rb_max, tn.plain_rows, k == 0);
        double best_eff = 0.0;
        for (int rb = 1; rb <= rb_max; ++rb)
            if (eff[rb] > best_eff)
                best_eff = eff[rb];
        // Items shorter than 32 steps (k != 0, fewer than 128 column entries) run the build without
        // the pipelined run; there three fp64 row blocks measured 1 to 8 % faster than four (more
        // registers left for steps in flight), while fp32 lost 10 %.
        if (sbytes == 8 && k != 0 && best == 4 && eff[3] >= 0.9 * best_eff) {
            int64_t col_entries = 1;
            for (int m = 1; m < ndim && col_entries < 128; ++m)
                if (m != k)
                    col_entries *= dims[m];
            if (col_entries < 128)
                best = 3;
        }
        if (tn.row_blocks >= 1 && tn.row_blocks <= rb_max)
            best = (int)tn.row_blocks;
        pl.RB = best;
    }
    pl.n_rowblk = (int)ceil_div(I0, 16 * pl.RB);

    // Column blocks of the output: at most four 16-column blocks per wavefront.
    {
        const int jb_total = (int)ceil_div(R, 16);
        const int cb_max = tn.max_col_blocks >= 1 && tn.max_col_blocks <= 4 ? (int)tn.max_col_blocks : 4;
        pl.n_jchunk = (int)ceil_div(jb_total, cb_max);
        pl.JB = (int)ceil_div(jb_total, pl.n_jchunk);
    }

    // Column modes: all but mode 0 and mode k.  Inner = lowest one with at
    // least 32 entries (eight steps per sweep), else the largest; the others are outer modes.
    int cols[MTTKRP_MAX_NDIM];
    int n_cols = 0;
    for (int m = 1; m < ndim; ++m)
        if (m != k)
            cols[n_cols++] = m;
    pl.inner = -1;
    if (pl.fuse_a >= 0)
        pl.inner = pl.fuse_a;       // two modes were fused to make the sweeps long: sweep over them
    for (int c = 0; c < n_cols && pl.inner < 0; ++c)
        if (dims[cols[c]] >= 32) { pl.inner = cols[c]; break; }
    if (pl.inner < 0)
        for (int c = 0; c < n_cols; ++c)
            if (pl.inner < 0 || dims[cols[c]] > dims[pl.inner])
                pl.inner = cols[c];
    pl.n_out = 0;
    pl.o_total = 1;
    for (int c = 0; c < n_cols; ++c)
        if (cols[c] != pl.inner) {
            pl.out_modes[pl.n_out++] = cols[c];
            pl.o_total *= dims[cols[c]];
        }
    pl.I_in = pl.inner >= 0 ? dims[pl.inner] : 1;
    pl.n_batch = k == 0 ? 1 : (int)dims[k];

    // Split the (outer x inner) column space so that about target_items
    // wavefront items exist, each with enough steps to amortise its epilogue.
    const int64_t steps_in = ceil_div(pl.I_in, 4);
    const int64_t steps_all = pl.o_total * steps_in;
    const int64_t base_items = (int64_t)pl.n_rowblk * pl.n_jchunk * pl.n_batch;
    const int64_t target = tn.target_items > 0 ? tn.target_items : 12288;   // four per resident wavefront slot at three per SIMD
    const int64_t min_steps = 16;
    int64_t max_steps = tn.max_steps > 0 ? tn.max_steps
                        : (sbytes == 4 ? 1024 : ((int64_t)1 << 40));   // fp32: short accumulation chains
    bool whole_rounds = false;      // F was chosen to fill whole rounds of the chip (first mode)
    const bool matrix_bound = pl.JB >= (sbytes == 8 ? 2 : 3);       // by the matrix cores rather than by HBM
    int64_t F = ceil_div(target, base_items);
    if (F > steps_all / min_steps)
        F = steps_all / min_steps;
    if (F < 1)
        F = 1;
    if (k == 0) {
        const int64_t waves = tn.waves > 0 ? tn.waves : stream_waves(sbytes, pl.RB, pl.JB);
        // One partial tile per workgroup (four splits) is written once and read once: keep
        // that traffic below ws_percent of the bytes of X, or 32 MiB if that is more.
        const double pct = tn.ws_percent > 0 ? (double)tn.ws_percent : 2.0;
        double budget = pct * 0.01 * (double)pl.N * sbytes;
        if (budget < 32.0 * 1048576.0)
            budget = 32.0 * 1048576.0;
        // The hand-scheduled fp64 instantiation gains more from fewer, longer items than from
        // the shared partial tile; every other one is faster with the LDS sum.
        const bool long_items = sbytes == 8 && pl.RB == 4 && pl.JB == 2;
        // Columns that do not start on 128-byte lines: neighbouring row blocks share the lines at
        // their boundaries (and the rows of the shifted last block), so they should run as the
        // wavefronts of one workgroup, where the second reader mostly hits in cache.  Measured
        // (fetched bytes 1.4 to 1.55 times X with the shared partial tile): 401 rows at R = 10
        // 0.74 -> 0.68 ms, 129 rows at R = 10 1.64 -> 1.44 ms.
        // (With several chunks of output columns the wavefronts of a workgroup are the chunks of one
        // piece of X, which matters more: 401 rows at R = 1000 16.7 against 19.3 ms.)
        const bool unaligned = (I0 * sbytes) % 128 != 0 && pl.n_rowblk > 1 && pl.n_jchunk == 1;
        pl.group = tn.first_group == 1 ? 1 : tn.first_group == 4 ? kWaves : (long_items || unaligned ? 1 : kWaves);
        // ... unless the traffic cap then leaves the chip under-filled: a partial tile per workgroup
        // allows four times the splits (100^4 at R = 32: 1310 items 0.229 ms, 5240 items 0.191 ms;
        // 1000 x 3 x 1000 x 100: 0.51 -> 0.45 ms; with the chip filled either way it loses 5 to 10 %)
        if (tn.first_group == 0 && pl.group == 1) {
            const double cap1 = budget / (2.0 * (double)I0 * (double)R * sbytes);
            const double resident = 1024.0 * (double)waves;
            if (cap1 < (double)F && (double)base_items * (cap1 < 1.0 ? 1.0 : cap1) < 0.9 * resident)
                pl.group = kWaves;
        }
        const double cap = pl.group * budget / (2.0 * (double)I0 * (double)R * sbytes);
        if ((double)F > cap)
            F = cap < 1.0 ? 1 : (int64_t)cap;
        // Ungrouped items are long and few: keep them to one round of the chip (256 compute
        // units x 4 SIMDs x 2 resident wavefronts), so that no second, partly filled round follows.
        if (pl.group == 1 && long_items) {
            const int64_t resident = 256 * 4 * 2;
            if (base_items <= resident && F > resident / base_items)
                F = resident / base_items;
        }
        // Few rounds of the chip: a partly filled last round costs a large share, so take whole
        // rounds (the nearest number; linear splits below make any count of equal items possible).
        // 48^5 fp32 at R = 64: 4608 items on 3072 slots -> 6144, 0.304 -> 0.284 ms.  Not where the
        // columns are not line-aligned: those launches are bound by the lines fetched twice, not by
        // the matrix cores, and ran 3 to 9 % slower with fewer, longer items.
        if (!unaligned) {
            const int64_t resident = 1024 * waves;
            const int64_t items = base_items * F;
            if (tn.linear != 2 && tn.target_items == 0 && items < 4 * resident && base_items <= resident) {
                const int64_t nearest = items < resident / 2 ? 1 : (items + resident / 2) / resident;
                // (one round fewer where the cap on memory forbids the nearest number, if the matrix cores bound the launch: 77 of
                // 82 such calls 0.85 times as long in the mean, 129^3 x 12 at R = 500 0.60 -> 0.46 ms; at lower ranks fewer, longer
                // items lose up to 1.5 times)
                for (int64_t rounds = nearest; rounds >= 1 && rounds >= nearest - (matrix_bound && sbytes == 8 ? 1 : 0) && !whole_rounds; --rounds) {
                    int64_t Fr = rounds * resident / base_items;
                    Fr -= Fr % pl.group;
                    if (Fr >= pl.group && (double)Fr <= 1.25 * cap && steps_all / Fr >= 32 && steps_all / Fr <= max_steps) {
                        F = Fr;
                        whole_rounds = true;
                    }
                }
            }
        }
    }
    if (pl.seg > 0) {
        // Paired rows: the kernel sees one batch value, so the splits carry all the parallelism, and
        // every split writes a slot (or a few) per output row.  Keep those partial sums, written once
        // and read once, below 4 % of the bytes of X (12^7 at R = 32: 37 MB of them for a 287 MB
        // tensor cost 20 % of the launch).
        const int64_t per_row = pl.seg_store ? dims[0] / pl.seg
                              : (pl.seg_first ? pl.n_rowblk : (pl.seg + 16 * pl.RB - 2) / (16 * pl.RB) + 1);
        const double per_split = (double)pl.out_rows * (double)per_row * (double)R * sbytes;
        double budget = (pl.seg_store ? 0.025 : 0.04) * (double)pl.N * sbytes;
        if (budget < 4.0 * 1048576.0)
            budget = 4.0 * 1048576.0;
        if ((double)F * per_split > budget)
            F = budget / per_split < 1.0 ? 1 : (int64_t)(budget / per_split);
    }
    if (F < ceil_div(steps_all, max_steps))
        F = ceil_div(steps_all, max_steps);
    if (F < ceil_div(pl.o_total, (int64_t)1 << 29))
        F = ceil_div(pl.o_total, (int64_t)1 << 29);
    // F = outer splits x inner splits.  Among the inner splits (each at least eight
    // steps long) take the pair whose largest item is closest to the average item, with the
    // fixed cost of a sweep counted in and a mild preference for reaching the wanted count.
    auto cut = [&](int64_t F) {
        double best_eff = -1.0;
        // (candidates: 1 .. 64, then steps of an eighth up to 16384: one long column mode next to few
        // row tiles needs thousands of pieces, 400 x 10^6 at R = 32: 448 items 0.95 ms)
        for (int64_t ni = 1, next = 2; ni <= 16384; ni = next) {
            next = ni + (ni < 64 ? 1 : ni / 8);
            if (ni > 1 && steps_in / ni < 8)
                break;
            const bool more = next <= 16384 && steps_in / next >= 8;     // a larger ni is possible
            if (tn.inner_splits > 0 && ni != tn.inner_splits && more)
                continue;
            int64_t no = F / ni;
            if (no < 1)
                no = 1;
            if (no > pl.o_total)
                no = pl.o_total;
            if (4 * ni * pl.o_total < 3 * F && more)
                continue;     // even every sweep on its own is too few: split the inner mode further
            const int64_t opi = ceil_div(pl.o_total, no);
            no = ceil_div(pl.o_total, opi);
            const int64_t in_steps = ceil_div(steps_in, ni);
            const int64_t n_in = ceil_div(pl.I_in, 4 * in_steps);
            const double avg = (double)steps_all / (double)(no * n_in);
            double eff = avg / (double)(opi * in_steps);
            const double ratio = (double)(no * n_in) / (double)F;    // stay near the wanted count
            if (ratio < 1.0)
                eff *= 0.85 + 0.15 * ratio;
            if (ratio < 0.75)
                eff *= ratio / 0.75;
            // every sweep drains and refills the pipeline: about twenty steps' worth (measured)
            eff *= (double)in_steps / (double)(in_steps + 20);
            if (eff > best_eff + 1e-9) {
                best_eff = eff;
                pl.n_osplit = no;
                pl.o_per_item = opi;
                pl.cols_per_isplit = (int)(4 * in_steps);
                pl.n_isplit = (int)n_in;
            }
        }
    };
    cut(F);
    // Every SIMD takes a whole number of items, and where the matrix cores bound the launch it takes equally long for
    // each: 8328 items run as long as 9216.  So a number of splits near F that leaves the least of the last item idle, an
    // item's start and end counted as twelve steps (65 x 66 x 36 x 24 at R = 36, last mode 28.1 -> 19.8 us; 159
    // calls that it changes 0.92 times as long in the mean, five more than 5 % slower).  Partial sums stay within what F
    // asked for, or within 5 % of X and 64 MiB, and fp32 chains no longer than with F.
    if (k != 0 && pl.seg == 0 && matrix_bound && tn.target_items == 0 && tn.linear == 0 && tn.inner_splits == 0) {
        auto simd_steps = [&]() {
            const double per_simd = (double)(base_items * pl.n_osplit * pl.n_isplit) / 1024.0;
            return per_simd < 16.0 ? ceil(per_simd) * (double)(pl.o_per_item * (pl.cols_per_isplit / 4) + 12) : -1.0;
        };
        const int64_t longest = sbytes == 4 ? pl.o_per_item * (pl.cols_per_isplit / 4) : max_steps;
        const double now = simd_steps(), row = (double)pl.n_rowblk * (double)dims[k] * (double)R * sbytes;
        double budget = 0.05 * (double)pl.N * sbytes < kNoallocBytes ? 0.05 * (double)pl.N * sbytes : kNoallocBytes;
        if (row * (double)(pl.n_osplit * pl.n_isplit) > budget)
            budget = row * (double)(pl.n_osplit * pl.n_isplit);
        double best = 0.97 * now;
        int64_t best_F = F;
        if (now > 0.0)
            for (int64_t f = F - F / 3 > 1 ? F - F / 3 : 1; f <= F + F / 3; f += 1 + F / 24) {
                cut(f);
                const int64_t steps = pl.o_per_item * (pl.cols_per_isplit / 4);
                const double t = simd_steps();
                if (t > 0.0 && t < best && steps >= 32 && steps <= longest && row * (double)(pl.n_osplit * pl.n_isplit) <= budget) {
                    best = t;
                    best_F = f;
                }
            }
        cut(best_F);
    }
    pl.steps_per_item = pl.o_per_item * (pl.cols_per_isplit / 4);
    // Linear splits: F balanced ranges of the whole step sequence, cutting sweeps where they fall.
    // Taken for the long first-mode items that fill the chip in one round, when whole sweeps and
    // inner splits leave them uneven or fewer than wanted (401 x 201 x 12 x 501 at R = 32: 251
    // splits of 1206 steps on 7 row blocks fill 1757 of the 2048 wavefront slots, 292 ranges of
    // 1035 steps fill 2044: 0.80 -> 0.75 ms).  With several rounds of shorter items the cut sweeps
    // cost more than the balance gains (129 rows, R = 32: 1.62 -> 1.89 ms).
    {
        const int64_t n_now = pl.n_osplit * pl.n_isplit;
        const double even = (double)steps_all / (double)n_now / (double)pl.steps_per_item;
        const bool one_round = k == 0 && pl.group == 1 && sbytes == 8 && pl.RB == 4 && pl.JB == 2 &&
                               base_items * F <= 256 * 4 * 2;
        const bool helps = (one_round || whole_rounds) && (n_now != F || even < 0.97);
        if ((tn.linear == 1 || (tn.linear == 0 && helps)) && F >= 1 && steps_all / F >= 1) {
            pl.linear = true;
            pl.n_osplit = F;
            pl.n_isplit = 1;
            pl.o_per_item = 1;
            pl.cols_per_isplit = (int)(4 * steps_in);
            pl.steps_per_item = ceil_div(steps_all, F);
        }
    }
    if (pl.steps_per_item >= ((int64_t)1 << 30))
        return MTTKRP_ERR_UNSUPPORTED;
    pl.n_splits = pl.n_osplit * pl.n_isplit;
    if (pl.n_splits >= ((int64_t)1 << 30))
        return MTTKRP_ERR_UNSUPPORTED;
    if (k == 0) {
        // One range of the column space: there is nothing to share, and three of four wavefronts of a group would be idle
        // (10^6 x 20 x 20 fp32 at R = 32 374 -> 342 us).
        if (pl.n_splits == 1 && tn.first_group == 0)
            pl.group = 1;
        pl.n_slots = ceil_div(pl.n_splits, pl.group);    // one partial tile per group of wavefronts
        pl.n_items = base_items * pl.n_slots * pl.group;
    } else if (pl.seg_store) {
        pl.n_slots = pl.n_splits * (dims[0] / pl.seg);      // (split, i_1)
        pl.n_items = base_items * pl.n_splits;
    } else if (pl.seg > 0 && !pl.seg_first) {
        // row tiles that can overlap the I_0 rows of one value of i_1, wherever those begin
        pl.seg_nblk = (int)((pl.seg + 16 * pl.RB - 2) / (16 * pl.RB) + 1);
        pl.n_slots = pl.n_splits * pl.seg_nblk;
        pl.n_items = base_items * pl.n_splits;
    } else {
        pl.n_slots = pl.n_splits * pl.n_rowblk;
        pl.n_items = base_items * pl.n_splits;
    }
    if (pl.n_items >= ((int64_t)1 << 31) - 64 || pl.n_slots >= ((int64_t)1 << 31))
        return MTTKRP_ERR_UNSUPPORTED;
    pl.part_bytes = pl.n_slots > 1
        ? (size_t)pl.n_slots * (size_t)(pl.seg > 0 ? pl.out_rows : dims[k]) * (size_t)R * (size_t)sbytes : 0;
    if (pl.seg > 0 && pl.part_bytes == 0)       // the paired epilogue always writes slots
        pl.part_bytes = (size_t)pl.out_rows * (size_t)R * (size_t)sbytes;
    if (pl.seg_first) {
        // every row tile writes a slot for every output row: fine while that stays small beside X
        double limit = 0.05 * (double)pl.N * sbytes;
        if (limit < 64.0 * 1048576.0)
            limit = 64.0 * 1048576.0;
        if ((double)pl.part_bytes > limit) {
            pl = Plan();
            return make_plan_for(ndim_in, dims_in, R, k_in, sbytes, tn, pl, prefer_rows, true);
        }
    }
    pl.ws_bytes = (pl.part_bytes + 255) / 256 * 256 + pl.fused_bytes;
    // First mode with several chunks of output columns: neighbouring workgroups read the same piece
    // of X; contiguous workgroup ranges per XCD put them behind one L2 (measured 3 % at R = 128).
    pl.xcd_remap = tn.xcd_remap == 1 || (tn.xcd_remap == 0 && k == 0 && pl.n_jchunk > 1);
    pl.wave_cap = (int)tn.waves_per_simd;
    // Several chunks of output columns read the same piece of X, which a non-temporal load lets the L2 drop before the next
    // one has come: fp64 with line-aligned columns, ten calls in a row of 16384 x 2048 x 64 at R = 128, first and last mode 8.63 ->
    // 8.06 and 8.14 -> 7.77 ms (on a card that clocks lower 8.84 -> 8.28 and 8.36 -> 7.99), 1024 x 1024 x 512 at R = 96, first mode
    // 1.64 -> 1.54; 18 calls at R = 96 to 500 0.963 times as long in the mean, none slower.
    pl.nt_off = tn.nt_loads == 1 || pl.n_jchunk > 1;
    // Short items: their prologue and epilogue dominate, more resident wavefronts win.  Where the run's offsets do not fit, its
    // build would be left with two-step batches at few wavefronts (tensors from 35 GB on, 100000 x 16 x 120 x 32 at R = 32, third
    // mode 10.3 ms, with the batches' own build 8.9; at R = 64 19.0 and 15.8; fp32 200000 x 16 x 140 x 30 at R = 64 19.2 and 18.3).
    pl.deep = tn.deep == 1 ? true : tn.deep == 2 ? false
              : pl.steps_per_item >= 32 &&
                    (pl.inner < 0 || run_of_lane_pointers(sbytes, pl.RB, pl.JB) || lane_offsets_fit(pl.strides[pl.inner], sbytes));
    return MTTKRP_OK;
}

// The streaming kernel's partial sums for k != 0 are one row of M per (row block, split) and
// batch value: with a short column space and a high rank that can approach the size of X.
// Then the second schedule, whose partial sums are a few rows per output row, takes over.
// The last mode with few entries in all other modes together (P of them): M = X^T K for X as a
// P x I_k matrix and K the Khatri-Rao product of the other factors (P x R, formed in the
// workspace), i.e. the contraction over the leading index.  Taken when K stays cache-resident
// (4 MiB) and mode 0 alone fills the streaming kernel's row tiles badly: then neither kernel has a
// plan with long work items (20 x 20 x 10^6 at R = 32: 2.1 ms on the second schedule, 0.68 ms here).
void maybe_lead_route(int ndim, const int64_t* dims, int R, int k, int sbytes, const Wanted& tn, Plan& pl)
{
    if (k != ndim - 1 || ndim < 2 || tn.lead_last == 2 || (tn.contract_rows == 1 && tn.lead_last != 1))
        return;
    int64_t P = 1;
    for (int m = 0; m < ndim - 1; ++m)
        P *= dims[m];
    const int64_t Q = dims[k];
    if (P < 2 || (double)P * R * sbytes > 4.0 * 1048576.0)
        return;
    if (tn.lead_last != 1) {
        double eff[5];
        int rb_max = 1;
        const int rb = choose_row_blocks(dims[0], R, sbytes, eff, rb_max, tn.plain_rows);
        if (eff[rb] >= 0.9 && rb > 2)
            return;
    }
    LeadingPlan lp;
    if (plan_leading(P, Q, R, sbytes, tn, lp) != MTTKRP_OK)
        return;
    // few output rows leave few work items, or need row splits with partial sums: not then
    // (16 x 16 x 16 x 50000 at R = 8 with six row splits: 0.34 ms against 0.30 ms on the streaming kernel)
    if (tn.lead_last != 1 && (Q < 256 || lp.plain_rsplit > 1))
        return;
    const size_t kbytes = ((size_t)P * (size_t)R * (size_t)sbytes + 255) / 256 * 256;
    Plan out;
    out.ndim = ndim; out.R = R; out.k = k; out.sbytes = sbytes;
    int64_t st = 1;
    for (int m = 0; m < ndim; ++m) {
        out.dims[m] = dims[m];
        out.strides[m] = st;
        st *= dims[m];
        out.orig[m] = m;
    }
    out.N = st;
    out.lead_route = true;
    out.lead = lp;
    out.lead_P = P;
    out.lead_Q = Q;
    out.n_items = lp.n_items;
    out.n_slots = lp.n_rsplit;
    out.steps_per_item = lp.rows_per_split / 16;
    out.part_bytes = lp.ws_bytes;
    out.fused_bytes = ndim == 2 ? 0 : kbytes;   // K
    out.ws_bytes = (out.part_bytes + 255) / 256 * 256 + out.fused_bytes;
    pl = out;
}

// Rough relative cost of a streaming plan, for choosing between two of them: the row tiles' cost
// per row of the tensor, what a partly filled last round of the chip wastes (half of it: the
// stragglers run faster), and the partial sums that are written and read again.
double plan_cost(const Plan& pl)
{
    const double eff = (double)pl.dims[0] / ((double)pl.n_rowblk * 16.0 * pl.RB);
    const double resident = 256.0 * 4.0 * stream_waves(pl.sbytes, pl.RB, pl.JB);
    const double rounds = (double)pl.n_items / resident;
    const double fill = rounds >= 4.0 ? 1.0 : ceil(rounds) / rounds;
    return per_row[pl.RB] / eff * (1.0 + 0.5 * (fill - 1.0)) *
           (1.0 + 2.0 * (double)pl.part_bytes / ((double)pl.N * pl.sbytes));
}

int make_general_plan(int ndim, const int64_t* dims, int R, int k, int sbytes, const Wanted& tn, Plan& pl)
{
    int rc = make_plan_for(ndim, dims, R, k, sbytes, tn, pl, false);
    if (rc == MTTKRP_OK && pl.seg_store) {
        // whole stored tiles cost traffic, and their cap can leave few items: compare with the plain plan
        // (129 x 257 x 12 x 500: 2076 items on 2048 slots, 0.39 against 0.35 ms; 40^5: 0.14 against 0.25 ms)
        Plan plain;
        if (tn.pair_rows != 1 && make_plan_for(ndim, dims, R, k, sbytes, tn, plain, false, true) == MTTKRP_OK &&
            !plain.contract_rows && plan_cost(plain) < plan_cost(pl))
            pl = plain;
    }
    if (rc == MTTKRP_OK)
        maybe_lead_route(ndim, dims, R, k, sbytes, tn, pl);
    if (rc != MTTKRP_OK || pl.contract_rows || pl.lead_route || k == 0)
        return rc;
    double limit = 0.05 * (double)pl.N * sbytes;
    if (limit < 64.0 * 1048576.0)
        limit = 64.0 * 1048576.0;
    if ((double)pl.part_bytes <= limit)
        return rc;
    Plan alt;
    if (make_plan_for(ndim, dims, R, k, sbytes, tn, alt, true) == MTTKRP_OK && alt.contract_rows && alt.ws_bytes < pl.ws_bytes)
        pl = alt;
    return MTTKRP_OK;
}

// One launch or few workgroups with a combine launch (small.hip) against the plan above: the two times on the GPU in us.  Up to
// kSmallFitValues the small kernel's is fitted to 17400 timings of graph replays (3800 calls, fp64 and fp32, three to seven modes, 2^15 to
// 2^23 values, R = 4 to 1000, each with up to six numbers of groups); on a half that was not fitted the median error is 7 %.  The general
// plan's is an older fit, 8 % off in the median.  2334 further calls of 2^8 to 2^19.8 values (two to eight modes): 734 run otherwise than by
// the older fit, 0.63 times as long in the mean, 2.6 % of them more than 5 % slower, the worst 1.33 times; their errors against extended
// precision are 0.78 (fp64) and 0.56 times (fp32) the former.  Beyond, an older fit of the small kernel stays (5650 calls; it gives times 1.15 to
// 1.47 times too long, from before its batches became as long as their remainders): the plans of many calls from 2^19.9 values on are pinned, the
// chosen streaming plans among them.  The new fit would take more calls there too (2^20 to 2^21 values: 0.80 against 0.90 times the general
// plan's time; to 2^22 0.89 against 0.97).
// By the number of column modes (up to one, two, three, four, more; the older fit one, two, others), per workgroup:
constexpr int64_t kSmallFitValues = (int64_t)7 << 17;
struct SmallFit {
    double base, mfma, loads, alu, sweep;      // launch; matrix cores, load instructions, address arithmetic; a sweep's start and end
    double crowd, rounds;                      // the share of each workgroup beyond one a compute unit; beyond what is resident
    double combine, part;                      // the second launch and its MB
    double cold, bytes, spill;                 // batches of loads from beyond L2; MB of X; four blocks of columns in fp64
};
const SmallFit small_fit[5] = {{2.69, 1.06, 0.00, 0.62, 0.83, 1.44, 0.78, 2.10, 2.24, 0.14, 0.056, 0.55},
                               {2.81, 1.24, 1.85, 0.53, 0.58, 1.38, 0.80, 2.22, 1.25, 0.00, 0.059, 0.72},
                               {3.36, 1.23, 7.59, 0.06, 0.16, 1.26, 0.93, 2.18, 1.05, 0.00, 0.062, 0.24},
                               {3.45, 1.44, 5.60, 0.27, 0.00, 1.13, 1.27, 2.44, 1.04, 0.00, 0.133, 0.77},
                               {4.13, 1.74, 5.69, 0.54, 0.00, 1.19, 0.90, 2.37, 0.73, 0.32, 0.054, 0.00}};
const SmallFit small_fit_large[3] = {{2.00, 1.67, 1.93, 0.00, 1.65, 1.92, 0.73, 2.46, 0.70, 0.03, 0.059, 1.09},
                                     {2.00, 1.27, 0.00, 0.75, 1.84, 1.72, 1.13, 2.59, 1.06, 0.00, 0.107, 5.72},
                                     {2.73, 0.71, 4.60, 1.35, 2.87, 1.72, 1.11, 3.12, 0.57, 1.25, 0.149, 3.55}};
double small_cost(const SmallPlan& sp, int sbytes, int n_modes, int64_t N, double part_bytes, bool first)
{
    const SmallFit& f = N <= kSmallFitValues ? small_fit[n_modes < 1 ? 0 : (n_modes < 5 ? n_modes - 1 : 4)]
                                             : small_fit_large[n_modes == 1 ? 0 : (n_modes == 2 ? 1 : 2)];
    const int batch = sp.RB * sp.JB <= 2 ? 8 : 4;
    const double units = (double)sp.n_tiles * sp.n_ranges, per = (double)(sp.cols_per_range / 4), steps = units * per / 2200.0;
    const double sweeps = ceil(units / sp.waves), mb = 1e-6 * (double)N * sbytes;
    const double busy = f.mfma * steps * sp.RB * sp.JB * (sbytes == 8 ? 16.0 : 8.0) +
                        f.loads * steps * (sp.RB + n_modes * (double)ceil_div(sp.JB, 16 / sbytes)) +
                        f.alu * steps * (n_modes * (6 + sp.JB * (sbytes / 4)) + 8 + 4 * sp.RB);
    const double groups = (double)sp.blocks * sp.n_jchunk * sp.n_groups / 256.0, rounds = groups / (16 / sp.waves);
    double t = f.base + busy + f.sweep * sweeps + f.crowd * (groups > 1.0 ? groups - 1.0 : 0.0) * busy +
               f.rounds * (rounds > 1.0 ? rounds - 1.0 : 0.0) * (f.base - 2.0 + f.sweep * sweeps) +
               f.cold * sweeps * ceil(per / batch) * (mb < 16.0 ? mb / 16.0 : 1.0) + f.bytes * mb;
    if (sp.n_groups > 1)
        t += f.combine + f.part * 1e-6 * part_bytes;
    if (sbytes == 8 && sp.JB == 4 && !first)
        t += f.spill * sweeps;
    return t;
}

double general_cost(const Plan& pl, int ndim)
{
    const bool paired_second = pl.seg > 0 && !pl.seg_first;
    const bool prepare = pl.fused_bytes > 0 || paired_second || pl.contract_rows;
    const bool combine = pl.n_slots > 1 || pl.seg > 0;
    const int tiles = (pl.contract_rows || pl.lead_route ? 1 : pl.RB) * (pl.lead_route ? pl.lead.JB : pl.JB);
    const double items = (double)pl.n_items, steps = (double)pl.steps_per_item;
    return 3.38 + (prepare ? 2.52 : 0.0) + (combine ? 2.45 : 0.0) + (pl.seg > 0 ? 2.71 : 0.0) + (pl.lead_route ? 0.78 : 0.0) +
           (ndim > 3 ? 0.92 : 0.0) + 0.045 * steps * (items > 3072.0 ? items / 3072.0 : 1.0) +
           1.31 * (items > 1024.0 ? items / 1024.0 : 1.0) * tiles * (pl.sbytes == 8 ? 64.0 : 32.0) * steps / 2200.0 +
           0.0406e-6 * (double)pl.N * pl.sbytes + 1.15e-3 * items + 0.837e-6 * (double)pl.ws_bytes + 0.197 * tiles;
}

// Above kSmallFitValues a fit of 2600 other calls timed with their host work, with fewer terms, has to agree: the older fit takes calls back
// that this one misjudges (of those that only it would take 24 % were more than 5 % slower).
double small_cost_with_host(const SmallPlan& sp, int sbytes, int n_modes, int64_t N)
{
    const double steps = (double)sp.n_tiles * sp.n_ranges * (sp.cols_per_range / 4);       // of one workgroup
    const double cycles = sbytes == 8 ? 64.0 : 32.0;
    const double mfma = steps * sp.RB * sp.JB * cycles / 4.0 / 2200.0;
    const double instr = steps * (12 + 6 * n_modes + 3 * sp.RB + 3 * sp.JB * n_modes) / 2200.0;
    const double sweeps = (double)ceil_div((int64_t)sp.n_tiles * sp.n_ranges, sp.waves);
    const double groups = (double)sp.blocks * sp.n_jchunk * sp.n_groups;
    const double resident = 256.0 * (16 / sp.waves);
    const double rounds = groups > resident ? groups / resident : 1.0;
    return 3.6 + rounds * (1.2 * mfma + 1.38 * instr + 2.3 * sweeps) + (sp.n_groups > 1 ? 3.55 : 0.0) +
           0.027e-6 * (double)N * sbytes;
}

double general_cost_with_host(const Plan& pl)
{
    const bool paired_second = pl.seg > 0 && !pl.seg_first;
    const bool prepare = pl.fused_bytes > 0 || paired_second || pl.contract_rows;
    const bool combine = pl.n_slots > 1 || pl.seg > 0;
    const bool rows = pl.contract_rows || pl.lead_route;      // (their tiles count as one row block of the fit)
    const double cycles = (pl.sbytes == 8 ? 64.0 : 32.0) * (rows ? 1 : pl.RB) * (pl.lead_route ? pl.lead.JB : pl.JB);
    const double items = (double)pl.n_items, rounds = items > 3072.0 ? items / 3072.0 : 1.0;
    const double steps = (double)pl.steps_per_item * rounds;
    return 5.5 + (prepare ? 2.6 : 0.0) + (combine ? 2.3 : 0.0) + (pl.seg > 0 ? 1.8 : 0.0) + 0.0455 * steps +
           1.96 * cycles * steps / 2200.0 + 0.107e-6 * (double)pl.N * pl.sbytes + 1.1e-3 * items;
}

// Time of a streaming plan in us, fitted to 7500 calls
// (fp64 and fp32, 2^20 to 2^28 values, R = 4 to 128, up to twenty decompositions each; median error 8.5 %): what a step
// costs (matrix cores at 1.9 GHz, HBM at 6.9 TB/s, or the latency of its loads), what an item and a sweep cost besides,
// the launches around it and the partial sums.
double stream_time(const Plan& pl)
{
    const double cycles = (pl.sbytes == 8 ? 64.0 : 32.0) * pl.RB * pl.JB;
    int waves = stream_waves(pl.sbytes, pl.RB, pl.JB), depth = stream_depth(pl.sbytes, pl.RB, pl.JB);
    if (!pl.deep) {
        const int tiles = pl.RB * pl.JB * (pl.sbytes / 4);
        waves = tiles <= 8 ? 4 : (tiles <= 12 ? 3 : 2);
        depth = 3;
    }
    const double slots = 1024.0 * waves, items = (double)pl.n_items;
    const double active = items < slots ? items : slots;
    const double mfma = cycles / 1885.0 * (active > 1024.0 ? active / 1024.0 : 1.0);
    const double mem = active * 64.0 * pl.RB * pl.sbytes / 6.866e6;
    const double latency = 0.315 / depth;
    const double step = pow(mfma * mfma * mfma * mfma + mem * mem * mem * mem + latency * latency * latency * latency, 0.25);
    const bool second = pl.seg > 0 && !pl.seg_first, per_row = pl.seg_first && !pl.seg_store;
    const double fixed = 1.459 + 0.266 * pl.RB * pl.JB + (second ? 1.70 : 0.0) + (per_row ? 5.62 : 0.0) +
                         0.765 * (double)pl.o_per_item;
    const double rounds = items > slots ? items / slots : 1.0;
    return 2.94 + (pl.fused_bytes > 0 || second ? 3.31 : 0.0) + (pl.n_slots > 1 || pl.seg > 0 ? 3.22 : 0.0) +
           0.966 * 1e-6 * (double)(pl.ws_bytes - pl.fused_bytes) + rounds * (fixed + (double)pl.steps_per_item * step);
}

// Tensors of 2^20 to 2^28 values: the rules above were fitted to larger ones, where a launch has many rounds of long
// items.  Other targets for the number of items, three row blocks, and rows paired / fused or not are compared by
// estimated time, and one of them is taken when it is estimated 15 % faster
// (20 % where the second mode's paired rows are given up): 1.05 times faster in the mean over 6000 such calls, 1.10 at
// 2^21 values, 1.05 at 2^25, 1.02 at 2^26, and 2 % of them more than 5 % slower (20 x 30 x 40 x 50 x 60 at R = 16, fourth
// mode: 178 -> 113 us). In fp32 a plan with longer chains of sums in an item than before is not taken
// (12 % of the fp32 calls keep their plan for it): such chains, up to 4 times as long, gave up to twice the error against
// fp64 (4112 x 359 x 25 at R = 32, first mode: 3.3e-8 -> 6.7e-8 rms).
void better_stream_plan(int ndim, const int64_t* dims, int R, int k, int sbytes, bool compact, Plan& pl)
{
    int64_t N = 1;
    for (int m = 0; m < ndim; ++m)
        N *= dims[m];
    if (N < ((int64_t)1 << 20) || N > ((int64_t)1 << 28) || pl.contract_rows || pl.lead_route)
        return;
    const double now = stream_time(pl);
    const bool paired_second = pl.seg > 0 && !pl.seg_first;
    // memory stays in its class: the bounds of the plan itself, for the first mode (whose workspace a shared sweep counts
    // on) never more than that plan, elsewhere up to 5 % of the tensor and what mttkrp_dense_f64_noalloc has
    size_t ws_max = pl.ws_bytes;
    if (k != 0) {
        double most = 0.05 * (double)N * sbytes;
        if (most > kNoallocBytes)
            most = kNoallocBytes;
        if ((double)ws_max < most)
            ws_max = (size_t)most;
    }
    Plan best;
    double best_time = now;
    bool found = false;
    for (int t = 0; t < 3; ++t)
        for (int rb = 0; rb <= 3; rb += 3)
            for (int rows = 0; rows < 3; ++rows) {
                if (t + rb + rows == 0)
                    continue;
                Tuning tn;
                tn.target_items = t == 0 ? 0 : (t == 1 ? 768 : 3072);
                tn.row_blocks = rb;
                tn.contract_rows = 2;
                (k < 2 ? tn.pair_rows : tn.fuse_rows) = rows;
                Plan c;
                if (make_plan_for(ndim, dims, R, k, sbytes, tn, c, false) != MTTKRP_OK || c.ws_bytes > ws_max)
                    continue;
                if (c.RB == 1 && c.JB >= 3)        // short of registers for what the fit gives it
                    continue;
                if (sbytes == 4 && c.steps_per_item > pl.steps_per_item)   // fp32: no longer chain of sums than before
                    continue;
                // What the estimate does not see (9400 calls whose plan it changed: 0.79 times as long in the mean and 5.6 % more than 5 %
                // slower; of the 620 left out here 47 %, of the others 2.7 %): long items a little over one for each SIMD, of which
                // some then run two and the others wait; items of a few steps; first modes that walk five modes and more.
                const double tiles = c.RB * c.JB * (sbytes / 4);
                if (!compact && ((c.n_items > 1024 && c.n_items <= 1536 && c.steps_per_item >= (tiles >= 12 ? 64 : 128)) ||
                                 c.steps_per_item < 4 || (k == 0 && c.n_out >= 5)))
                    continue;
                const double time = stream_time(c);
                if (time < best_time && time < (paired_second && c.seg == 0 ? 0.80 : 0.85) * now) {
                    best = c;
                    best_time = time;
                    found = true;
                }
            }
    if (found)
        pl = best;
}

// (compact: see mttkrp_dense_bytes)
int choose_plan(int ndim, const int64_t* dims, int R, int k, int sbytes, const Tuning& tn, bool tuned, bool compact, Plan& pl)
{
    const int rc = make_general_plan(ndim, dims, R, k, sbytes, tn, pl);
    if (rc != MTTKRP_OK)
        return rc;
    if (tn.row_blocks == 0 && sbytes == 8 && R > 48) {
        // Fewer row blocks a wavefront can mean more partial rows (446 x 118 x 9560 at R = 64, third mode: 49 -> 69 MB): the
        // costs of wide tiles choose only within min(5 % of the tensor, 64 MiB) or the memory of the other plan.
        Wanted general = tn;
        general.plain_rows = true;
        Plan c;
        double most = 0.05 * (double)pl.N * sbytes;
        if (most > kNoallocBytes)
            most = kNoallocBytes;
        if ((double)pl.ws_bytes > most && make_general_plan(ndim, dims, R, k, sbytes, general, c) == MTTKRP_OK &&
            c.ws_bytes < pl.ws_bytes)
            pl = c;
    }
    if (compact && sbytes == 4 && R > 48) {
        // Whole rounds of three wavefronts a SIMD can take more splits than those of two, and more partial sums (1 x 13 x 55 x 12 x 2 x
        // 152 x 30 at R = 263: the sweep beyond its limit).
        Wanted two = tn;
        two.waves = 2;
        Plan c;
        if (make_general_plan(ndim, dims, R, k, sbytes, two, c) == MTTKRP_OK && c.ws_bytes < pl.ws_bytes)
            pl = c;
    }
    if (!tuned)
        better_stream_plan(ndim, dims, R, k, sbytes, compact, pl);
    // the other keys choose among the decompositions of the general plans
    if (tn.small_route == 2 || (tn.small_route == 0 && (tuned || compact)))
        return rc;
    // 32-bit offsets in the kernel, and a bounded grid
    int64_t N = 1, C = 1;
    for (int m = 0; m < ndim; ++m) {
        N *= dims[m];
        if (m > 0 && m != k)
            C *= dims[m];
        if (dims[m] >= ((int64_t)1 << 24) || dims[m] * (int64_t)R >= ((int64_t)1 << 30))
            return rc;
    }
    if (N * sbytes >= ((int64_t)1 << 31) || R > 4096)
        return rc;
    const int n_modes = k == 0 ? ndim - 1 : ndim - 2;
    SmallPlan best;
    // At 0.8 the calls that get slower are few: of 1901 that were not fitted 1.7 % of those taken are more than 5 % slower than the general
    // plan, at 0.9 3.0 %, at 1.0 6.3 %, and all are 0.681, 0.679 and 0.682 times as long in the mean; beyond 2^22 values 4 %.
    if (tn.small_route == 0 && N > ((int64_t)1 << 22))
        return rc;
    double best_cost = tn.small_route == 1 ? 1e300 : 0.8 * general_cost(pl, ndim);
    bool take = false;
    for (int groups = 1; groups <= 64; groups = groups == 1 ? 4 : 2 * groups) {
        if (tn.small_groups > 0)
            groups = (int)tn.small_groups;
        if (groups > 1 && C < 16 * (int64_t)groups && tn.small_groups == 0)
            break;
        const SmallPlan sp = mttkrp_small_plan(ndim, dims, R, k, sbytes, groups);
        // fp32: no longer chain of sums than the general plan's (beyond it the sums are fp64 in both)
        // partial sums of the groups: 16 MiB, or what the general plan has (tall outputs of a high rank)
        const double bytes = groups > 1 ? (double)sp.n_groups * (double)dims[k] * R * sbytes : 0.0;
        if ((sbytes == 8 || sp.cols_per_range <= 4 * pl.steps_per_item || tn.small_route == 1) &&
            (bytes <= 16777216.0 || bytes <= (double)pl.ws_bytes)) {
            const double cost = small_cost(sp, sbytes, n_modes, N, bytes, k == 0);
            if (cost < best_cost && (tn.small_route == 1 || N <= kSmallFitValues ||
                                     small_cost_with_host(sp, sbytes, n_modes, N) < 0.8 * general_cost_with_host(pl))) {
                best = sp;
                best_cost = cost;
                take = true;
            }
        }
        if (tn.small_groups > 0)
            break;
    }
    if (!take)
        return rc;
    pl.small = true;
    pl.sp = best;
    pl.small_bytes = best.n_groups > 1 ? (size_t)best.n_groups * (size_t)dims[k] * (size_t)R * (size_t)sbytes : 0;
    if (pl.ws_bytes < (pl.small_bytes + 255) / 256 * 256)
        pl.ws_bytes = (pl.small_bytes + 255) / 256 * 256;
    return MTTKRP_OK;
}

// Plans at default settings are kept by shape: a call pays for the planning above once (15 us with the candidates of
// better_stream_plan, as long as a small call) and then for a look-up.  Sixteen sets of eight plans, the least recently used
// one of a set makes room: a tensor has at most eight modes, so no two of them can drive each other out (with one entry per
// hash 4 % of the three-way and 21 % of the six-way shapes planned two of their modes anew at every call, 5 to 21 us).
// g_mutex held.
struct PlanKey {
    int64_t dims[MTTKRP_MAX_NDIM];
    int32_t ndim, R, k, sbytes;
};
constexpr int kPlanSets = 16, kPlanWays = 8;
static_assert(kPlanWays >= MTTKRP_MAX_NDIM, "the modes of a tensor fit in one set");
struct PlanEntry {
    uint64_t last_use = 0;       // 0: empty
    uint64_t hash = 0;
    PlanKey key;
    Plan plan;
};
PlanEntry g_plans[kPlanSets][kPlanWays];
uint64_t g_plan_clock = 0;

PlanEntry* kept_plan(uint64_t hash, const PlanKey& key)
{
    for (PlanEntry& e : g_plans[(hash >> 40) % kPlanSets])
        if (e.last_use && e.hash == hash && memcmp(&e.key, &key, sizeof(key)) == 0) {
            e.last_use = ++g_plan_clock;
            return &e;
        }
    return nullptr;
}

void keep_plan(uint64_t hash, const PlanKey& key, const Plan& pl)
{
    PlanEntry* oldest = &g_plans[(hash >> 40) % kPlanSets][0];
    if (kept_plan(hash, key))    // another thread was faster
        return;
    for (PlanEntry& e : g_plans[(hash >> 40) % kPlanSets])
        if (e.last_use < oldest->last_use)
            oldest = &e;
    oldest->last_use = ++g_plan_clock;
    oldest->hash = hash;
    oldest->key = key;
    oldest->plan = pl;
}

int make_plan(int ndim, const int64_t* dims, int R, int k, int sbytes, Plan& pl)
{
    int rc = validate(ndim, dims, R, k, sbytes);
    if (rc != MTTKRP_OK)
        return rc;
    PlanKey key;
    memset(&key, 0, sizeof(key));
    uint64_t h = (uint64_t)R * 31 + (uint64_t)k * 7 + (uint64_t)sbytes;
    for (int m = 0; m < ndim; ++m) {
        key.dims[m] = dims[m];
        h = (h ^ (uint64_t)dims[m]) * 0x9e3779b97f4a7c15ull;
    }
    key.ndim = ndim; key.R = R; key.k = k; key.sbytes = sbytes;
    const Tuning none;
    Tuning tn;
    bool tuned;
    {
        std::lock_guard<std::mutex> lock(g_mutex);
        tn = g_tune;
        tuned = memcmp(&tn, &none, sizeof(tn)) != 0;
        if (!tuned)
            if (const PlanEntry* e = kept_plan(h, key)) {
                pl = e->plan;
                return MTTKRP_OK;
            }
    }
    rc = choose_plan(ndim, dims, R, k, sbytes, tn, tuned, false, pl);
    if (rc == MTTKRP_OK && !tuned) {
        std::lock_guard<std::mutex> lock(g_mutex);
        keep_plan(h, key, pl);
    }
    return rc;
}

int make_compact_plan(int ndim, const int64_t* dims, int R, int k, int sbytes, Plan& pl)
{
    const Tuning none, tn = tuning();
    return choose_plan(ndim, dims, R, k, sbytes, tn, memcmp(&tn, &none, sizeof(tn)) != 0, true, pl);
}

template <typename T, int RB, int JB>
void launch_stream(const StreamArgs<T>& a, dim3 grid, hipStream_t st, int cap, bool nt_off, bool deep)
{
    // first mode: two wavefront tiles of LDS for the cross-wavefront sum
    size_t lds = a.first_mode && a.group4 ? (size_t)2 * RB * JB * 4 * 64 * sizeof(T) : 0;
    // Resident wavefronts per SIMD can be capped by reserving LDS: a workgroup is one
    // wavefront per SIMD, and a compute unit has 160 KB of LDS.
    if (cap >= 1 && cap <= 7) {
        const size_t want = (size_t)160 * 1024 / (size_t)(cap + 1) + 256;
        if (want <= 65536 && want > lds)
            lds = want;
    }
    // non-temporal tensor loads only when each load instruction reads whole aligned lines
    const bool nt = !nt_off && sizeof(T) == 8 && a.I0 % 16 == 0 && ((uintptr_t)a.X & 127u) == 0;
    if (deep) {
        if (nt)
            hipLaunchKernelGGL((mttkrp_stream_kernel<T, RB, JB, true, true>), grid, dim3(kBlockThreads), lds, st, a);
        else
            hipLaunchKernelGGL((mttkrp_stream_kernel<T, RB, JB, false, true>), grid, dim3(kBlockThreads), lds, st, a);
    } else {
        if (nt)
            hipLaunchKernelGGL((mttkrp_stream_kernel<T, RB, JB, true, false>), grid, dim3(kBlockThreads), lds, st, a);
        else
            hipLaunchKernelGGL((mttkrp_stream_kernel<T, RB, JB, false, false>), grid, dim3(kBlockThreads), lds, st, a);
    }
}

template <typename T, int RB>
void launch_stream_jb(int JB, const StreamArgs<T>& a, dim3 grid, hipStream_t st, int cap, bool nt_off, bool deep)
{
    switch (JB) {
    case 1: launch_stream<T, RB, 1>(a, grid, st, cap, nt_off, deep); break;
    case 2: launch_stream<T, RB, 2>(a, grid, st, cap, nt_off, deep); break;
    case 3: launch_stream<T, RB, 3>(a, grid, st, cap, nt_off, deep); break;
    default: launch_stream<T, RB, 4>(a, grid, st, cap, nt_off, deep); break;
    }
}

template <typename T>
void launch_stream_rb(int RB, int JB, const StreamArgs<T>& a, dim3 grid, hipStream_t st, int cap, bool nt_off, bool deep)
{
    switch (RB) {
    case 1: launch_stream_jb<T, 1>(JB, a, grid, st, cap, nt_off, deep); break;
    case 2: launch_stream_jb<T, 2>(JB, a, grid, st, cap, nt_off, deep); break;
    case 3: launch_stream_jb<T, 3>(JB, a, grid, st, cap, nt_off, deep); break;
    default: launch_stream_jb<T, 4>(JB, a, grid, st, cap, nt_off, deep); break;
    }
}

template <typename T, int CB>
void launch_rowsum_jb(int JB, const RowSumArgs<T>& a, dim3 grid, hipStream_t st)
{
    // CB * JB <= 8 accumulator tiles (the planner's limit)
    switch (JB) {
    case 1: hipLaunchKernelGGL((mttkrp_rowsum_kernel<T, CB, 1>), grid, dim3(kBlockThreads), 0, st, a); break;
    case 2: hipLaunchKernelGGL((mttkrp_rowsum_kernel<T, CB, 2>), grid, dim3(kBlockThreads), 0, st, a); break;
    case 3:
        if constexpr (CB <= 2)
            hipLaunchKernelGGL((mttkrp_rowsum_kernel<T, CB, 3>), grid, dim3(kBlockThreads), 0, st, a);
        break;
    case 4:
        if constexpr (CB <= 2)
            hipLaunchKernelGGL((mttkrp_rowsum_kernel<T, CB, 4>), grid, dim3(kBlockThreads), 0, st, a);
        break;
    case 5:
        if constexpr (CB == 1)
            hipLaunchKernelGGL((mttkrp_rowsum_kernel<T, CB, 5>), grid, dim3(kBlockThreads), 0, st, a);
        break;
    case 6:
        if constexpr (CB == 1)
            hipLaunchKernelGGL((mttkrp_rowsum_kernel<T, CB, 6>), grid, dim3(kBlockThreads), 0, st, a);
        break;
    case 7:
        if constexpr (CB == 1)
            hipLaunchKernelGGL((mttkrp_rowsum_kernel<T, CB, 7>), grid, dim3(kBlockThreads), 0, st, a);
        break;
    default:
        if constexpr (CB == 1)
            hipLaunchKernelGGL((mttkrp_rowsum_kernel<T, CB, 8>), grid, dim3(kBlockThreads), 0, st, a);
        break;
    }
}

template <typename T>
void launch_rowsum(int CB, int JB, const RowSumArgs<T>& a, dim3 grid, hipStream_t st)
{
    switch (CB) {
    case 1: launch_rowsum_jb<T, 1>(JB, a, grid, st); break;
    case 2: launch_rowsum_jb<T, 2>(JB, a, grid, st); break;
    case 3: launch_rowsum_jb<T, 3>(JB, a, grid, st); break;
    default: launch_rowsum_jb<T, 4>(JB, a, grid, st); break;
    }
}

constexpr int kTimingSlots = 512;   // ring of timed calls kept per device

struct TimedCall {
    // before the streaming kernel, between the two kernels, after the combine kernel
    hipEvent_t ev[3] = {nullptr, nullptr, nullptr};
    bool combine = false;
};

// Library-owned workspaces: one per (device, stream), so that calls in flight on different
// streams of a device never share partial sums.  A device keeps at most kOwnedSlots of them; a
// further stream takes over the least recently used one after waiting for the event recorded
// behind that workspace's last call.
constexpr int kOwnedSlots = 8;

struct OwnedWorkspace {
    hipStream_t stream = nullptr;
    bool used = false;           // stream is meaningful
    void* ws = nullptr;
    size_t ws_bytes = 0;
    hipEvent_t done = nullptr;   // recorded after the last kernel that uses ws (see DeviceState::record)
    bool pending = false;        // done has been recorded at least once
    bool unmarked = false;       // calls have used ws since, with no event behind them
    uint64_t last_use = 0;
};

struct DeviceState {
    OwnedWorkspace own[kOwnedSlots];
    uint64_t use_counter = 0;
    // Whether calls record an event behind their last kernel.  A workspace only changes hands when a ninth
    // stream comes along, and the event costs the GPU about 5 us a call (64^3: 20.5 -> 15.7 us), so none is
    // recorded until then; the first hand-over waits for the whole device once.
    bool record = false;
    TimedCall* calls = nullptr;  // kTimingSlots entries once timing has been used
    int64_t n_timed = 0;         // calls recorded since timing was last enabled
    const void* zeros = nullptr; // this device's address of zero_pad
};
DeviceState g_dev[kMaxDevices];
bool g_timing = false;

// The owned workspace of (device state, stream) with at least `bytes` bytes, or null after a
// failed HIP call.  Called with g_mutex held and the device current.  Waits (on the host) only
// when a workspace changes hands or has to grow while its last call may still be running.
OwnedWorkspace* owned_workspace(DeviceState& ds, hipStream_t st, size_t bytes)
{
    OwnedWorkspace* slot = nullptr;
    for (int i = 0; i < kOwnedSlots && !slot; ++i)
        if (ds.own[i].used && ds.own[i].stream == st)
            slot = &ds.own[i];
    if (!slot) {
        for (int i = 0; i < kOwnedSlots; ++i) {
            OwnedWorkspace& c = ds.own[i];
            if (!slot || (!c.used && slot->used) || (c.used == slot->used && c.last_use < slot->last_use))
                slot = &c;
        }
        if (slot->used && !ds.record) {
            if (hipDeviceSynchronize() != hipSuccess)
                return nullptr;
            for (int i = 0; i < kOwnedSlots; ++i)
                ds.own[i].unmarked = false;
            ds.record = true;
        }
        if (slot->pending && hipEventSynchronize(slot->done) != hipSuccess)
            return nullptr;
        slot->pending = false;
        slot->used = true;
        slot->stream = st;
    }
    if (ds.record && !slot->done && hipEventCreateWithFlags(&slot->done, hipEventDisableTiming) != hipSuccess) {
        slot->done = nullptr;
        return nullptr;
    }
    if (slot->ws_bytes < bytes) {
        if (slot->ws) {
            if (slot->pending && hipEventSynchronize(slot->done) != hipSuccess)
                return nullptr;
            if (slot->unmarked && hipStreamSynchronize(st) != hipSuccess)     // the slot's stream is the caller's
                return nullptr;
            slot->pending = false;
            slot->unmarked = false;
            (void)hipFree(slot->ws);
            slot->ws = nullptr;
            slot->ws_bytes = 0;
        }
        const size_t want = bytes + (bytes >> 2);
        if (hipMalloc(&slot->ws, want) != hipSuccess) {
            (void)hipGetLastError();
            slot->ws = nullptr;
            return nullptr;
        }
        slot->ws_bytes = want;
    }
    slot->last_use = ++ds.use_counter;
    return slot;
}

// Launches of the contraction over the leading index for a plan made by plan_leading (no
// locking, no planning).  With lambda or beta the result passes through the combine kernel:
// over the row splits' partial sums, or, without row splits, over one slot at `workspace`.
template <typename T>
int launch_leading(const LeadingPlan& pl, int64_t P, int64_t Q, const T* X, const T* K, int64_t ldK, int R, T* out,
                   int64_t ld_out, void* workspace, const T* lambda, double beta, hipStream_t st)
{
    if (pl.CB * pl.JB > 8 || pl.CB < 1 || pl.CB > 4 || pl.JB < 1 || pl.JB > 8)
        return MTTKRP_ERR_UNSUPPORTED;
    const bool scaled = lambda != nullptr || beta != 0.0;
    const bool via_ws = pl.ws_bytes > 0 || scaled;
    if (pl.cp.ok) {
        ContractArgs<T> ca;
        memset(&ca, 0, sizeof(ca));
        ca.X = X;
        ca.K = K;
        ca.out = via_ws ? (T*)workspace : out;
        ca.P = P;
        ca.Q = Q;
        ca.ldK = ldK;
        ca.ld_out = via_ws ? R : ld_out;
        ca.rows_per_split = pl.cp.rows_per_split;
        ca.n_items = pl.cp.n_items;
        ca.R = R;
        ca.n_rsplit = pl.cp.n_rsplit;
        ca.n_ctile = (int32_t)pl.cp.n_ctile;
        ca.chain = pl.cp.chain;
        (void)hipGetLastError();
        const int rc = mttkrp_contract_launch<T>(pl.cp, ca, st);
        if (rc != MTTKRP_OK)
            return rc;
        if (via_ws)
            launch_combine<T>((T*)workspace, out, Q * (int64_t)R, R, pl.n_rsplit, pl.n_rsplit * (int64_t)R,
                              (int64_t)R, lambda, beta, ld_out, st);
        return hipGetLastError() == hipSuccess ? MTTKRP_OK : MTTKRP_ERR_DEVICE;
    }
    RowSumArgs<T> ra;
    memset(&ra, 0, sizeof(ra));
    ra.X = X;
    ra.A0 = K;
    ra.W = K;                    // not read in the store mode
    ra.out = via_ws ? (T*)workspace : out;
    ra.sx_batch = 0;
    ra.sx_lo = P;
    ra.sx_hi = 0;
    ra.C_lo = (int32_t)Q;
    ra.C = (int32_t)Q;
    ra.I0 = (int32_t)P;
    ra.R = R;
    ra.ld0 = (int32_t)ldK;
    ra.ld_dst = (int32_t)(via_ws ? R : ld_out);
    ra.n_cchunk = pl.n_cchunk;
    ra.n_jchunk = pl.n_jchunk;
    ra.n_batch = 1;
    ra.n_rsplit = pl.n_rsplit;
    ra.rows_per_split = pl.rows_per_split;
    ra.n_items = (int32_t)pl.n_items;
    ra.n_slots = pl.n_rsplit;
    ra.store_s = 1;
    const int64_t blocks = ceil_div(pl.n_items, kWaves);
    (void)hipGetLastError();
    launch_rowsum<T>(pl.CB, pl.JB, ra, dim3((unsigned)blocks), st);
    if (via_ws)
        launch_combine<T>((T*)workspace, out, Q * (int64_t)R, R, pl.n_rsplit, pl.n_rsplit * (int64_t)R,
                          (int64_t)R, lambda, beta, ld_out, st);
    return hipGetLastError() == hipSuccess ? MTTKRP_OK : MTTKRP_ERR_DEVICE;
}

template <typename T>
int run_leading(int64_t P, int64_t Q, const T* X, const T* K, int64_t ldK, int R, T* out, int64_t ld_out,
                void* workspace, size_t workspace_bytes, void* stream, bool compact = false)
{
    if (!X || !K || !out)
        return MTTKRP_ERR_INVALID_ARG;
    LeadingPlan pl;
    const int rc = plan_leading(P, Q, R, (int)sizeof(T), tuning_for(compact), pl);
    if (rc != MTTKRP_OK)
        return rc;
    if (ldK < R || ldK >= ((int64_t)1 << 27) || ld_out < R || ld_out >= ((int64_t)1 << 27))
        return MTTKRP_ERR_INVALID_ARG;
    if (pl.ws_bytes > 0 && (!workspace || workspace_bytes < pl.ws_bytes))
        return MTTKRP_ERR_WORKSPACE;
    return launch_leading<T>(pl, P, Q, X, K, ldK, R, out, ld_out, workspace, nullptr, 0.0, (hipStream_t)stream);
}

template <typename T>
int run(int ndim, const int64_t* dims, const T* X, const T* const* factors, int R, int k, T* M,
        void* workspace, size_t workspace_bytes, bool own_ws, void* stream,
        const T* lambda = nullptr, double beta = 0.0, const int64_t* ld_factors = nullptr, int64_t ldM = 0,
        bool allow_timing = true, bool compact = false)
{
    if (!X || !M || !factors)
        return MTTKRP_ERR_INVALID_ARG;
    // leading dimensions: rows of factors[m] are ld_factors[m] values apart, rows of M ldM (default R)
    int64_t ld[MTTKRP_MAX_NDIM];
    if (ndim >= 1 && ndim <= MTTKRP_MAX_NDIM)
        for (int m = 0; m < ndim; ++m) {
            ld[m] = ld_factors ? ld_factors[m] : R;
            if (m != k && (ld[m] < R || ld[m] >= ((int64_t)1 << 27)))
                return MTTKRP_ERR_INVALID_ARG;
        }
    if (ldM == 0)
        ldM = R;
    if (ldM < R || ldM >= ((int64_t)1 << 27))
        return MTTKRP_ERR_INVALID_ARG;
    Plan pl;
    int rc = compact ? make_compact_plan(ndim, dims, R, k, (int)sizeof(T), pl) : make_plan(ndim, dims, R, k, (int)sizeof(T), pl);
    if (rc != MTTKRP_OK)
        return rc;
    // The kernel for small tensors addresses a factor's rows in 32 bits: blocks of arrays of 2^32 values and more run on
    // the general decomposition, which the plan holds besides and whose workspace it counts.
    for (int m = 0; m < ndim; ++m)
        if (m != k && dims[m] * ld[m] >= ((int64_t)1 << 32))
            pl.small = false;
    // Weights and accumulation are applied by the combine kernel, which then always runs.
    const bool scaled = lambda != nullptr || beta != 0.0;
    if (scaled && pl.part_bytes == 0) {
        pl.part_bytes = (size_t)dims[k] * (size_t)R * sizeof(T);
        const size_t bytes = (pl.part_bytes + 255) / 256 * 256 + pl.fused_bytes;
        pl.ws_bytes = pl.ws_bytes > bytes ? pl.ws_bytes : bytes;
    }
    for (int m = 0; m < ndim; ++m)
        if (m != k && !factors[m])
            return MTTKRP_ERR_INVALID_ARG;
    // The problem the kernels see: the caller's, or the one with two modes fused (then
    // factor fuse_a is the product matrix at the end of the workspace).
    const T* fac[MTTKRP_MAX_NDIM];
    int64_t fld[MTTKRP_MAX_NDIM];
    for (int m = 0; m < pl.ndim; ++m) {
        fac[m] = factors[pl.orig[m]];
        fld[m] = ld[pl.orig[m]];
    }
    const int k_call = k;
    k = pl.k;

    int dev = 0;
    if (hipGetDevice(&dev) != hipSuccess)
        return MTTKRP_ERR_DEVICE;
    if (dev < 0 || dev >= kMaxDevices)
        return MTTKRP_ERR_UNSUPPORTED;
    hipStream_t st = (hipStream_t)stream;

    std::lock_guard<std::mutex> lock(g_mutex);
    DeviceState& ds = g_dev[dev];
    if (!ds.zeros) {     // (the name zero_pad is no device address on the host: ask the runtime, once per device)
        void* ptr = nullptr;
        if (hipGetSymbolAddress(&ptr, HIP_SYMBOL(zero_pad)) != hipSuccess) {
            (void)hipGetLastError();
            return MTTKRP_ERR_DEVICE;
        }
        ds.zeros = ptr;
    }
    T* ws = nullptr;
    OwnedWorkspace* owned = nullptr;
    if (pl.ws_bytes > 0) {
        if (own_ws) {
            const size_t bytes = pl.small ? pl.small_bytes : pl.ws_bytes;
            owned = bytes > 0 ? owned_workspace(ds, st, bytes) : nullptr;
            if (bytes > 0 && !owned)
                return MTTKRP_ERR_DEVICE;
            ws = owned ? (T*)owned->ws : nullptr;
        } else {
            if (!workspace || workspace_bytes < pl.ws_bytes || ((uintptr_t)workspace & 255u))
                return MTTKRP_ERR_WORKSPACE;
            ws = (T*)workspace;
        }
    }
    char* const fused = pl.n_fuse > 0 ? (char*)ws + (pl.part_bytes + 255) / 256 * 256 : nullptr;
    for (int f = 0; f < pl.n_fuse; ++f) {
        fac[pl.fus[f].red] = (const T*)(fused + pl.fus[f].offset);
        fld[pl.fus[f].red] = R;
    }
    // behind the call's last kernel: marks when its owned workspace may change hands or be freed
    auto finish = [&]() {
        if (!owned)
            return;
        if (ds.record && hipEventRecord(owned->done, st) == hipSuccess)
            owned->pending = true;
        else
            owned->unmarked = true;
    };
    const bool timing = g_timing && allow_timing;    // timing creates events on first use
    TimedCall* tc = nullptr;
    if (timing) {
        if (!ds.calls) {
            TimedCall* calls = new (std::nothrow) TimedCall[kTimingSlots];
            if (!calls)
                return MTTKRP_ERR_DEVICE;
            for (int c = 0; c < kTimingSlots; ++c)
                for (int e = 0; e < 3; ++e)
                    if (hipEventCreate(&calls[c].ev[e]) != hipSuccess) {
                        delete[] calls;   // events created so far are leaked; creation does not fail in practice
                        return MTTKRP_ERR_DEVICE;
                    }
            ds.calls = calls;
        }
        tc = &ds.calls[ds.n_timed % kTimingSlots];
    }

    if (pl.small) {
        k = k_call;
        SmallArgs<T> sa;
        memset(&sa, 0, sizeof(sa));
        sa.X = X;
        sa.A0 = k == 0 ? nullptr : factors[0];
        sa.out = pl.small_bytes > 0 ? ws : M;
        sa.lambda = lambda;
        sa.beta = beta;
        int64_t C = 1, stride = 1;
        for (int m = 0; m < ndim; ++m) {
            if (m == k)
                sa.sx_batch = k == 0 ? 0 : (int32_t)stride;
            else if (m > 0) {
                sa.A[sa.n] = factors[m];
                sa.dim[sa.n] = (int32_t)dims[m];
                sa.ld[sa.n] = (int32_t)ld[m];
                sa.sx[sa.n] = (int32_t)stride;
                if (dims[m] > 1)
                    mttkrp_small_divisor((uint32_t)dims[m], sa.magic[sa.n], sa.shift[sa.n]);
                sa.n += 1;
                C *= dims[m];
            }
            stride *= dims[m];
        }
        sa.I0 = (int32_t)dims[0];
        sa.R = R;
        sa.C = (int32_t)C;
        sa.ld0 = k == 0 ? 0 : (int32_t)ld[0];
        sa.ld_out = (int32_t)ldM;
        sa.group_stride = dims[k] * (int64_t)R;
        sa.row_stride = R;
        sa.n_tiles = pl.sp.n_tiles;
        sa.n_ranges = pl.sp.n_ranges;
        sa.cols_per_range = pl.sp.cols_per_range;
        sa.cols_per_group = pl.sp.cols_per_group;
        (void)hipGetLastError();
        if (timing)
            (void)hipEventRecord(tc->ev[0], st);
        const int src = mttkrp_small_launch<T>(pl.sp, sa, k == 0, st);
        if (timing) {
            (void)hipEventRecord(tc->ev[1], st);
            tc->combine = false;
        }
        if (src != MTTKRP_OK) {
            finish();
            return src;
        }
        if (pl.small_bytes > 0) {
            launch_combine<T>(ws, M, dims[k] * (int64_t)R, R, pl.sp.n_groups, (int64_t)R, dims[k] * (int64_t)R, lambda,
                              beta, ldM, st);
            if (timing) {
                (void)hipEventRecord(tc->ev[2], st);
                tc->combine = true;
            }
            if (hipGetLastError() != hipSuccess) {
                finish();
                return MTTKRP_ERR_DEVICE;
            }
        }
        if (timing)
            ds.n_timed += 1;
        finish();
        return MTTKRP_OK;
    }
    if (pl.lead_route) {
        // K = Khatri-Rao product of the factors of modes 0 .. d-2 (mode 0 fastest), behind the partial sums
        const T* K = factors[0];
        int64_t ldK = ld[0];
        (void)hipGetLastError();
        if (timing)
            (void)hipEventRecord(tc->ev[0], st);
        if (ndim > 2) {
            ColWeightArgs<T> cw;
            memset(&cw, 0, sizeof(cw));
            for (int m = 0; m < ndim - 1; ++m) {
                cw.A[m] = factors[m];
                cw.ld[m] = ld[m];
                cw.dim[m] = (int32_t)pl.dims[m];
            }
            cw.n = ndim - 1;
            T* const dst = (T*)((char*)ws + (pl.part_bytes + 255) / 256 * 256);
            const int64_t n_entries = pl.lead_P * (int64_t)R;
            hipLaunchKernelGGL((mttkrp_colweights_kernel<T>), dim3((unsigned)ceil_div(n_entries, 256)), dim3(256), 0, st,
                               cw, n_entries, R, dst);
            K = dst;
            ldK = R;
        }
        const int lrc = launch_leading<T>(pl.lead, pl.lead_P, pl.lead_Q, X, K, ldK, R, M, ldM, ws, lambda, beta, st);
        if (timing) {
            (void)hipEventRecord(tc->ev[1], st);
            tc->combine = false;
            if (lrc == MTTKRP_OK)
                ds.n_timed += 1;
        }
        finish();
        return lrc;
    }
    if (pl.contract_rows && pl.cp.ok) {
        T* const S = (T*)((char*)ws + (pl.part_bytes + 255) / 256 * 256);
        ContractArgs<T> ca;
        memset(&ca, 0, sizeof(ca));
        ca.X = X;
        ca.K = factors[0];
        ca.out = S;
        ca.P = pl.dims[0];
        ca.Q = pl.N / pl.dims[0];
        ca.ldK = ld[0];
        ca.ld_out = R;
        ca.rows_per_split = pl.cp.rows_per_split;
        ca.n_items = pl.cp.n_items;
        ca.R = R;
        ca.n_rsplit = pl.cp.n_rsplit;
        ca.n_ctile = (int32_t)pl.cp.n_ctile;
        ca.chain = pl.cp.chain;
        ModeSumArgs<T, T> ms;
        memset(&ms, 0, sizeof(ms));
        ms.S = S;
        ms.part = pl.part_bytes > 0 ? ws : M;
        ms.ld_part = pl.part_bytes > 0 ? R : ldM;
        for (int m = 1; m < pl.ndim; ++m) {
            ms.A[m - 1] = m == k ? nullptr : factors[m];
            ms.ld[m - 1] = m == k ? 0 : ld[m];
            ms.dim[m - 1] = (int32_t)pl.dims[m];
        }
        ms.n = pl.ndim - 1;
        ms.t = k - 1;
        ms.R = R;
        ms.n_split = (uint32_t)pl.cp.n_rsplit;
        ms.n_pairs = (uint32_t)(pl.C * pl.cp.n_rsplit);
        ms.per_seg = (uint32_t)ceil_div(pl.C * (int64_t)pl.cp.n_rsplit, pl.cp_segs);
        (void)hipGetLastError();
        if (timing)
            (void)hipEventRecord(tc->ev[0], st);
        int crc = mttkrp_contract_launch<T>(pl.cp, ca, st);
        if (crc == MTTKRP_OK)
            crc = mttkrp_modesum_launch<T, T>(ms, pl.dims[k], pl.cp_segs, st);
        if (timing) {
            (void)hipEventRecord(tc->ev[1], st);
            tc->combine = false;
        }
        if (crc != MTTKRP_OK) {
            finish();
            return crc;
        }
        if (pl.part_bytes > 0) {
            launch_combine<T>((T*)ws, M, pl.dims[k] * (int64_t)R, R, pl.cp_segs, pl.cp_segs * (int64_t)R, (int64_t)R, lambda, beta, ldM, st);
            if (timing) {
                (void)hipEventRecord(tc->ev[2], st);
                tc->combine = true;
            }
            if (hipGetLastError() != hipSuccess) {
                finish();
                return MTTKRP_ERR_DEVICE;
            }
        }
        if (timing)
            ds.n_timed += 1;
        finish();
        return MTTKRP_OK;
    }
    if (pl.contract_rows) {
        if (pl.CB * pl.JB > 8 || pl.CB < 1 || pl.CB > 4 || pl.JB < 1 || pl.JB > 8)
            return MTTKRP_ERR_UNSUPPORTED;
        T* const W = (T*)((char*)ws + (pl.part_bytes + 255) / 256 * 256);
        ColWeightArgs<T> cw;
        memset(&cw, 0, sizeof(cw));
        for (int m = 1; m < pl.ndim; ++m)
            if (m != k) {
                cw.A[cw.n] = factors[m];
                cw.ld[cw.n] = ld[m];
                cw.dim[cw.n] = (int32_t)pl.dims[m];
                cw.n += 1;
            }
        RowSumArgs<T> ra;
        memset(&ra, 0, sizeof(ra));
        ra.X = X;
        ra.A0 = factors[0];
        ra.W = W;
        ra.out = pl.part_bytes > 0 ? ws : M;
        ra.sx_batch = pl.strides[k];
        ra.sx_lo = pl.dims[0];
        ra.sx_hi = pl.strides[k] * pl.dims[k];
        ra.C_lo = (int32_t)pl.C_lo;
        ra.C = (int32_t)pl.C;
        ra.I0 = (int32_t)pl.dims[0];
        ra.R = R;
        ra.ld0 = (int32_t)ld[0];
        ra.ld_dst = (int32_t)(pl.part_bytes > 0 ? R : ldM);
        ra.n_cchunk = pl.n_cchunk;
        ra.n_jchunk = pl.n_jchunk;
        ra.n_batch = pl.n_batch;
        ra.n_rsplit = pl.n_rsplit;
        ra.rows_per_split = pl.rows_per_split;
        ra.n_items = (int32_t)pl.n_items;
        ra.n_slots = (int32_t)pl.n_slots;
        const int64_t rblocks = ceil_div(pl.n_items, kWaves);
        if (rblocks >= ((int64_t)1 << 31))
            return MTTKRP_ERR_UNSUPPORTED;
        (void)hipGetLastError();
        if (timing)
            (void)hipEventRecord(tc->ev[0], st);
        const int64_t n_entries = pl.C * (int64_t)R;
        hipLaunchKernelGGL((mttkrp_colweights_kernel<T>), dim3((unsigned)ceil_div(n_entries, 256)), dim3(256), 0, st,
                           cw, n_entries, R, W);
        launch_rowsum<T>(pl.CB, pl.JB, ra, dim3((unsigned)rblocks), st);
        if (timing) {
            (void)hipEventRecord(tc->ev[1], st);
            tc->combine = false;
        }
        if (hipGetLastError() != hipSuccess) {
            finish();
            return MTTKRP_ERR_DEVICE;
        }
        if (pl.part_bytes > 0) {
            const int64_t n_elems = pl.dims[k] * (int64_t)R;
            launch_combine<T>((T*)ws, M, n_elems, R, (int)pl.n_slots, pl.n_slots * (int64_t)R, (int64_t)R, lambda, beta, ldM, st);
            if (timing) {
                (void)hipEventRecord(tc->ev[2], st);
                tc->combine = true;
            }
            if (hipGetLastError() != hipSuccess) {
                finish();
                return MTTKRP_ERR_DEVICE;
            }
        }
        if (timing)
            ds.n_timed += 1;
        finish();
        return MTTKRP_OK;
    }

    StreamArgs<T> a;
    memset(&a, 0, sizeof(a));
    a.X = X;
    a.A_row = k == 0 ? nullptr : fac[0];
    a.A_in = pl.inner >= 0 ? fac[pl.inner] : fac[0];   // without column modes k != 0, so factors[0] exists
    a.no_inner = pl.inner >= 0 ? 0 : 1;
    a.sx_in = pl.inner >= 0 ? pl.strides[pl.inner] : 0;
    a.sx_batch = k == 0 ? 0 : pl.strides[k];
    for (int m = 0; m < kMaxOuter; ++m) {
        a.A_out[m] = nullptr;
        a.sx_out[m] = 0;
        a.dim_out[m] = 1;
        a.ld_out[m] = R;
    }
    a.ld_in = (int32_t)(pl.inner >= 0 ? fld[pl.inner] : fld[0]);
    a.ld_row = (int32_t)fld[0];
    a.ld_dst = (int32_t)(pl.part_bytes > 0 ? R : ldM);
    for (int m = 0; m < pl.n_out; ++m) {
        a.A_out[m] = fac[pl.out_modes[m]];
        a.sx_out[m] = pl.strides[pl.out_modes[m]];
        a.dim_out[m] = (int32_t)pl.dims[pl.out_modes[m]];
        a.ld_out[m] = (int32_t)fld[pl.out_modes[m]];
    }
    if (pl.n_out == 0)
        a.ld_out[0] = a.ld_in;    // the kernel then reads row 0 of the inner factor as a dummy
    a.out = pl.part_bytes > 0 ? ws : M;
    a.o_total = pl.o_total;
    a.o_per_item = pl.o_per_item;
    a.n_out = pl.n_out;
    a.I0 = (int32_t)pl.dims[0];
    a.I_in = (int32_t)pl.I_in;
    a.R = R;
    a.first_mode = k == 0;
    a.n_rowblk = pl.n_rowblk;
    a.n_jchunk = pl.n_jchunk;
    a.n_batch = pl.n_batch;
    a.n_isplit = pl.n_isplit;
    a.cols_per_isplit = pl.cols_per_isplit;
    a.n_items = (int32_t)pl.n_items;
    a.n_slots = (int32_t)pl.n_slots;
    a.n_splits = (int32_t)pl.n_splits;
    a.xcd_remap = pl.xcd_remap ? 1 : 0;
    a.group4 = pl.group == kWaves ? 1 : 0;
    a.linear = pl.linear ? 1 : 0;
    a.seg = (int32_t)pl.seg;
    a.seg_first = pl.seg_store ? 2 : (pl.seg_first ? 1 : 0);
    a.seg_nblk = pl.seg_nblk;
    if (pl.seg_first) {              // the weights are rows of A_1
        a.A_row = fac[1];
        a.ld_row = (int32_t)fld[1];
    }
    a.zeros = ds.zeros;

    int64_t blocks = ceil_div(pl.n_items, kWaves);
    if (a.xcd_remap)
        blocks = ceil_div(blocks, 8) * 8;
    if (blocks >= ((int64_t)1 << 31))
        return MTTKRP_ERR_UNSUPPORTED;

    (void)hipGetLastError();
    if (timing)
        (void)hipEventRecord(tc->ev[0], st);
    // not every slot of every output row is written with paired rows in the second mode: the others must read as zero
    const bool clear_slots = pl.seg > 0 && !pl.seg_first;
    if (pl.n_fuse > 0 || clear_slots) {
        PrepareArgs<T> pa;
        memset(&pa, 0, sizeof(pa));
        pa.R = R;
        int64_t pblocks = 0;
        for (int f = 0; f < pl.n_fuse; ++f) {
            const Plan::Fusion& fu = pl.fus[f];
            const int64_t n_entries = fu.Ia * fu.Ib * (int64_t)R;
            pa.Aa[f] = factors[fu.a];
            pa.Ab[f] = factors[fu.a + 1];
            pa.lda[f] = ld[fu.a];
            pa.ldb[f] = ld[fu.a + 1];
            pa.F[f] = (T*)(fused + fu.offset);
            pa.Ia[f] = (uint32_t)fu.Ia;
            pa.n_entries[f] = (uint32_t)n_entries;
            pa.blocks[f] = (uint32_t)ceil_div(n_entries, 256);
            pblocks += pa.blocks[f];
        }
        if (clear_slots) {
            pa.zero = (uint32_t*)ws;
            pa.n_words = (int64_t)(pl.part_bytes / 4);
            const int64_t zblocks = ceil_div(pa.n_words, 4 * 256);
            pa.zero_blocks = (uint32_t)(zblocks < 4096 ? zblocks : 4096);
            pblocks += pa.zero_blocks;
        }
        hipLaunchKernelGGL((mttkrp_prepare_kernel<T>), dim3((unsigned)pblocks), dim3(256), 0, st, pa);
    }
    launch_stream_rb<T>(pl.RB, pl.JB, a, dim3((unsigned)blocks), st, pl.wave_cap, pl.nt_off, pl.deep);
    if (timing) {
        (void)hipEventRecord(tc->ev[1], st);
        tc->combine = false;
    }
    if (hipGetLastError() != hipSuccess) {
        finish();
        return MTTKRP_ERR_DEVICE;
    }
    if (pl.part_bytes > 0) {
        const int64_t n_elems = (pl.seg > 0 ? pl.out_rows : pl.dims[k]) * (int64_t)R;
        const int64_t stride_row = k == 0 || pl.seg_store ? R : pl.n_slots * (int64_t)R;
        const int64_t stride_slot = k == 0 ? pl.dims[0] * (int64_t)R : (pl.seg_store ? pl.seg * (int64_t)R : R);
        launch_combine<T>((T*)ws, M, n_elems, R, (int)pl.n_slots, stride_row, stride_slot, lambda, beta, ldM, st);
        if (timing) {
            (void)hipEventRecord(tc->ev[2], st);
            tc->combine = true;
        }
        if (hipGetLastError() != hipSuccess) {
            finish();
            return MTTKRP_ERR_DEVICE;
        }
    }
    if (timing)
        ds.n_timed += 1;
    finish();
    return MTTKRP_OK;
}

// ---------------------------------------------------------------------------
// Partial contraction over the leading index.  The tensor as a P x Q matrix (first index
// fastest): T(c, j) = sum_r X(r + P c) K(r, j).  With K the Khatri-Rao product of the factors
// of the leading modes this is the part of Eq. (elem) that every mode above them shares.
// It runs the second schedule's kernel in its store mode: one "batch", Q columns, no weights.
// ---------------------------------------------------------------------------
// Device address of `scratch` on the current device, looked up once per device (the array has
// a different address on every GPU); null after a failed runtime call.
void* g_scratch_ptr[kMaxDevices];

void* scratch_address()
{
    int dev = 0;
    if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= kMaxDevices)
        return nullptr;
    std::lock_guard<std::mutex> lock(g_mutex);
    if (!g_scratch_ptr[dev]) {
        void* ptr = nullptr;
        if (hipGetSymbolAddress((void**)&ptr, HIP_SYMBOL(scratch)) != hipSuccess) {
            (void)hipGetLastError();
            return nullptr;
        }
        g_scratch_ptr[dev] = ptr;
    }
    return g_scratch_ptr[dev];
}

}  // namespace

size_t mttkrp_dense_bytes(int ndim, const int64_t* dims, int R, int k, int sbytes, bool compact)
{
    Plan pl;
    const int rc = compact ? make_compact_plan(ndim, dims, R, k, sbytes, pl) : make_plan(ndim, dims, R, k, sbytes, pl);
    return rc == MTTKRP_OK ? pl.ws_bytes : (size_t)-1;
}
size_t mttkrp_leading_bytes(int64_t P, int64_t Q, int R, int sbytes, bool compact)
{
    LeadingPlan pl;
    if (plan_leading(P, Q, R, sbytes, tuning_for(compact), pl) != MTTKRP_OK)
        return (size_t)-1;
    return pl.ws_bytes;
}
template <typename T>
int mttkrp_dense_run(int ndim, const int64_t* dims, const T* X, const T* const* factors, int R, int k, T* M, void* workspace,
                     size_t workspace_bytes, void* stream, bool compact)
{
    return run<T>(ndim, dims, X, factors, R, k, M, workspace, workspace_bytes, false, stream, nullptr, 0.0, nullptr, 0, true, compact);
}
template <typename T>
int mttkrp_leading_run(int64_t P, int64_t Q, const T* X, const T* K, int R, T* out, void* workspace, size_t workspace_bytes,
                       void* stream, bool compact)
{
    return run_leading<T>(P, Q, X, K, R, R, out, R, workspace, workspace_bytes, stream, compact);
}
template int mttkrp_dense_run<double>(int, const int64_t*, const double*, const double* const*, int, int, double*, void*, size_t, void*, bool);
template int mttkrp_dense_run<float>(int, const int64_t*, const float*, const float* const*, int, int, float*, void*, size_t, void*, bool);
template int mttkrp_leading_run<double>(int64_t, int64_t, const double*, const double*, int, double*, void*, size_t, void*, bool);
template int mttkrp_leading_run<float>(int64_t, int64_t, const float*, const float*, int, float*, void*, size_t, void*, bool);

extern "C" {

int mttkrp_dense_f64_noalloc(int ndim, const int64_t* dims, const double* X, const double* const* factors,
                             int R, int k, double* M, void* stream)
{
    void* const ptr = scratch_address();
    if (!ptr)
        return MTTKRP_ERR_DEVICE;
    // the kernels get the looked-up device address as their workspace, exactly as they get a
    // caller's buffer in mttkrp_dense_f64_ws; a plan that needs more is rejected there
    return run<double>(ndim, dims, X, factors, R, k, M, ptr, (size_t)MTTKRP_NOALLOC_SCRATCH_BYTES, false, stream,
                       nullptr, 0.0, nullptr, 0, false);
}

int mttkrp_dense_f64(int ndim, const int64_t* dims, const double* X, const double* const* factors,
                     int R, int k, double* M, void* stream)
{
    return run<double>(ndim, dims, X, factors, R, k, M, nullptr, 0, true, stream);
}

int mttkrp_dense_f32(int ndim, const int64_t* dims, const float* X, const float* const* factors,
                     int R, int k, float* M, void* stream)
{
    return run<float>(ndim, dims, X, factors, R, k, M, nullptr, 0, true, stream);
}

size_t mttkrp_dense_workspace_bytes(int ndim, const int64_t* dims, int R, int k, int dtype_bytes)
{
    return mttkrp_dense_bytes(ndim, dims, R, k, dtype_bytes, false);
}

int mttkrp_dense_f64_ws(int ndim, const int64_t* dims, const double* X,
                        const double* const* factors, int R, int k, double* M, void* workspace,
                        size_t workspace_bytes, void* stream)
{
    return run<double>(ndim, dims, X, factors, R, k, M, workspace, workspace_bytes, false, stream);
}

int mttkrp_dense_f32_ws(int ndim, const int64_t* dims, const float* X, const float* const* factors,
                        int R, int k, float* M, void* workspace, size_t workspace_bytes,
                        void* stream)
{
    return run<float>(ndim, dims, X, factors, R, k, M, workspace, workspace_bytes, false, stream);
}

size_t mttkrp_dense_ex_workspace_bytes(int ndim, const int64_t* dims, int R, int k, int dtype_bytes)
{
    Plan pl;
    if (make_plan(ndim, dims, R, k, dtype_bytes, pl) != MTTKRP_OK)
        return (size_t)-1;
    const size_t part = pl.part_bytes > 0 ? pl.part_bytes : (size_t)pl.dims[pl.k] * (size_t)R * (size_t)dtype_bytes;
    const size_t bytes = (part + 255) / 256 * 256 + pl.fused_bytes;
    return bytes > pl.ws_bytes ? bytes : pl.ws_bytes;
}

int mttkrp_dense_f64_ex(int ndim, const int64_t* dims, const double* X,
                        const double* const* factors, int R, int k, const double* lambda,
                        double beta, double* M, void* workspace, size_t workspace_bytes,
                        void* stream)
{
    return run<double>(ndim, dims, X, factors, R, k, M, workspace, workspace_bytes,
                       workspace == nullptr, stream, lambda, beta);
}

int mttkrp_dense_f32_ex(int ndim, const int64_t* dims, const float* X, const float* const* factors,
                        int R, int k, const float* lambda, float beta, float* M, void* workspace,
                        size_t workspace_bytes, void* stream)
{
    return run<float>(ndim, dims, X, factors, R, k, M, workspace, workspace_bytes,
                      workspace == nullptr, stream, lambda, (double)beta);
}

int mttkrp_dense_f64_ld(int ndim, const int64_t* dims, const double* X, const double* const* factors,
                        const int64_t* ld_factors, int R, int k, const double* lambda, double beta,
                        double* M, int64_t ldM, void* workspace, size_t workspace_bytes, void* stream)
{
    if (!ld_factors)
        return MTTKRP_ERR_INVALID_ARG;
    return run<double>(ndim, dims, X, factors, R, k, M, workspace, workspace_bytes,
                       workspace == nullptr, stream, lambda, beta, ld_factors, ldM);
}

int mttkrp_dense_f32_ld(int ndim, const int64_t* dims, const float* X, const float* const* factors,
                        const int64_t* ld_factors, int R, int k, const float* lambda, float beta,
                        float* M, int64_t ldM, void* workspace, size_t workspace_bytes, void* stream)
{
    if (!ld_factors)
        return MTTKRP_ERR_INVALID_ARG;
    return run<float>(ndim, dims, X, factors, R, k, M, workspace, workspace_bytes,
                      workspace == nullptr, stream, lambda, (double)beta, ld_factors, ldM);
}

size_t mttkrp_contract_leading_workspace_bytes(int64_t P, int64_t Q, int R, int dtype_bytes)
{
    return mttkrp_leading_bytes(P, Q, R, dtype_bytes, false);
}

int mttkrp_contract_leading_f64(int64_t P, int64_t Q, const double* X, const double* K, int64_t ldK, int R,
                                double* T_out, int64_t ldT, void* workspace, size_t workspace_bytes, void* stream)
{
    return run_leading<double>(P, Q, X, K, ldK, R, T_out, ldT, workspace, workspace_bytes, stream);
}

int mttkrp_contract_leading_f32(int64_t P, int64_t Q, const float* X, const float* K, int64_t ldK, int R,
                                float* T_out, int64_t ldT, void* workspace, size_t workspace_bytes, void* stream)
{
    return run_leading<float>(P, Q, X, K, ldK, R, T_out, ldT, workspace, workspace_bytes, stream);
}

const char* mttkrp_status_string(int status)
{
    switch (status) {
    case MTTKRP_OK: return "ok";
    case MTTKRP_ERR_INVALID_ARG: return "invalid argument";
    case MTTKRP_ERR_UNSUPPORTED: return "unsupported size or number of modes";
    case MTTKRP_ERR_WORKSPACE: return "workspace too small or misaligned";
    case MTTKRP_ERR_DEVICE: return "HIP runtime call failed";
    case MTTKRP_ERR_NUMERICAL: return "numerical breakdown (a matrix that must be positive definite is not)";
    default: return "unknown status";
    }
}

int mttkrp_version(void) { return 100; }

void mttkrp_release(void)
{
    std::lock_guard<std::mutex> lock(g_mutex);
    int cur = 0;
    if (hipGetDevice(&cur) != hipSuccess)
        return;
    for (int d = 0; d < kMaxDevices; ++d) {
        DeviceState& ds = g_dev[d];
        bool any = ds.calls != nullptr;
        for (int i = 0; i < kOwnedSlots; ++i)
            any = any || ds.own[i].ws || ds.own[i].done;
        if (!any)
            continue;
        if (hipSetDevice(d) != hipSuccess)
            continue;
        (void)hipDeviceSynchronize();
        for (int i = 0; i < kOwnedSlots; ++i) {
            OwnedWorkspace& o = ds.own[i];
            if (o.ws)
                (void)hipFree(o.ws);
            if (o.done)
                (void)hipEventDestroy(o.done);
            o = OwnedWorkspace();
        }
        if (ds.calls) {
            for (int c = 0; c < kTimingSlots; ++c)
                for (int e = 0; e < 3; ++e)
                    (void)hipEventDestroy(ds.calls[c].ev[e]);
            delete[] ds.calls;
        }
        ds.calls = nullptr;
        ds.n_timed = 0;
        ds.record = false;
    }
    (void)hipSetDevice(cur);
}

int mttkrp_timing_enable(int enable)
{
    std::lock_guard<std::mutex> lock(g_mutex);
    g_timing = enable != 0;
    if (g_timing)
        for (int d = 0; d < kMaxDevices; ++d)
            g_dev[d].n_timed = 0;
    return MTTKRP_OK;
}

int64_t mttkrp_timing_count(void)
{
    int dev = 0;
    if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= kMaxDevices)
        return 0;
    std::lock_guard<std::mutex> lock(g_mutex);
    return g_dev[dev].n_timed;
}

int mttkrp_timing_get(int64_t index, float* stream_ms, float* combine_ms)
{
    if (!stream_ms || !combine_ms)
        return MTTKRP_ERR_INVALID_ARG;
    int dev = 0;
    if (hipGetDevice(&dev) != hipSuccess)
        return MTTKRP_ERR_DEVICE;
    if (dev < 0 || dev >= kMaxDevices)
        return MTTKRP_ERR_UNSUPPORTED;
    std::lock_guard<std::mutex> lock(g_mutex);
    DeviceState& ds = g_dev[dev];
    if (!ds.calls || index < 0 || index >= ds.n_timed || index < ds.n_timed - kTimingSlots)
        return MTTKRP_ERR_INVALID_ARG;
    TimedCall& tc = ds.calls[index % kTimingSlots];
    *combine_ms = 0.0f;
    if (hipEventSynchronize(tc.combine ? tc.ev[2] : tc.ev[1]) != hipSuccess)
        return MTTKRP_ERR_DEVICE;
    if (hipEventElapsedTime(stream_ms, tc.ev[0], tc.ev[1]) != hipSuccess)
        return MTTKRP_ERR_DEVICE;
    if (tc.combine && hipEventElapsedTime(combine_ms, tc.ev[1], tc.ev[2]) != hipSuccess)
        return MTTKRP_ERR_DEVICE;
    return MTTKRP_OK;
}

int mttkrp_timing_last(float* stream_ms, float* combine_ms)
{
    return mttkrp_timing_get(mttkrp_timing_count() - 1, stream_ms, combine_ms);
}

int mttkrp_tune_set(const char* key, int64_t value)
{
    if (!key || value < 0)
        return MTTKRP_ERR_INVALID_ARG;
    std::lock_guard<std::mutex> lock(g_mutex);
    if (!strcmp(key, "row_blocks")) {
        if (value > 4) return MTTKRP_ERR_INVALID_ARG;
        g_tune.row_blocks = value;
    } else if (!strcmp(key, "target_items")) {
        g_tune.target_items = value;
    } else if (!strcmp(key, "max_steps")) {
        g_tune.max_steps = value;
    } else if (!strcmp(key, "xcd_remap")) {
        if (value > 2) return MTTKRP_ERR_INVALID_ARG;
        g_tune.xcd_remap = value;
    } else if (!strcmp(key, "max_col_blocks")) {
        if (value > 8) return MTTKRP_ERR_INVALID_ARG;
        g_tune.max_col_blocks = value;
    } else if (!strcmp(key, "first_group")) {
        if (value != 0 && value != 1 && value != 4) return MTTKRP_ERR_INVALID_ARG;
        g_tune.first_group = value;
    } else if (!strcmp(key, "waves_per_simd")) {
        if (value > 8) return MTTKRP_ERR_INVALID_ARG;
        g_tune.waves_per_simd = value;
    } else if (!strcmp(key, "small_route")) {
        if (value > 2) return MTTKRP_ERR_INVALID_ARG;
        g_tune.small_route = value;
    } else if (!strcmp(key, "lds_contract")) {
        if (value > 2) return MTTKRP_ERR_INVALID_ARG;
        g_tune.lds_contract = value;
    } else if (!strcmp(key, "small_groups")) {
        if (value > 1024) return MTTKRP_ERR_INVALID_ARG;
        g_tune.small_groups = value;
    } else if (!strcmp(key, "lead_last")) {
        if (value > 2) return MTTKRP_ERR_INVALID_ARG;
        g_tune.lead_last = value;
    } else if (!strcmp(key, "fuse_rows")) {
        if (value > 2) return MTTKRP_ERR_INVALID_ARG;
        g_tune.fuse_rows = value;
    } else if (!strcmp(key, "pair_rows")) {
        if (value > 2) return MTTKRP_ERR_INVALID_ARG;
        g_tune.pair_rows = value;
    } else if (!strcmp(key, "fuse_bytes")) {
        g_tune.fuse_bytes = value;
    } else if (!strcmp(key, "rows_col_blocks")) {
        if (value > 4) return MTTKRP_ERR_INVALID_ARG;
        g_tune.rows_col_blocks = value;
    } else if (!strcmp(key, "contract_rows")) {
        if (value > 2) return MTTKRP_ERR_INVALID_ARG;
        g_tune.contract_rows = value;
    } else if (!strcmp(key, "inner_splits")) {
        if (value > 64) return MTTKRP_ERR_INVALID_ARG;
        g_tune.inner_splits = value;
    } else if (!strcmp(key, "linear")) {
        if (value > 2) return MTTKRP_ERR_INVALID_ARG;
        g_tune.linear = value;
    } else if (!strcmp(key, "deep")) {
        if (value > 2) return MTTKRP_ERR_INVALID_ARG;
        g_tune.deep = value;
    } else if (!strcmp(key, "nt_loads")) {
        if (value > 1) return MTTKRP_ERR_INVALID_ARG;
        g_tune.nt_loads = value;
    } else if (!strcmp(key, "ws_percent")) {
        if (value > 100) return MTTKRP_ERR_INVALID_ARG;
        g_tune.ws_percent = value;
    } else {
        return MTTKRP_ERR_INVALID_ARG;
    }
    return MTTKRP_OK;
}

int mttkrp_plan_describe(int ndim, const int64_t* dims, int R, int k, int dtype_bytes, char* buf,
                         size_t buflen)
{
    if (!buf || buflen == 0)
        return MTTKRP_ERR_INVALID_ARG;
    buf[0] = 0;
    Plan pl;
    int rc = make_plan(ndim, dims, R, k, dtype_bytes, pl);
    if (rc != MTTKRP_OK)
        return rc;
    // small tensors: the line of the general decomposition, then what runs instead of it
    if (pl.small) {
        const int used = snprintf(buf, buflen, "small_route=1 small_rows=%d small_groups=%d small_waves=%d small_steps=%d | ",
                                  16 * pl.sp.RB, pl.sp.n_groups, pl.sp.waves, pl.sp.cols_per_range / 4);
        if (used < 0 || (size_t)used >= buflen)
            return MTTKRP_OK;
        buf += used;
        buflen -= (size_t)used;
    }
    if (pl.lead_route) {
        snprintf(buf, buflen,
                 "shape=leading P=%lld Q=%lld cols_per_wave=%d col_blocks=%d j_chunks=%d row_splits=%d "
                 "items=%lld steps_per_item=%lld slots=%lld ws_bytes=%zu fused_modes=-1 fused_rows=0 fused_bytes=%zu "
                 "paired_rows=0",
                 (long long)pl.lead_P, (long long)pl.lead_Q, 16 * pl.lead.CB, pl.lead.JB, pl.lead.n_jchunk,
                 pl.lead.n_rsplit, (long long)pl.n_items, (long long)pl.steps_per_item, (long long)pl.n_slots,
                 pl.ws_bytes, pl.fused_bytes);
        return MTTKRP_OK;
    }
    if (pl.contract_rows) {
        snprintf(buf, buflen,
                 "shape=rows cols_per_wave=%d col_chunks=%d col_blocks=%d j_chunks=%d batch=%d "
                 "row_splits=%d outer_splits=1 inner_splits=1 "
                 "items=%lld steps_per_item=%lld slots=%lld ws_bytes=%zu fused_modes=-1 fused_rows=0 fused_bytes=%zu "
                 "lds=%d segments=%d",
                 16 * pl.CB, pl.n_cchunk, pl.JB, pl.n_jchunk, pl.n_batch, pl.n_rsplit, (long long)pl.n_items,
                 (long long)pl.steps_per_item, (long long)pl.n_slots, pl.ws_bytes, pl.fused_bytes, pl.cp.ok ? 1 : 0,
                 pl.cp.ok ? pl.cp_segs : 0);
        return MTTKRP_OK;
    }
    snprintf(buf, buflen,
             "shape=%s rows_per_wave=%d row_blocks=%d col_blocks=%d j_chunks=%d inner_mode=%d "
             "outer_modes=%d batch=%d o_per_item=%lld outer_splits=%lld inner_splits=%d "
             "items=%lld steps_per_item=%lld slots=%lld ws_bytes=%zu fused_modes=%d fused_rows=%d fused_bytes=%zu "
             "paired_rows=%d deep=%d",
             k == 0 ? "first" : (k == ndim - 1 ? "last" : "middle"), 16 * pl.RB, pl.n_rowblk,
             pl.JB, pl.n_jchunk, pl.inner, pl.n_out, pl.n_batch, (long long)pl.o_per_item,
             (long long)pl.n_osplit, pl.n_isplit, (long long)pl.n_items,
             (long long)pl.steps_per_item, (long long)pl.n_slots, pl.ws_bytes,
             pl.fuse_a >= 0 ? pl.orig[pl.fuse_a] : -1, pl.n_fuse > 0 && pl.fus[0].red == 0 ? 1 : 0, pl.fused_bytes,
             pl.seg > 0 ? (pl.seg_store ? 3 : (pl.seg_first ? 2 : 1)) : 0, pl.deep ? 1 : 0);
    return MTTKRP_OK;
}

}  // extern "C"
