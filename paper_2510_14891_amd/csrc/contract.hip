// Contraction over the leading index:  S(c, j) = sum_r X(r, c) K(r, j),  X as a P x Q matrix, first index fastest.
//
// The operand that the MFMAs need (16 columns of X side by side, four rows apart) lies across memory.
// mttkrp_rowsum_kernel loads it directly: a wavefront reads 16 CB columns in pieces of 128 bytes, holds one tile for a
// whole column, drains between tiles, and reads K for itself.  Here a workgroup of eight wavefronts (four from three
// blocks of output columns on) walks 128 (64) columns in stages of 256 bytes per column (32 fp64 or 64 fp32 rows): its
// threads load whole 256-byte pieces (16 lanes each), keep two stages in registers on their way, and pass them through
// LDS, K's rows beside them, so that K is read once per workgroup.  Workgroups are persistent and the loads of the next
// tile start while the last stages of a tile are consumed, so short columns cost no drain.
//
// What bounds it: at R <= 16 HBM; fp64 at R = 32 reads 5.0 TB/s beside 40 TFLOP/s of the matrix cores (72 in a large product),
// and neither goes faster beside the other.  Against mttkrp_rowsum_kernel, 20 to 80 calls in a row: 1024 x 524288 (4.3 GB) 0.863 ->
// 0.777 ms at R = 8 (5.5 TB/s), 0.954 -> 0.866 at R = 32; 16641 x 60372 (8 GB) at R = 10 1.63 -> 1.37; 10^6 x 400, fp32, R = 32 0.410 ->
// 0.409.  The barrier before a stage's last quarter instead of at its end, where all wavefronts waited for LDS at once: 70
// contractions 0.98 times as long in the mean (the last of these 0.425 -> 0.409, 1024 x 524288 at R = 32 0.875 -> 0.866).
#include "mttkrp_contract.h"

#include <math.h>

namespace {

typedef double double2_t __attribute__((ext_vector_type(2)));
typedef double double4_t __attribute__((ext_vector_type(4)));
typedef float float4_t __attribute__((ext_vector_type(4)));

template <typename T> struct Types;
template <> struct Types<double> {
    typedef double4_t acc_t;
    typedef double2_t piece_t;                 // 16 bytes
    static __device__ __forceinline__ acc_t mfma(double a, double b, acc_t c) { return __builtin_amdgcn_mfma_f64_16x16x4f64(a, b, c, 0, 0, 0); }
    static __device__ __forceinline__ int row(int lane, int q) { return 4 * q + (lane >> 4); }
};
template <> struct Types<float> {
    typedef float4_t acc_t;
    typedef float4_t piece_t;
    static __device__ __forceinline__ acc_t mfma(float a, float b, acc_t c) { return __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, 0, 0, 0); }
    static __device__ __forceinline__ int row(int lane, int q) { return 4 * (lane >> 4) + q; }
};

constexpr int kPieces = 16;                    // 16-byte pieces of a column per stage

// 16 bytes from memory that is only aligned to a value
template <typename T> __device__ __forceinline__ typename Types<T>::piece_t load_piece(const T* p)
{
    typename Types<T>::piece_t v;
    __builtin_memcpy(&v, p, 16);
    return v;
}

template <typename T, int JB, int CW, bool CHAINS>
__global__ void __launch_bounds__(64 * CW, CW == 4 && JB <= 2 ? 3 : 2) mttkrp_contract_kernel(const ContractArgs<T> p)
{
    typedef Types<T> TT;
    typedef typename TT::acc_t acc_t;
    typedef typename TT::piece_t piece_t;
    constexpr int THREADS = 64 * CW;
    constexpr int kCols = 16 * CW;             // tensor columns of the workgroup
    constexpr int G = 16 / (int)sizeof(T);     // values per piece
    constexpr int SR = kPieces * G;            // rows per stage
    constexpr int NC = 16 * JB;                // output columns of the workgroup
    constexpr int KP = NC / G;                 // pieces per row of K
    constexpr int XL = kCols * kPieces / THREADS, KN = SR * KP, KL = (KN + THREADS - 1) / THREADS;   // pieces a thread loads per stage
    extern __shared__ __align__(16) unsigned char lds_raw[];
    piece_t* const Xs = reinterpret_cast<piece_t*>(lds_raw);                         // [2][column][piece ^ (column & 15)]
    T* const Ks = reinterpret_cast<T*>(lds_raw + 2 * kCols * kPieces * 16);          // [2][row][NC]

    const int tid = (int)threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int cw = wave, il = lane & 15, kq = lane >> 4;
    // contiguous item ranges per XCD: tiles that share the lines at their boundary meet behind one L2
    const int64_t wg = (int64_t)(blockIdx.x & 7) * (gridDim.x >> 3) + (blockIdx.x >> 3);

    struct Item { int64_t c0, r0, r1; int split; };
    auto item_of = [&](int64_t it) {
        Item o;
        const int64_t ct = it % p.n_ctile;
        o.split = (int)(it / p.n_ctile);
        o.c0 = ct * kCols;
        o.r0 = o.split * p.rows_per_split;
        o.r1 = o.split == p.n_rsplit - 1 ? p.P : o.r0 + p.rows_per_split;
        return o;
    };

    // stages of an item (whole ones and one that is shifted back to end with the range: the rows it repeats are masked)
    auto stages_of = [&](const Item& o) { return (int)((o.r1 - o.r0 + SR - 1) / SR); };

    // --- producer: loads of (item, stage), two stages ahead of the consumer
    int64_t p_item = wg, p_row = 0, p_last = 0;
    int p_left = 0;                            // stages of the item not yet requested
    const T* xsrc[XL];
    const T* ksrc[KL];
    auto enter = [&]() {
        const Item o = item_of(p_item);
        p_row = o.r0;
        p_last = o.r1 - SR;
        p_left = stages_of(o);
#pragma unroll
        for (int i = 0; i < XL; ++i) {
            const int id = tid + i * THREADS;
            const int64_t c = o.c0 + (id >> 4) < p.Q ? o.c0 + (id >> 4) : p.Q - 1;     // columns past Q repeat the last one
            xsrc[i] = p.X + c * p.P + (id & 15) * G;
        }
#pragma unroll
        for (int i = 0; i < KL; ++i) {
            const int id = (tid + i * THREADS) % KN, row = id / KP, pc = id % KP;      // (more threads than pieces: some load twice)
            const int j = pc * G;
            ksrc[i] = p.K + (int64_t)row * p.ldK + (j + G <= p.R ? j : p.R - G);       // pieces past R end at R
        }
    };
    // (never skipped: behind a branch the compiler could not tell these loads from the older ones it waits for; past
    // the last item the last stage is read again and dropped)
    auto issue = [&](piece_t (&x)[XL], piece_t (&k)[KL]) {
        const int64_t r = p_left > 1 ? p_row : p_last;
#pragma unroll
        for (int i = 0; i < XL; ++i)
            x[i] = load_piece<T>(xsrc[i] + r);
        const int64_t kr = r * p.ldK;
#pragma unroll
        for (int i = 0; i < KL; ++i)
            k[i] = load_piece<T>(ksrc[i] + kr);
        if (p_left > 1) {
            p_row += SR;
            --p_left;
        } else if (p_item + gridDim.x < p.n_items) {
            p_item += gridDim.x;
            enter();
        }
    };
    auto stash = [&](const piece_t (&x)[XL], const piece_t (&k)[KL], int buf) {
#pragma unroll
        for (int i = 0; i < XL; ++i) {
            const int id = tid + i * THREADS, c = id >> 4;
            Xs[(buf * kCols + c) * kPieces + ((id & 15) ^ (c & 15))] = x[i];
        }
#pragma unroll
        for (int i = 0; i < KL; ++i) {
            const int id = (tid + i * THREADS) % KN;
            reinterpret_cast<piece_t*>(Ks)[(buf * SR * KP) + id] = k[i];
        }
    };

    // --- consumer
    acc_t acc[JB];
    // CHAINS (fp32): after p.chain stages the accumulators go into fp64 sums, so that no chain of fp32 sums is longer than
    // the row splits of the kernel this one replaces, however few its own are
    double sum[CHAINS ? JB : 1][4];
    int chain = p.chain;
    auto clear_acc = [&]() {
#pragma unroll
        for (int jb = 0; jb < JB; ++jb)
            acc[jb] = (acc_t)(0);
        chain = p.chain;
    };
    auto clear = [&]() {
        clear_acc();
        if constexpr (CHAINS) {
#pragma unroll
            for (int jb = 0; jb < JB; ++jb)
#pragma unroll
                for (int q = 0; q < 4; ++q)
                    sum[jb][q] = 0.0;
        }
    };
    auto end_chain = [&]() {
        if constexpr (CHAINS) {
#pragma unroll
            for (int jb = 0; jb < JB; ++jb)
#pragma unroll
                for (int q = 0; q < 4; ++q)
                    sum[jb][q] += (double)acc[jb][q];
            clear_acc();
        }
    };
    // natural output column (inside the workgroup's NC) of block jb in this lane: chunks of G blocks, consecutive
    // columns per lane inside a chunk, so that one LDS read fetches a chunk's entries
    auto natural = [&](int jb) {
        constexpr int last = JB % G;
        const int ch = jb / G, n = ch < JB / G ? G : last;
        return 16 * G * ch + n * il + (jb - G * ch);
    };
    // Operands of quarter t of a stage: a[t], and b[t & 1] (read one quarter ahead of its MFMAs).
    constexpr int NTQ = kPieces / 4;
    static_assert(NTQ == 4, "the order of a stage below");
    piece_t a[NTQ];
    T b[2][G][JB];
    auto read_a = [&](int buf, int t) { a[t] = (Xs + (buf * kCols + 16 * cw + il) * kPieces)[(4 * t + kq) ^ il]; };
    auto read_b = [&](int buf, int t) {
        const T* const kb = Ks + buf * SR * NC;
#pragma unroll
        for (int e = 0; e < G; ++e) {
            const T* const row = kb + ((4 * t + kq) * G + e) * NC;
#pragma unroll
            for (int jb = 0; jb < JB; ++jb)
                b[t & 1][e][jb] = row[natural(jb)];
        }
    };
    // rows below `skip` are masked (zeros for both operands)
    auto multiply = [&](int t, int skip) {
        if (skip > 0) {
#pragma unroll
            for (int e = 0; e < G; ++e) {
                const bool ok = (4 * t + kq) * G + e >= skip;
                a[t][e] = ok ? a[t][e] : (T)0;
#pragma unroll
                for (int jb = 0; jb < JB; ++jb)
                    b[t & 1][e][jb] = ok ? b[t & 1][e][jb] : (T)0;
            }
        }
#pragma unroll
        for (int e = 0; e < G; ++e)
#pragma unroll
            for (int jb = 0; jb < JB; ++jb)
                acc[jb] = TT::mfma(a[t][e], b[t & 1][e][jb], acc[jb]);
    };
    auto store = [&](const Item& o) {
        auto value = [&](int jb, int q) {
            if constexpr (CHAINS)
                return (T)(sum[jb][q] + (double)acc[jb][q]);
            else
                return acc[jb][q];
        };
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            const int64_t c = o.c0 + 16 * cw + TT::row(lane, q);
            if (c < p.Q) {
                T* const dst = p.out + (c * p.n_rsplit + o.split) * p.ld_out;
#pragma unroll
                for (int jb = 0; jb < JB; ++jb) {
                    const int nat = natural(jb), first = nat / G * G;                   // of its piece
                    const int j = (first + G <= p.R ? first : p.R - G) + nat % G;
                    if (j >= first)                                                     // else it belongs to another piece
                        dst[j] = value(jb, q);
                }
            }
        }
    };

    if (wg >= p.n_items)
        return;
    enter();
    Item cur = item_of(wg);
    int64_t c_item = wg;
    int c_left = stages_of(cur);
    piece_t xr[2][XL], kr[2][KL];
    issue(xr[0], kr[0]);
    issue(xr[1], kr[1]);
    stash(xr[0], kr[0], 0);
    __syncthreads();
    clear();
    read_a(0, 0);
    read_b(0, 0);
    // Stage n lies in buffer n & 1, stage n + 1 in register set (n + 1) & 1, stage n + 2 is requested.  LDS is filled and the
    // first operands of the next stage are read while MFMAs of this one run, the barrier lies before its last quarter: at the end of
    // a stage nothing is left to wait for (all wavefronts of a compute unit may be in this one workgroup).  The empty asm keeps
    // the compiler from moving the reads down to their use.
    auto stage = [&](int par) -> bool {
        issue(xr[par], kr[par]);
        const int skip = c_left > 1 ? 0 : (int)(cur.r0 + (int64_t)stages_of(cur) * SR - cur.r1);
        read_a(par, 1);
        read_b(par, 1);
        read_a(par, 2);
        read_a(par, 3);
        asm volatile("" ::: "memory");
        multiply(0, skip);
        read_b(par, 2);
        asm volatile("" ::: "memory");
        multiply(1, skip);
        stash(xr[par ^ 1], kr[par ^ 1], par ^ 1);
        read_b(par, 3);
        asm volatile("" ::: "memory");
        multiply(2, skip);
        __syncthreads();
        read_a(par ^ 1, 0);
        read_b(par ^ 1, 0);
        asm volatile("" ::: "memory");
        multiply(3, skip);
        bool more = true;
        if (--c_left == 0) {
            store(cur);
            clear();
            c_item += gridDim.x;
            more = c_item < p.n_items;
            if (more) {
                cur = item_of(c_item);
                c_left = stages_of(cur);
            }
        } else if (CHAINS && --chain == 0) {
            end_chain();
        }
        return more;
    };
    while (stage(0) && stage(1)) {
    }
}

// part[i_t][segment][R] = this segment's share of  sum_o w(o, j) sum_s S(q, s, j),  w(o, j) = the product of the other modes'
// factor rows: the mode-t result from the contraction over the leading index.  q runs over the modes in `p`
// (lowest fastest), o over all of them but t, s over the row splits of the contraction.  A workgroup owns (i_t, a
// segment of the pairs (o, s), TJ output columns); a thread has JV consecutive columns (the last group ends at R, columns that
// two groups share are stored by the first) and adds the pairs te, te + TE, ... in fp64, then the first wavefront adds the TE
// subtotals, several lanes a column (one lane: 128 dependent additions up to R = 8, 0 to 5 % of a sweep over small tensors).  Decoding a pair takes some fifty instructions: for one column a thread it bounded the kernel, for four
// 16 to 32 bytes come with it (134 MB at R = 32: 46 -> 27 us; 51 MB in fp32 27 -> 14).  Four pairs are requested before the first is added.
template <typename T, typename TP, int TJ, int JV>
__global__ void __launch_bounds__(256) mttkrp_modesum_kernel(const ModeSumArgs<T, TP> p)
{
    constexpr int LJ = TJ / JV, TE = 256 / LJ, U = 4;
    __shared__ double red[TE][TJ + 1];
    const int tj = (int)threadIdx.x % LJ, te = (int)threadIdx.x / LJ;
    const uint32_t it = blockIdx.x;
    const int j = (int)blockIdx.z * TJ + tj * JV, jj = min(j, p.R - JV);
    const uint32_t e0 = blockIdx.y * p.per_seg, e1 = min(p.n_pairs, e0 + p.per_seg);
    auto load = [](const T* src, T (&v)[JV]) { __builtin_memcpy(v, src, sizeof(v)); };     // (rows are only aligned to a value)
    double acc[JV];
#pragma unroll
    for (int c = 0; c < JV; ++c)
        acc[c] = 0.0;
    for (uint32_t e = e0 + te; e < e1; e += U * TE) {
        T v[U][JV];
        double w[U][JV];
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const bool ok = e + u * TE < e1;
            const uint32_t pair = ok ? e + u * TE : e, o = p.n_split > 1 ? pair / p.n_split : pair;
            uint32_t rem = o, q = 0, stride = 1;
#pragma unroll
            for (int c = 0; c < JV; ++c)
                w[u][c] = 1.0;
            for (int m = 0; m < p.n; ++m) {
                if (m == p.t) {
                    q += it * stride;
                } else {
                    const uint32_t d = (uint32_t)p.dim[m], nx = rem / d, im = rem - nx * d;
                    rem = nx;
                    q += im * stride;
                    T a[JV];
                    load(p.A[m] + (int64_t)im * p.ld[m] + jj, a);
#pragma unroll
                    for (int c = 0; c < JV; ++c)
                        w[u][c] *= (double)a[c];
                }
                stride *= (uint32_t)p.dim[m];
            }
            load(p.S + ((int64_t)q * p.n_split + (pair - o * p.n_split)) * p.R + jj, v[u]);
        }
#pragma unroll
        for (int u = 0; u < U; ++u)
#pragma unroll
            for (int c = 0; c < JV; ++c) {
                const double t = (double)v[u][c] * w[u][c];
                acc[c] += e + u * TE < e1 ? t : 0.0;
            }
    }
#pragma unroll
    for (int c = 0; c < JV; ++c)
        red[te][tj * JV + c] = acc[c];
    __syncthreads();
    if (threadIdx.x < 64) {
        constexpr int TG = 64 / TJ;                   // lanes that share a column's subtotals
        const int c = (int)threadIdx.x % TJ, g = (int)threadIdx.x / TJ, first = (int)blockIdx.z * TJ + c / JV * JV;        // of the column's group
        const int col = min(first, p.R - JV) + c % JV;
        double v = 0.0;
#pragma unroll
        for (int q = 0; q < TE / TG; ++q)
            v += red[g * (TE / TG) + q][c];
#pragma unroll
        for (int d = TJ; d < 64; d <<= 1)
            v += __shfl_xor(v, d);
        if (g == 0 && first < p.R && col >= first) {
            p.part[((int64_t)it * gridDim.y + blockIdx.y) * p.ld_part + col] = (TP)v;
        }
    }
}

// The same for many rows with few pairs each and one segment: a thread has a row and JV columns and takes the pairs one after the
// other, four requested at a time and added in four sums; the pair is the same in all threads.  A workgroup of the kernel above would
// leave most of its threads without a pair and wait for their subtotals.  fp64, us, with the sum of one segment that the other needed:
// 43334 rows of 16 pairs at R = 4 99 -> 7.4, 131072 of 4 at R = 8 280 -> 9.8, 20000 of 12 at R = 20 50 -> 10.
template <typename T, typename TP, int JV>
__global__ void __launch_bounds__(256) mttkrp_modesum_rows_kernel(const ModeSumArgs<T, TP> p, int64_t n_threads, uint32_t groups)
{
    constexpr int U = 4;
    const int64_t id = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (id >= n_threads)
        return;
    const uint32_t it = (uint32_t)(id / groups);
    const int j = (int)(id - (int64_t)it * groups) * JV, jj = min(j, p.R - JV);
    auto load = [](const T* src, T (&v)[JV]) { __builtin_memcpy(v, src, sizeof(v)); };
    double acc[U][JV];
#pragma unroll
    for (int u = 0; u < U; ++u)
#pragma unroll
        for (int c = 0; c < JV; ++c)
            acc[u][c] = 0.0;
    for (uint32_t e = 0; e < p.n_pairs; e += U) {
        T v[U][JV];
        double w[U][JV];
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const uint32_t pair = min(e + u, p.n_pairs - 1), o = p.n_split > 1 ? pair / p.n_split : pair;
            uint32_t rem = o, q = 0, stride = 1;
#pragma unroll
            for (int c = 0; c < JV; ++c)
                w[u][c] = 1.0;
            for (int m = 0; m < p.n; ++m) {
                if (m == p.t) {
                    q += it * stride;
                } else {
                    const uint32_t d = (uint32_t)p.dim[m], nx = rem / d, im = rem - nx * d;
                    rem = nx;
                    q += im * stride;
                    T a[JV];
                    load(p.A[m] + (int64_t)im * p.ld[m] + jj, a);
#pragma unroll
                    for (int c = 0; c < JV; ++c)
                        w[u][c] *= (double)a[c];
                }
                stride *= (uint32_t)p.dim[m];
            }
            load(p.S + ((int64_t)q * p.n_split + (pair - o * p.n_split)) * p.R + jj, v[u]);
        }
#pragma unroll
        for (int u = 0; u < U; ++u)
#pragma unroll
            for (int c = 0; c < JV; ++c) {
                const double t = (double)v[u][c] * w[u][c];
                acc[u][c] += e + u < p.n_pairs ? t : 0.0;
            }
    }
#pragma unroll
    for (int c = 0; c < JV; ++c)
        if (jj + c >= j)                              // else it belongs to the group before
            p.part[(int64_t)it * p.ld_part + jj + c] = (TP)((acc[0][c] + acc[1][c]) + (acc[2][c] + acc[3][c]));
}

int lds_bytes(int JB, int CW) { return 2 * (16 * CW * kPieces * 16 + 4096 * JB); }

template <typename T, int JB, int CW, bool CHAINS>
void launch_kernel(const ContractPlan& pl, const ContractArgs<T>& a, hipStream_t st)
{
    const size_t lds = (size_t)lds_bytes(JB, CW);
    if (lds > 65536)
        (void)hipFuncSetAttribute((const void*)mttkrp_contract_kernel<T, JB, CW, CHAINS>, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
    hipLaunchKernelGGL((mttkrp_contract_kernel<T, JB, CW, CHAINS>), dim3((unsigned)pl.grid), dim3(64 * CW), lds, st, a);
}
template <typename T, int JB, int CW>
void launch(const ContractPlan& pl, const ContractArgs<T>& a, hipStream_t st)
{
    // (at two blocks of output columns and four wavefronts the fp64 sums spill: 10^6 x 400 at R = 32 0.356 -> 0.428 ms, the
    // same as with as many more row splits)
    if constexpr (sizeof(T) == 4)
        if (pl.chain > 0)
            return launch_kernel<T, JB, CW, true>(pl, a, st);
    launch_kernel<T, JB, CW, false>(pl, a, st);
}

}  // namespace

ContractPlan mttkrp_contract_plan(int64_t P, int64_t Q, int R, int sbytes, int64_t max_splits, int64_t target_items, int64_t max_rows,
                                  int64_t max_chain)
{
    ContractPlan pl;
    const int G = 16 / sbytes, SR = kPieces * G;
    const int jb_total = (R + 15) / 16;
    // Where it pays (against mttkrp_rowsum_kernel; 2 GB tensors, P = 40 to 400 000, R = 8 to 64): fp64 up to R = 32 from
    // 384 rows on 0.9 to 1.4 times faster (1.12 in the mean; columns that do not begin on lines gain most: 16641 rows
    // 0.468 -> 0.380 ms at R = 16, 2573 rows 0.584 -> 0.426 at R = 32), up to R = 48 only where columns are not
    // line-aligned (1.03 to 1.2; 0.85 to 1.0 aligned), above that the matrix cores bound both and the barriers cost 10 %.
    // fp32 from 256 rows on and up to R = 64 1.02 to 1.5 (16641 rows at R = 16 0.603 -> 0.413 ms).
    const bool unaligned = (P * sbytes) % 128 != 0;
    // Not for fp64 columns of a multiple of 32 KB (4096 x 131072 at R = 32 0.747 -> 0.851 ms, 16384 x 131072 at R = 8 2.77 ->
    // 2.82), which the other kernel streams at 5.7 to 6.2 TB/s.
    const bool power = sbytes == 8 && (P * sbytes) % 32768 == 0;
    if (R < G || Q < 1 || P < (sbytes == 8 ? 384 : 256) || power || jb_total > 4 || (sbytes == 8 && jb_total > (unaligned ? 3 : 2)))
        return pl;
    pl.JB = jb_total;
    // Eight wavefronts (128 columns) share K's rows where registers allow: 2 to 10 % over four at two blocks and fewer,
    // unless the last tile wastes more (10^6 x 400, fp32: 0.425 against 0.370 ms).
    pl.CW = pl.JB <= 2 && (Q + 127) / 128 * 128 <= 1.05 * (double)((Q + 63) / 64 * 64) ? 8 : 4;
    pl.n_ctile = (Q + 16 * pl.CW - 1) / (16 * pl.CW);
    const int64_t slots = 256 * (pl.CW == 8 ? 1 : (pl.JB <= 2 ? 3 : 2));      // two wavefronts per SIMD, or three
    const int64_t stages = (P + SR - 1) / SR;
    if (max_rows <= 0 || max_rows > ((int64_t)1 << 40))
        max_rows = (int64_t)1 << 40;
    if (sbytes == 4 && max_rows > 4096)
        max_rows = 4096;
    if (sbytes == 8 || max_chain <= 0)
        max_chain = max_rows;
    int64_t best = 1;
    if (target_items > 0) {
        best = (target_items + pl.n_ctile - 1) / pl.n_ctile;
    } else {
        // row splits only where the tiles do not fill the resident workgroups evenly, and never more of them (of their
        // partial sums) than the other kernel would make; every split is written and read once more (R / rows of the
        // tensor's bytes, twice), and eight stages are the least an item is worth
        double best_cost = 1e300;
        for (int64_t s = 1; s <= max_splits && s * 8 <= stages + 7; s = s < 16 ? s + 1 : s + s / 8) {
            const int64_t per = (stages + s - 1) / s;
            const double rounds = ceil((double)(pl.n_ctile * s) / (double)slots);
            const double cost = rounds * (double)per * (1.0 + (s > 1 ? 2.0 * (double)s * R / (double)P : 0.0)) + (s > 1 ? 2.0 : 0.0);
            if (cost < best_cost * 0.98) {
                best_cost = cost;
                best = s;
            }
        }
    }
    pl.rows_per_split = (stages + best - 1) / best * SR;
    if (pl.rows_per_split > max_rows) {
        // whole stages, unless that makes more splits (partial sums) than asked for; one stage at least
        pl.rows_per_split = max_rows / SR * SR;
        if (pl.rows_per_split < SR || (P + pl.rows_per_split - 1) / pl.rows_per_split > max_splits)
            pl.rows_per_split = max_rows > SR ? max_rows : SR;
    }
    if (pl.rows_per_split > max_chain && P > max_chain)
        pl.chain = max_chain / SR > 0 ? (int)(max_chain / SR) : 1;
    const int64_t n = (P + pl.rows_per_split - 1) / pl.rows_per_split;
    if (n >= (1 << 20) || pl.n_ctile >= ((int64_t)1 << 31) || pl.n_ctile * n >= ((int64_t)1 << 40))
        return pl;
    pl.n_rsplit = (int)n;
    pl.n_items = pl.n_ctile * n;
    int64_t grid = pl.n_items < slots ? pl.n_items : slots;
    grid = (grid + 7) / 8 * 8;
    pl.grid = (int)grid;
    pl.ok = true;
    return pl;
}

template <typename T> int mttkrp_contract_launch(const ContractPlan& pl, const ContractArgs<T>& a, hipStream_t st)
{
    switch (pl.JB) {
    case 1: pl.CW == 8 ? launch<T, 1, 8>(pl, a, st) : launch<T, 1, 4>(pl, a, st); break;
    case 2: pl.CW == 8 ? launch<T, 2, 8>(pl, a, st) : launch<T, 2, 4>(pl, a, st); break;
    case 3: launch<T, 3, 4>(pl, a, st); break;
    default:
        if constexpr (sizeof(T) == 4) {
            launch<T, 4, 4>(pl, a, st);
            break;
        }
        return MTTKRP_ERR_UNSUPPORTED;
    }
    return hipGetLastError() == hipSuccess ? MTTKRP_OK : MTTKRP_ERR_DEVICE;
}
template int mttkrp_contract_launch<double>(const ContractPlan&, const ContractArgs<double>&, hipStream_t);
template int mttkrp_contract_launch<float>(const ContractPlan&, const ContractArgs<float>&, hipStream_t);

// Where a row's pairs are a thread's: the fewest rows that give every compute unit a wavefront (4096 rows at R = 16 of 16 pairs 16.3 -> 7.2 us, of 64
// 16.1 -> 7.3; 16384 rows of 100 at R = 4 41.9 -> 7.4), and pairs that a thread has in 64 rounds of requests.
constexpr uint32_t kRowPairs = 256;
constexpr int64_t kRowThreads = 16384;
template <typename T, typename TP, int JV> void modesum(const ModeSumArgs<T, TP>& a, int64_t I_t, int n_seg, hipStream_t st)
{
    const int64_t groups = (a.R + JV - 1) / JV, threads = I_t * groups;
    if (n_seg == 1 && a.n_pairs <= kRowPairs && threads >= kRowThreads && threads < ((int64_t)1 << 38)) {
        hipLaunchKernelGGL((mttkrp_modesum_rows_kernel<T, TP, JV>), dim3((unsigned)((threads + 255) / 256)), dim3(256), 0, st, a, threads,
                           (uint32_t)groups);
        return;
    }
    if (a.R > 16)
        hipLaunchKernelGGL((mttkrp_modesum_kernel<T, TP, 32, JV>), dim3((unsigned)I_t, (unsigned)n_seg, (unsigned)((a.R + 31) / 32)), dim3(256), 0, st, a);
    else if (a.R > 8)
        hipLaunchKernelGGL((mttkrp_modesum_kernel<T, TP, 16, JV>), dim3((unsigned)I_t, (unsigned)n_seg, 1), dim3(256), 0, st, a);
    else
        hipLaunchKernelGGL((mttkrp_modesum_kernel<T, TP, 8, JV>), dim3((unsigned)I_t, (unsigned)n_seg, 1), dim3(256), 0, st, a);
}
template <typename T, typename TP> int mttkrp_modesum_launch(const ModeSumArgs<T, TP>& a, int64_t I_t, int n_seg, hipStream_t st)
{
    if (a.R >= 4)
        modesum<T, TP, 4>(a, I_t, n_seg, st);
    else
        modesum<T, TP, 1>(a, I_t, n_seg, st);
    return hipGetLastError() == hipSuccess ? MTTKRP_OK : MTTKRP_ERR_DEVICE;
}
template int mttkrp_modesum_launch<double, double>(const ModeSumArgs<double, double>&, int64_t, int, hipStream_t);
template int mttkrp_modesum_launch<float, float>(const ModeSumArgs<float, float>&, int64_t, int, hipStream_t);
template int mttkrp_modesum_launch<float, double>(const ModeSumArgs<float, double>&, int64_t, int, hipStream_t);
