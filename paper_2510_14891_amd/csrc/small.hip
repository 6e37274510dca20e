// MTTKRP in one launch, for tensors so small that a call is bound by launches and by latency.
//
//   M(n, j) = sum_{i: i_k = n} X(i) prod_{m != k} A_m(i_m, j)          (paper Sec. II-B, Eq. (elem))
//
// The streaming kernel (mttkrp.hip) spreads one output row over many workgroups and adds up their partial
// sums in a second launch; each launch takes about 4 us whatever it does, and its items of 16 steps and more
// leave most of the chip idle on a 2 MB tensor.  Here a workgroup owns whole output rows: one i_k (k != 0) or 16
// rows of mode 0 (k = 0).  Its up to 16 wavefronts take pieces of the column space (and row tiles), keep their
// sums in MFMA accumulators and add them up in LDS in a fixed order; weights and accumulation are applied on the way
// out.  With few output rows several workgroups share a row's columns, leave partial sums in a workspace, and the combine kernel
// adds them in a second launch (two launches instead of three).
//
// Columns are decoded by every lane for itself (a multiply-high per mode above the lowest): that hides
// behind the loads, and short modes need no fused product matrices.  fp64, us a call, before and now: 64^3 at R = 16 15.7 /
// 8.4 / 8.4 -> 8.3 / 5.1 / 5.0; 100 x 80 x 60 at R = 10, CP-ALS, 12 sweeps 1482 -> 1190; 4947 calls that take it 0.55 times as
// long in the mean.  mttkrp.hip says where the line between the two paths lies.
#include "mttkrp_small.h"

namespace {

typedef double double4_t __attribute__((ext_vector_type(4)));
typedef float float4_t __attribute__((ext_vector_type(4)));

template <typename T> struct Mfma;
template <> struct Mfma<double> {
    typedef double4_t acc_t;
    static __device__ __forceinline__ acc_t run(double a, double b, acc_t c) { return __builtin_amdgcn_mfma_f64_16x16x4f64(a, b, c, 0, 0, 0); }
    static __device__ __forceinline__ int row(int lane, int q) { return 4 * q + (lane >> 4); }
};
template <> struct Mfma<float> {
    typedef float4_t acc_t;
    static __device__ __forceinline__ acc_t run(float a, float b, acc_t c) { return __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, 0, 0, 0); }
    static __device__ __forceinline__ int row(int lane, int q) { return 4 * (lane >> 4) + q; }
};

// steps (of four columns) whose loads are in flight together
template <int RB, int JB> constexpr int kSteps = RB * JB <= 2 ? 8 : 4;

// Output columns of a lane, as in the streaming kernel: JB consecutive ones, so that one wide load (two for more
// than 16 bytes) fetches its entries of a factor row.  A group that would cross R is moved back to end at R and
// stores only the columns it owns.
template <typename T, int N> struct Lay {
    static constexpr int G = 16 / (int)sizeof(T);
    static constexpr int n0 = N < G ? N : G;
    static constexpr int n1 = N - n0;
};

// NM: column modes (1 or 2), 0: any number.
template <typename T, int RB, int JB, int NM, bool FIRST>
__global__ void __launch_bounds__(64 * kSmallWaves) mttkrp_small_kernel(const SmallArgs<T> p)
{
    typedef Mfma<T> MF;
    typedef typename MF::acc_t acc_t;
    typedef Lay<T, JB> LC;
    constexpr int U = kSteps<RB, JB>;
    extern __shared__ double red[];
    const int lane = (int)threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    const int n_waves = (int)(blockDim.x >> 6);
    const int il = lane & 15, kk = lane >> 4;
    const int R = p.R, j_first = (int)blockIdx.y * 16 * JB;
    const int jt0 = j_first + LC::n0 * il, jt1 = j_first + 16 * LC::n0 + LC::n1 * il;
    const int js0 = min(jt0, R - LC::n0), js1 = LC::n1 > 0 ? min(jt1, R - LC::n1) : 0;
    auto column = [&](int jb) { return jb < LC::n0 ? js0 + jb : js1 + (jb - LC::n0); };
    auto owned = [&](int jb) { return jb < LC::n0 ? column(jb) >= jt0 : column(jb) >= jt1; };
    // (the first entry's address is formed before the others are counted from it: a 32-bit index for each of them could
    // wrap as far as the compiler knows, and they stay separate loads)
    auto load_cols = [&](const T* a, uint32_t off, T (&v)[JB]) {
        const T* const a0 = a + (off + (uint32_t)js0);
#pragma unroll
        for (int jb = 0; jb < LC::n0; ++jb)
            v[jb] = a0[jb];
        if constexpr (LC::n1 > 0) {
            const T* const a1 = a + (off + (uint32_t)js1);
#pragma unroll
            for (int jb = 0; jb < LC::n1; ++jb)
                v[LC::n0 + jb] = a1[jb];
        }
    };
    const T* const xb = FIRST ? p.X : p.X + (int64_t)blockIdx.x * p.sx_batch;
    const int g0 = (int)blockIdx.z * p.cols_per_group, g1 = min(p.C, g0 + p.cols_per_group);   // this group's columns

    acc_t acc[RB][JB];
    // acc = X(rows row0 .., columns [c0, c1)) * Khatri-Rao rows.  Lanes past c1 enter zeros for both operands (exact
    // zeros whatever the tensor holds), rows past I_0 repeat the last one and are dropped by the caller.
    auto sweep = [&](int row0, int c0, int c1) {
#pragma unroll
        for (int r = 0; r < RB; ++r)
#pragma unroll
            for (int jb = 0; jb < JB; ++jb)
                acc[r][jb] = (acc_t)(0);
        uint32_t row[RB];
#pragma unroll
        for (int r = 0; r < RB; ++r)
            row[r] = (uint32_t)min(row0 + 16 * r + il, p.I0 - 1);
        auto batch = [&](int c, bool masked) {
            T xs[U][RB], bs[U][JB];
#pragma unroll
            for (int u = 0; u < U; ++u) {
                uint32_t rem = (uint32_t)(c + 4 * u + kk);
                if (masked)
                    rem = min(rem, (uint32_t)(c1 - 1));
                uint32_t off = 0;
                auto mode = [&](int m, bool last, bool first) {
                    uint32_t i = rem;
                    if (!last && p.dim[m] > 1) {
                        const uint32_t q = __umulhi(rem, p.magic[m]) >> p.shift[m];
                        i = rem - q * (uint32_t)p.dim[m];
                        rem = q;
                    } else if (!last) {
                        i = 0;
                    }
                    off += i * (uint32_t)p.sx[m];
                    T v[JB];
                    load_cols(p.A[m], i * (uint32_t)p.ld[m], v);
#pragma unroll
                    for (int jb = 0; jb < JB; ++jb)
                        bs[u][jb] = first ? v[jb] : bs[u][jb] * v[jb];
                };
                if constexpr (NM == 1) {
                    mode(0, true, true);
                } else if constexpr (NM == 2) {
                    mode(0, false, true);
                    mode(1, true, false);
                } else {
#pragma unroll
                    for (int jb = 0; jb < JB; ++jb)
                        bs[u][jb] = (T)1;
#pragma unroll
                    for (int m = 0; m < kSmallModes; ++m)
                        if (m < p.n)
                            mode(m, m == p.n - 1, false);
                }
#pragma unroll
                for (int r = 0; r < RB; ++r)
                    xs[u][r] = xb[off + row[r]];
            }
            if (masked) {
#pragma unroll
                for (int u = 0; u < U; ++u) {
                    const bool ok = c + 4 * u + kk < c1;
#pragma unroll
                    for (int r = 0; r < RB; ++r)
                        xs[u][r] = ok ? xs[u][r] : (T)0;
#pragma unroll
                    for (int jb = 0; jb < JB; ++jb)
                        bs[u][jb] = ok ? bs[u][jb] : (T)0;
                }
            }
#pragma unroll
            for (int u = 0; u < U; ++u)
#pragma unroll
                for (int r = 0; r < RB; ++r)
#pragma unroll
                    for (int jb = 0; jb < JB; ++jb)
                        acc[r][jb] = MF::run(xs[u][r], bs[u][jb], acc[r][jb]);
        };
        int c = c0;
        for (; c + 4 * U <= c1; c += 4 * U)
            batch(c, false);
        if (c < c1)
            batch(c, true);
    };
    auto store = [&](int64_t row, int j, double v) {
        if (gridDim.z > 1) {       // the combine kernel applies weights and accumulation
            p.out[(int64_t)blockIdx.z * p.group_stride + row * p.row_stride + j] = (T)v;
            return;
        }
        if (p.lambda)
            v *= (double)p.lambda[j];
        T* const o = p.out + row * p.ld_out + j;
        if (p.beta != 0.0)
            v += p.beta * (double)*o;
        *o = (T)v;
    };

    if constexpr (FIRST) {
        // one row tile; wavefront w holds the sum over piece w of the group's columns
        const int row0 = (int)blockIdx.x * 16;
        const int c0 = g0 + wave * p.cols_per_range;
        sweep(row0, c0, min(g1, c0 + p.cols_per_range));
#pragma unroll
        for (int jb = 0; jb < JB; ++jb) {
            if (jb > 0)
                __syncthreads();
#pragma unroll
            for (int q = 0; q < 4; ++q)
                red[wave * 256 + MF::row(lane, q) * 16 + il] = (double)acc[0][jb][q];
            __syncthreads();
            for (int t = (int)threadIdx.x; t < 256; t += (int)blockDim.x) {
                // (entry t & 15 belongs to lane t & 15 of the layout above: this thread's own il)
                const int r = row0 + (t >> 4);
                double v = 0.0;
                for (int w = 0; w < n_waves; ++w)
                    v += red[w * 256 + t];
                if (r < p.I0 && owned(jb))
                    store(r, column(jb), v);
            }
        }
    } else {
        // every (row tile, piece of the columns): weighted with A_0 and summed over the rows
        double v[JB];
#pragma unroll
        for (int jb = 0; jb < JB; ++jb)
            v[jb] = 0.0;
        for (int u = wave; u < p.n_tiles * p.n_ranges; u += n_waves) {
            const int rng = u / p.n_tiles, row0 = (u - rng * p.n_tiles) * 16 * RB;
            T w[RB][4][JB];          // under way before the sweep
#pragma unroll
            for (int r = 0; r < RB; ++r)
#pragma unroll
                for (int q = 0; q < 4; ++q)
                    load_cols(p.A0, (uint32_t)min(row0 + 16 * r + MF::row(lane, q), p.I0 - 1) * (uint32_t)p.ld0, w[r][q]);
            const int c0 = g0 + rng * p.cols_per_range;
            sweep(row0, c0, min(g1, c0 + p.cols_per_range));
#pragma unroll
            for (int r = 0; r < RB; ++r)
#pragma unroll
                for (int q = 0; q < 4; ++q) {
                    const bool in = row0 + 16 * r + MF::row(lane, q) < p.I0;
#pragma unroll
                    for (int jb = 0; jb < JB; ++jb) {
                        const double t = (double)acc[r][jb][q] * (double)w[r][q][jb];
                        v[jb] += in ? t : 0.0;
                    }
                }
        }
#pragma unroll
        for (int jb = 0; jb < JB; ++jb) {
            double t = v[jb];
            t += __shfl_xor(t, 16);
            t += __shfl_xor(t, 32);
            if (kk == 0)
                red[wave * (16 * JB) + 16 * jb + il] = t;
        }
        __syncthreads();
        if (wave == 0 && kk == 0) {
#pragma unroll
            for (int jb = 0; jb < JB; ++jb) {
                double t = 0.0;
                for (int w = 0; w < n_waves; ++w)
                    t += red[w * (16 * JB) + 16 * jb + il];
                if (owned(jb))
                    store((int64_t)blockIdx.x, column(jb), t);
            }
        }
    }
}

template <typename T, int RB, int JB, bool FIRST>
void launch(const SmallPlan& pl, const SmallArgs<T>& a, hipStream_t st)
{
    const dim3 grid((unsigned)pl.blocks, (unsigned)pl.n_jchunk, (unsigned)pl.n_groups), block(64 * pl.waves);
    const size_t lds = (size_t)pl.waves * (FIRST ? 256 : 16 * JB) * sizeof(double);
    if (a.n == 1)
        hipLaunchKernelGGL((mttkrp_small_kernel<T, RB, JB, 1, FIRST>), grid, block, lds, st, a);
    else if (a.n == 2)
        hipLaunchKernelGGL((mttkrp_small_kernel<T, RB, JB, 2, FIRST>), grid, block, lds, st, a);
    else
        hipLaunchKernelGGL((mttkrp_small_kernel<T, RB, JB, 0, FIRST>), grid, block, lds, st, a);
}

}  // namespace

SmallPlan mttkrp_small_plan(int ndim, const int64_t* dims, int R, int k, int sbytes, int groups)
{
    SmallPlan pl;
    const int jb_total = (R + 15) / 16;
    pl.n_jchunk = (jb_total + 3) / 4;
    pl.JB = (jb_total + pl.n_jchunk - 1) / pl.n_jchunk;
    int64_t C = 1;
    for (int m = 1; m < ndim; ++m)
        if (m != k)
            C *= dims[m];
    int64_t tiles = 1;
    if (k == 0) {
        pl.blocks = (dims[0] + 15) / 16;
    } else {
        // at most four accumulator tiles: registers for the weights and the loads beside them
        pl.RB = pl.JB == 1 ? (sbytes == 8 ? 2 : 4) : (pl.JB == 2 ? 2 : 1);
        if (dims[0] <= 16)
            pl.RB = 1;
        else if (dims[0] <= 32 && pl.RB > 2)
            pl.RB = 2;
        tiles = (dims[0] + 16 * pl.RB - 1) / (16 * pl.RB);
        pl.blocks = dims[k];
    }
    const int batch = pl.RB * pl.JB <= 2 ? 8 : 4;      // steps whose loads are in flight together (kSteps)
    int64_t steps = (C + 3) / 4;
    if (groups > 1) {
        const int64_t per_group = (steps + groups - 1) / groups;
        pl.n_groups = (int)((steps + per_group - 1) / per_group);
        pl.cols_per_group = (int)(4 * per_group);
        steps = per_group;
    } else {
        pl.cols_per_group = (int)(4 * steps);
    }
    // as many pieces as the workgroup has wavefronts for, each at least half a batch of loads
    int64_t ranges = tiles < kSmallWaves ? kSmallWaves / tiles : 1;
    if (ranges > (2 * steps + batch - 1) / batch)
        ranges = (2 * steps + batch - 1) / batch;
    const int64_t per = (steps + ranges - 1) / ranges;
    pl.cols_per_range = (int)(4 * per);
    pl.n_ranges = (int)((steps + per - 1) / per);
    pl.n_tiles = (int)tiles;
    const int64_t units = tiles * pl.n_ranges;
    pl.waves = (int)(units < kSmallWaves ? units : kSmallWaves);
    return pl;
}

void mttkrp_small_divisor(uint32_t d, uint32_t& magic, uint32_t& shift)
{
    // With l = ceil(log2 d) and m = floor(2^(31 + l) / d) + 1 the error m d - 2^(31 + l) is at most d <= 2^l, so
    // floor(n m / 2^(31 + l)) = floor(n / d) for every n < 2^31 (Granlund and Montgomery); m < 2^32 from d = 2 on.
    uint32_t l = 1;
    while (((uint64_t)1 << l) < d)
        ++l;
    magic = (uint32_t)((((uint64_t)1 << (31 + l)) / d) + 1);
    shift = l - 1;
}

template <typename T> int mttkrp_small_launch(const SmallPlan& pl, const SmallArgs<T>& a, bool first_mode, hipStream_t st)
{
    if (first_mode) {
        switch (pl.JB) {
        case 1: launch<T, 1, 1, true>(pl, a, st); break;
        case 2: launch<T, 1, 2, true>(pl, a, st); break;
        case 3: launch<T, 1, 3, true>(pl, a, st); break;
        default: launch<T, 1, 4, true>(pl, a, st); break;
        }
    } else if (pl.JB == 1) {
        if constexpr (sizeof(T) == 4)
            if (pl.RB == 4) {
                launch<T, 4, 1, false>(pl, a, st);
                return hipGetLastError() == hipSuccess ? MTTKRP_OK : MTTKRP_ERR_DEVICE;
            }
        if (pl.RB == 2)
            launch<T, 2, 1, false>(pl, a, st);
        else
            launch<T, 1, 1, false>(pl, a, st);
    } else if (pl.JB == 2) {
        if (pl.RB == 2)
            launch<T, 2, 2, false>(pl, a, st);
        else
            launch<T, 1, 2, false>(pl, a, st);
    } else if (pl.JB == 3) {
        launch<T, 1, 3, false>(pl, a, st);
    } else {
        launch<T, 1, 4, false>(pl, a, st);
    }
    return hipGetLastError() == hipSuccess ? MTTKRP_OK : MTTKRP_ERR_DEVICE;
}
template int mttkrp_small_launch<double>(const SmallPlan&, const SmallArgs<double>&, bool, hipStream_t);
template int mttkrp_small_launch<float>(const SmallPlan&, const SmallArgs<float>&, bool, hipStream_t);
