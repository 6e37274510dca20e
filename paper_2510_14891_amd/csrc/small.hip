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
// behind the loads, and short modes need no fused product matrices.  fp64, us a call, general plan and this kernel: 64^3 at R = 16 15.7 /
// 8.4 / 8.4 -> 8.3 / 5.1 / 5.0; 100 x 80 x 60 at R = 10, CP-ALS, 12 sweeps 1482 -> 1190; 4947 calls that take it 0.55 times as
// long in the mean.  mttkrp.hip says where the line between the two paths lies.
//
// A wavefront has one or two batches of loads, so each wait counts: a remainder runs as a batch of its own length (the padding of a
// full one cost loads and MFMAs: 64^3 5.4 -> 4.6 us), all column modes' loads are under way before the first product (8^5, third
// mode 6.7 -> 3.7: a branch per mode had made each load wait for the one before), consecutive rows share a load (4.6 -> 4.2), the
// weights come after the sweep, when their registers are free (64^3 at R = 32 7.8 -> 5.6, 128 x 128 x 64 at R = 64 12.9 -> 7.9 where
// registers had been spilled), the wavefronts' sums are read eight at a time (100 x 80 x 60, first mode 5.6 -> 4.2 with the
// remainders).
#include "mttkrp_small.h"

#include <type_traits>

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

// steps (of four columns) whose loads are in flight together: fewer where those of three or four column modes, the accumulators
// and the weights would pass the 128 registers of a lane
template <typename T, int RB, int JB, int NM> constexpr int steps_in_flight()
{
    constexpr int words = (int)sizeof(T) / 4, most = RB * JB <= 2 ? 8 : 4;
    constexpr int held = words * 4 * RB * JB, step = words * (RB + (NM > 0 ? NM : 3) * JB);
    return NM != 1 && held + most * step > 115 ? most / 2 : most;
}

// Output columns of a lane, as in the streaming kernel: JB consecutive ones, so that one wide load (two for more
// than 16 bytes) fetches its entries of a factor row.  A group that would cross R is moved back to end at R and
// stores only the columns it owns.
template <typename T, int N> struct Lay {
    static constexpr int G = 16 / (int)sizeof(T);
    static constexpr int n0 = N < G ? N : G;
    static constexpr int n1 = N - n0;
};

// NM: column modes (1 to 4: their loads are all under way before the first product is formed), 0: none or more.
template <typename T, int RB, int JB, int NM, bool FIRST>
__global__ void __launch_bounds__(64 * kSmallWaves) mttkrp_small_kernel(const SmallArgs<T> p)
{
    typedef Mfma<T> MF;
    typedef typename MF::acc_t acc_t;
    typedef Lay<T, JB> LC;
    constexpr int U = steps_in_flight<T, RB, JB, NM>();
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

    // Rows of MFMA index i: RB consecutive ones (one load), block r holding the r-th.  Rows that would pass I_0 are moved back
    // to end there; those that another index holds as well are dropped.
    auto first_row = [&](int row0, int i) { return min(row0 + RB * i, p.I0 - RB); };
    acc_t acc[RB][JB];
    // acc = X(rows row0 .., columns [c0, c1)) * Khatri-Rao rows.  Lanes past c1 enter zeros for both operands (exact
    // zeros whatever the tensor holds).
    auto sweep = [&](int row0, int c0, int c1) {
#pragma unroll
        for (int r = 0; r < RB; ++r)
#pragma unroll
            for (int jb = 0; jb < JB; ++jb)
                acc[r][jb] = (acc_t)(0);
        const uint32_t row = (uint32_t)first_row(row0, il);
        auto batch = [&](int c, auto count, bool masked) {
            constexpr int N = decltype(count)::value;
            T xs[N][RB], bs[N][JB];
            uint32_t rem[N], off[N];
#pragma unroll
            for (int u = 0; u < N; ++u) {
                rem[u] = (uint32_t)(c + 4 * u + kk);
                if (masked)
                    rem[u] = min(rem[u], (uint32_t)(c1 - 1));
                off[u] = 0;
            }
            // index of mode m in step u's column, and its entries of the factor
            auto mode = [&](int m, int u, bool last, T (&v)[JB]) {
                uint32_t i = rem[u];
                if (!last) {
                    const uint32_t q = p.dim[m] > 1 ? __umulhi(i, p.magic[m]) >> p.shift[m] : i;
                    i -= q * (uint32_t)p.dim[m];
                    rem[u] = q;
                }
                off[u] += i * (uint32_t)p.sx[m];
                load_cols(p.A[m], i * (uint32_t)p.ld[m], v);
            };
            auto tensor = [&](int u) {
                const T* const x = xb + (off[u] + row);
#pragma unroll
                for (int r = 0; r < RB; ++r)
                    xs[u][r] = x[r];
            };
            if constexpr (NM > 0) {
#pragma unroll
                for (int u = 0; u < N; ++u) {
#pragma unroll
                    for (int m = 0; m < NM; ++m) {
                        T v[JB];
                        mode(m, u, m == NM - 1, v);
#pragma unroll
                        for (int jb = 0; jb < JB; ++jb)
                            bs[u][jb] = m == 0 ? v[jb] : bs[u][jb] * v[jb];
                    }
                    tensor(u);
                }
            } else {
                // a mode at a time, all its loads before the first product (no mode at all: columns of ones)
#pragma unroll
                for (int u = 0; u < N; ++u)
#pragma unroll
                    for (int jb = 0; jb < JB; ++jb)
                        bs[u][jb] = (T)1;
                if (p.n == 0)
#pragma unroll
                    for (int u = 0; u < N; ++u)
                        tensor(u);
                for (int m = 0; m < p.n; ++m) {
                    T v[N][JB];
#pragma unroll
                    for (int u = 0; u < N; ++u)
                        mode(m, u, m == p.n - 1, v[u]);
                    if (m == p.n - 1)
#pragma unroll
                        for (int u = 0; u < N; ++u)
                            tensor(u);
#pragma unroll
                    for (int u = 0; u < N; ++u)
#pragma unroll
                        for (int jb = 0; jb < JB; ++jb)
                            bs[u][jb] *= v[u][jb];
                }
            }
            if (masked) {
#pragma unroll
                for (int u = 0; u < N; ++u) {
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
            for (int u = 0; u < N; ++u)
#pragma unroll
                for (int r = 0; r < RB; ++r)
#pragma unroll
                    for (int jb = 0; jb < JB; ++jb)
                        acc[r][jb] = MF::run(xs[u][r], bs[u][jb], acc[r][jb]);
        };
        int c = c0;
        for (; c + 4 * U <= c1; c += 4 * U)
            batch(c, std::integral_constant<int, U>(), false);
        // the remainder in a batch of its own length: pieces of half a batch are the rule where a call is small
        const int left = (c1 - c + 3) / 4, part = (U + 3) / 4;
        if (left > 3 * part)
            batch(c, std::integral_constant<int, U>(), true);
        else if (left > 2 * part)
            batch(c, std::integral_constant<int, U < 3 * part ? U : 3 * part>(), true);
        else if (left > part)
            batch(c, std::integral_constant<int, 2 * part>(), true);
        else if (left > 0)
            batch(c, std::integral_constant<int, part>(), true);
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

    // the wavefronts' values in their order, requested eight at a time: one after the other they cost an LDS latency each
    auto add_up = [&](const double* a, int stride) {
        double v = 0.0;
        for (int w0 = 0; w0 < n_waves; w0 += 8) {
            double x[8];
#pragma unroll
            for (int h = 0; h < 8; ++h)
                x[h] = a[min(w0 + h, n_waves - 1) * stride];
#pragma unroll
            for (int h = 0; h < 8; ++h)
                v += w0 + h < n_waves ? x[h] : 0.0;
        }
        return v;
    };
    if constexpr (FIRST) {
        // one row tile; wavefront w holds the sum over piece w of the group's columns
        const int row0 = (int)blockIdx.x * 16;
        const int c0 = g0 + wave * p.cols_per_range;
        sweep(row0, c0, min(g1, c0 + p.cols_per_range));
#pragma unroll
        for (int jb = 0; jb < JB; ++jb) {
            double* const tile = red + (jb & 1) * n_waves * 256;     // two in turn: one barrier a block of columns
#pragma unroll
            for (int q = 0; q < 4; ++q)
                tile[wave * 256 + MF::row(lane, q) * 16 + il] = (double)acc[0][jb][q];
            __syncthreads();
            for (int t = (int)threadIdx.x; t < 256; t += (int)blockDim.x) {
                // (entry t & 15 belongs to lane t & 15 of the layout above: this thread's own il)
                const int r = row0 + (t >> 4);
                const double v = add_up(tile + t, 256);
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
            const int c0 = g0 + rng * p.cols_per_range;
            sweep(row0, c0, min(g1, c0 + p.cols_per_range));
            T w[RB][4][JB];
#pragma unroll
            for (int r = 0; r < RB; ++r)
#pragma unroll
                for (int q = 0; q < 4; ++q)
                    load_cols(p.A0, (uint32_t)(first_row(row0, MF::row(lane, q)) + r) * (uint32_t)p.ld0, w[r][q]);
#pragma unroll
            for (int r = 0; r < RB; ++r)
#pragma unroll
                for (int q = 0; q < 4; ++q) {
                    const bool in = first_row(row0, MF::row(lane, q)) + r >= row0 + RB * MF::row(lane, q);
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
        if (wave == 0 && kk < JB && owned(kk))      // (lane group kk takes block kk)
            store((int64_t)blockIdx.x, column(kk), add_up(red + lane, 16 * JB));
    }
}

template <typename T, int RB, int JB, bool FIRST>
void launch(const SmallPlan& pl, const SmallArgs<T>& a, hipStream_t st)
{
    const dim3 grid((unsigned)pl.blocks, (unsigned)pl.n_jchunk, (unsigned)pl.n_groups), block(64 * pl.waves);
    const size_t lds = (size_t)pl.waves * (FIRST ? (JB > 1 ? 512 : 256) : 16 * JB) * sizeof(double);
    switch (a.n) {
    case 1: hipLaunchKernelGGL((mttkrp_small_kernel<T, RB, JB, 1, FIRST>), grid, block, lds, st, a); break;
    case 2: hipLaunchKernelGGL((mttkrp_small_kernel<T, RB, JB, 2, FIRST>), grid, block, lds, st, a); break;
    case 3: hipLaunchKernelGGL((mttkrp_small_kernel<T, RB, JB, 3, FIRST>), grid, block, lds, st, a); break;
    case 4: hipLaunchKernelGGL((mttkrp_small_kernel<T, RB, JB, 4, FIRST>), grid, block, lds, st, a); break;
    default: hipLaunchKernelGGL((mttkrp_small_kernel<T, RB, JB, 0, FIRST>), grid, block, lds, st, a); break;
    }
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
    const int batch = pl.RB * pl.JB <= 2 ? 8 : 4;      // steps whose loads are in flight together (mostly)
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
