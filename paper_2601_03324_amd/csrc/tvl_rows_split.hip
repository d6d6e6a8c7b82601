// tvl_rows_split.hip -- one-vector GEMV over fp32 or fp16 weights, plain or
// with RMSNorm / SwiGLU: wavefronts of a workgroup share 1 to 8 weight rows and
// split their columns.  The default for launches of one weight dtype where it
// is the faster form (rows_split in tvl_abi.cpp says where, and why).
//
// What bounds it: HBM in long launches; in short ones the dependent rounds of
// a wavefront and the CUs the launch reaches.  x (and the RMSNorm weight) comes
// from the caches next to the weights and shares the rate at which a CU takes
// in lines, 4 (8) bytes per column against R rows of weights: with one or two
// rows per wavefront, what a whole-row launch needs to fill the GPU, x is as
// much as half of what a CU reads.  With the columns split, R can be 4 (fp32) or 8
// (fp16) and a launch still has as many wavefronts, each with a quarter of the
// rounds.  Two chunks in flight per wavefront, in registers of their own; no
// LDS but for the sums at the end.
//
// Measured (us, against the whole-row forms): 300 x 20000 fp32 8.8 -> 5.9, 4096 x
// 11008 fp32 30.8 -> 28.5 (6.3 TB/s), fp16 16.7 -> 14.0 (6.4 TB/s); 32000 x 768
// fp16 10.3 -> 8.4; 110M token fp16 51 -> 34; RMSNorm + SwiGLU pair of 1000 x 8000
// fp32 19.1 -> 11.7, fp16 15.1 -> 7.7; one fused 70B-shaped layer, fp32 547 -> 495
// (6.9 TB/s), fp16 265 -> 250 (6.9 TB/s).
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "tvl_device.h"

namespace tvl {
namespace {

__device__ __forceinline__ __amdgpu_buffer_rsrc_t rsrc_of(const void *base, int64_t bytes)
{
    const int n = bytes > 0x7fffffff ? 0x7fffffff : (int)bytes;
    return __builtin_amdgcn_make_buffer_rsrc(const_cast<void *>(base), (short)0, n, 0x00020000);
}

// R weight rows (of a SwiGLU pair R / 2 rows of W, then the same of W3).  A
// chunk is one 16-byte load of every lane: 64 N columns.  Every load's whole
// offset is range-checked, and lanes past the row's end (or a chunk past the
// last) take an offset past every descriptor: no memory access, zeros.
template <typename T, int R, bool NORM, bool SWIGLU>
struct SplitRowsOf {
    using V = typename Vec<T>::type;
    static constexpr int ES = (int)sizeof(T);
    static constexpr int N = Vec<T>::N;
    static constexpr int NX = N / 4;
    static constexpr int CH = kWave * N;
    static constexpr int kNone = (int)0x80000000u;
    static constexpr int RO = SWIGLU ? R / 2 : R; // output rows

    struct Chunk {
        V w[R];
        f4 x[NX], g[NX];
    };

    __amdgpu_buffer_rsrc_t wr, w3r, xr, gr;
    int vw[RO], K, col; // col: the lane's first column

    __device__ __forceinline__ SplitRowsOf(const DevItem &it, int row0, int lane)
        : K(it.K), col(lane * N)
    {
        const int left = min(it.M - row0, RO);
        const int64_t pitch = it.ldw * ES, xbytes = ((int64_t)it.K * 4 + 15) & ~(int64_t)15;
        wr = rsrc_of(static_cast<const char *>(it.W) + (int64_t)row0 * pitch, left * pitch);
        if constexpr (SWIGLU)
            w3r = rsrc_of(static_cast<const char *>(it.W3) + (int64_t)row0 * pitch, left * pitch);
        xr = rsrc_of(it.x, xbytes);
        if constexpr (NORM) gr = rsrc_of(it.g, xbytes);
#pragma unroll
        for (int r = 0; r < RO; ++r) // rows past M repeat the last (not stored)
            vw[r] = (int)(min(r, left - 1) * pitch) + lane * 16;
    }

    __device__ __forceinline__ void load(int c, Chunk &t) const
    {
        const bool on = col + c * CH < K;
#pragma unroll
        for (int h = 0; h < NX; ++h) {
            const int vx = on ? 4 * (col + c * CH) + 16 * h : kNone;
            t.x[h] = __builtin_bit_cast(f4, __builtin_amdgcn_raw_buffer_load_b128(xr, vx, 0, 0));
            if constexpr (NORM)
                t.g[h] = __builtin_bit_cast(f4, __builtin_amdgcn_raw_buffer_load_b128(gr, vx, 0, 0));
        }
#pragma unroll
        for (int r = 0; r < R; ++r)
            t.w[r] = __builtin_bit_cast(
                V, __builtin_amdgcn_raw_buffer_load_b128(SWIGLU && r >= RO ? w3r : wr,
                                                         on ? vw[r % RO] + c * (16 * kWave) : kNone,
                                                         0, 2));
    }

    __device__ __forceinline__ void multiply(int c, Chunk &t, f4 (&acc)[R], f4 &ssq) const
    {
        if ((c + 1) * CH > K) { // wavefront-uniform: the ragged last chunk
            const int valid = K - c * CH - col;
#pragma unroll
            for (int h = 0; h < NX; ++h) {
                t.x[h] = mask_from<f4, 4>(t.x[h], valid - 4 * h);
                if constexpr (NORM) t.g[h] = mask_from<f4, 4>(t.g[h], valid - 4 * h);
            }
#pragma unroll
            for (int r = 0; r < R; ++r)
                t.w[r] = mask_from<V, N>(t.w[r], valid);
        }
        if constexpr (NORM) {
#pragma unroll
            for (int h = 0; h < NX; ++h) {
                fma4(ssq, t.x[h], t.x[h]);
                t.x[h] *= t.g[h];
            }
        }
#pragma unroll
        for (int r = 0; r < R; ++r)
            mac_x(acc[r], t.w[r], t.x[0], t.x[NX - 1]);
    }

    // chunks c0, c0 + step, ...: the next chunk's loads are in flight while one
    // is multiplied, each in registers of its own
    __device__ __forceinline__ void run(int c0, int step, f4 (&acc)[R], f4 &ssq) const
    {
        const int nc = (K + CH - 1) / CH;
        Chunk a, b;
        int c = c0;
        load(c, a);
        for (; c + step < nc; c += 2 * step) {
            load(c + step, b);
            __builtin_amdgcn_sched_barrier(0);
            multiply(c, a, acc, ssq);
            __builtin_amdgcn_sched_barrier(0);
            load(c + 2 * step, a);
            __builtin_amdgcn_sched_barrier(0);
            multiply(c + step, b, acc, ssq);
            __builtin_amdgcn_sched_barrier(0);
        }
        if (c < nc) multiply(c, a, acc, ssq);
    }
};

// KS of the WV wavefronts share each set of R weight rows.
template <typename T, int R, int KS, int WV, bool NORM, bool SWIGLU>
__device__ __forceinline__ void tile_rows_split(const DevItem &it, int row0)
{
    using Rows = SplitRowsOf<T, R, NORM, SWIGLU>;
    constexpr int RO = Rows::RO, SETS = WV / KS;
    const int lane = threadIdx.x & (kWave - 1);
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave);
    const int wrow0 = row0 + wave / KS * RO;
    __shared__ float part[WV * R], squares[WV];
    f4 acc[R], ssq = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int r = 0; r < R; ++r)
        acc[r] = f4{0.f, 0.f, 0.f, 0.f};
    if (wrow0 < it.M) { // wavefront-uniform
        const Rows rows(it, wrow0, lane);
        rows.run(wave % KS, KS, acc, ssq);
    }
    const float v = reduce_rows<R>(acc, lane);
    constexpr int G = kWave / R;
    if (lane % G == 0) part[wave * R + lane / G] = v;
    if constexpr (NORM) {
        const float s = wave_sum((ssq.x + ssq.y) + (ssq.z + ssq.w));
        if (lane == 0) squares[wave] = s;
    }
    __syncthreads();
    const int t = threadIdx.x, set = t / RO, r = t % RO;
    if (set < SETS && row0 + t < it.M) {
        float a = 0.f, b = 0.f, s = 0.f;
#pragma unroll
        for (int w = 0; w < KS; ++w) {
            a += part[(set * KS + w) * R + r];
            if constexpr (SWIGLU) b += part[(set * KS + w) * R + RO + r];
            if constexpr (NORM) s += squares[set * KS + w];
        }
        if constexpr (NORM) {
            const float inv = 1.0f / sqrtf(s / (float)it.K + it.eps);
            a *= inv;
            b *= inv;
        }
        it.y[row0 + t] = SWIGLU ? silu(a) * b : a;
    }
}

template <typename T, int R, int KS, int WV, bool FUSED>
__device__ __forceinline__ void tile_any_split(const DevItem &it, int row0)
{
    if constexpr (FUSED) {
        if (it.op == kOpSwiglu) {
            if constexpr (R > 1) {
                if (it.g)
                    tile_rows_split<T, R, KS, WV, true, true>(it, row0);
                else
                    tile_rows_split<T, R, KS, WV, false, true>(it, row0);
            }
            return;
        }
        if (it.g) {
            tile_rows_split<T, R, KS, WV, true, false>(it, row0);
            return;
        }
    }
    tile_rows_split<T, R, KS, WV, false, false>(it, row0);
}

template <typename T, int R, int KS, int WV, bool FUSED>
__global__ __launch_bounds__(WV *kWave) void k_sweep_rows_split(const DevItem *__restrict__ items,
                                                                 const DevTile *__restrict__ tiles)
{
    const DevTile tl = tiles[blockIdx.x];
    const DevItem it = items[tl.item];
    tile_any_split<T, R, KS, WV, FUSED>(it, tl.row0);
}

template <typename T, int R, int KS, int WV, bool FUSED>
__global__ __launch_bounds__(WV *kWave) void k_item_rows_split(const DevItem it)
{
    const int rows = (FUSED && it.op == kOpSwiglu ? R / 2 : R) * (WV / KS);
    tile_any_split<T, R, KS, WV, FUSED>(it, (int)blockIdx.x * rows);
}

template <typename T, int R, int KS, int WV, bool FUSED>
hipError_t launch(const RowsSplit &s, const DevItem *items, const DevTile *tiles, int n,
                  const DevItem *one, hipStream_t st)
{
    if (one) {
        const int rows = s.rows(one->op);
        hipLaunchKernelGGL((k_item_rows_split<T, R, KS, WV, FUSED>),
                           dim3((one->M + rows - 1) / rows), dim3(WV * kWave), 0, st, *one);
    } else {
        hipLaunchKernelGGL((k_sweep_rows_split<T, R, KS, WV, FUSED>), dim3(n), dim3(WV * kWave), 0,
                           st, items, tiles);
    }
    return hipGetLastError();
}

// (weight rows per set, wavefronts per set, wavefronts per workgroup) of each
// kind of launch that rows_split can choose
#define TVL_ROWS_SPLIT_F32(X) X(1, 4, 4) X(2, 4, 4) X(4, 2, 2) X(4, 4, 4)
#define TVL_ROWS_SPLIT_F16(X) X(2, 1, 4) X(8, 1, 4) X(4, 2, 2) X(8, 2, 2) X(2, 4, 4) X(8, 4, 4)
#define TVL_ROWS_SPLIT_F32_FUSED(X) X(2, 1, 4) X(4, 1, 4) X(4, 4, 4)
#define TVL_ROWS_SPLIT_F16_FUSED(X) X(4, 1, 4) X(4, 2, 2) X(4, 2, 4) X(8, 2, 2) X(4, 4, 4)

template <typename T, bool FUSED>
hipError_t pick(const RowsSplit &s, const DevItem *items, const DevTile *tiles, int n,
                const DevItem *one, hipStream_t st)
{
#define X(R_, K_, W_)                                                                             \
    if (s.set == R_ && s.split == K_ && s.waves == W_)                                             \
        return launch<T, R_, K_, W_, FUSED>(s, items, tiles, n, one, st);
    if constexpr (sizeof(T) == 4 && !FUSED) {
        TVL_ROWS_SPLIT_F32(X)
    } else if constexpr (sizeof(T) == 4) {
        TVL_ROWS_SPLIT_F32_FUSED(X)
    } else if constexpr (!FUSED) {
        TVL_ROWS_SPLIT_F16(X)
    } else {
        TVL_ROWS_SPLIT_F16_FUSED(X)
    }
#undef X
    return hipErrorInvalidValue;
}

hipError_t any(const RowsSplit &s, const DevItem *items, const DevTile *tiles, int n,
               const DevItem *one, hipStream_t st)
{
    if (s.f16)
        return s.fused ? pick<_Float16, true>(s, items, tiles, n, one, st)
                       : pick<_Float16, false>(s, items, tiles, n, one, st);
    return s.fused ? pick<float, true>(s, items, tiles, n, one, st)
                   : pick<float, false>(s, items, tiles, n, one, st);
}

}  // namespace

hipError_t launch_sweep_rows_split(const RowsSplit &s, const DevItem *items, const DevTile *tiles,
                                   int ntiles, hipStream_t st)
{
    return any(s, items, tiles, ntiles, nullptr, st);
}

hipError_t launch_item_rows_split(const RowsSplit &s, const DevItem &item, hipStream_t st)
{
    return any(s, nullptr, nullptr, 0, &item, st);
}

}  // namespace tvl
