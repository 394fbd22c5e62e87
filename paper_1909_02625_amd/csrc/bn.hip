// Training-mode batch normalisation fused with the residual add and the ReLU that follow it,
// forward and backward, on NHWC tensors x[M][C] (M = N*H*W rows, channels contiguous).
//
// These layers carry no reuse: each is a stream over HBM, so the kernels are built around
// 16-byte coalesced row segments.  Thread t of a 256-thread workgroup owns the channel vector
// (t mod CV) and walks rows t/CV, t/CV + RL, ...; per-channel sums are accumulated in fp64
// registers (free in an HBM-bound kernel, and it removes the cancellation in E[x^2]-E[x]^2),
// combined through LDS, written as one partial per workgroup, and merged by a one-wave-per-
// channel kernel in a fixed order, so results are identical from run to run.
//
//   forward :  stats-partial -> finalize (mean, invstd, scale/shift) -> apply (+res, ReLU)
//   backward:  reduce-partial (sum dz, sum dz*xhat) -> finalize (dgamma, dbeta, coefficients)
//              -> apply (dx, and dz into the residual branch)
#include "common.h"

namespace dsp {
namespace {

constexpr int kThreads = 256;
constexpr int kMaxPartialBlocks = 512;
typedef __attribute__((ext_vector_type(4))) float f32x4;
typedef __attribute__((ext_vector_type(4))) uint32_t u32x4;
typedef __attribute__((ext_vector_type(2))) uint32_t u32x2;

// Layout of a workgroup over x[M][C]: CV channel vectors per row, RL row lanes.
struct RowLayout {
    int cv;   // channel vectors per row (C / VW)
    int cvb;  // channel vectors handled by one workgroup column (min(cv, 256))
    int rl;   // row lanes per workgroup (256 / cvb)
};
inline RowLayout make_layout(int C, int VW)
{
    RowLayout L;
    L.cv = C / VW;
    L.cvb = L.cv < kThreads ? L.cv : kThreads;
    L.rl = kThreads / L.cvb;
    return L;
}

// scale * x + shift as the forward pass stores it (one fused multiply-add, rounded to the storage type): the backward
// kernels that decide the ReLU from x call this too, and get the forward pass's decision
template <typename T>
__device__ inline float bn_value(float x, float scale, float shift)
{
    return to_float<T>(from_float<T>(__builtin_fmaf(x, scale, shift)));
}

// Sums over the lanes of a wave: lanes of equal lane % VPR hold the same VW channels (of channel vector lane % VPR); the wave's
// sums go to dst[channel][2].  Each exchange hands half of a lane's channels to the lane across, so that they cost VW - 1
// exchanges and not VW * log2(64 / VPR); the order of additions is fixed.
template <int VW, int MASK, int COUNT>
__device__ inline void reduce_wave_step(double (&s0)[VW], double (&s1)[VW], int lane, int& off, bool& writes)
{
    if constexpr (MASK < 64) {
        const bool up = (lane & MASK) != 0;
        if constexpr (COUNT > 1) {
            constexpr int HALF = COUNT / 2;
#pragma unroll
            for (int i = 0; i < HALF; ++i) {
                const double k0 = up ? s0[i + HALF] : s0[i], g0 = up ? s0[i] : s0[i + HALF];
                const double k1 = up ? s1[i + HALF] : s1[i], g1 = up ? s1[i] : s1[i + HALF];
                s0[i] = k0 + __shfl_xor(g0, MASK, 64);
                s1[i] = k1 + __shfl_xor(g1, MASK, 64);
            }
            if (up) off += HALF;
            reduce_wave_step<VW, MASK * 2, HALF>(s0, s1, lane, off, writes);
        } else {
            s0[0] += __shfl_xor(s0[0], MASK, 64);
            s1[0] += __shfl_xor(s1[0], MASK, 64);
            writes = writes && !up;
            reduce_wave_step<VW, MASK * 2, 1>(s0, s1, lane, off, writes);
        }
    }
}
template <int VW, int VPR>
__device__ inline void reduce_wave(double (&s0)[VW], double (&s1)[VW], double (*dst)[2])
{
    const int lane = threadIdx.x & 63;
    int off = 0;
    bool writes = true;
    reduce_wave_step<VW, VPR, VW>(s0, s1, lane, off, writes);
    constexpr int LEFT = VW * VPR > 64 ? VW * VPR / 64 : 1;
    if (writes)
#pragma unroll
        for (int i = 0; i < LEFT; ++i) {
            double* d = dst[(lane % VPR) * VW + off + i];
            d[0] = s0[i];
            d[1] = s1[i];
        }
}

// The tail of the summing kernels: combines the row lanes of each channel vector in a fixed order (all channels of the
// vector at once) and writes the workgroup's partial row part_row[c][2].  Where a wave holds whole rows (a power of two of
// channel vectors, at most 64) its lanes exchange their sums and only the four waves meet in LDS; the tree through LDS that
// serves the others takes a barrier and 2 VW double additions in LDS per level, a third of the launch on small maps.  Together
// with loads that stay packed until they are used (registers, eight bf16 channels: ReLU from sign bytes 126 instead of 171, from x
// 117 instead of 153, four waves per SIMD instead of two or three; from y 140 instead of 177, three waves), backward sums with
// sign bytes: 131072 x 16 bf16 8.9 -> 5.5 us, 12544 x 256 8.2 -> 6.7, 200704 x 128 23.8 -> 18.4 (5.6 TB/s); from x 7.5 -> 5.0,
// 7.9 -> 7.2, 21.8 -> 17.6.
template <int VW>
__device__ inline void combine_row_lanes(double (&s0)[VW], double (&s1)[VW], double (&red)[VW][kThreads][2],
                                         bool active, int rlane, const RowLayout& L, double* __restrict__ part_row, int c0)
{
    const int tid = threadIdx.x;
    // (then every thread has a row lane, and one workgroup column holds all channels; 8 channels and more come as vectors)
    if (L.cvb <= (VW == 1 ? 4 : 64) && (L.cvb & (L.cvb - 1)) == 0) {
        const int C = L.cvb * VW;
        double(*sums)[2] = &red[0][0];
        double(*mine)[2] = sums + (tid >> 6) * C;
        switch (L.cvb) {
        case 1: reduce_wave<VW, 1>(s0, s1, mine); break;
        case 2: reduce_wave<VW, 2>(s0, s1, mine); break;
        case 4: reduce_wave<VW, 4>(s0, s1, mine); break;
        default:
            if constexpr (VW > 1) {
                if (L.cvb == 8) reduce_wave<VW, 8>(s0, s1, mine);
                else if (L.cvb == 16) reduce_wave<VW, 16>(s0, s1, mine);
                else if (L.cvb == 32) reduce_wave<VW, 32>(s0, s1, mine);
                else reduce_wave<VW, 64>(s0, s1, mine);
            }
        }
        __syncthreads();
        for (int i = tid; i < 2 * C; i += kThreads) {
            double a = 0.0;
#pragma unroll
            for (int w = 0; w < kThreads / 64; ++w) a += sums[w * C + (i >> 1)][i & 1];
            part_row[i] = a;
        }
        return;
    }
#pragma unroll
    for (int i = 0; i < VW; ++i) {
        red[i][tid][0] = s0[i];
        red[i][tid][1] = s1[i];
    }
    __syncthreads();
    int w = 1;
    while (w < L.rl) w <<= 1;
    for (w >>= 1; w > 0; w >>= 1) {
        if (active && rlane < w && rlane + w < L.rl) {
            const int other = tid + w * L.cvb;
#pragma unroll
            for (int i = 0; i < VW; ++i) {
                red[i][tid][0] += red[i][other][0];
                red[i][tid][1] += red[i][other][1];
            }
        }
        __syncthreads();
    }
    if (active && rlane == 0) {
#pragma unroll
        for (int i = 0; i < VW; ++i) {
            double* dst = part_row + (c0 + i) * 2;
            dst[0] = red[i][tid][0];
            dst[1] = red[i][tid][1];
        }
    }
}

// How tensors whose apply kernels merge the partial sums themselves are dealt out (see "finalize inside the apply kernels").
constexpr int kMergeEntries = 2048;  // partial rows x channels of a group
constexpr int64_t kMergeTensorBytes = (int64_t)3 << 19;
// With kWideChannels and more the sums come by channel groups and in few rows (bn_group_sums_kernel):
constexpr int kWideChannels = 128;
constexpr int kWideConvEntries = 3072;       // partial rows x channels of a group where a convolution left them
constexpr int kWideBackwardWgs = 96;         // workgroups of the largest such backward sums, at least
constexpr int kWideRunBytes = 96 << 10;      // of a tensor, per workgroup that sums
constexpr int kBnThreads = 512;
struct BnLayout {
    int cg, groups;              // channels per group, groups
    int rows_per_wg, row_blocks;
};
__device__ inline int bn_work_item(const BnLayout& L, int* g0)
{
    const unsigned b = blockIdx.x, nb = gridDim.x, q = nb / 8, r = nb % 8, xcd = b % 8;
    const unsigned item = xcd * q + (xcd < r ? xcd : r) + b / 8;
    *g0 = (int)(item % (unsigned)L.groups) * L.cg;
    return (int)(item / (unsigned)L.groups);
}

// ---- per-channel sums ---------------------------------------------------------------------------
// MODE 0: s0 = sum x, s1 = sum x^2.
// MODE 1: dz = dy * [y > 0] (if RM != 0); s0 = sum dz, s1 = sum dz * (x - mean) * invstd.  RM = 1 reads the stored y;
//         RM = 2 (a batch norm without residual) forms y again from x and the forward pass's {scale, shift} with the
//         forward kernel's own expression and rounding, so the decision is the same and y is never read.
//         RM = 3 (vector paths): `y` points at the sign bytes the forward apply kernel left instead -- one byte per
//         channel vector, bit k = element k of the stored output is positive: an eighth (bf16: a sixteenth) of y.
// MODE 2: out = x + dy as stored (the element-wise sum of two feature maps); s0 = sum out, s1 = sum out^2:
//         the sum layer together with the statistics pass of the batch norm that reads it.
// part[blockIdx.x][c][2]; blockIdx.y walks channel groups when C/VW > 256.
template <typename T>
struct AddOut {
    T* out;        // MODE 2: the sum
    const T* b1;   // second instance: the other operand and the sum
    T* out1;
};
template <int VW>
struct BnSumCoef {
    float mu[VW], is[VW], fsc[VW], fsh[VW];
};
template <int VW, int MODE, int RM>
__device__ inline void load_sum_coef(BnSumCoef<VW>& k, const float* __restrict__ mean, const float* __restrict__ invstd,
                                     const float* __restrict__ fcoef, int C, int c0)
{
#pragma unroll
    for (int i = 0; i < VW; ++i) {
        if (MODE == 1) {
            k.mu[i] = mean[c0 + i];
            k.is[i] = invstd[c0 + i];
        }
        if (MODE == 1 && RM == 2) {
            k.fsc[i] = fcoef[c0 + i];
            k.fsh[i] = fcoef[C + c0 + i];
        }
    }
}
// Adds the rows r, r + rl, .. below r_end of channel vector cvi (channels c0 ..) of cv to s0 and s1.
template <typename T, int VW, int MODE, int RM>
__device__ inline void add_rows(const T* __restrict__ x, const T* __restrict__ dy, const T* __restrict__ y, T* __restrict__ out,
                                const BnSumCoef<VW>& k, int64_t r, int64_t r_end, int rl, int C, int c0, int cv, int cvi,
                                double (&s0)[VW], double (&s1)[VW])
{
    typedef typename VecIO<T, VW>::Raw Raw;
    // U rows per trip with all their loads issued before the first add: the loop is bound by load
    // latency, not by bandwidth, unless several rows are in flight per thread (three where the ReLU is decided from x in
    // bf16: beside the constants of eight channels a fourth spills, 131072 x 16 5.5 -> 5.0 us, 30000 x 40 7.5 -> 6.7)
    constexpr int U = RM == 2 && VW == 8 ? 3 : 4;
    for (; r < r_end; r += (int64_t)U * rl) {
        Raw xr[U], gr[U], yr[U];
        uint32_t bits[U];
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int64_t ru = r + (int64_t)u * rl;
            if (ru < r_end) {
                xr[u] = VecIO<T, VW>::raw(x + ru * C + c0);
                if (MODE >= 1) gr[u] = VecIO<T, VW>::raw(dy + ru * C + c0);
                if (MODE == 1 && RM == 1) yr[u] = VecIO<T, VW>::raw(y + ru * C + c0);
                if (MODE == 1 && RM == 3) bits[u] = ((const uint8_t*)y)[ru * cv + cvi];
            }
        }
#pragma unroll
        for (int u = 0; u < U; ++u) {
            if (r + (int64_t)u * rl >= r_end) break;
            float xv[VW], gv[VW], yv[VW];
            VecIO<T, VW>::unpack(xr[u], xv);
            if (MODE >= 1) VecIO<T, VW>::unpack(gr[u], gv);
            if (MODE == 1 && RM == 1) VecIO<T, VW>::unpack(yr[u], yv);
#pragma unroll
            for (int i = 0; i < VW; ++i) {
                if (MODE == 2) xv[i] = to_float<T>(from_float<T>(xv[i] + gv[i]));  // the value as stored
                if (MODE == 0 || MODE == 2) {
                    s0[i] += (double)xv[i];
                    s1[i] += (double)xv[i] * (double)xv[i];
                } else {
                    const bool on = RM == 0 ? true
                                    : RM == 1 ? yv[i] > 0.f
                                    : RM == 2 ? bn_value<T>(xv[i], k.fsc[i], k.fsh[i]) > 0.f : ((bits[u] >> i) & 1u) != 0;
                    const float dz = on ? gv[i] : 0.f;
                    s0[i] += (double)dz;
                    s1[i] += (double)(dz * ((xv[i] - k.mu[i]) * k.is[i]));
                }
            }
            if (MODE == 2) VecIO<T, VW>::store(out + (r + (int64_t)u * rl) * C + c0, xv);
        }
    }
}
template <typename T, int VW, int MODE, int RM>
__global__ __launch_bounds__(kThreads) __attribute__((amdgpu_waves_per_eu(RM == 1 ? 3 : 4))) void bn_sums_kernel(const T* __restrict__ x, const T* __restrict__ dy,
                                                           const T* __restrict__ y, const float* __restrict__ mean,
                                                           const float* __restrict__ invstd, double* __restrict__ part,
                                                           int64_t M, int C, RowLayout L, int rows_per_block,
                                                           const T* __restrict__ x1, double* __restrict__ part1,
                                                           AddOut<T> add, const float* __restrict__ fcoef)
{
    // blockIdx.z = 1: the second instance of a twin launch (other tensor, same shape)
    T* __restrict__ out = add.out;
    if (blockIdx.z) {
        x = x1;
        part = part1;
        if (MODE == 2) {
            dy = add.b1;
            out = add.out1;
        }
    }
    __shared__ double red[VW][kThreads][2];  // one 16-byte pair per thread and channel, neighbouring lanes side by side: no bank conflicts
    const int tid = threadIdx.x;
    const int cvi = blockIdx.y * L.cvb + tid % L.cvb;
    const int rlane = tid / L.cvb;
    const bool active = rlane < L.rl && cvi < L.cv;
    const int c0 = cvi * VW;
    double s0[VW], s1[VW];
#pragma unroll
    for (int i = 0; i < VW; ++i) s0[i] = s1[i] = 0.0;
    BnSumCoef<VW> k;
    if (active) load_sum_coef<VW, MODE, RM>(k, mean, invstd, fcoef, C, c0);
    const int64_t r_begin = (int64_t)blockIdx.x * rows_per_block;
    const int64_t r_end = r_begin + rows_per_block < M ? r_begin + rows_per_block : M;
    if (active) add_rows<T, VW, MODE, RM>(x, dy, y, out, k, r_begin + rlane, r_end, L.rl, C, c0, L.cv, cvi, s0, s1);
    combine_row_lanes<VW>(s0, s1, red, active, rlane, L, part + (int64_t)blockIdx.x * C * 2, c0);
}

// The same sums with few partial rows, for tensors whose apply kernels merge them: a workgroup takes a group of L.cg channels over a
// run of rows (the work items of those kernels), so that what each of their workgroups reads back, rows x channels of a
// group, stays at kMergeEntries.  That is kMergeEntries / cg runs, so at most 32 x C / 64 workgroups of 64 channels, 64 at C = 128 and 256
// from C = 512 on in bf16, and 64 x C / 32 in fp32; a run of kWideRunBytes ends it at 48 KB x C of a tensor (6 MB at C = 128 in bf16).
template <typename T, int VW, int MODE, int RM>
__global__ __launch_bounds__(kBnThreads) __attribute__((amdgpu_waves_per_eu(RM == 1 ? 3 : 4))) void bn_group_sums_kernel(
    const T* __restrict__ x, const T* __restrict__ dy, const T* __restrict__ y, const float* __restrict__ mean,
    const float* __restrict__ invstd, double* __restrict__ part, int64_t M, int C, BnLayout L, const T* __restrict__ x1,
    double* __restrict__ part1, const float* __restrict__ fcoef)
{
    if (blockIdx.y) {  // the second instance of a twin launch
        x = x1;
        part = part1;
    }
    constexpr int NW = kBnThreads / 64;
    __shared__ double sums[NW][64][2];
    int g0;
    const int rb = bn_work_item(L, &g0);
    const int tid = threadIdx.x, vpr = L.cg / VW, rpp = kBnThreads / vpr, c0 = g0 + (tid % vpr) * VW;
    const bool active = c0 < C;  // (channels come in whole vectors)
    double s0[VW], s1[VW];
#pragma unroll
    for (int i = 0; i < VW; ++i) s0[i] = s1[i] = 0.0;
    BnSumCoef<VW> k;
    if (active) {
        load_sum_coef<VW, MODE, RM>(k, mean, invstd, fcoef, C, c0);
        const int64_t r_begin = (int64_t)rb * L.rows_per_wg, r_end = r_begin + L.rows_per_wg < M ? r_begin + L.rows_per_wg : M;
        add_rows<T, VW, MODE, RM>(x, dy, y, (T*)nullptr, k, r_begin + tid / vpr, r_end, rpp, C, c0, C / VW, c0 / VW, s0, s1);
    }
    double(*mine)[2] = sums[tid >> 6];
    if (L.cg == 64) reduce_wave<VW, 64 / VW>(s0, s1, mine);
    else if (L.cg == 32) reduce_wave<VW, 32 / VW>(s0, s1, mine);
    else reduce_wave<VW, 16 / VW>(s0, s1, mine);
    __syncthreads();
    if (tid < 2 * L.cg && g0 + (tid >> 1) < C) {
        double a = 0.0;
#pragma unroll
        for (int w = 0; w < NW; ++w) a += sums[w][tid >> 1][tid & 1];
        part[((int64_t)rb * C + g0) * 2 + tid] = a;
    }
}

// Merging the partials.  The partials of a conv epilogue can be thousands of rows (one per row tile), so a
// workgroup of kMergeLanes x 4 threads takes 4 channels and reads whole 64-byte row segments, up to 8 loads
// in flight per thread and added in row order; then a fixed tree over the row lanes: the sums cross LDS behind one barrier,
// the first wave adds the lanes 32 and 16 apart as it reads them and the others by exchanges.  Returns the two sums
// of channel blockIdx.x * 4 + (threadIdx.x & 3) to the threads of row lane 0; the waves but the first return nothing.
// What bounds these launches is the chain load -> tree -> coefficients -> store, each load a miss to memory behind a launch
// that wrote from other dies; the channel's parameters are fetched with the partials.  (One barrier instead of six and that
// early fetch gain nothing measurable in the finalize launches, 0.999-1.003x over seven networks and layers; they have the form of
// merge_group below, where the merge stands in front of every workgroup's rows.)
constexpr int kMergeLanes = 64;
typedef __attribute__((ext_vector_type(2))) double f64x2;
__device__ inline void merge_partials(const double* __restrict__ part, int nblk, int C, f64x2 (&red)[kMergeLanes * 4], double* sa, double* sb)
{
    const int tid = threadIdx.x, cq = tid & 3, r = tid >> 2;
    const int c = blockIdx.x * 4 + cq;
    double a = 0.0, b = 0.0;
    if (c < C)
        for (int k0 = r; k0 < nblk; k0 += kMergeLanes * 8) {
            f64x2 v[8];
#pragma unroll
            for (int u = 0; u < 8; ++u) {
                const int k = k0 + kMergeLanes * u;
                v[u] = k < nblk ? *(const f64x2*)(part + ((int64_t)k * C + c) * 2) : f64x2{0.0, 0.0};
            }
#pragma unroll
            for (int u = 0; u < 8; ++u) {
                a += v[u][0];
                b += v[u][1];
            }
        }
    red[tid] = f64x2{a, b};
    __syncthreads();
    if (tid >= 64) return;
    f64x2 t = (red[tid] + red[tid + 128]) + (red[tid + 64] + red[tid + 192]);
#pragma unroll
    for (int w = 32; w >= 4; w >>= 1) {
        t[0] += __shfl_xor(t[0], w, 64);
        t[1] += __shfl_xor(t[1], w, 64);
    }
    *sa = t[0];
    *sb = t[1];
}

// Forward: mean, invstd, coef = {scale, shift}.
struct BnStatOut {
    const double* part;
    float *mean, *invstd, *coef;
};
__device__ inline void bn_forward_coef(double a, double b, double inv_M, float eps, float gamma, float beta, const BnStatOut& o, int c,
                                       int C, bool store, float* scale, float* shift)
{
    const double mu = a * inv_M;
    double var = b * inv_M - mu * mu;
    if (var < 0.0) var = 0.0;
    const double is = rsqrt(var + (double)eps);  // (1 / sqrt is a chain twice as long; the statistics of 120 calls kept their bits)
    const double sc = (double)gamma * is;
    *scale = (float)sc;
    *shift = (float)((double)beta - mu * sc);
    if (store) {
        o.mean[c] = (float)mu;
        o.invstd[c] = (float)is;
        o.coef[c] = *scale;
        o.coef[C + c] = *shift;
    }
}
__global__ __launch_bounds__(kMergeLanes * 4) void bn_fwd_finalize_kernel(BnStatOut o0, BnStatOut o1, int nblk, int C,
                                                                          double inv_M, float eps,
                                                                          const float* __restrict__ gamma,
                                                                          const float* __restrict__ beta)
{
    __shared__ f64x2 red[kMergeLanes * 4];
    const BnStatOut o = blockIdx.y ? o1 : o0;
    const int c = blockIdx.x * 4 + (threadIdx.x & 3);
    const bool mine = threadIdx.x < 4 && c < C;
    const float ga = mine ? gamma[c] : 0.f, be = mine ? beta[c] : 0.f;
    double a, b;
    merge_partials(o.part, nblk, C, red, &a, &b);
    float scale, shift;
    if (mine) bn_forward_coef(a, b, inv_M, eps, ga, be, o, c, C, true, &scale, &shift);
}

// Backward: dgamma, dbeta and dx = c1*dz - c2*x + c0 with
// c1 = gamma*invstd, c2 = c1*invstd*dgamma/M, c0 = c2*mean - c1*dbeta/M.
struct BnGradOut {
    const double* part;
    const float *gamma, *mean, *invstd;
    float *dgamma, *dbeta, *coef;
};
struct BnChannel {
    float gamma, mean, invstd;
};
__device__ inline BnChannel bn_channel(const BnGradOut& o, bool mine, int c)
{
    return mine ? BnChannel{o.gamma[c], o.mean[c], o.invstd[c]} : BnChannel{};
}
__device__ inline void bn_backward_coef(double a, double b, double inv_M, const BnGradOut& o, const BnChannel& p, int c, bool store,
                                        float* k1, float* k2, float* k0)
{
    const double c1 = (double)p.gamma * (double)p.invstd;
    const double c2 = c1 * (double)p.invstd * b * inv_M;
    *k1 = (float)c1;
    *k2 = (float)c2;
    *k0 = (float)(c2 * (double)p.mean - c1 * a * inv_M);
    if (store) {
        o.dbeta[c] = (float)a;
        o.dgamma[c] = (float)b;
    }
}
__global__ __launch_bounds__(kMergeLanes * 4) void bn_bwd_finalize_kernel(BnGradOut o, int nblk, int C, double inv_M)
{
    __shared__ f64x2 red[kMergeLanes * 4];
    const int c = blockIdx.x * 4 + (threadIdx.x & 3);
    const bool mine = threadIdx.x < 4 && c < C;
    const BnChannel p = bn_channel(o, mine, c);
    double a, b;
    merge_partials(o.part, nblk, C, red, &a, &b);
    if (mine) bn_backward_coef(a, b, inv_M, o, p, c, true, o.coef + c, o.coef + C + c, o.coef + 2 * C + c);
}

// y = [relu](scale*x + shift [+ res]); blockIdx.y selects the instance of a twin launch
struct BnApplyIo {
    const void* x;
    const void* res;
    void* y;
    const float* coef;
    uint8_t* bits;  // if set (vector paths, ReLU): one byte per channel vector, bit k = element k of y as stored is positive
};
template <typename T, int VW, bool RELU, bool HAS_RES>
__global__ __launch_bounds__(kThreads) void bn_fwd_apply_kernel(BnApplyIo io0, BnApplyIo io1, int64_t nvec, int C, int cv)
{
    const BnApplyIo io = blockIdx.y ? io1 : io0;
    const T* __restrict__ x = (const T*)io.x;
    const T* __restrict__ res = (const T*)io.res;
    T* __restrict__ y = (T*)io.y;
    const float* __restrict__ coef = io.coef;
    // channel vector of element i = i mod cv, carried along the grid-stride loop instead of divided out each trip
    const uint32_t step = gridDim.x * kThreads, step_c = step % (uint32_t)cv;
    uint32_t cvi = (blockIdx.x * kThreads + threadIdx.x) % (uint32_t)cv;
    for (int64_t i = (int64_t)blockIdx.x * kThreads + threadIdx.x; i < nvec;
         i += step, cvi = cvi + step_c >= (uint32_t)cv ? cvi + step_c - (uint32_t)cv : cvi + step_c) {
        const int c0 = (int)cvi * VW;
        float xv[VW], rv[VW], ov[VW];
        VecIO<T, VW>::load(x + i * VW, xv);
        if (HAS_RES) VecIO<T, VW>::load(res + i * VW, rv);
#pragma unroll
        for (int k = 0; k < VW; ++k) {
            float v = __builtin_fmaf(xv[k], coef[c0 + k], coef[C + c0 + k]);
            if (HAS_RES) v += rv[k];
            if (RELU) v = v > 0.f ? v : 0.f;
            ov[k] = v;
        }
        VecIO<T, VW>::store(y + i * VW, ov);
        if (RELU && VW > 1 && io.bits) {
            uint32_t bits = 0u;
#pragma unroll
            for (int k = 0; k < VW; ++k) bits |= (to_float<T>(from_float<T>(ov[k])) > 0.f ? 1u : 0u) << k;
            io.bits[i] = (uint8_t)bits;
        }
    }
}

// dz = dy*[y>0] (y as stored, or formed again from x: RM as in bn_sums_kernel);  dx = [dx_prev +] c1*dz - c2*x + c0;  dres (+)= dz.  dx_prev is dx itself (accumulate in place)
// or another tensor's gradient that reaches the same input (the shortcut of a pre-activation unit).
template <typename T, int VW, int RM, bool HAS_RES, bool RES_ACC, bool DX_ACC>
__global__ __launch_bounds__(kThreads) void bn_bwd_apply_kernel(const T* __restrict__ dy, const T* __restrict__ x,
                                                                const T* __restrict__ y, T* dx, const T* dx_prev,
                                                                T* __restrict__ dres, const float* __restrict__ coef,
                                                                int64_t nvec, int C, int cv, const float* __restrict__ fcoef)
{
    // channel vector of element i = i mod cv, carried along the grid-stride loop instead of divided out each trip
    const uint32_t step = gridDim.x * kThreads, step_c = step % (uint32_t)cv;
    uint32_t cvi = (blockIdx.x * kThreads + threadIdx.x) % (uint32_t)cv;
    for (int64_t i = (int64_t)blockIdx.x * kThreads + threadIdx.x; i < nvec;
         i += step, cvi = cvi + step_c >= (uint32_t)cv ? cvi + step_c - (uint32_t)cv : cvi + step_c) {
        const int c0 = (int)cvi * VW;
        float gv[VW], xv[VW], yv[VW], ov[VW], rv[VW];
        VecIO<T, VW>::load(dy + i * VW, gv);
        VecIO<T, VW>::load(x + i * VW, xv);
        if (RM == 1) VecIO<T, VW>::load(y + i * VW, yv);
        if (RM == 3) {
            const uint32_t bits = ((const uint8_t*)y)[i];
#pragma unroll
            for (int k = 0; k < VW; ++k) yv[k] = (bits >> k) & 1u ? 1.f : 0.f;
        }
        if (DX_ACC) VecIO<T, VW>::load(dx_prev + i * VW, ov);
        if (HAS_RES && RES_ACC) VecIO<T, VW>::load(dres + i * VW, rv);
#pragma unroll
        for (int k = 0; k < VW; ++k) {
            if (RM == 2) yv[k] = bn_value<T>(xv[k], fcoef[c0 + k], fcoef[C + c0 + k]);
            const float dz = (RM == 0 || yv[k] > 0.f) ? gv[k] : 0.f;
            const float d = coef[c0 + k] * dz - coef[C + c0 + k] * xv[k] + coef[2 * C + c0 + k];
            ov[k] = DX_ACC ? ov[k] + d : d;
            if (HAS_RES) rv[k] = RES_ACC ? rv[k] + dz : dz;
        }
        VecIO<T, VW>::store(dx + i * VW, ov);
        if (HAS_RES) VecIO<T, VW>::store(dres + i * VW, rv);
    }
}

// ---- finalize inside the apply kernels --------------------------------------------------------------
// On small tensors with few partial rows every apply workgroup merges the partials of its own channels instead of waiting for
// a launch that does it once.  A workgroup owns a group of cg channels (a power of two, 128 bytes of a row where there are
// that many), so that its share of the partials is short, over a run of rows; the first rows of its tensor are on their way
// while it merges.  Its first row block also leaves the statistics.  Consecutive work items (the groups of one run of rows,
// which share cache lines and partial rows) go to one XCD.  The sums are taken in merge_partials' order (64 row lanes, then a
// tree), so which of the two forms a shape takes does not show in the results.
// Bound by latency: the partials and the first rows come from memory, the coefficients depend on the former and the stores on both.
// Two rows in flight a thread and 256 workgroups: with four rows the registers leave one workgroup per compute unit, with 512
// workgroups the partials are read twice as often (resnet20 1.5 %, resnet56 0.5 % slower).
// Up to 127 channels, forward and backward with their sums, six launches against four: 2664 x 72 fp32 27.8 -> 20.9 us, 2048 x 16
// fp32 27.7 -> 21.1.  The line lies where the gain ends inside a network, where other streams' kernels fill the chip during
// the extra launch anyway while every workgroup's merge reads L2: with merging up to 8192 partials (rows x channels of a group)
// and 32 MB resnet20 was 8 % slower and conv4_x 4.5 %, up to 4096 and 2 MB resnet20 still 1 %.
// From 128 channels on the sums are dealt out by channel groups and leave at most 2048 partials.  Forward / backward with sign
// bytes, sums included: 12544 x 256 bf16 12.7 -> 10.3 / 14.7 -> 12.8 us, 4864 x 1024 bf16 18.8 -> 12.1 / 21.5 -> 15.4, 11956 x 256 fp32
// 15.1 -> 11.9 / 18.6 -> 14.4; conv4_x driven by separate calls 1856 -> 1774 us a step.  The far lines are where 11500 calls of 128 to
// 2048 channels and up to 32 MB, timed in graphs against three launches, stop gaining (whole groups of 128 bytes / a ragged last group / an
// odd number of channels); the backward ones serve every form of the ReLU, which all have to take their sums in one order:
//   forward   8-12 MB 1.48 / 1.25 / 1.18, 16-20 MB 1.13 / 1.07 / 0.98, 28-32 MB 1.06 / 1.02 / 0.94; lines at 32, 16 and 12 MB.  Beyond 20 MB
//             a residual in fp32 leaves 0.95-1.07 (7163 x 768 22.5 -> 23.4 us), without one 1.01-1.19.
//   backward  8-12 MB 1.27 / 1.19 / 1.06, 12-16 MB 1.14 / 1.12 / 0.98, 16-20 MB 1.06 / 1.01 / 0.93, 24-28 MB 0.98 / 0.92 / 0.85: x and dy, which both
//             launches read, are 32 MB at 16, what the L2s of the dies hold together; lines at 16, 12 and 8 MB.  From x alone the gain ends
//             later (16-20 MB 1.11), from y with a residual earlier (12697 x 576 bf16, 14 MB, 27.2 -> 28.9 us).  Powers of two gain
//             up to the end (24-32 MB 1.03-1.08 in fp32, 1.05-1.24 in bf16; why, no counter was asked).
// Groups of 64 bytes end at 8 MB, backward with a ragged last one at 6 (bf16, 18912 x 200, from y with a residual: 18.3 -> 20.8 us at 7.2 MB,
// 1.1x at 6.2).  The backward sums of two groups, 64 workgroups, lose at any size (16384 x 128 bf16 from x 11.1 -> 13.1 us, from sign
// bytes 11.0 -> 11.7), three gain (1.05-1.2x; at 16384 rows from x 0.97).
// A convolution's rows are merged up to 3072 partials.  Alone, a batch norm behind a 1x1 convolution gains beyond that as well (128 to 2048
// channels, 3072-4096 partials 1.08x in bf16 and 1.13x in fp32, 6144-8192 1.07 and 1.11, 8192-12288 1.04 and 1.05), but inside conv4_x at
// batch 64, whose convolutions leave 49 rows x 64 channels (3136), the step is 2 % slower with them merged (32 steps 77.0
// -> 78.7 ms, up to 4096 or 8192 alike); at batch 19 the 38 rows (2432) gain 4 %, resnet18 and resnext29 do not move.
// Sums of channel g0 + tid % CG to the threads of row group 0 (tid < CG).  Thread = (channel, row group rg of RG): it holds the
// row lanes rg, rg + RG, .. of the 64; the lanes 32, 16, .. RG apart meet in its registers, the others cross LDS behind one
// barrier and meet in the first wave, eight of them as they are read, the rest by exchanges.
template <int CG>
__device__ inline void merge_group(const double* __restrict__ part, int nblk, int C, int g0, f64x2 (&red)[kBnThreads], double* sa,
                                   double* sb)
{
    constexpr int RG = kBnThreads / CG, NL = kMergeLanes / RG;
    const int tid = threadIdx.x, c = g0 + tid % CG, rg = tid / CG;
    double a[NL], b[NL];
#pragma unroll
    for (int j = 0; j < NL; ++j) a[j] = b[j] = 0.0;
    if (c < C)
        for (int k0 = rg; k0 < nblk; k0 += kMergeLanes) {
            f64x2 v[NL];
#pragma unroll
            for (int j = 0; j < NL; ++j) {
                const int k = k0 + RG * j;
                v[j] = k < nblk ? *(const f64x2*)(part + ((int64_t)k * C + c) * 2) : f64x2{0.0, 0.0};
            }
#pragma unroll
            for (int j = 0; j < NL; ++j) {
                a[j] += v[j][0];
                b[j] += v[j][1];
            }
        }
#pragma unroll
    for (int w = NL / 2; w > 0; w >>= 1)
#pragma unroll
        for (int j = 0; j < w; ++j) {
            a[j] += a[j + w];
            b[j] += b[j + w];
        }
    red[tid] = f64x2{a[0], b[0]};
    __syncthreads();
    if (tid >= 64) return;
    // (lane tid reads the row groups tid / CG + (64 / CG) j of its channel)
    const f64x2 s04 = red[tid] + red[tid + 256], s15 = red[tid + 64] + red[tid + 320], s26 = red[tid + 128] + red[tid + 384],
                s37 = red[tid + 192] + red[tid + 448];
    f64x2 t = (s04 + s26) + (s15 + s37);
#pragma unroll
    for (int w = 32; w >= CG; w >>= 1) {
        t[0] += __shfl_xor(t[0], w, 64);
        t[1] += __shfl_xor(t[1], w, 64);
    }
    *sa = t[0];
    *sb = t[1];
}
__device__ inline void merge_channels(const BnLayout& L, const double* part, int nblk, int C, int g0, f64x2 (&red)[kBnThreads],
                                      double* sa, double* sb)
{
    if (L.cg == 64) merge_group<64>(part, nblk, C, g0, red, sa, sb);
    else if (L.cg == 32) merge_group<32>(part, nblk, C, g0, red, sa, sb);
    else merge_group<16>(part, nblk, C, g0, red, sa, sb);
}

template <typename T, int VW, bool RELU, bool HAS_RES>
__global__ __launch_bounds__(kBnThreads) void bn_fwd_merge_apply_kernel(BnApplyIo io0, BnApplyIo io1, BnStatOut o0, BnStatOut o1, BnLayout L,
                                                                  int nblk, int64_t M, int C, double inv_M, float eps,
                                                                  const float* __restrict__ gamma, const float* __restrict__ beta)
{
    typedef typename VecIO<T, VW>::Raw Raw;
    __shared__ f64x2 red[kBnThreads];
    __shared__ float coef[2][64];
    const BnApplyIo io = blockIdx.y ? io1 : io0;
    const BnStatOut o = blockIdx.y ? o1 : o0;
    const T* __restrict__ x = (const T*)io.x;
    const T* __restrict__ res = (const T*)io.res;
    T* __restrict__ y = (T*)io.y;
    int g0;
    const int rb = bn_work_item(L, &g0);
    const int tid = threadIdx.x, vpr = L.cg / VW, rpp = kBnThreads / vpr;
    const int cl = (tid % vpr) * VW, c0 = g0 + cl;
    const bool active = c0 < C;  // (channels come in whole vectors)
    const int64_t r_end = (int64_t)(rb + 1) * L.rows_per_wg < M ? (int64_t)(rb + 1) * L.rows_per_wg : M;
    constexpr int U = 2;
    int64_t r = (int64_t)rb * L.rows_per_wg + tid / vpr;
    Raw xr[U], rr[U];
    auto load = [&]() {
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int64_t ru = r + (int64_t)u * rpp;
            if (!active || ru >= r_end) continue;
            xr[u] = VecIO<T, VW>::raw(x + ru * C + c0);
            if (HAS_RES) rr[u] = VecIO<T, VW>::raw(res + ru * C + c0);
        }
    };
    const bool mine = tid < L.cg && g0 + tid < C;
    const float ga = mine ? gamma[g0 + tid] : 0.f, be = mine ? beta[g0 + tid] : 0.f;
    load();  // on their way while the partials are merged
    double a, b;
    merge_channels(L, o.part, nblk, C, g0, red, &a, &b);
    if (mine) bn_forward_coef(a, b, inv_M, eps, ga, be, o, g0 + tid, C, rb == 0, &coef[0][tid], &coef[1][tid]);
    __syncthreads();
    float sc[VW], sh[VW];
#pragma unroll
    for (int k = 0; k < VW; ++k) {
        sc[k] = active ? coef[0][cl + k] : 0.f;
        sh[k] = active ? coef[1][cl + k] : 0.f;
    }
    while (r < r_end) {
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int64_t ru = r + (int64_t)u * rpp;
            if (!active || ru >= r_end) continue;
            float xv[VW], rv[VW], ov[VW];
            VecIO<T, VW>::unpack(xr[u], xv);
            if (HAS_RES) VecIO<T, VW>::unpack(rr[u], rv);
#pragma unroll
            for (int k = 0; k < VW; ++k) {
                float v = __builtin_fmaf(xv[k], sc[k], sh[k]);
                if (HAS_RES) v += rv[k];
                if (RELU) v = v > 0.f ? v : 0.f;
                ov[k] = v;
            }
            VecIO<T, VW>::store(y + ru * C + c0, ov);
            if (RELU && VW > 1 && io.bits) {
                uint32_t bits = 0u;
#pragma unroll
                for (int k = 0; k < VW; ++k) bits |= (to_float<T>(from_float<T>(ov[k])) > 0.f ? 1u : 0u) << k;
                io.bits[ru * (C / VW) + c0 / VW] = (uint8_t)bits;
            }
        }
        r += (int64_t)U * rpp;
        if (r < r_end) load();
    }
}

// dz = dy*[y>0] (y as stored, or formed again from x: RM as in bn_sums_kernel);  dx = [dx_prev +] c1*dz - c2*x + c0;  dres (+)= dz.  dx_prev is dx itself (accumulate in place)
// or another tensor's gradient that reaches the same input (the shortcut of a pre-activation unit).
template <typename T, int VW, int RM, bool HAS_RES, bool RES_ACC, bool DX_ACC>
__global__ __launch_bounds__(kBnThreads) void bn_bwd_merge_apply_kernel(const T* __restrict__ dy, const T* __restrict__ x,
                                                                  const T* __restrict__ y, T* dx, const T* dx_prev,
                                                                  T* __restrict__ dres, BnGradOut o, BnLayout L, int nblk, int64_t M,
                                                                  int C, double inv_M, const float* __restrict__ fcoef)
{
    typedef typename VecIO<T, VW>::Raw Raw;
    __shared__ f64x2 red[kBnThreads];
    __shared__ float coef[3][64];
    int g0;
    const int rb = bn_work_item(L, &g0);
    const int tid = threadIdx.x, vpr = L.cg / VW, rpp = kBnThreads / vpr;
    const int cl = (tid % vpr) * VW, c0 = g0 + cl;
    const bool active = c0 < C;
    const int64_t r_end = (int64_t)(rb + 1) * L.rows_per_wg < M ? (int64_t)(rb + 1) * L.rows_per_wg : M;
    constexpr int U = 2;
    int64_t r = (int64_t)rb * L.rows_per_wg + tid / vpr;
    Raw gr[U], xr[U], yr[U], pr[U], rr[U];
    uint32_t bits[U];
    auto load = [&]() {
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int64_t ru = r + (int64_t)u * rpp;
            if (!active || ru >= r_end) continue;
            gr[u] = VecIO<T, VW>::raw(dy + ru * C + c0);
            xr[u] = VecIO<T, VW>::raw(x + ru * C + c0);
            if (RM == 1) yr[u] = VecIO<T, VW>::raw(y + ru * C + c0);
            if (RM == 3) bits[u] = ((const uint8_t*)y)[ru * (C / VW) + c0 / VW];
            if (DX_ACC) pr[u] = VecIO<T, VW>::raw(dx_prev + ru * C + c0);
            if (HAS_RES && RES_ACC) rr[u] = VecIO<T, VW>::raw(dres + ru * C + c0);
        }
    };
    const bool mine = tid < L.cg && g0 + tid < C;
    const BnChannel p = bn_channel(o, mine, g0 + tid);
    float c1[VW], c2[VW], c3[VW], fsc[VW], fsh[VW];
    if (RM == 2)
#pragma unroll
        for (int k = 0; k < VW; ++k) {
            fsc[k] = active ? fcoef[c0 + k] : 0.f;
            fsh[k] = active ? fcoef[C + c0 + k] : 0.f;
        }
    load();
    double a, b;
    merge_channels(L, o.part, nblk, C, g0, red, &a, &b);
    if (mine) bn_backward_coef(a, b, inv_M, o, p, g0 + tid, rb == 0, &coef[0][tid], &coef[1][tid], &coef[2][tid]);
    __syncthreads();
#pragma unroll
    for (int k = 0; k < VW; ++k) {
        c1[k] = active ? coef[0][cl + k] : 0.f;
        c2[k] = active ? coef[1][cl + k] : 0.f;
        c3[k] = active ? coef[2][cl + k] : 0.f;
    }
    while (r < r_end) {
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int64_t ru = r + (int64_t)u * rpp;
            if (!active || ru >= r_end) continue;
            float gv[VW], xv[VW], yv[VW], pv[VW], rv[VW], ov[VW];
            VecIO<T, VW>::unpack(gr[u], gv);
            VecIO<T, VW>::unpack(xr[u], xv);
            if (RM == 1) VecIO<T, VW>::unpack(yr[u], yv);
            if (DX_ACC) VecIO<T, VW>::unpack(pr[u], pv);
            if (HAS_RES && RES_ACC) VecIO<T, VW>::unpack(rr[u], rv);
#pragma unroll
            for (int k = 0; k < VW; ++k) {
                const bool on = RM == 0 ? true
                                : RM == 1 ? yv[k] > 0.f
                                : RM == 2 ? bn_value<T>(xv[k], fsc[k], fsh[k]) > 0.f : ((bits[u] >> k) & 1u) != 0;
                const float dz = on ? gv[k] : 0.f;
                const float d = c1[k] * dz - c2[k] * xv[k] + c3[k];
                ov[k] = DX_ACC ? pv[k] + d : d;
                if (HAS_RES) rv[k] = RES_ACC ? rv[k] + dz : dz;
            }
            VecIO<T, VW>::store(dx + ru * C + c0, ov);
            if (HAS_RES) VecIO<T, VW>::store(dres + ru * C + c0, rv);
        }
        r += (int64_t)U * rpp;
        if (r < r_end) load();
    }
}

// ---- batch norm + ReLU + max pool in one pass (bf16) ---------------------------------------------------------
// For a batch norm whose only reader is a max pool: y = relu(scale * x + shift) is formed per window tap exactly as
// bn_fwd_apply_kernel would store it (same expression, same rounding) and never written; the pooled tensor and the
// chosen taps are the same bits the two separate kernels leave.  After the ReLU every value is a non-negative bf16, so
// values order like their bit patterns: per channel the kernel keeps one 32-bit key = value bits << 16 | (15 - tap) and
// takes the unsigned maximum, which is the largest value and, among equal ones, the first tap of the row-major window
// scan (the rule of maxpool_fwd_kernel).  A thread owns 8 consecutive channels of one output pixel; all taps of a
// window are loaded before the first is used (out-of-image taps read a clamped address and are masked out).
// Workgroup ids are dealt round-robin to the 8 XCDs; the remap gives each XCD one contiguous eighth of the output per
// grid-stride trip, so the input rows two neighbouring output rows share are fetched into one L2, once.
template <int K>
__global__ __launch_bounds__(kThreads) void bn_relu_maxpool_bf16_kernel(const bf16_t* __restrict__ x,
                                                                        const float* __restrict__ coef,
                                                                        bf16_t* __restrict__ y, uint8_t* __restrict__ arg,
                                                                        int N, int H, int W, int C, int Ho, int Wo, int k_rt,
                                                                        int stride, int pad)
{
    const int k = K ? K : k_rt;
    const uint32_t cv = (uint32_t)(C / 8);
    const uint32_t total = (uint32_t)N * Ho * Wo * cv;
    const uint32_t nb = gridDim.x, lb = (blockIdx.x & 7u) * (nb >> 3) + (blockIdx.x >> 3);
    for (uint32_t i = lb * kThreads + threadIdx.x; i < total; i += nb * kThreads) {
        const uint32_t t = i / cv;
        const int c = (int)(i - t * cv) * 8;
        const uint32_t t2 = t / (uint32_t)Wo;
        const int wo = (int)(t - t2 * Wo);
        const int n = (int)(t2 / (uint32_t)Ho), ho = (int)(t2 - (uint32_t)n * Ho);
        float sc[8], sh[8];
#pragma unroll
        for (int e = 0; e < 8; e += 4) {
            const f32x4 a = *(const f32x4*)(coef + c + e), b = *(const f32x4*)(coef + C + c + e);
            sc[e] = a.x; sc[e + 1] = a.y; sc[e + 2] = a.z; sc[e + 3] = a.w;
            sh[e] = b.x; sh[e + 1] = b.y; sh[e + 2] = b.z; sh[e + 3] = b.w;
        }
        uint32_t key[8];
#pragma unroll
        for (int e = 0; e < 8; ++e) key[e] = 0u;
        auto tap = [&](int r, int s, u32x4 v) {
            const int hi = ho * stride + r - pad, wi = wo * stride + s - pad;
            const bool valid = (unsigned)hi < (unsigned)H && (unsigned)wi < (unsigned)W;
            // A tap outside the image was loaded from the clamped address, which is a pixel of this same window (pad < k)
            // whose own tap is inside: its value is in the race anyway, and with code 0 the copy loses every tie.
            const uint32_t code = valid ? (uint32_t)(15 - (r * k + s)) : 0u;
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                float lo = __builtin_fmaf(__uint_as_float(v[e] << 16), sc[2 * e], sh[2 * e]);
                float hi2 = __builtin_fmaf(__uint_as_float(v[e] & 0xffff0000u), sc[2 * e + 1], sh[2 * e + 1]);
                lo = lo > 0.f ? lo : 0.f;
                hi2 = hi2 > 0.f ? hi2 : 0.f;
                const uint32_t pk = pack_bf16x2(lo, hi2);
                const uint32_t k0 = (pk << 16) | code, k1 = (pk & 0xffff0000u) | code;
                key[2 * e] = key[2 * e] > k0 ? key[2 * e] : k0;
                key[2 * e + 1] = key[2 * e + 1] > k1 ? key[2 * e + 1] : k1;
            }
        };
        auto addr = [&](int r, int s) {
            int hi = ho * stride + r - pad, wi = wo * stride + s - pad;
            hi = hi < 0 ? 0 : (hi >= H ? H - 1 : hi);
            wi = wi < 0 ? 0 : (wi >= W ? W - 1 : wi);
            return (const u32x4*)(x + (((int64_t)n * H + hi) * W + wi) * C + c);
        };
        if (K) {
            // element offsets of the window's (clamped) rows and columns: one sum per tap
            uint32_t roff[K ? K : 1], coff[K ? K : 1];
#pragma unroll
            for (int r = 0; r < K; ++r) {
                int hi = ho * stride + r - pad, wi = wo * stride + r - pad;
                hi = hi < 0 ? 0 : (hi >= H ? H - 1 : hi);
                wi = wi < 0 ? 0 : (wi >= W ? W - 1 : wi);
                roff[r] = (uint32_t)((n * H + hi) * W) * (uint32_t)C + (uint32_t)c;
                coff[r] = (uint32_t)wi * (uint32_t)C;
            }
            u32x4 v[K ? K * K : 1];
#pragma unroll
            for (int r = 0; r < K; ++r)
#pragma unroll
                for (int s = 0; s < K; ++s) v[r * K + s] = *(const u32x4*)(x + (roff[r] + coff[s]));
#pragma unroll
            for (int r = 0; r < K; ++r)
#pragma unroll
                for (int s = 0; s < K; ++s) tap(r, s, v[r * K + s]);
        } else {
            for (int r = 0; r < k; ++r)
                for (int s = 0; s < k; ++s) tap(r, s, *addr(r, s));
        }
        u32x4 o;
        uint32_t a0 = 0u, a1 = 0u;
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            o[e] = (key[2 * e] >> 16) | (key[2 * e + 1] & 0xffff0000u);
            a0 |= (15u - (key[e] & 15u)) << (8 * e);
            a1 |= (15u - (key[4 + e] & 15u)) << (8 * e);
        }
        *(u32x4*)(y + (int64_t)i * 8) = o;
        if (arg) *(u32x2*)(arg + (int64_t)i * 8) = u32x2{a0, a1};
    }
}

// ---- backward of batch norm + ReLU + (3 x 3 / stride 2 / pad 1 max pool) without the pool's input gradient ----------
// The pool's backward gives input pixel (hi, wi) the sum of the output gradients of the windows whose recorded tap is that
// pixel.  Seen from a 2 x 2 cell of input pixels (2a + i, 2b + j) only the four windows (a + u, b + v), u, v in {0, 1},
// can have chosen one of them, each with a fixed tap code r * 3 + s per pixel:
//     pixel (0,0): window (0,0) tap 4                       pixel (0,1): windows (0,1) tap 3, (0,0) tap 5
//     pixel (1,0): windows (1,0) tap 1, (0,0) tap 7         pixel (1,1): windows (1,1) tap 0, (1,0) tap 2, (0,1) tap 6, (0,0) tap 8
// (listed in the order maxpool_bwd_kernel adds them: window rows, then columns, descending).  A thread owns 8 channels
// of one cell: it loads the four windows' gradients and taps once, forms the four pixels' gradients -- rounded to bf16,
// the values maxpool_bwd_kernel would have stored -- and goes on with the batch norm's backward for those pixels.  The
// ReLU is decided from x (RM = 2 of bn_sums_kernel).  Windows past the last row / column do not exist (Ho = H / 2).
struct PoolCells {
    const bf16_t* dpool;   // [N][Ho][Wo][C]
    const uint8_t* arg;    // [N][Ho][Wo][C]
    int H, W, Ho, Wo;
    uint32_t wo_mul, wo_sh, ho_mul, ho_sh;  // cell / Wo and (cell / Wo) / Ho by multiplication
};
__device__ inline void pool_cell_grad(const PoolCells& p, int n, int a, int b, int c0, int C, float (&g)[4][8])
{
    u32x4 gw[4];
    u32x2 aw[4];
    bool ok[4];
#pragma unroll
    for (int q = 0; q < 4; ++q) {
        const int ho = a + (q >> 1), wo = b + (q & 1);
        ok[q] = ho < p.Ho && wo < p.Wo;
        const int64_t o = (((int64_t)n * p.Ho + (ho < p.Ho ? ho : a)) * p.Wo + (wo < p.Wo ? wo : b)) * C + c0;
        gw[q] = *(const u32x4*)(p.dpool + o);
        aw[q] = *(const u32x2*)(p.arg + o);
    }
#pragma unroll
    for (int v = 0; v < 8; ++v) {
        float gq[4];
        uint32_t tq[4];
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            const uint32_t w = gw[q][v >> 1];
            gq[q] = __uint_as_float((v & 1) ? (w & 0xffff0000u) : (w << 16));
            tq[q] = ok[q] ? ((aw[q][v >> 2] >> (8 * (v & 3))) & 0xffu) : 255u;
        }
        float s;
        s = tq[0] == 4u ? gq[0] : 0.f;
        g[0][v] = to_float<bf16_t>(from_float<bf16_t>(s));
        s = tq[1] == 3u ? gq[1] : 0.f;
        if (tq[0] == 5u) s += gq[0];
        g[1][v] = to_float<bf16_t>(from_float<bf16_t>(s));
        s = tq[2] == 1u ? gq[2] : 0.f;
        if (tq[0] == 7u) s += gq[0];
        g[2][v] = to_float<bf16_t>(from_float<bf16_t>(s));
        s = tq[3] == 0u ? gq[3] : 0.f;
        if (tq[2] == 2u) s += gq[2];
        if (tq[1] == 6u) s += gq[1];
        if (tq[0] == 8u) s += gq[0];
        g[3][v] = to_float<bf16_t>(from_float<bf16_t>(s));
    }
}

// s0 = sum dz, s1 = sum dz * xhat over the cells of a workgroup (thread = channel vector tid % cv, cell lane tid / cv)
__global__ __launch_bounds__(kThreads) void bn_pool_bwd_reduce_kernel(const bf16_t* __restrict__ x, PoolCells p,
                                                                      const float* __restrict__ mean,
                                                                      const float* __restrict__ invstd,
                                                                      const float* __restrict__ fcoef,
                                                                      double* __restrict__ part, uint32_t cells, int C,
                                                                      RowLayout L, int cells_per_block)
{
    __shared__ double red[8][kThreads][2];
    const int tid = threadIdx.x;
    const int cvi = blockIdx.y * L.cvb + tid % L.cvb;
    const int clane = tid / L.cvb;
    const bool active = clane < L.rl && cvi < L.cv;
    const int c0 = cvi * 8;
    double s0[8], s1[8];
    float mu[8], is[8], fsc[8], fsh[8];
#pragma unroll
    for (int i = 0; i < 8; ++i) {
        s0[i] = s1[i] = 0.0;
        if (active) {
            mu[i] = mean[c0 + i];
            is[i] = invstd[c0 + i];
            fsc[i] = fcoef[c0 + i];
            fsh[i] = fcoef[C + c0 + i];
        }
    }
    const uint32_t c_begin = blockIdx.x * (uint32_t)cells_per_block;
    const uint32_t c_end = c_begin + cells_per_block < cells ? c_begin + cells_per_block : cells;
    if (active)
        for (uint32_t cell = c_begin + clane; cell < c_end; cell += L.rl) {
            const uint32_t t2 = fast_div(cell, p.wo_mul, p.wo_sh);
            const int b = (int)(cell - t2 * p.Wo);
            const int n = (int)fast_div(t2, p.ho_mul, p.ho_sh), a = (int)(t2 - (uint32_t)n * p.Ho);
            const bf16_t* x0 = x + (((int64_t)n * p.H + 2 * a) * p.W + 2 * b) * C + c0;
            float xv[4][8], g[4][8];
#pragma unroll
            for (int q = 0; q < 4; ++q) VecIO<bf16_t, 8>::load(x0 + ((int64_t)(q >> 1) * p.W + (q & 1)) * C, xv[q]);
            pool_cell_grad(p, n, a, b, c0, C, g);
#pragma unroll
            for (int q = 0; q < 4; ++q)
#pragma unroll
                for (int i = 0; i < 8; ++i) {
                    const float dz = bn_value<bf16_t>(xv[q][i], fsc[i], fsh[i]) > 0.f ? g[q][i] : 0.f;
                    s0[i] += (double)dz;
                    s1[i] += (double)(dz * ((xv[q][i] - mu[i]) * is[i]));
                }
        }
    combine_row_lanes<8>(s0, s1, red, active, clane, L, part + (int64_t)blockIdx.x * C * 2, c0);
}

// dx = [dx_prev +] c1*dz - c2*x + c0 for the four pixels of a cell; item i = (cell i / cv, channel vector i % cv)
template <bool DX_ACC>
__global__ __launch_bounds__(kThreads) void bn_pool_bwd_apply_kernel(const bf16_t* __restrict__ x, PoolCells p, bf16_t* dx,
                                                                     const bf16_t* dx_prev, const float* __restrict__ coef,
                                                                     const float* __restrict__ fcoef, uint32_t items, int C,
                                                                     uint32_t cv, uint32_t cv_mul, uint32_t cv_sh)
{
    const uint32_t nb = gridDim.x, lb = (blockIdx.x & 7u) * (nb >> 3) + (blockIdx.x >> 3);  // an XCD walks neighbouring cells
    for (uint32_t i = lb * kThreads + threadIdx.x; i < items; i += nb * kThreads) {
        const uint32_t cell = fast_div(i, cv_mul, cv_sh);
        const int c0 = (int)(i - cell * cv) * 8;
        const uint32_t t2 = fast_div(cell, p.wo_mul, p.wo_sh);
        const int b = (int)(cell - t2 * p.Wo);
        const int n = (int)fast_div(t2, p.ho_mul, p.ho_sh), a = (int)(t2 - (uint32_t)n * p.Ho);
        const int64_t o0 = (((int64_t)n * p.H + 2 * a) * p.W + 2 * b) * C + c0;
        float xv[4][8], g[4][8], ov[4][8];
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            const int64_t o = o0 + ((int64_t)(q >> 1) * p.W + (q & 1)) * C;
            VecIO<bf16_t, 8>::load(x + o, xv[q]);
            if (DX_ACC) VecIO<bf16_t, 8>::load(dx_prev + o, ov[q]);
        }
        pool_cell_grad(p, n, a, b, c0, C, g);
#pragma unroll
        for (int q = 0; q < 4; ++q) {
#pragma unroll
            for (int k = 0; k < 8; ++k) {
                const float dz = bn_value<bf16_t>(xv[q][k], fcoef[c0 + k], fcoef[C + c0 + k]) > 0.f ? g[q][k] : 0.f;
                const float d = coef[c0 + k] * dz - coef[C + c0 + k] * xv[q][k] + coef[2 * C + c0 + k];
                ov[q][k] = DX_ACC ? ov[q][k] + d : d;
            }
            VecIO<bf16_t, 8>::store(dx + o0 + ((int64_t)(q >> 1) * p.W + (q & 1)) * C, ov[q]);
        }
    }
}

// Channels per group: 128 bytes of a row (16 channels at least), smaller where that pads the channel count by less.
int bn_channel_group(int C, int VW)
{
    int best = VW == 8 ? 64 : 32;
    for (int cg = best / 2; cg >= 16; cg /= 2)
        if (ceil_div(C, cg) * cg * 9 < ceil_div(C, best) * best * 8) best = cg;
    return best;
}
BnLayout bn_layout(int64_t M, int C, int VW, int64_t blocks)
{
    BnLayout L;
    L.cg = bn_channel_group(C, VW);
    L.groups = ceil_div(C, L.cg);
    const int rpp = kBnThreads / (L.cg / VW);
    const int64_t trips = (M + blocks * rpp - 1) / (blocks * rpp);
    L.rows_per_wg = (int)trips * rpp;
    L.row_blocks = ceil_div(M, L.rows_per_wg);
    return L;
}
// Up to 256 workgroups over all groups and instances, fewer where a thread would get less than two vectors.
BnLayout merge_layout(int64_t M, int C, int VW, int instances)
{
    const int cg = bn_channel_group(C, VW), groups = ceil_div(C, cg);
    const int64_t rpp = kBnThreads / (cg / VW);
    int64_t blocks = (256 + groups * instances - 1) / (groups * instances);
    const int64_t most = (M + 2 * rpp - 1) / (2 * rpp);
    if (blocks > most) blocks = most;
    return bn_layout(M, C, VW, blocks < 1 ? 1 : blocks);
}
// The largest tensor whose sums are taken by channel groups or, behind a convolution, merged by the apply kernel (the lines: see
// "finalize inside the apply kernels").
int64_t wide_tensor_bytes(int C, int VW, int cg, int esz, bool backward)
{
    constexpr int64_t MB = 1 << 20;
    const bool whole = C % cg == 0;  // no group shares a cache line with the next
    if (cg * esz < 128) return (whole || !backward ? 8 : 6) * MB * (cg * esz) / 64;
    if (!backward) return (whole ? 32 : VW > 1 ? 16 : 12) * MB;
    return ((C & (C - 1)) == 0 ? 32 : whole ? 16 : VW > 1 ? 12 : 8) * MB;
}
// wide: the partials are those of bn_group_sums_kernel or of a convolution.
inline bool merges(int64_t M, int C, int VW, int esz, int nblk, bool wide, bool backward)
{
    const int cg = bn_channel_group(C, VW);
    wide = wide && C >= kWideChannels;
    return M * C * esz <= (wide ? wide_tensor_bytes(C, VW, cg, esz, backward) : kMergeTensorBytes) &&
           (int64_t)nblk * cg <= (wide ? kWideConvEntries : kMergeEntries);
}
// Work items of bn_group_sums_kernel: at most kMergeEntries / cg runs of rows, two rows a thread or more; false where the tensor has
// too few channels or is too large for so few.
bool group_sums_layout(int64_t M, int C, int VW, int esz, bool backward, BnLayout* L)
{
    const int cg = bn_channel_group(C, VW), rpp = kBnThreads / (cg / VW);
    int64_t runs = kMergeEntries / cg;
    const int64_t most = (M + 2 * rpp - 1) / (2 * rpp);
    if (runs > most) runs = most;
    *L = bn_layout(M, C, VW, runs);
    if (backward && L->groups * (kMergeEntries / cg) < kWideBackwardWgs) return false;
    return C >= kWideChannels && M * C * esz <= wide_tensor_bytes(C, VW, cg, esz, backward) && (int64_t)L->rows_per_wg * cg * esz <= kWideRunBytes;
}

int plan_rows(int64_t M, const RowLayout& L, int* nblk)
{
    // every thread should see >= 4 rows (one trip of the summing loop); at most kMaxPartialBlocks workgroups
    int64_t rows = (int64_t)L.rl * 4;
    int64_t blocks = (M + rows - 1) / rows;
    if (blocks > kMaxPartialBlocks) {
        blocks = kMaxPartialBlocks;
        rows = (M + blocks - 1) / blocks;
        blocks = (M + rows - 1) / rows;
    }
    *nblk = (int)blocks;
    return (int)rows;
}

inline int apply_grid(int64_t nvec)
{
    int64_t g = (nvec + kThreads - 1) / kThreads;
    const int64_t cap = 256 * 16;
    return (int)(g < cap ? (g < 1 ? 1 : g) : cap);
}

template <typename T, int VW>
int bn_forward_t(const void* x, const void* res, void* y, const float* gamma, const float* beta, float eps, int64_t M,
                 int C, bool relu, const BnBuffers& buf, hipStream_t st, int presummed, const BnForwardTwin* tw, bool stats_only,
                 uint8_t* relu_bits)
{
    const RowLayout L = make_layout(C, VW);
    int nblk;
    const int rows = plan_rows(M, L, &nblk);
    const unsigned ni = tw ? 2 : 1;
    const dim3 grid(nblk, ceil_div(L.cv, L.cvb), ni);
    const double tensor_bytes = (double)M * C * sizeof(T) * ni;
    BnLayout gl;
    if (presummed > 0) {
        nblk = presummed;
    } else if (group_sums_layout(M, C, VW, sizeof(T), false, &gl)) {  // (of every form: the bits of the statistics do not depend on it)
        nblk = gl.row_blocks;
        ProfScope ps(sizeof(T) == 2 ? "bn_stats<bf16>" : "bn_stats<fp32>", tensor_bytes, 1);
        DSP_LAUNCH(ps, (bn_group_sums_kernel<T, VW, 0, 0>), dim3((unsigned)(gl.groups * gl.row_blocks), ni), dim3(kBnThreads), 0, st,
                   (const T*)x, (const T*)nullptr, (const T*)nullptr, (const float*)nullptr, (const float*)nullptr, buf.partial, M, C,
                   gl, (const T*)(tw ? tw->x : nullptr), tw ? tw->buf.partial : nullptr, (const float*)nullptr);
    } else {
        ProfScope ps(sizeof(T) == 2 ? "bn_stats<bf16>" : "bn_stats<fp32>", tensor_bytes, 1);
        DSP_LAUNCH(ps, (bn_sums_kernel<T, VW, 0, 0>), grid, dim3(kThreads), 0, st, (const T*)x, (const T*)nullptr,
                   (const T*)nullptr, (const float*)nullptr, (const float*)nullptr, buf.partial, M, C, L, rows,
                   (const T*)(tw ? tw->x : nullptr), tw ? tw->buf.partial : nullptr, AddOut<T>{}, (const float*)nullptr);
    }
    const BnStatOut o0{buf.partial, buf.mean, buf.invstd, buf.coef};
    const BnStatOut o1 = tw ? BnStatOut{tw->buf.partial, tw->buf.mean, tw->buf.invstd, tw->buf.coef} : o0;
    const BnApplyIo io0{x, res, y, buf.coef, relu_bits};
    const BnApplyIo io1 = tw ? BnApplyIo{tw->x, tw->res, tw->y, tw->buf.coef, tw->relu_bits} : io0;
    if (!stats_only && merges(M, C, VW, sizeof(T), nblk, true, false)) {
        const BnLayout ml = merge_layout(M, C, VW, (int)ni);
        ProfScope ps(sizeof(T) == 2 ? "bn_merge_apply_relu<bf16>" : "bn_merge_apply_relu<fp32>", tensor_bytes * (res ? 3 : 2), 1);
#define BN_APPLY(R, H)                                                                                                             \
    DSP_LAUNCH(ps, (bn_fwd_merge_apply_kernel<T, VW, R, H>), dim3((unsigned)(ml.groups * ml.row_blocks), ni), dim3(kBnThreads), 0, st, \
               io0, io1, o0, o1, ml, nblk, M, C, 1.0 / (double)M, eps, gamma, beta)
        if (relu) {
            if (res) BN_APPLY(true, true); else BN_APPLY(true, false);
        } else {
            if (res) BN_APPLY(false, true); else BN_APPLY(false, false);
        }
#undef BN_APPLY
        DSP_HIP(hipGetLastError());
        return DSP_OK;
    }
    {
        ProfScope ps("bn_fwd_finalize", (double)nblk * C * 16.0 * ni, 1);
        DSP_LAUNCH(ps, bn_fwd_finalize_kernel, dim3(ceil_div(C, 4), ni), dim3(kMergeLanes * 4), 0, st, o0, o1, nblk, C,
                   1.0 / (double)M, eps, gamma, beta);
    }
    if (stats_only) {
        DSP_HIP(hipGetLastError());
        return DSP_OK;
    }
    const int64_t nvec = M * (C / VW);
    const dim3 ag(apply_grid(nvec), ni);
    ProfScope ps(sizeof(T) == 2 ? "bn_apply_relu<bf16>" : "bn_apply_relu<fp32>", tensor_bytes * (res ? 3 : 2), 1);
#define BN_APPLY(R, H) \
    DSP_LAUNCH(ps, (bn_fwd_apply_kernel<T, VW, R, H>), ag, dim3(kThreads), 0, st, io0, io1, nvec, C, L.cv)
    if (relu) {
        if (res) BN_APPLY(true, true); else BN_APPLY(true, false);
    } else {
        if (res) BN_APPLY(false, true); else BN_APPLY(false, false);
    }
#undef BN_APPLY
    DSP_HIP(hipGetLastError());
    return DSP_OK;
}

template <typename T, int VW, int RM>
int bn_backward_t(const void* dy, const void* x, const void* y, void* dx, void* dres, bool racc, bool xacc,
                  const float* gamma, float* dgamma, float* dbeta, int64_t M, int C, const BnBuffers& buf, hipStream_t st,
                  const void* dx_prev, const float* fcoef)
{
    const RowLayout L = make_layout(C, VW);
    int nblk;
    const int rows = plan_rows(M, L, &nblk);
    const dim3 grid(nblk, ceil_div(L.cv, L.cvb));
    const double tensor_bytes = (double)M * C * sizeof(T);
    BnLayout gl;
    const bool grouped = group_sums_layout(M, C, VW, sizeof(T), true, &gl);
    if (grouped) nblk = gl.row_blocks;
    {
        ProfScope ps(sizeof(T) == 2 ? "bn_bwd_reduce<bf16>" : "bn_bwd_reduce<fp32>", tensor_bytes * (RM == 1 ? 3 : 2) + (RM == 3 ? tensor_bytes / (VW * sizeof(T)) : 0.0), 1);
        if (grouped)
            DSP_LAUNCH(ps, (bn_group_sums_kernel<T, VW, 1, RM>), dim3((unsigned)(gl.groups * gl.row_blocks)), dim3(kBnThreads), 0, st,
                       (const T*)x, (const T*)dy, (const T*)y, (const float*)buf.mean, (const float*)buf.invstd, buf.partial, M, C, gl,
                       (const T*)nullptr, (double*)nullptr, fcoef);
        else
            DSP_LAUNCH(ps, (bn_sums_kernel<T, VW, 1, RM>), grid, dim3(kThreads), 0, st, (const T*)x, (const T*)dy,
                   (const T*)y, (const float*)buf.mean, (const float*)buf.invstd, buf.partial, M, C, L, rows,
                   (const T*)nullptr, (double*)nullptr, AddOut<T>{}, fcoef);
    }
    const BnGradOut o{buf.partial, gamma, buf.mean, buf.invstd, dgamma, dbeta, buf.coef};
    // reads dy, x (y too where the ReLU is decided from the stored output, and the old values where it accumulates);
    // writes dx (and dres)
    const double apply_bytes = tensor_bytes * (2 + (RM == 1 ? 1 : 0) + 1 + (xacc ? 1 : 0) + (dres ? 1 + (racc ? 1 : 0) : 0)) +
                               (RM == 3 ? tensor_bytes / (VW * sizeof(T)) : 0.0);
    if (merges(M, C, VW, sizeof(T), nblk, grouped, true)) {
        const BnLayout ml = merge_layout(M, C, VW, 1);
        ProfScope ps(sizeof(T) == 2 ? "bn_bwd_merge_apply<bf16>" : "bn_bwd_merge_apply<fp32>", apply_bytes, 1);
#define BN_BAPPLY(H, RA, XA)                                                                                               \
    DSP_LAUNCH(ps, (bn_bwd_merge_apply_kernel<T, VW, (H && RM == 2) ? 1 : RM, H, RA, XA>),                                 \
               dim3((unsigned)(ml.groups * ml.row_blocks)), dim3(kBnThreads), 0, st, (const T*)dy, (const T*)x, (const T*)y, \
               (T*)dx, (const T*)dx_prev, (T*)dres, o, ml, nblk, M, C, 1.0 / (double)M, fcoef)
        if (dres) {
            if (racc) { if (xacc) BN_BAPPLY(true, true, true); else BN_BAPPLY(true, true, false); }
            else      { if (xacc) BN_BAPPLY(true, false, true); else BN_BAPPLY(true, false, false); }
        } else {
            if (xacc) BN_BAPPLY(false, false, true); else BN_BAPPLY(false, false, false);
        }
#undef BN_BAPPLY
        DSP_HIP(hipGetLastError());
        return DSP_OK;
    }
    {
        ProfScope ps("bn_bwd_finalize", (double)nblk * C * 16.0, 1);
        DSP_LAUNCH(ps, bn_bwd_finalize_kernel, dim3(ceil_div(C, 4)), dim3(kMergeLanes * 4), 0, st, o, nblk, C, 1.0 / (double)M);
    }
    const int64_t nvec = M * (C / VW);
    const dim3 ag(apply_grid(nvec));
    ProfScope ps(sizeof(T) == 2 ? "bn_bwd_apply<bf16>" : "bn_bwd_apply<fp32>", apply_bytes, 1);
#define BN_BAPPLY(H, RA, XA)                                                                                   \
    DSP_LAUNCH(ps, (bn_bwd_apply_kernel<T, VW, (H && RM == 2) ? 1 : RM, H, RA, XA>), ag, dim3(kThreads), 0, st, \
               (const T*)dy, (const T*)x, (const T*)y, (T*)dx, (const T*)dx_prev, (T*)dres, (const float*)buf.coef,   \
               nvec, C, L.cv, fcoef)
    if (dres) {
        if (racc) { if (xacc) BN_BAPPLY(true, true, true); else BN_BAPPLY(true, true, false); }
        else      { if (xacc) BN_BAPPLY(true, false, true); else BN_BAPPLY(true, false, false); }
    } else {
        if (xacc) BN_BAPPLY(false, false, true); else BN_BAPPLY(false, false, false);
    }
#undef BN_BAPPLY
    DSP_HIP(hipGetLastError());
    return DSP_OK;
}

}  // namespace

int bn_max_partial_blocks() { return kMaxPartialBlocks; }

template <typename T, int VW>
int add_stats_t(const void* a, const void* b, void* y, int64_t M, int C, double* partial, hipStream_t st,
                const AddStatsTwin* tw)
{
    const RowLayout L = make_layout(C, VW);
    int nblk;
    const int rows = plan_rows(M, L, &nblk);
    const unsigned ni = tw ? 2 : 1;
    const dim3 grid(nblk, ceil_div(L.cv, L.cvb), ni);
    ProfScope ps("add_fwd_stats", (double)M * C * sizeof(T) * 3.0 * ni, 1);
    DSP_LAUNCH(ps, (bn_sums_kernel<T, VW, 2, 0>), grid, dim3(kThreads), 0, st, (const T*)a, (const T*)b, (const T*)nullptr,
               (const float*)nullptr, (const float*)nullptr, partial, M, C, L, rows, (const T*)(tw ? tw->a : nullptr),
               tw ? tw->partial : nullptr, (AddOut<T>{(T*)y, (const T*)(tw ? tw->b : nullptr), (T*)(tw ? tw->y : nullptr)}),
               (const float*)nullptr);
    DSP_HIP(hipGetLastError());
    return DSP_OK;
}

static bool add_stats_vec(int dtype, int C) { return C % (dtype == DSP_BF16 ? 8 : 4) == 0; }

int add_stats_blocks(int dtype, int64_t M, int C)
{
    const int vw = add_stats_vec(dtype, C) ? (dtype == DSP_BF16 ? 8 : 4) : 1;
    int nblk;
    (void)plan_rows(M, make_layout(C, vw), &nblk);
    return nblk;
}

int launch_add_forward_stats(int dtype, const void* a, const void* b, void* y, int64_t M, int C, double* partial,
                             hipStream_t st, const AddStatsTwin* twin)
{
    DSP_REQUIRE(a && b && y && partial && M > 0 && C > 0, DSP_EINVAL, "add + statistics: bad argument");
    if (twin) DSP_REQUIRE(twin->a && twin->b && twin->y && twin->partial, DSP_EINVAL, "add + statistics: incomplete second instance");
    if (dtype == DSP_BF16) {
        if (add_stats_vec(dtype, C)) return add_stats_t<bf16_t, 8>(a, b, y, M, C, partial, st, twin);
        return add_stats_t<bf16_t, 1>(a, b, y, M, C, partial, st, twin);
    }
    if (add_stats_vec(dtype, C)) return add_stats_t<float, 4>(a, b, y, M, C, partial, st, twin);
    return add_stats_t<float, 1>(a, b, y, M, C, partial, st, twin);
}

int launch_bn_forward(int dtype, const void* x, const void* res, void* y, const float* gamma, const float* beta,
                      float eps, int64_t M, int C, bool relu, const BnBuffers& buf, hipStream_t st, int presummed,
                      const BnForwardTwin* twin, bool stats_only, uint8_t* relu_bits)
{
    DSP_REQUIRE(M > 0 && C > 0 && presummed >= 0, DSP_EINVAL, "bn: bad shape");
    DSP_REQUIRE(!relu_bits || (relu && bn_relu_bits_bytes(dtype, M, C) > 0), DSP_EINVAL, "bn forward: sign bytes need a ReLU and channels in whole 16-byte runs");
    if (twin)
        DSP_REQUIRE(twin->x && (twin->y || stats_only) && (twin->res != nullptr) == (res != nullptr), DSP_EINVAL,
                    "bn forward: incomplete second instance");
    if (dtype == DSP_BF16) {
        if (C % 8 == 0) return bn_forward_t<bf16_t, 8>(x, res, y, gamma, beta, eps, M, C, relu, buf, st, presummed, twin, stats_only, relu_bits);
        return bn_forward_t<bf16_t, 1>(x, res, y, gamma, beta, eps, M, C, relu, buf, st, presummed, twin, stats_only, nullptr);
    }
    if (C % 4 == 0) return bn_forward_t<float, 4>(x, res, y, gamma, beta, eps, M, C, relu, buf, st, presummed, twin, stats_only, relu_bits);
    return bn_forward_t<float, 1>(x, res, y, gamma, beta, eps, M, C, relu, buf, st, presummed, twin, stats_only, nullptr);
}

int launch_bn_apply(int dtype, const void* x, void* y, const float* coef, int64_t M, int C, bool relu, hipStream_t st)
{
    DSP_REQUIRE(M > 0 && C > 0 && x && y && coef, DSP_EINVAL, "bn apply: bad argument");
    const BnApplyIo io{x, nullptr, y, coef, nullptr};
    const double bytes = (double)M * C * dtype_size(dtype) * 2;
#define BN_APPLY1(T, VW)                                                                                               \
    do {                                                                                                               \
        const int64_t nvec = M * (C / VW);                                                                             \
        ProfScope ps(sizeof(T) == 2 ? "bn_apply_relu<bf16>" : "bn_apply_relu<fp32>", bytes, 1);                        \
        if (relu) DSP_LAUNCH(ps, (bn_fwd_apply_kernel<T, VW, true, false>), dim3(apply_grid(nvec)), dim3(kThreads), 0, st, io, io, nvec, C, C / VW); \
        else DSP_LAUNCH(ps, (bn_fwd_apply_kernel<T, VW, false, false>), dim3(apply_grid(nvec)), dim3(kThreads), 0, st, io, io, nvec, C, C / VW);    \
    } while (0)
    if (dtype == DSP_BF16) {
        if (C % 8 == 0) BN_APPLY1(bf16_t, 8); else BN_APPLY1(bf16_t, 1);
    } else {
        if (C % 4 == 0) BN_APPLY1(float, 4); else BN_APPLY1(float, 1);
    }
#undef BN_APPLY1
    DSP_HIP(hipGetLastError());
    return DSP_OK;
}

bool bn_relu_maxpool_supported(int dtype, int C, int k) { return dtype == DSP_BF16 && C % 8 == 0 && k >= 1 && k <= 4; }

int launch_bn_relu_maxpool_forward(int dtype, const void* x, const float* coef, void* y, uint8_t* argmax, int N, int H, int W,
                                   int C, int k, int stride, int pad, hipStream_t st)
{
    DSP_REQUIRE(bn_relu_maxpool_supported(dtype, C, k), DSP_EINVAL, "bn + relu + max pool: bf16, channels in runs of 8, window <= 4 x 4");
    DSP_REQUIRE(x && coef && y && N > 0 && stride >= 1 && pad >= 0 && pad < k && H + 2 * pad >= k && W + 2 * pad >= k, DSP_EINVAL,
                "bn + relu + max pool: bad argument");
    DSP_REQUIRE((int64_t)N * H * W * C < (1ll << 31), DSP_EINVAL, "bn + relu + max pool: tensors of 2^31 elements or more are not supported");
    DSP_REQUIRE(((uintptr_t)x % 16) == 0 && ((uintptr_t)y % 16) == 0 && ((uintptr_t)argmax % 8) == 0 && ((uintptr_t)coef % 16) == 0,
                DSP_EINVAL, "bn + relu + max pool: unaligned tensor");
    const int Ho = (H + 2 * pad - k) / stride + 1, Wo = (W + 2 * pad - k) / stride + 1;
    const int64_t total = (int64_t)N * Ho * Wo * (C / 8);
    int64_t grid = (total + kThreads - 1) / kThreads;
    grid = (grid + 7) / 8 * 8;
    if (grid > 256 * 32) grid = 256 * 32;
    ProfScope ps("bn_relu_maxpool_fwd<bf16>", ((double)N * H * W * C + (double)N * Ho * Wo * C) * 2.0 + (double)N * Ho * Wo * C, 1);
    if (k == 3)
        DSP_LAUNCH(ps, (bn_relu_maxpool_bf16_kernel<3>), dim3((unsigned)grid), dim3(kThreads), 0, st, (const bf16_t*)x, coef, (bf16_t*)y,
                   argmax, N, H, W, C, Ho, Wo, k, stride, pad);
    else
        DSP_LAUNCH(ps, (bn_relu_maxpool_bf16_kernel<0>), dim3((unsigned)grid), dim3(kThreads), 0, st, (const bf16_t*)x, coef, (bf16_t*)y,
                   argmax, N, H, W, C, Ho, Wo, k, stride, pad);
    DSP_HIP(hipGetLastError());
    return DSP_OK;
}

size_t bn_relu_bits_bytes(int dtype, int64_t M, int C)
{
    const int vw = dtype == DSP_BF16 ? 8 : 4;
    return C % vw == 0 ? (size_t)(M * (C / vw)) : 0;
}

bool bn_pool_backward_supported(int dtype, int C, int H, int W, int k, int stride, int pad)
{
    return dtype == DSP_BF16 && C % 8 == 0 && k == 3 && stride == 2 && pad == 1 && H >= 2 && W >= 2 && H % 2 == 0 && W % 2 == 0;
}

static int bn_pool_backward(const PoolGrad& pg, const void* x, void* dx, bool xacc, const void* dx_prev, const float* gamma,
                            float* dgamma, float* dbeta, int64_t M, int C, const BnBuffers& buf, hipStream_t st, const float* fcoef)
{
    PoolCells p{};
    p.dpool = (const bf16_t*)pg.dpool;
    p.arg = pg.argmax;
    p.H = pg.H;
    p.W = pg.W;
    p.Ho = pg.H / 2;
    p.Wo = pg.W / 2;
    fast_div_constants((uint32_t)p.Wo, &p.wo_mul, &p.wo_sh);
    fast_div_constants((uint32_t)p.Ho, &p.ho_mul, &p.ho_sh);
    const int64_t cells = M / 4;
    const RowLayout L = make_layout(C, 8);
    int nblk;
    const int cells_per_block = plan_rows(cells, L, &nblk);
    const double tensor_bytes = (double)M * C * 2.0, pool_bytes = (double)cells * C * 3.0;
    {
        ProfScope ps("bn_pool_bwd_reduce<bf16>", tensor_bytes + pool_bytes, 1);
        DSP_LAUNCH(ps, bn_pool_bwd_reduce_kernel, dim3(nblk, ceil_div(L.cv, L.cvb)), dim3(kThreads), 0, st, (const bf16_t*)x, p,
                   (const float*)buf.mean, (const float*)buf.invstd, fcoef, buf.partial, (uint32_t)cells, C, L, cells_per_block);
    }
    {
        ProfScope ps("bn_bwd_finalize", (double)nblk * C * 16.0, 1);
        const BnGradOut o{buf.partial, gamma, buf.mean, buf.invstd, dgamma, dbeta, buf.coef};
        DSP_LAUNCH(ps, bn_bwd_finalize_kernel, dim3(ceil_div(C, 4)), dim3(kMergeLanes * 4), 0, st, o, nblk, C, 1.0 / (double)M);
    }
    const int64_t items = cells * L.cv;
    int64_t grid = (items + kThreads - 1) / kThreads;
    grid = (grid + 7) / 8 * 8;
    if (grid > 256 * 16) grid = 256 * 16;
    uint32_t cv_mul, cv_sh;
    fast_div_constants((uint32_t)L.cv, &cv_mul, &cv_sh);
    ProfScope ps("bn_pool_bwd_apply<bf16>", tensor_bytes * (2 + (xacc ? 1 : 0)) + pool_bytes, 1);
    if (xacc)
        DSP_LAUNCH(ps, bn_pool_bwd_apply_kernel<true>, dim3((unsigned)grid), dim3(kThreads), 0, st, (const bf16_t*)x, p, (bf16_t*)dx,
                   (const bf16_t*)dx_prev, (const float*)buf.coef, fcoef, (uint32_t)items, C, (uint32_t)L.cv, cv_mul, cv_sh);
    else
        DSP_LAUNCH(ps, bn_pool_bwd_apply_kernel<false>, dim3((unsigned)grid), dim3(kThreads), 0, st, (const bf16_t*)x, p, (bf16_t*)dx,
                   (const bf16_t*)dx_prev, (const float*)buf.coef, fcoef, (uint32_t)items, C, (uint32_t)L.cv, cv_mul, cv_sh);
    DSP_HIP(hipGetLastError());
    return DSP_OK;
}

int launch_bn_backward(int dtype, const void* dy, const void* x, const void* y, void* dx, void* dres,
                       bool dres_accumulate, bool dx_accumulate, const float* gamma, float* dgamma, float* dbeta,
                       int64_t M, int C, bool relu, const BnBuffers& buf, hipStream_t st, const void* dx_add,
                       const float* fwd_coef, const PoolGrad* pool, const uint8_t* relu_bits)
{
    DSP_REQUIRE(M > 0 && C > 0, DSP_EINVAL, "bn: bad shape");
    if (pool) {
        DSP_REQUIRE(relu && fwd_coef && !dres && pool->dpool && pool->argmax && x && dx &&
                        bn_pool_backward_supported(dtype, C, pool->H, pool->W, pool->k, pool->stride, pool->pad) &&
                        M % ((int64_t)pool->H * pool->W) == 0 && M * C < (1ll << 31) && ((uintptr_t)pool->dpool % 16) == 0 &&
                        ((uintptr_t)pool->argmax % 8) == 0 && ((uintptr_t)x % 16) == 0 && ((uintptr_t)dx % 16) == 0 &&
                        ((uintptr_t)dx_add % 16) == 0,
                    DSP_EINVAL, "bn backward behind a max pool: bf16, channels in runs of 8, 3 x 3 / 2 / 1 windows over an even map, "
                                "ReLU without residual, 16-byte aligned tensors");
        return bn_pool_backward(*pool, x, dx, dx_accumulate || dx_add, dx_add ? dx_add : dx, gamma, dgamma, dbeta, M, C, buf, st,
                                fwd_coef);
    }
    const void* dx_prev = dx_add ? dx_add : dx;
    if (dx_add) dx_accumulate = true;
    // the ReLU of a batch norm without residual can be decided from x (no read of y) when the caller still has the
    // forward pass's {scale, shift}
    const bool from_x = relu && fwd_coef && !dres;
    const bool from_bits = relu && !from_x && relu_bits && bn_relu_bits_bytes(dtype, M, C) > 0;
    if (from_bits) y = relu_bits;
    DSP_REQUIRE(!relu || from_x || y, DSP_EINVAL, "bn backward: the ReLU needs the stored output");
#define BN_BWD_RM(T, VW, RM)                                                                                        \
    bn_backward_t<T, VW, RM>(dy, x, y, dx, dres, dres_accumulate, dx_accumulate, gamma, dgamma, dbeta, M, C, buf, st, \
                             dx_prev, fwd_coef)
#define BN_BWD(T, VW) (!relu ? BN_BWD_RM(T, VW, 0) : from_x ? BN_BWD_RM(T, VW, 2) : (from_bits && VW > 1) ? BN_BWD_RM(T, VW, 3) : BN_BWD_RM(T, VW, 1))
    if (dtype == DSP_BF16) {
        if (C % 8 == 0) return BN_BWD(bf16_t, 8);
        return BN_BWD(bf16_t, 1);
    }
    if (C % 4 == 0) return BN_BWD(float, 4);
    return BN_BWD(float, 1);
#undef BN_BWD
#undef BN_BWD_RM
}

}  // namespace dsp
