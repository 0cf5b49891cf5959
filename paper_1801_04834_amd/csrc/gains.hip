// Gain-applied visibilities and their adjoint with respect to the complex gains.
//
// Per-input complex gains (station, polarisation, subband, channel) are constant over a
// block, so applying them to the channelised samples before the X stage equals scaling each
// stored visibility:  V'_ab = g_a conj(g_b) V0_ab.  For a real loss with upstream gradient
// G = dL/dRe V' + i dL/dIm V', the gradient with respect to g_k (same convention) is
//     sum_{entries with b = k} conj(G_ab) g_a V0_ab + sum_{entries with a = k} G_ab g_b conj(V0_ab).
// Both kernels are bandwidth-bound passes over the visibilities in their own order.  With
// P = G conj(V0) the gradient is a product with the Hermitian matrix whose stored half P is:
//     grad_a += P_ab g_b,    grad_b += conj(P_ab) g_a,
// so the adjoint reads every entry once: a workgroup walks the baselines (s1, 0 .. s1) of a channel,
// thread (s2, q) keeping the column sums of its input in registers and the row sums going through a
// reduction over the threads of equal p1.  No atomics; the order of the sums is fixed
// (bit-reproducible).
#include "cobalt_internal.h"

namespace cobalt {
namespace {

__device__ __forceinline__ float2 cmul(float2 x, float2 y) {
    return make_float2(x.x * y.x - x.y * y.y, x.x * y.y + x.y * y.x);
}
__device__ __forceinline__ float2 cconj(float2 x) { return make_float2(x.x, -x.y); }

// Two neighbouring entries (one station pair and p1) per thread: 16-byte loads and stores, one 32-bit
// division (48 stations, 1024 channels: 17.2 -> 13.3 us; 76 stations: 40 -> 30).  The threads run
// through the entries of all channels: with whole workgroups per channel a few stations leave most
// of their threads idle (one station, 131072 channels: 34 us against 7).
__global__ __launch_bounds__(256) void apply_gains_kernel(const float4* __restrict__ vis0, const float2* __restrict__ gains,
                                                          float4* __restrict__ vis, unsigned per_ch, int M, unsigned n) {
    const unsigned id = blockIdx.x * 256u + threadIdx.x;
    if (id >= n) return;
    const unsigned ch = id / per_ch;
    const int e = (int)(id - ch * per_ch);         // baseline * 2 + p1
    const int bl = e >> 1, p1 = e & 1;
    int s1 = (int)((sqrtf(8.f * bl + 1.f) - 1.f) * 0.5f);
    while (s1 * (s1 + 1) / 2 > bl) --s1;
    while ((s1 + 1) * (s1 + 2) / 2 <= bl) ++s1;
    const int s2 = bl - s1 * (s1 + 1) / 2;
    const float2* g = gains + (int64_t)ch * M;
    const float2 ga = g[2 * s1 + p1], g0 = g[2 * s2], g1 = g[2 * s2 + 1];
    const float4 v = vis0[id];
    const float2 x = cmul(cmul(ga, cconj(g0)), make_float2(v.x, v.y)), y = cmul(cmul(ga, cconj(g1)), make_float2(v.z, v.w));
    vis[id] = make_float4(x.x, x.y, y.x, y.y);
}

// v of this lane plus those of all lanes of the wave with the same lane bit 1
__device__ __forceinline__ float add_same_p1(float v) {
    v += __builtin_bit_cast(float, __builtin_amdgcn_mov_dpp(__builtin_bit_cast(int, v), 0xb1, 0xf, 0xf, true));   // lane ^ 1
    v += __builtin_bit_cast(float, __builtin_amdgcn_mov_dpp(__builtin_bit_cast(int, v), 0x124, 0xf, 0xf, true));  // row rotated by 4
    v += __builtin_bit_cast(float, __builtin_amdgcn_mov_dpp(__builtin_bit_cast(int, v), 0x128, 0xf, 0xf, true));  // row rotated by 8
    const auto r16 = __builtin_amdgcn_permlane16_swap(__float_as_uint(v), __float_as_uint(v), false, false);
    v = __uint_as_float(r16[0]) + __uint_as_float(r16[1]);
    const auto r32 = __builtin_amdgcn_permlane32_swap(__float_as_uint(v), __float_as_uint(v), false, false);
    return __uint_as_float(r32[0]) + __uint_as_float(r32[1]);
}

// One workgroup of >= 4 S threads per channel: thread j = 4 s2 + q, q = 2 p1 + p2 (the entries of a
// row s1 are 4 (s1 + 1) consecutive ones).  48 stations, 1024 channels: 37.4 us with one thread per
// input walking its row and its column, 19.2 us in this form (77 MB read: 12.5 us at the copy rate).
// LDS for up to 16 NW stations, so that small arrays have as many channels in flight as a CU holds
// waves (one station, 131072 channels: 89 us with LDS for 128 stations, 37 so; 42 with one thread per input).
template <int NW>
__global__ __launch_bounds__(64 * NW) void apply_gains_adjoint_kernel(const float2* __restrict__ vis0, const float2* __restrict__ gains,
                                                                  const float2* __restrict__ grad_vis, float2* __restrict__ grad_gains,
                                                                  int S) {
    __shared__ float2 part[16 * NW][NW][2];        // row sums [s1][wave][p1]
    __shared__ float2 col[64 * NW];                // column sums [thread]
    const int j = threadIdx.x, wave = j >> 6, n_wave = blockDim.x >> 6;
    const int s2 = j >> 2, p1 = (j >> 1) & 1, p2 = j & 1;
    const int64_t ch = blockIdx.x;
    const int64_t n4 = (int64_t)S * (S + 1) * 2;   // entries of a channel
    const float2* v0 = vis0 + ch * n4 + j;
    const float2* G = grad_vis + ch * n4 + j;
    const float2* g = gains + ch * 2 * S;
    const float2 gb = s2 < S ? g[2 * s2 + p2] : make_float2(0.f, 0.f);
    float2 acc = make_float2(0.f, 0.f);
    // rows below this wave's first station hold no entry of its threads
    constexpr int kU = 8;                          // rows in flight
    for (int r0 = 16 * wave; r0 < S; r0 += kU) {
        float2 v[kU], w[kU], ga[kU];
#pragma unroll
        for (int u = 0; u < kU; ++u) {
            const int s1 = r0 + u;
            const bool ok = s1 < S && s2 <= s1;
            const int at = 2 * s1 * (s1 + 1);
            v[u] = ok ? v0[at] : make_float2(0.f, 0.f);
            w[u] = ok ? G[at] : make_float2(0.f, 0.f);
            ga[u] = ok ? g[2 * s1 + p1] : make_float2(0.f, 0.f);
        }
#pragma unroll
        for (int u = 0; u < kU; ++u) {
            const int s1 = r0 + u;
            if (s1 >= S) break;
            const bool ok = s2 <= s1;
            const float2 P = cmul(w[u], cconj(v[u]));
            const float2 t = cmul(cconj(P), ga[u]), rsum = cmul(P, gb);
            acc.x += ok ? t.x : 0.f;
            acc.y += ok ? t.y : 0.f;
            const float x = add_same_p1(ok ? rsum.x : 0.f), y = add_same_p1(ok ? rsum.y : 0.f);
            if ((j & 63) == 2 * p1) part[s1][wave][p1] = make_float2(x, y);
        }
    }
    col[j] = acc;
    __syncthreads();
    if (j >= 2 * S) return;
    // input j = (station, pol): its row sums over the waves that hold entries of the row, then its
    // column sums over p1
    const int s = j >> 1, p = j & 1;
    float2 r = make_float2(0.f, 0.f);
    for (int w = 0; w < n_wave && 16 * w <= s; ++w) {
        r.x += part[s][w][p].x;
        r.y += part[s][w][p].y;
    }
    const float2 c0 = col[4 * s + p], c1 = col[4 * s + 2 + p];
    grad_gains[ch * 2 * S + j] = make_float2(r.x + (c0.x + c1.x), r.y + (c0.y + c1.y));
}

}  // namespace

hipError_t launch_apply_gains(const void* vis0, const void* gains, void* vis, int n_chan, int S, hipStream_t st) {
    const int per_ch = S * (S + 1);                // entry pairs of a channel
    // millions of channels in pieces: a launch holds fewer than 2^32 work-items
    const int piece = (1 << 30) / per_ch;
    hipError_t e = hipSuccess;
    for (int64_t c0 = 0; c0 < n_chan && e == hipSuccess; c0 += piece) {
        const unsigned n = (unsigned)((n_chan - c0 < piece ? n_chan - c0 : piece) * per_ch);
        hipLaunchKernelGGL(apply_gains_kernel, dim3((n + 255) / 256), dim3(256), 0, st, (const float4*)vis0 + c0 * per_ch,
                           (const float2*)gains + c0 * 2 * S, (float4*)vis + c0 * per_ch, (unsigned)per_ch, 2 * S, n);
        e = hipGetLastError();
    }
    return e;
}

hipError_t launch_apply_gains_adjoint(const void* vis0, const void* gains, const void* grad_vis, void* grad_gains, int n_chan,
                                      int S, hipStream_t st) {
    if (n_chan == 0) return hipSuccess;
    const dim3 grid((unsigned)n_chan), block((unsigned)((4 * S + 63) / 64 * 64));
    const float2 *v = (const float2*)vis0, *g = (const float2*)gains, *G = (const float2*)grad_vis;
    float2* out = (float2*)grad_gains;
    if (S <= 16) hipLaunchKernelGGL(apply_gains_adjoint_kernel<1>, grid, block, 0, st, v, g, G, out, S);
    else if (S <= 32) hipLaunchKernelGGL(apply_gains_adjoint_kernel<2>, grid, block, 0, st, v, g, G, out, S);
    else if (S <= 64) hipLaunchKernelGGL(apply_gains_adjoint_kernel<4>, grid, block, 0, st, v, g, G, out, S);
    else if (S <= kMaxStations) hipLaunchKernelGGL(apply_gains_adjoint_kernel<8>, grid, block, 0, st, v, g, G, out, S);
    else return hipErrorInvalidValue;
    return hipGetLastError();
}

}  // namespace cobalt
