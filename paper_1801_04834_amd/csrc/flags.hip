// Lost-sample flags: which channel samples read a lost input sample, and per-baseline
// weights (channel samples valid for both stations).
//
// Lost or late input is recorded and travels with the data product ("Processing steps",
// sec. 3.2; "Dealing with jitter and hardware failure", sec. 7.2).  Channel sample j of a
// stream is the FIR output over input rows j-T+1 .. j of C samples each (rows before the
// block come from the previous block), so it is flagged when any of those T rows holds a
// lost sample.  The F stage writes flagged channel samples as zero, so they drop out of every
// visibility, and the weights count what remains per baseline.
//
// Bit conventions: a wave takes 64 rows as one mask (bit i = row R0 + i); the carried history word
// holds rows -15 .. -1 in bits 17 .. 31, i.e. as a mask of rows -64 .. -1 it is the word << 32.  The
// flagged channel samples of the 64 rows are the upper half of  OR_{d<16} ((mask : rows before) << d).
//
// Both kernels are tiny next to the F stage and bound by latency, so they are cut fine: one wave per
// 64 rows with a row per lane (neighbouring lanes read neighbouring words; a wave per stream with 32
// rows per lane took 14.6 us for 407 streams of 1501 rows, this form 7.5), and 16 lanes per baseline
// (one thread per baseline took 13.9 us for 11 x 703 baselines, this form 5).
#include "cobalt_internal.h"

namespace cobalt {
namespace {

static_assert(kHistRows == 15, "history bits 17..31 of the row word before the block");

// Rows of one stream that hold a lost sample, one row per lane.
__device__ __forceinline__ uint64_t row_mask(const FlagArgs& a, const uint32_t* __restrict__ fl, int64_t base, int b, int row,
                                             bool wanted) {
    // row r covers samples g + Cr .. g + Cr + C-1 of the input row: bits b..31 of word i0, all of
    // words i0+1 .. i0+C/32-1 and bits 0..b-1 of word i0+C/32 (present when b > 0, since the window
    // ends inside the row)
    uint32_t any = 0;
    if (fl && wanted) {
        const int wr = a.C >> 5;
        const uint32_t* w = fl + base + (int64_t)row * wr;
        any = w[0] >> b;
        for (int k = 1; k < wr; ++k) any |= w[k];
        if (b) any |= w[wr] & ((1u << b) - 1u);
    }
    return __ballot(any != 0u);
}

__global__ __launch_bounds__(256) void chanflag_kernel(FlagArgs a) {
    const int lane = threadIdx.x & 63;
    const int n_seg = (a.n_c + 63) >> 6;                      // waves per stream
    const int64_t id = (int64_t)blockIdx.x * 4 + (threadIdx.x >> 6);
    const int64_t sst = id / n_seg;                           // s * SB + sb
    if (sst >= (int64_t)a.S * a.SB) return;
    const int r0 = (int)(id % n_seg) * 64;
    const int64_t g = a.coarse[(int)(sst / a.SB)];            // window start in the row
    const uint32_t* __restrict__ fl = a.flags ? a.flags + sst * a.flag_words : nullptr;
    const uint64_t m = row_mask(a, fl, g >> 5, (int)(g & 31), r0 + lane, r0 + lane < a.n_c);
    const uint64_t prev = r0 == 0 ? (uint64_t)a.hist_old[sst] << 32
                                  : row_mask(a, fl, g >> 5, (int)(g & 31), r0 - 64 + lane, lane >= 64 - kHistRows);
    uint64_t hi = m, lo = prev;
#pragma unroll
    for (int sh = 1; sh < 16; sh <<= 1) {                     // OR over shifts 0 .. 15
        hi |= hi << sh | lo >> (64 - sh);
        lo |= lo << sh;
    }
    const int left = a.n_c - r0;
    if (left < 64) hi &= ((uint64_t)1 << left) - 1u;
    const int w = (r0 >> 5) + lane;
    if (lane < 2 && w < a.n_words) a.cflag[sst * a.n_words + w] = (uint32_t)(lane ? hi >> 32 : hi);
    if (left <= 64 && lane == 0) {
        // rows n_c-15 .. n_c-1 are bits e-14 .. e, e = left - 1, of the mask with the rows before below it
        const int sh = left - kHistRows;
        const uint64_t last = sh >= 0 ? m >> sh : m << -sh | prev >> (64 + sh);
        a.hist_new[sst] = (uint32_t)(last & 0x7fffu) << 17;
    }
}

// 16 lanes per (subband, baseline): popcount of the channel samples valid for both stations.
// Without flags every baseline has all N_c.
__global__ __launch_bounds__(256) void weights_kernel(const uint32_t* __restrict__ cflag, int32_t* __restrict__ weights,
                                                      int S, int SB, int n_c, int n_words) {
    const int B = S * (S + 1) / 2;
    const int bl = blockIdx.x * 16 + (threadIdx.x >> 4), l = threadIdx.x & 15;
    const int sb = blockIdx.y;
    int cnt = 0;
    if (bl < B && cflag) {
        int s1 = (int)((sqrtf(8.f * bl + 1.f) - 1.f) * 0.5f);
        while (s1 * (s1 + 1) / 2 > bl) --s1;
        while ((s1 + 1) * (s1 + 2) / 2 <= bl) ++s1;
        const int s2 = bl - s1 * (s1 + 1) / 2;
        const uint32_t* f1 = cflag + ((int64_t)s1 * SB + sb) * n_words;
        const uint32_t* f2 = cflag + ((int64_t)s2 * SB + sb) * n_words;
        for (int w = l; w < n_words; w += 16) {
            const int left = n_c - 32 * w;
            const uint32_t valid = left >= 32 ? 0xffffffffu : (1u << left) - 1u;
            cnt += __popc(~(f1[w] | f2[w]) & valid);
        }
    }
    for (int m = 1; m < 16; m <<= 1) cnt += __shfl_xor(cnt, m, 16);
    if (bl < B && l == 0) weights[(int64_t)sb * B + bl] = cflag ? cnt : n_c;
}

}  // namespace

hipError_t launch_chanflags(const FlagArgs& a, hipStream_t st) {
    if (a.n_c == 0) return hipSuccess;
    const int64_t waves = (int64_t)a.S * a.SB * ((a.n_c + 63) / 64);
    hipLaunchKernelGGL(chanflag_kernel, dim3((unsigned)((waves + 3) / 4)), dim3(256), 0, st, a);
    return hipGetLastError();
}

hipError_t launch_weights(const uint32_t* cflag, int32_t* weights, int S, int SB, int n_c, int n_words, hipStream_t st) {
    const int B = S * (S + 1) / 2;
    hipLaunchKernelGGL(weights_kernel, dim3((unsigned)((B + 15) / 16), (unsigned)SB), dim3(256), 0, st, cflag, weights, S, SB,
                       n_c, n_words);
    return hipGetLastError();
}

}  // namespace cobalt
