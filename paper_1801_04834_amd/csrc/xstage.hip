// X stage of the FX correlator for gfx950: per channel, V = Z Z^H over all inputs
// (station x polarisation), integrated over the block ("Signal processing with GPU
// kernels", sec. 7.5: correlations of all pairs of antenna fields, averaged to ~1 s).
//
// MFMA form (FP16-split and int8): a complex Hermitian rank-K update written as two real
// contractions over K = 2 N_c interleaved (re, im) values:
//     Re V[a][b] = sum_k A[a][k] A[b][k]         (A = interleaved rows of Z)
//     Im V[a][b] = sum_k A[a][k] A'[b][k]        (A' = per sample (re, im) -> (-im, re))
// One workgroup owns one channel and keeps every lower-triangle 16x16 tile of V in accumulators;
// channel rows stream through LDS once.  An MFMA fragment of row block I (lane i: row 16I + i%16,
// 16 bytes of K) is simultaneously an A operand (row I) and a B operand (column I), so both
// operands of a tile come from the same LDS reads and the k order inside a fragment never matters.
// A' is built in registers from the B-role fragments.
//   FP16-split: Z*2^k = hi + lo (two fp16 planes); V ~= hh + hl + lh accumulated in FP32
//   (the dropped lo*lo term is below 2^-22 of |Z|^2), scaled back by 2^-2k.  A diagonal tile (I = J)
//   needs h h^T + h l^T + l h^T: it accumulates h h^T and X = h l^T in two products and adds
//   X + X^T (real part) or X - X^T (imaginary part) at the end.  X has accumulators of its own: one
//   sum of h (h + 2 l)^T would need none, but 2 l overflows FP16 for lo values above 32752, which a
//   channelised buffer filled by the caller may hold, and the MFMAs round towards zero, twice per
//   k-step of the long sums of the autos (relative error against 64 bits at 76 stations 7.3e-7
//   instead of 4.7e-7).
//   int8: exact int32 sums.
// Plain FP32 form: the same two contractions on FP32 operands and FP32 MFMAs over 16x16 tiles, with
// partial sums over 128 channel samples folded into running totals.
#include <type_traits>

#include "cobalt_internal.h"
#include "xring.h"

namespace cobalt {
namespace {

typedef _Float16 half8 __attribute__((ext_vector_type(8)));
typedef float floatx4 __attribute__((ext_vector_type(4)));
typedef int intx4 __attribute__((ext_vector_type(4)));
typedef unsigned uintx4 __attribute__((ext_vector_type(4)));

template <int I, int N, class F>
__device__ __forceinline__ void static_for_impl(F& f) {
    if constexpr (I < N) {
        f(std::integral_constant<int, I>{});
        static_for_impl<I + 1, N>(f);
    }
}
template <int N, class F>
__device__ __forceinline__ void static_for(F&& f) { static_for_impl<0, N>(f); }

// Lower-triangle tiles of an R x R block grid, column-major: (0,0),(1,0)..(R-1,0),(1,1)..
constexpr int tile_J(int R, int idx) {
    int J = 0;
    while (idx >= R - J) { idx -= R - J; ++J; }
    return J;
}
constexpr int tile_I(int R, int idx) {
    int J = 0;
    while (idx >= R - J) { idx -= R - J; ++J; }
    return J + idx;
}

// LDS rows are XOR-swizzled in 16-byte granules (granule g of row r is stored at g ^ (r%16)),
// so the 16 rows of one MFMA fragment read hit distinct banks without padding.
__device__ __forceinline__ int lds_off(int row, int g) { return row * kRowB + ((g ^ (row & 15)) << 4); }

// (re, im) -> (-im, re) on packed fp16 pairs
__device__ __forceinline__ uintx4 swapneg_f16(uintx4 d) {
    uintx4 r;
#pragma unroll
    for (int e = 0; e < 4; ++e) r[e] = __builtin_amdgcn_alignbit(d[e], d[e], 16) ^ 0x00008000u;
    return r;
}
// (re, im) -> (-im, re) on packed int8 pairs; inputs lie in [-127, 127]
__device__ __forceinline__ uintx4 swapneg_i8(uintx4 d) {
    uintx4 r;
#pragma unroll
    for (int e = 0; e < 4; ++e) {
        const unsigned t = __builtin_amdgcn_perm(d[e], d[e], 0x02030001u);   // bytes (im, re) pairs
        const unsigned lo = t & 0x00ff00ffu;
        r[e] = (t & 0xff00ff00u) | ((0x01000100u - lo) & 0x00ff00ffu);
    }
    return r;
}

typedef __attribute__((address_space(3))) void* lds_ptr_t;

// ------------------------------------------------------------------ LDS ring ---
// Wait until at most n of this wave's transfers are outstanding (rounded down to the counts
// built: a smaller count waits longer, never shorter).
__device__ __forceinline__ void wait_transfers(int n) {
    if (n >= 32) asm volatile("s_waitcnt vmcnt(32)" ::: "memory");
    else if (n >= 24) asm volatile("s_waitcnt vmcnt(24)" ::: "memory");
    else if (n >= 16) asm volatile("s_waitcnt vmcnt(16)" ::: "memory");
    else if (n >= 12) asm volatile("s_waitcnt vmcnt(12)" ::: "memory");
    else if (n >= 8) asm volatile("s_waitcnt vmcnt(8)" ::: "memory");
    else if (n >= 6) asm volatile("s_waitcnt vmcnt(6)" ::: "memory");
    else if (n >= 4) asm volatile("s_waitcnt vmcnt(4)" ::: "memory");
    else if (n >= 3) asm volatile("s_waitcnt vmcnt(3)" ::: "memory");
    else if (n >= 2) asm volatile("s_waitcnt vmcnt(2)" ::: "memory");
    else if (n >= 1) asm volatile("s_waitcnt vmcnt(1)" ::: "memory");
    else asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
}
// Workgroup barrier that leaves the transfers in flight (a __syncthreads() would wait for them);
// this wave's LDS reads and writes are complete before it.
__device__ __forceinline__ void lds_barrier() { asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory"); }

// Issue stage s into its ring slot at buf.  Every wave issues exactly ipw transfers of a full stage (the
// last ones repeat the stage's final transfer), so that counted waits hold for every wave; the
// last, partial stage may issue fewer.
template <int MODE, int NWV>
__device__ __forceinline__ void ring_issue(const XArgs& a, const XRing& q, const char* __restrict__ chan, char* buf, int s, int wave,
                                           int lane) {
    const int c0 = s * q.nch, nch = min(q.nch, q.n_chunk - c0);
    const int rsub = lane >> 4, p = lane & 15;
    int ck = 0, i = wave;
    for (int k = 0; k < q.ipw; ++k, i += NWV) {
        while (i >= q.n_inst) { i -= q.n_inst; ++ck; }
        if (ck >= nch) {
            if (nch < q.nch) break;
            ck = nch - 1;
            i = q.n_inst - 1;
        }
        const int row = 4 * i + rsub, g = p ^ (row & 15);
        bool ok = row < a.M;
        const char* src;
        if constexpr (MODE == XM_FP32) {
            src = chan + (int64_t)(c0 + ck) * (a.M * 256) + (row * 256 + g * 16);
        } else if constexpr (MODE == XM_FP16_SPLIT) {
            src = chan + (int64_t)(c0 + ck) * (2 * a.M * 128) + ((g >> 3) * (a.M * 128) + row * 128 + (g & 7) * 16);
        } else {
            const int kb = 4 * (c0 + ck) + (g >> 2);
            ok = ok && kb < a.n_kb;
            src = chan + (int64_t)kb * (a.M * 64) + (row * 64 + (g & 3) * 16);
        }
        if (ok) __builtin_amdgcn_global_load_lds((const void*)src, (lds_ptr_t)(buf + ck * q.chunk_b + i * 1024), 16, 0, 2);
    }
}

// Zero columns >= n_c of the last chunk, of which `first` > 0 are kept, for rows < M: whole granules, the
// granule that holds both kinds by mask (its samples have landed).
template <int MODE>
__device__ __forceinline__ void zero_columns(const XArgs& a, char* buf, int first, int tid, int nthr) {
    constexpr int kPer = MODE == XM_FP32 ? 2 : MODE == XM_FP16_SPLIT ? 4 : 8;   // samples per granule
    constexpr int kPlane = MODE == XM_FP16_SPLIT ? 8 : 16;                      // granules of a row and plane
    const int g0 = first / kPer, keep = first % kPer * (16 / kPer);   // bytes kept of granule g0
    const int n = kPlane - g0;
    for (int id = tid; id < a.M * n; id += nthr) {
        const int row = id / n, g = g0 + id % n;
        uintx4 mask = {};
        if (g == g0) {
#pragma unroll
            for (int e = 0; e < 4; ++e) mask[e] = keep >= 4 * e + 4 ? 0xffffffffu : keep > 4 * e ? 0xffffu : 0u;
        }
#pragma unroll
        for (int p = 0; p < 16; p += kPlane) *(uintx4*)(buf + lds_off(row, p + g)) &= mask;
    }
}

// The ring's loop over a channel: body(stage buffer, chunks in the stage) runs with
// every chunk of the stage in LDS.
template <int MODE, int NWV, class F>
__device__ __forceinline__ void ring_loop(const XArgs& a, const XRing& q, const char* __restrict__ chan, char* lds, int tid, F&& body) {
    constexpr int kc = MODE == XM_INT8 ? 128 : 32;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6), lane = tid & 63;
    const int slot_b = q.nch * q.chunk_b;
    for (int s = 0; s < ring_ahead(q); ++s) ring_issue<MODE, NWV>(a, q, chan, lds + s * slot_b, s, wave, lane);
    int slot = 0, freed = q.depth - 1;        // slots of stage s and of stage s - 1 (and s + depth - 1)
    for (int s = 0; s < q.n_stage; ++s) {
        wait_transfers(ring_may_fly(q, s));
        lds_barrier();                        // ... for every wave; the slot of stage s - 1 is free
        if (s + q.depth - 1 < q.n_stage) ring_issue<MODE, NWV>(a, q, chan, lds + freed * slot_b, s + q.depth - 1, wave, lane);
        char* buf = lds + slot * slot_b;
        freed = slot;
        if (++slot == q.depth) slot = 0;
        const int nch = min(q.nch, q.n_chunk - s * q.nch);
        if (s == q.n_stage - 1 && a.n_c % kc != 0) {
            zero_columns<MODE>(a, buf + (nch - 1) * q.chunk_b, a.n_c % kc, tid, 64 * NWV);
            lds_barrier();
        }
        body(buf, nch);
    }
    lds_barrier();                            // every wave is done with the chunks
}

// ------------------------------------------------------------------ MFMA forms ---
// One workgroup of NWV waves per channel.  The lower triangle of 16 x 16 tiles (NB row blocks) goes
// to ks_groups wave groups as runs of a column-major tile list; the waves of a group split the
// k-steps of a stage among them, so that a few tiles keep every wave busy.
// Bound by the channel's HBM stream and, with many channels, by the chip's power: both the stream
// and the matrix pipes draw on it (24 stations x 2048 channels holds 1.70 GHz), so work that is not
// needed costs time also where no pipe is full.  Hence tiles of 16 (48 inputs: 30 MFMAs of 16x16x32
// per 16 samples against 28 of twice the length with tiles of 32), zeros for the padding rows and
// two instead of three products on the diagonal.  Four waves per workgroup and two or more
// workgroups per CU; with at most one channel per CU eight waves and the whole LDS as ring; one wave for
// the shortest blocks of small arrays.  Groups are as few as the accumulators and fragments allow without spilling.
// Measured against one workgroup of four waves with up to four 32 x 32 tiles each (waves idle below
// 5 row blocks of 32), us, FP16-split: 24 st x 32 SB 604 -> 428 (5.7 TB/s); 48 x 16 640 -> 545;
// 52 x 61 2905 -> 2240; 76 x 64 4030 -> 3780; 24 x 1 125 -> 49; 48 x 1 at 256 channels 54 -> 36;
// 80 x 32 2094 -> 1972.  int8: 24 x 32 118 -> 108; 28 x 32 128 -> 125; 76 x 64 910 -> 884.
template <int MODE, int NB, int NWV> constexpr int ks_per() {
    return (tile_count(NB) + ks_groups(MODE == XM_INT8, NB, NWV) - 1) / ks_groups(MODE == XM_INT8, NB, NWV);
}
template <int MODE, int NB, int NWV, int G> constexpr int ks_tiles() {
    const int left = tile_count(NB) - G * ks_per<MODE, NB, NWV>();
    return left < ks_per<MODE, NB, NWV>() ? left : ks_per<MODE, NB, NWV>();
}
template <int NB, int NWV> constexpr int ks_waves_per_simd() { return NWV == 8 ? 2 : NWV == 1 || NB <= 2 ? 4 : NB == 3 ? 3 : 2; }
// row blocks used by tiles [t0, t0 + n)
constexpr unsigned ks_blocks(int NB, int t0, int n) {
    unsigned m = 0;
    for (int t = t0; t < t0 + n; ++t) m |= 1u << tile_I(NB, t) | 1u << tile_J(NB, t);
    return m;
}

template <int MODE> struct KCfg;
template <> struct KCfg<XM_FP16_SPLIT> {
    static constexpr int kSteps = ks_steps(false);
    using acc_t = floatx4;
};
template <> struct KCfg<XM_INT8> {
    static constexpr int kSteps = ks_steps(true);
    using acc_t = intx4;
};

// Halve the k parts of a group's sums: of waves p and p ^ half (half a power of two), the lower
// keeps the first (N + 1) / 2 tiles and the upper the rest, each adding what the other sent through
// LDS; the tiles a wave keeps move to the front and t_own follows.  Ends with a barrier.
template <int N, class ACC>
__device__ __forceinline__ void ks_halve(ACC* re, ACC* im, ACC* area, int kpart, int half, int stride, int lane, int& t_own, int& n_own) {
    constexpr int H = (N + 1) / 2;
    const bool upper = (kpart & half) != 0;
    ACC* mine = area + lane;                                            // this wave's outgoing tiles
    const ACC* theirs = area + (upper ? -half : half) * stride + lane;  // the partner's
    if (upper) {
#pragma unroll
        for (int t = 0; t < H; ++t) { mine[2 * t * 64] = re[t]; mine[(2 * t + 1) * 64] = im[t]; }
#pragma unroll
        for (int t = H; t < N; ++t) { re[t - H] = re[t]; im[t - H] = im[t]; }
    } else {
#pragma unroll
        for (int t = H; t < N; ++t) { mine[2 * (t - H) * 64] = re[t]; mine[(2 * (t - H) + 1) * 64] = im[t]; }
    }
    lds_barrier();
#pragma unroll
    for (int t = 0; t < H; ++t) {
        if (t < N - H || !upper) {
            re[t] += theirs[2 * t * 64];
            im[t] += theirs[(2 * t + 1) * 64];
        }
    }
    t_own += upper ? H : 0;
    n_own = upper ? n_own - H : min(n_own, H);
    lds_barrier();
}
template <int N, int P, class ACC>
__device__ __forceinline__ void ks_reduce(ACC* re, ACC* im, ACC* area, int kpart, int stride, int lane, int& t_own, int& n_own) {
    if constexpr (P > 1) {
        ks_halve<N>(re, im, area, kpart, P / 2, stride, lane, t_own, n_own);
        ks_reduce<(N + 1) / 2, P / 2>(re, im, area, kpart, stride, lane, t_own, n_own);
    }
}
constexpr int ks_left(int n, int parts) { return parts > 1 ? ks_left((n + 1) / 2, parts / 2) : n; }

template <int MODE, int NB, int NWV, int G>
__device__ __forceinline__ void xks_wave(const XArgs& a, const XRing& q, const char* __restrict__ chan, char* lds, int tid) {
    using acc_t = typename KCfg<MODE>::acc_t;
    constexpr int kSteps = KCfg<MODE>::kSteps;
    constexpr int kTG = ks_groups(MODE == XM_INT8, NB, NWV), kPer = ks_per<MODE, NB, NWV>(), T0 = G * kPer, NT = ks_tiles<MODE, NB, NWV, G>(), kKP = ks_parts(MODE == XM_INT8, NB, NWV);
    constexpr unsigned kUsed = ks_blocks(NB, T0, NT);
    constexpr bool kSplit = MODE == XM_FP16_SPLIT;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6), lane = tid & 63, kpart = wave / kTG;
    const int row = lane & 15, kg = lane >> 4;

    acc_t re[kPer], im[kPer];
#pragma unroll
    for (int t = 0; t < kPer; ++t) re[t] = im[t] = acc_t{};
    acc_t xre[kSplit ? kPer : 1], xim[kSplit ? kPer : 1];               // h l^T of diagonal tiles
#pragma unroll
    for (int t = 0; t < (kSplit ? kPer : 1); ++t) xre[t] = xim[t] = acc_t{};
    // the last row block's padding rows: the row of zeros behind the ring, or, where the chunks hold
    // them, rows of every slot that no transfer writes
    const int kept = 4 * q.n_inst - a.M;                                // padding rows in a chunk
    const bool behind = 4 * q.n_inst < 16 * NB, pad = behind && 16 * (NB - 1) + row >= a.M;
    const char* zeros = lds + q.lds_b - kRowB;
    if (behind) {
        if (tid < 16) *(uint4*)(lds + q.lds_b - kRowB + tid * 16) = make_uint4(0, 0, 0, 0);
    } else {
        for (int i = tid; i < ring_slots(q) * kept * 16; i += 64 * NWV)
            *(uint4*)(lds + i / (kept * 16) * q.chunk_b + a.M * kRowB + i % (kept * 16) * 16) = make_uint4(0, 0, 0, 0);
    }

    ring_loop<MODE, NWV>(a, q, chan, lds, tid, [&](char* buf, int nch) {
        for (int id = kpart; id < nch * kSteps; id += kKP) {
            const char* base = buf + (id / kSteps) * q.chunk_b + row * kRowB + (((4 * (id % kSteps) + kg) ^ row) << 4);
            const char* last = pad ? zeros : base + 16 * (NB - 1) * kRowB;
            if constexpr (MODE == XM_FP16_SPLIT) {
                const int to_lo = pad ? 0 : (base - buf) & 128 ? -128 : 128;       // granule 8 + g
                const char* base_lo = buf + ((base - buf) ^ 128);
                uintx4 fh[NB], fl[NB];
                static_for<NB>([&](auto bi) {
                    constexpr int b = decltype(bi)::value;
                    if constexpr ((kUsed >> b) & 1u) {
                        fh[b] = *(const uintx4*)(b == NB - 1 ? last : base + 16 * b * kRowB);
                        fl[b] = *(const uintx4*)(b == NB - 1 ? last + to_lo : base_lo + 16 * b * kRowB);
                    }
                });
                // column by column, kept apart: the swapped operands of one column are live at a time
                // (all at once spill at 5 row blocks; 40 stations x 16 subbands 685 us against 379)
                static_for<NB>([&](auto ji) {
                    constexpr int J = decltype(ji)::value;
                    static_for<3>([&](auto pi) {
                        constexpr int pr = decltype(pi)::value;
                        static_for<NT>([&](auto t_) {
                            constexpr int t = decltype(t_)::value;
                            constexpr int I = tile_I(NB, T0 + t);
                            if constexpr (tile_J(NB, T0 + t) == J && !(I == J && pr == 2)) {
                                const half8 A = __builtin_bit_cast(half8, pr == 2 ? fl[I] : fh[I]);
                                const half8 B = __builtin_bit_cast(half8, pr == 1 ? fl[J] : fh[J]);
                                const half8 Bs = __builtin_bit_cast(half8, swapneg_f16(__builtin_bit_cast(uintx4, B)));
                                acc_t& R = I == J && pr == 1 ? xre[t] : re[t];
                                acc_t& Q = I == J && pr == 1 ? xim[t] : im[t];
                                R = __builtin_amdgcn_mfma_f32_16x16x32_f16(A, B, R, 0, 0, 0);
                                Q = __builtin_amdgcn_mfma_f32_16x16x32_f16(A, Bs, Q, 0, 0, 0);
                            }
                        });
                    });
                    __builtin_amdgcn_sched_barrier(0);
                });
            } else {
                uintx4 f[NB];
                static_for<NB>([&](auto bi) {
                    constexpr int b = decltype(bi)::value;
                    if constexpr ((kUsed >> b) & 1u) f[b] = *(const uintx4*)(b == NB - 1 ? last : base + 16 * b * kRowB);
                });
                static_for<NT>([&](auto t_) {
                    constexpr int t = decltype(t_)::value;
                    constexpr int I = tile_I(NB, T0 + t), J = tile_J(NB, T0 + t);
                    const intx4 A = __builtin_bit_cast(intx4, f[I]), B = __builtin_bit_cast(intx4, f[J]);
                    const intx4 Bs = __builtin_bit_cast(intx4, swapneg_i8(f[J]));
                    re[t] = __builtin_amdgcn_mfma_i32_16x16x64_i8(A, B, re[t], 0, 0, 0);
                    im[t] = __builtin_amdgcn_mfma_i32_16x16x64_i8(A, Bs, im[t], 0, 0, 0);
                });
            }
        }
    });

    // several k parts: W = h h^T + 2 X takes one place in the sums, and W + W^T = 2 (h h^T + X + X^T)
    if constexpr (kSplit && kKP > 1) {
        static_for<NT>([&](auto t_) {
            constexpr int t = decltype(t_)::value;
            if constexpr (tile_I(NB, T0 + t) == tile_J(NB, T0 + t)) {
                re[t] += 2.f * xre[t];
                im[t] += 2.f * xim[t];
            }
        });
    }

    // ---- sums over the k parts; every wave ends with a share of its group's tiles ----
    constexpr int kStride = kTG * ((kPer + 1) / 2) * 2 * 64;            // accumulators between k parts' areas
    static_assert(kKP == 1 || kKP * kStride * 16 <= ks_sums(MODE == XM_INT8, NB, NWV), "partial sums inside LDS");
    int t_own = T0, n_own = NT;
    ks_reduce<kPer, kKP>(re, im, (acc_t*)lds + kpart * kStride + G * (kStride / kTG), kpart, kStride, lane, t_own, n_own);

    // ---- stored baselines s1 >= s2, all four polarisation products ----
    const int64_t ch = blockIdx.x;
    const int64_t n_bl = (int64_t)a.S * (a.S + 1) / 2;
    float* tr = (float*)lds + wave * (2 * 16 * 17);
#pragma unroll
    for (int t = 0; t < ks_left(kPer, kKP); ++t) {
        if (t >= n_own) continue;
        int J = 0, I = t_own + t;                                       // tile t_own + t of the column-major list
        while (I >= NB - J) { I -= NB - J; ++J; }
        I += J;
        // lane: column b, rows aa0 .. aa0 + 3 (both polarisations of stations aa0 / 2 and aa0 / 2 + 1)
        const int b = 16 * J + row, aa0 = 16 * I + 4 * kg;
        acc_t vr = re[t], vi = im[t];
        if constexpr (MODE == XM_FP16_SPLIT) {
            if (I == J) {
                // h h^T + X + X^T and h h^T + X - X^T, or (W + W^T) / 2 and (W - W^T) / 2; the same
                // wave reads its transpose back (its LDS operations complete in order)
                const acc_t wr = kKP == 1 ? xre[t] : vr, wi = kKP == 1 ? xim[t] : vi;
#pragma unroll
                for (int r = 0; r < 4; ++r) {
                    tr[(4 * kg + r) * 17 + row] = wr[r];
                    tr[16 * 17 + (4 * kg + r) * 17 + row] = wi[r];
                }
#pragma unroll
                for (int r = 0; r < 4; ++r) {
                    const float sr = wr[r] + tr[row * 17 + 4 * kg + r], si = wi[r] - tr[16 * 17 + row * 17 + 4 * kg + r];
                    vr[r] = kKP == 1 ? vr[r] + sr : 0.5f * sr;
                    vi[r] = kKP == 1 ? vi[r] + si : 0.5f * si;
                }
            }
            vr *= a.out_scale;
            vi *= a.out_scale;
        }
#pragma unroll
        for (int r = 0; r < 4; ++r)
            if (aa0 + r == b) vi[r] = 0;
        // lanes of an even and the next odd column exchange, so that each stores two neighbouring
        // polarisation products (16 bytes): even columns XX, XY, odd columns YX, YY
#pragma unroll
        for (int u = 0; u < 2; ++u) {
            const uintx4 wr = __builtin_bit_cast(uintx4, vr), wi = __builtin_bit_cast(uintx4, vi);
            const unsigned r0 = wr[2 * u], i0 = wi[2 * u], r1 = wr[2 * u + 1], i1 = wi[2 * u + 1];
            const bool odd = (row & 1) != 0;
            const unsigned sr = odd ? r0 : r1, si = odd ? i0 : i1;      // what the neighbour stores
            const unsigned gr = __builtin_amdgcn_mov_dpp(sr, 0xb1, 0xf, 0xf, true);   // quad_perm 1, 0, 3, 2
            const unsigned gi = __builtin_amdgcn_mov_dpp(si, 0xb1, 0xf, 0xf, true);
            const int s1 = (aa0 >> 1) + u, s2 = b >> 1;
            if (s1 < a.S && s2 <= s1) {
                const uintx4 v = odd ? uintx4{gr, gi, r1, i1} : uintx4{r0, i0, gr, gi};
                ((uintx4*)a.vis)[(ch * n_bl + (int64_t)s1 * (s1 + 1) / 2 + s2) * 2 + (odd ? 1 : 0)] = v;
            }
        }
    }
}

template <int MODE, int NB, int NWV>
__global__ __launch_bounds__(64 * NWV, (ks_waves_per_simd<NB, NWV>())) void xstage_ksplit_kernel(XArgs a, XRing q) {
    extern __shared__ __attribute__((aligned(1024))) char lds[];        // q.lds_b bytes
    const int tid = threadIdx.x;
    const char* chan = (const char*)a.chan + (int64_t)blockIdx.x * a.chan_stride;
    const int g = __builtin_amdgcn_readfirstlane(tid >> 6) % ks_groups(MODE == XM_INT8, NB, NWV);
    static_for<ks_groups(MODE == XM_INT8, NB, NWV)>([&](auto gi) {
        constexpr int G = decltype(gi)::value;
        if (g == G) xks_wave<MODE, NB, NWV, G>(a, q, chan, lds, tid);
    });
}

template <int MODE, int NB, int NWV>
hipError_t launch_ksplit(const XArgs& a, hipStream_t st) {
    const XRing q = ks_ring(MODE == XM_INT8, NB, NWV, a.M, a.n_c);
    if (!ring_ok(q, KCfg<MODE>::kSteps)) return hipErrorInvalidConfiguration;
    hipLaunchKernelGGL((xstage_ksplit_kernel<MODE, NB, NWV>), dim3((unsigned)a.n_chan), dim3(64 * NWV), q.lds_b, st, a, q);
    return hipGetLastError();
}
template <int MODE, int NB>
hipError_t launch_ksplit(const XArgs& a, hipStream_t st) {
    const int nwv = ks_waves(MODE == XM_INT8, NB, a.n_c, a.n_chan, kCUs);
    if constexpr (NB <= 2) {
        if (nwv == 1) return launch_ksplit<MODE, NB, 1>(a, st);
    }
    return nwv == 8 ? launch_ksplit<MODE, NB, 8>(a, st) : launch_ksplit<MODE, NB, 4>(a, st);
}

template <int MODE>
hipError_t launch_mode(const XArgs& a, hipStream_t st) {
    switch ((a.M + 15) / 16) {
        case 1: return launch_ksplit<MODE, 1>(a, st);
        case 2: return launch_ksplit<MODE, 2>(a, st);
        case 3: return launch_ksplit<MODE, 3>(a, st);
        case 4: return launch_ksplit<MODE, 4>(a, st);
        case 5: return launch_ksplit<MODE, 5>(a, st);
        case 6: return launch_ksplit<MODE, 6>(a, st);
        case 7: return launch_ksplit<MODE, 7>(a, st);
        case 8: return launch_ksplit<MODE, 8>(a, st);
        case 9: return launch_ksplit<MODE, 9>(a, st);
        case 10: return launch_ksplit<MODE, 10>(a, st);
        default: return hipErrorInvalidValue;
    }
}

// ------------------------------------------------------------------ plain FP32 form ---
// FP32 samples and FP32 products on v_mfma_f32_16x16x4_f32 (one FP32 multiply-add per element, as
// the vector units do, at twice their rate without packed FP32).  The lower triangle of 16 x 16
// tiles (re and im accumulators) is dealt out as tile lists: `groups` workgroups per channel,
// n_tg wave groups in each and TPW tiles per wave; the 8 / n_tg waves of a group split the k-steps
// among them (8 samples each) and add their sums through LDS at the end, in a fixed order.  A
// 16-byte fragment of lane i (row i % 16, samples 2 (i / 16) and 2 (i / 16) + 1 of a k-step) is
// four k values of an A and of a B operand; Im takes (-im, re) as B.  On a diagonal tile the two
// products of Im are each other's negative transposes, so only Q = im re^T is formed and Im = Q - Q^T.
// Bound by the FP32 matrix pipes (a library product reaches 154 TFLOP/s here).  Tiles of 16 waste
// less of the triangle than tiles of 32 (24 stations: 6 x 256 against 3 x 1024 products per k), and
// the k-split keeps all eight waves busy at any station count.  Against complex FMAs on the vector
// units (one thread per 4 x 8 inputs, one workgroup per channel): 60 stations, 512 channels, 3072 samples
// 1777 -> 1045 us; 8 stations, 64 channels 1472 -> 29 us (that form had one wave per channel).
// Blocked accumulation: a wave's products over kF32Fold k-steps go into partial sums, which are
// then added to its running totals.  A single running sum over all N_c samples leaves a relative
// rounding error of about u sqrt(N_c) / 6 (u = 2^-24; the additions round at the size of the
// growing sum); partial sums of b samples folded into the totals leave about
// u (b / sqrt(N_c) + sqrt(N_c / b)) / 6, smallest near b = sqrt(N_c): 7.7 times less at
// N_c = 3072 and b = 128.
constexpr int kF32Fold = 16;                  // k-steps of 8 samples

template <int TPW>
__global__ __launch_bounds__(64 * kF32Waves, 2) void xstage_f32_kernel(XArgs a, XRing q, XF32 f) {
    extern __shared__ __attribute__((aligned(1024))) char lds[];        // q.lds_b bytes
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int64_t ch = blockIdx.x / f.groups;
    const int tg = wave % f.n_tg, kpart = wave / f.n_tg, n_kp = kF32Waves / f.n_tg;
    const char* chan = (const char*)a.chan + ch * a.chan_stride;

    // this wave's tiles: TPW consecutive ones of the column-major lower triangle (tiles past the
    // end repeat the last one and are not stored)
    const int t0 = ((int)(blockIdx.x % f.groups) * f.n_tg + tg) * TPW;
    const int nt = min(TPW, f.n_tiles - t0);  // <= 0: an idle wave (it still moves data)
    int ti[TPW], tj[TPW];
    {
        int J = 0, left = min(t0, f.n_tiles - 1);
        while (left >= f.nb - J) { left -= f.nb - J; ++J; }
        int I = J + left;
#pragma unroll
        for (int t = 0; t < TPW; ++t) {
            ti[t] = I;
            tj[t] = J;
            if (t + 1 < nt) {
                if (++I == f.nb) { ++J; I = J; }
            }
        }
    }
    floatx4 re[TPW], im[TPW], tre[TPW], tim[TPW];   // partial sums, running totals
#pragma unroll
    for (int t = 0; t < TPW; ++t) re[t] = im[t] = tre[t] = tim[t] = floatx4{};
    int step = kpart, since = 0;              // k-step inside the stage, k-steps since the last fold

    ring_loop<XM_FP32, kF32Waves>(a, q, chan, lds, tid, [&](char* buf, int nch) {
        if (nt > 0) {
            for (step = kpart; step < 4 * nch; step += n_kp) {
                const char* base = buf + (step >> 2) * q.chunk_b + (lane & 15) * kRowB +
                                   (((4 * (step & 3) + (lane >> 4)) ^ (lane & 15)) << 4);
                // each tile's fragments are read before the products of the tile before it
                floatx4 An = *(const floatx4*)(base + ti[0] * (16 * kRowB));
                floatx4 Bn = *(const floatx4*)(base + tj[0] * (16 * kRowB));
#pragma unroll
                for (int t = 0; t < TPW; ++t) {
                    const floatx4 A = An, B = Bn;
                    if (t + 1 < TPW) {
                        An = *(const floatx4*)(base + ti[t + 1] * (16 * kRowB));
                        Bn = *(const floatx4*)(base + tj[t + 1] * (16 * kRowB));
                        __builtin_amdgcn_sched_barrier(0);
                    }
                    re[t] = __builtin_amdgcn_mfma_f32_16x16x4f32(A[0], B[0], re[t], 0, 0, 0);
                    im[t] = __builtin_amdgcn_mfma_f32_16x16x4f32(A[1], B[0], im[t], 0, 0, 0);
                    re[t] = __builtin_amdgcn_mfma_f32_16x16x4f32(A[1], B[1], re[t], 0, 0, 0);
                    im[t] = __builtin_amdgcn_mfma_f32_16x16x4f32(A[3], B[2], im[t], 0, 0, 0);
                    re[t] = __builtin_amdgcn_mfma_f32_16x16x4f32(A[2], B[2], re[t], 0, 0, 0);
                    re[t] = __builtin_amdgcn_mfma_f32_16x16x4f32(A[3], B[3], re[t], 0, 0, 0);
                    if (ti[t] != tj[t]) {
                        im[t] = __builtin_amdgcn_mfma_f32_16x16x4f32(A[0], -B[1], im[t], 0, 0, 0);
                        im[t] = __builtin_amdgcn_mfma_f32_16x16x4f32(A[2], -B[3], im[t], 0, 0, 0);
                    }
                }
                if (++since == kF32Fold) {
                    since = 0;
#pragma unroll
                    for (int t = 0; t < TPW; ++t) {
                        tre[t] += re[t];
                        tim[t] += im[t];
                        re[t] = im[t] = floatx4{};
                    }
                }
            }
        }
    });
#pragma unroll
    for (int t = 0; t < TPW; ++t) {
        tre[t] += re[t];
        tim[t] += im[t];
    }
    // sums over the k parts, halving their number per round
    floatx4* red = (floatx4*)lds;             // [k part][wave group][tile][re, im][lane]
    for (int half = n_kp / 2; half >= 1; half >>= 1) {
        if (kpart >= half && kpart < 2 * half) {
            floatx4* dst = red + (size_t)((kpart - half) * f.n_tg + tg) * TPW * 2 * 64 + lane;
#pragma unroll
            for (int t = 0; t < TPW; ++t) {
                dst[(2 * t) * 64] = tre[t];
                dst[(2 * t + 1) * 64] = tim[t];
            }
        }
        lds_barrier();
        if (kpart < half) {
            const floatx4* src = red + (size_t)(kpart * f.n_tg + tg) * TPW * 2 * 64 + lane;
#pragma unroll
            for (int t = 0; t < TPW; ++t) {
                tre[t] += src[(2 * t) * 64];
                tim[t] += src[(2 * t + 1) * 64];
            }
        }
        lds_barrier();
    }
    if (kpart != 0) return;
    const int64_t B = (int64_t)a.S * (a.S + 1) / 2;
    float* tr = (float*)lds + tg * (16 * 17);
#pragma unroll
    for (int t = 0; t < TPW; ++t) {
        const int b = 16 * tj[t] + (lane & 15);
        if (ti[t] == tj[t]) {
            // the same wave reads its transpose back (its LDS operations complete in order)
#pragma unroll
            for (int r = 0; r < 4; ++r) tr[(4 * (lane >> 4) + r) * 17 + (lane & 15)] = tim[t][r];
#pragma unroll
            for (int r = 0; r < 4; ++r) tim[t][r] -= tr[(lane & 15) * 17 + 4 * (lane >> 4) + r];
        }
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            const int aa = 16 * ti[t] + 4 * (lane >> 4) + r;
            const int s1 = aa >> 1, s2 = b >> 1;
            if (t < nt && aa < a.M && b < a.M && s1 >= s2) {
                const int64_t idx = (ch * B + (int64_t)s1 * (s1 + 1) / 2 + s2) * 4 + 2 * (aa & 1) + (b & 1);
                ((float2*)a.vis)[idx] = make_float2(tre[t][r], aa == b ? 0.f : tim[t][r]);
            }
        }
    }
}

}  // namespace

hipError_t launch_xstage_mfma(int x_mode, const XArgs& a, hipStream_t st) {
    if (a.n_chan <= 0) return hipSuccess;
    if (x_mode == XM_FP16_SPLIT) return launch_mode<XM_FP16_SPLIT>(a, st);
    if (x_mode == XM_INT8) return launch_mode<XM_INT8>(a, st);
    return hipErrorInvalidValue;
}

hipError_t launch_xstage_fp32(const XArgs& a, hipStream_t st) {
    if (a.n_chan <= 0) return hipSuccess;
    const XF32 f = f32_split(a.M, a.n_c, a.n_chan, kCUs);
    if (f.n_tg < 1) return hipErrorInvalidConfiguration;
    const XRing q = f32_ring(f, a.M, a.n_c);
    if (!ring_ok(q, kF32Steps)) return hipErrorInvalidConfiguration;
    const dim3 grid((unsigned)((int64_t)a.n_chan * f.groups)), block(64 * kF32Waves);
    switch (f.tpw) {
        case 1: hipLaunchKernelGGL(xstage_f32_kernel<1>, grid, block, q.lds_b, st, a, q, f); break;
        case 2: hipLaunchKernelGGL(xstage_f32_kernel<2>, grid, block, q.lds_b, st, a, q, f); break;
        case 3: hipLaunchKernelGGL(xstage_f32_kernel<3>, grid, block, q.lds_b, st, a, q, f); break;
        case 4: hipLaunchKernelGGL(xstage_f32_kernel<4>, grid, block, q.lds_b, st, a, q, f); break;
        case 5: hipLaunchKernelGGL(xstage_f32_kernel<5>, grid, block, q.lds_b, st, a, q, f); break;
        case 6: hipLaunchKernelGGL(xstage_f32_kernel<6>, grid, block, q.lds_b, st, a, q, f); break;
        case 7: hipLaunchKernelGGL(xstage_f32_kernel<7>, grid, block, q.lds_b, st, a, q, f); break;
        case 8: hipLaunchKernelGGL(xstage_f32_kernel<8>, grid, block, q.lds_b, st, a, q, f); break;
        case 9: hipLaunchKernelGGL(xstage_f32_kernel<9>, grid, block, q.lds_b, st, a, q, f); break;
        default: return hipErrorInvalidValue;
    }
    return hipGetLastError();
}

}  // namespace cobalt
