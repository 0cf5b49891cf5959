// X stage of the FX correlator for gfx950: per channel, V = Z Z^H over all inputs
// (station x polarisation), integrated over the block ("Signal processing with GPU
// kernels", sec. 7.5: correlations of all pairs of antenna fields, averaged to ~1 s).
//
// MFMA form (FP16-split and int8): a complex Hermitian rank-K update written as two real
// contractions over K = 2 N_c interleaved (re, im) values:
//     Re V[a][b] = sum_k A[a][k] A[b][k]         (A = interleaved rows of Z)
//     Im V[a][b] = sum_k A[a][k] A'[b][k]        (A' = per sample (re, im) -> (-im, re))
// One workgroup owns one channel and keeps every lower-triangle 32x32 tile of V in
// accumulators; channel rows stream through LDS once.  An MFMA fragment of row block I
// (lane i: row 32I + i%32, 8 halves / 16 bytes of K) is simultaneously an A operand (row
// I) and a B operand (column I), so both operands of a tile come from the same LDS reads
// and the k order inside a fragment never matters.  A' is built in registers from the
// B-role fragments.
//   FP16-split: Z*2^k = hi + lo (two fp16 planes); V ~= hh + hl + lh accumulated in FP32
//   (the dropped lo*lo term is below 2^-22 of |Z|^2), scaled back by 2^-2k.  On a diagonal
//   tile (I = J) the lh product is the transpose of hl (real part) and minus its transpose
//   (imaginary part), so it is not multiplied but added from hl at the end (where registers
//   allow: every diagonal tile of the 152-input grid).
//   int8: exact int32 sums.
// Plain FP32 form: the same two contractions on FP32 operands and FP32 MFMAs over 16x16 tiles, with
// partial sums over 128 channel samples folded into running totals.
#include <type_traits>

#include "cobalt_internal.h"

namespace cobalt {
namespace {

typedef _Float16 half8 __attribute__((ext_vector_type(8)));
typedef float floatx4 __attribute__((ext_vector_type(4)));
typedef float floatx16 __attribute__((ext_vector_type(16)));
typedef int intx16 __attribute__((ext_vector_type(16)));
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
constexpr int tile_count(int R) { return R * (R + 1) / 2; }
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
constexpr int kTilesPerWave = 4;
// blocks used by wave W as A (row) or B (column) operands
constexpr unsigned wave_blocks(int R, int W, bool as_b) {
    unsigned m = 0;
    for (int t = kTilesPerWave * W; t < kTilesPerWave * W + kTilesPerWave && t < tile_count(R); ++t)
        m |= 1u << (as_b ? tile_J(R, t) : tile_I(R, t));
    return m;
}

// Whether wave W of an R-block grid forms lh of its diagonal tiles from hl (FP16-split): each
// such tile holds one more accumulator pair, so only where at most 5 pairs fit in registers.
constexpr bool diag_from_hl(int R, int W) {
    int n = 0, d = 0;
    for (int t = kTilesPerWave * W; t < kTilesPerWave * W + kTilesPerWave && t < tile_count(R); ++t) {
        ++n;
        if (tile_I(R, t) == tile_J(R, t)) ++d;
    }
    return n + d <= 5;
}

template <int MODE> struct XCfg;
template <> struct XCfg<XM_FP16_SPLIT> {
    static constexpr int kKc = 32;            // complex samples per chunk (one K block)
    static constexpr int kSteps = 4;          // k-steps of 16 halves per chunk
    using acc_t = floatx16;
    using frag_t = half8;
};
template <> struct XCfg<XM_INT8> {
    static constexpr int kKc = 128;           // complex samples per chunk (four K blocks)
    static constexpr int kSteps = 8;          // k-steps of 32 bytes per chunk
    using acc_t = intx16;
    using frag_t = intx4;
};
constexpr int kRowB = 256;                    // LDS bytes per row and chunk (16 granules of 16 B)

// LDS rows are XOR-swizzled in 16-byte granules (granule g of row r is stored at g ^ (r%16)),
// so the 32 rows of one MFMA fragment read hit distinct banks without padding.
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

// Issue the global -> LDS transfers of one chunk (rows < M) into LDS buffer `buf`.  One
// instruction moves 64 lanes x 16 B into 1 KB of consecutive LDS (4 rows); lane L of
// instruction i fills row 4i + L/16, stored granule L%16.  Rows >= M are never written.
//   FP16-split chunk = K block kb: [hi: M rows x 128 B][lo: M rows x 128 B]; logical granule
//   g < 8 is hi bytes 16g.., g >= 8 lo bytes 16(g-8)...
//   int8 chunk = K blocks kb..kb+3, each [M rows x 64 B]; logical granule g is block g/4,
//   bytes 16(g%4)...  Blocks past the last one are not loaded.
template <int MODE>
__device__ __forceinline__ void issue_chunk(const XArgs& a, const char* __restrict__ chan, char* buf, int kc0, int wave, int lane) {
    const int n_inst = (a.M + 3) / 4;
    const int rsub = lane >> 4, p = lane & 15;
    for (int i = wave; i < n_inst; i += 4) {
        const int row = 4 * i + rsub;
        const int g = p ^ (row & 15);
        const char* src;
        bool ok = row < a.M;
        if constexpr (MODE == XM_FP16_SPLIT) {
            const char* blk = chan + (int64_t)(kc0 / kKBlock) * (2 * a.M * 128);
            src = blk + (g >> 3) * (a.M * 128) + row * 128 + (g & 7) * 16;
        } else {
            const int kb = kc0 / kKBlock + (g >> 2);
            ok = ok && kb < a.n_kb;
            src = chan + (int64_t)kb * (a.M * 64) + row * 64 + (g & 3) * 16;
        }
        // non-temporal: each byte of the channelised data is read once (measured ~1.5 % faster)
        if (ok) __builtin_amdgcn_global_load_lds((const void*)src, (lds_ptr_t)(buf + i * 1024), 16, 0, 2);
    }
}

// Zero the LDS entries of columns >= N_c (the last, partial chunk) and of K blocks that were
// not loaded, for rows < M.
template <int MODE>
__device__ __forceinline__ void zero_tail(const XArgs& a, char* buf, int kc0, int tid) {
    constexpr int kKc = XCfg<MODE>::kKc;
    const int first = a.n_c - kc0;                     // first column to clear
    const int cols = kKc - first;
    for (int id = tid; id < a.M * cols; id += 256) {
        const int row = id / cols, c = first + id % cols;
        if constexpr (MODE == XM_FP16_SPLIT) {
            *(unsigned*)(buf + lds_off(row, c >> 2) + (c & 3) * 4) = 0u;        // hi
            *(unsigned*)(buf + lds_off(row, 8 + (c >> 2)) + (c & 3) * 4) = 0u;  // lo
        } else {
            *(unsigned short*)(buf + lds_off(row, c >> 3) + (c & 7) * 2) = 0;
        }
    }
}

template <int MODE, int R, int W>
__device__ __forceinline__ void xwave(const XArgs& a, const char* __restrict__ chan, char* lds, int tid) {
    using C_ = XCfg<MODE>;
    using acc_t = typename C_::acc_t;
    using frag_t = typename C_::frag_t;
    constexpr int NT = tile_count(R);
    constexpr int T0 = kTilesPerWave * W;
    constexpr int NW = NT - T0 <= 0 ? 0 : (NT - T0 > kTilesPerWave ? kTilesPerWave : NT - T0);
    constexpr unsigned useA = wave_blocks(R, W, false) | wave_blocks(R, W, true);
    constexpr unsigned useB = wave_blocks(R, W, true);
    constexpr bool kDiagHl = MODE == XM_FP16_SPLIT && diag_from_hl(R, W);
    constexpr int kBufB = R * 32 * kRowB;
    const int lane = tid & 63;

    acc_t vre[kTilesPerWave], vim[kTilesPerWave];
    acc_t xre[kTilesPerWave], xim[kTilesPerWave];     // hl of diagonal tiles (FP16-split)
#pragma unroll
    for (int t = 0; t < kTilesPerWave; ++t) {
        vre[t] = acc_t{};
        vim[t] = acc_t{};
        xre[t] = acc_t{};
        xim[t] = acc_t{};
    }

    // rows M .. 32R-1 stay zero in both buffers
    for (int off = a.M * kRowB + tid * 16; off < kBufB; off += 256 * 16) {
        *(uint4*)(lds + off) = make_uint4(0, 0, 0, 0);
        *(uint4*)(lds + kBufB + off) = make_uint4(0, 0, 0, 0);
    }
    __syncthreads();
    if (a.n_c > 0) issue_chunk<MODE>(a, chan, lds, 0, W, lane);

    int cur = 0;
    for (int kc0 = 0; kc0 < a.n_c; kc0 += C_::kKc) {
        char* buf = lds + cur * kBufB;
        __builtin_amdgcn_s_waitcnt(0);        // this wave's transfers of chunk kc0 have landed
        __syncthreads();                      // ... and everyone's; the other buffer is free
        if (kc0 + C_::kKc < a.n_c) issue_chunk<MODE>(a, chan, lds + (cur ^ 1) * kBufB, kc0 + C_::kKc, W, lane);
        if (kc0 + C_::kKc > a.n_c) {          // last, partial chunk (uniform)
            zero_tail<MODE>(a, buf, kc0, tid);
            __syncthreads();
        }
        if constexpr (NW > 0) {
#pragma unroll
            for (int ks = 0; ks < C_::kSteps; ++ks) {
                const int row = lane & 31;
                const int g = 2 * ks + (lane >> 5);
                if constexpr (MODE == XM_FP16_SPLIT) {
                    uintx4 fh[R], fl[R], gh[R], gl[R];
                    static_for<R>([&](auto bi) {
                        constexpr int b = decltype(bi)::value;
                        if constexpr ((useA >> b) & 1u) {
                            fh[b] = *(const uintx4*)(buf + lds_off(32 * b + row, g));
                            fl[b] = *(const uintx4*)(buf + lds_off(32 * b + row, 8 + g));
                        }
                        if constexpr ((useB >> b) & 1u) {
                            gh[b] = swapneg_f16(fh[b]);
                            gl[b] = swapneg_f16(fl[b]);
                        }
                    });
                    // three products (hh, hl, lh), each over all tiles: independent accumulators
                    // between dependent MFMAs; diagonal tiles keep hl apart and skip lh
                    static_for<3>([&](auto pi) {
                        constexpr int pr = decltype(pi)::value;
                        static_for<NW>([&](auto ti) {
                            constexpr int t = decltype(ti)::value;
                            constexpr int I = tile_I(R, T0 + t), J = tile_J(R, T0 + t);
                            constexpr bool dg = kDiagHl && I == J;
                            if constexpr (!(dg && pr == 2)) {
                                const frag_t A = __builtin_bit_cast(frag_t, pr == 2 ? fl[I] : fh[I]);
                                const frag_t B = __builtin_bit_cast(frag_t, pr == 1 ? fl[J] : fh[J]);
                                const frag_t Bs = __builtin_bit_cast(frag_t, pr == 1 ? gl[J] : gh[J]);
                                if constexpr (dg && pr == 1) {
                                    xre[t] = __builtin_amdgcn_mfma_f32_32x32x16_f16(A, B, xre[t], 0, 0, 0);
                                    xim[t] = __builtin_amdgcn_mfma_f32_32x32x16_f16(A, Bs, xim[t], 0, 0, 0);
                                } else {
                                    vre[t] = __builtin_amdgcn_mfma_f32_32x32x16_f16(A, B, vre[t], 0, 0, 0);
                                    vim[t] = __builtin_amdgcn_mfma_f32_32x32x16_f16(A, Bs, vim[t], 0, 0, 0);
                                }
                            }
                        });
                    });
                } else {
                    uintx4 f[R], gg[R];
                    static_for<R>([&](auto bi) {
                        constexpr int b = decltype(bi)::value;
                        if constexpr ((useA >> b) & 1u) f[b] = *(const uintx4*)(buf + lds_off(32 * b + row, g));
                        if constexpr ((useB >> b) & 1u) gg[b] = swapneg_i8(f[b]);
                    });
                    static_for<NW>([&](auto ti) {
                        constexpr int t = decltype(ti)::value;
                        constexpr int I = tile_I(R, T0 + t), J = tile_J(R, T0 + t);
                        const frag_t A = __builtin_bit_cast(frag_t, f[I]);
                        const frag_t B = __builtin_bit_cast(frag_t, f[J]);
                        const frag_t Bs = __builtin_bit_cast(frag_t, gg[J]);
                        vre[t] = __builtin_amdgcn_mfma_i32_32x32x32_i8(A, B, vre[t], 0, 0, 0);
                        vim[t] = __builtin_amdgcn_mfma_i32_32x32x32_i8(A, Bs, vim[t], 0, 0, 0);
                    });
                }
            }
        }
        cur ^= 1;
    }

    // ---- diagonal tiles (FP16-split): Re += hl + hl^T, Im += hl - hl^T, through LDS ----
    if constexpr (MODE == XM_FP16_SPLIT) {
        __syncthreads();                      // every wave is done with the chunk buffers
        constexpr int kTw = 2 * 32 * 33;      // floats per wave: two padded 32 x 32 tiles
        float* tr = (float*)lds + W * kTw;
        static_for<NW>([&](auto ti) {
            constexpr int t = decltype(ti)::value;
            constexpr int I = tile_I(R, T0 + t), J = tile_J(R, T0 + t);
            if constexpr (kDiagHl && I == J) {
                static_assert((W + 1) * kTw * 4 <= 2 * R * 32 * kRowB, "transpose area inside LDS");
                const int col = lane & 31;
#pragma unroll
                for (int r = 0; r < 16; ++r) {
                    const int row = 8 * (r >> 2) + 4 * (lane >> 5) + (r & 3);
                    tr[row * 33 + col] = xre[t][r];
                    tr[32 * 33 + row * 33 + col] = xim[t][r];
                }
                // the same wave reads the transpose back (its LDS operations complete in order)
#pragma unroll
                for (int r = 0; r < 16; ++r) {
                    const int row = 8 * (r >> 2) + 4 * (lane >> 5) + (r & 3);
                    vre[t][r] += xre[t][r] + tr[col * 33 + row];
                    vim[t][r] += xim[t][r] - tr[32 * 33 + col * 33 + row];
                }
            }
        });
    }

    // ---- epilogue: stored baselines s1 >= s2, all four polarisation products ----
    if constexpr (NW > 0) {
        const int64_t ch = blockIdx.x;
        const int64_t B = (int64_t)a.S * (a.S + 1) / 2;
        static_for<NW>([&](auto ti) {
            constexpr int t = decltype(ti)::value;
            constexpr int I = tile_I(R, T0 + t), J = tile_J(R, T0 + t);
            const int b = 32 * J + (lane & 31);
#pragma unroll
            for (int r = 0; r < 16; ++r) {
                const int aa = 32 * I + 8 * (r >> 2) + 4 * (lane >> 5) + (r & 3);
                if (aa < a.M && b < a.M) {
                    const int s1 = aa >> 1, s2 = b >> 1;
                    if (s1 >= s2) {
                        const int64_t idx = (ch * B + (int64_t)s1 * (s1 + 1) / 2 + s2) * 4 + 2 * (aa & 1) + (b & 1);
                        if constexpr (MODE == XM_FP16_SPLIT) {
                            const float re = vre[t][r] * a.out_scale;
                            const float im = aa == b ? 0.f : vim[t][r] * a.out_scale;
                            ((float2*)a.vis)[idx] = make_float2(re, im);
                        } else {
                            ((int2*)a.vis)[idx] = make_int2(vre[t][r], aa == b ? 0 : vim[t][r]);
                        }
                    }
                }
            }
        });
    }
}

template <int MODE, int R>
__global__ __launch_bounds__(256, 2) void xstage_mfma_kernel(XArgs a) {
    __shared__ __attribute__((aligned(1024))) char lds[2 * R * 32 * kRowB];   // two chunk buffers
    const int tid = threadIdx.x;
    const char* chan = (const char*)a.chan + (int64_t)blockIdx.x * a.chan_stride;
    switch (tid >> 6) {
        case 0: xwave<MODE, R, 0>(a, chan, lds, tid); break;
        case 1: xwave<MODE, R, 1>(a, chan, lds, tid); break;
        case 2: xwave<MODE, R, 2>(a, chan, lds, tid); break;
        default: xwave<MODE, R, 3>(a, chan, lds, tid); break;
    }
}

template <int MODE>
hipError_t launch_mode(const XArgs& a, hipStream_t st) {
    const int R = (a.M + 31) / 32;
    const dim3 grid((unsigned)a.n_chan), block(256);
    switch (R) {
        case 1: hipLaunchKernelGGL((xstage_mfma_kernel<MODE, 1>), grid, block, 0, st, a); break;
        case 2: hipLaunchKernelGGL((xstage_mfma_kernel<MODE, 2>), grid, block, 0, st, a); break;
        case 3: hipLaunchKernelGGL((xstage_mfma_kernel<MODE, 3>), grid, block, 0, st, a); break;
        case 4: hipLaunchKernelGGL((xstage_mfma_kernel<MODE, 4>), grid, block, 0, st, a); break;
        case 5: hipLaunchKernelGGL((xstage_mfma_kernel<MODE, 5>), grid, block, 0, st, a); break;
        default: return hipErrorInvalidValue;
    }
    return hipGetLastError();
}

// ------------------------------------------------------------------ LDS ring ---
// Chunks (one K block in FP32 and FP16-split mode, four in int8 mode; 256 bytes per row) stream
// global -> LDS through a ring of `depth` stages of `nch` chunks, depth - 1 of them in flight.
// Only ceil(M/4)*4 rows are kept per chunk; fragment reads of a row block's padding rows fall on
// whatever follows inside the LDS array, and only reach outputs that are never stored.
struct XRing {
    int nch, depth;          // chunks per stage, stages
    int n_inst, ipw;         // 1 KB transfers per chunk, transfers per wave and (full) stage
    int chunk_b;             // bytes per chunk
    int n_chunk;             // chunks of a channel
};

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

// Issue stage s into its ring slot.  Every wave issues exactly ipw transfers of a full stage (the
// last ones repeat the stage's final transfer), so that counted waits hold for every wave; the
// last, partial stage may issue fewer.
template <int MODE, int NWV>
__device__ __forceinline__ void ring_issue(const XArgs& a, const XRing& q, const char* __restrict__ chan, char* lds, int s, int wave,
                                           int lane) {
    const int c0 = s * q.nch, nch = min(q.nch, q.n_chunk - c0);
    char* buf = lds + (s % q.depth) * (q.nch * q.chunk_b);
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

// Host: ring of at most lds_b bytes (minus `slack` bytes that fragment reads may run past the
// last chunk).  Stages of about 8 KB per wave keep the barriers few; the depth takes the rest.
XRing make_ring(int mode, const XArgs& a, int waves, int lds_b, int slack, int nch_multiple) {
    XRing q{};
    const int kc = mode == XM_INT8 ? 128 : 32;
    q.n_chunk = (a.n_c + kc - 1) / kc;
    q.n_inst = (a.M + 3) / 4;
    q.chunk_b = q.n_inst * 1024;
    const int room = (lds_b - slack) / q.chunk_b;                  // chunks that fit
    int nch = room / 3;                                            // three stages or more
    nch = nch / nch_multiple * nch_multiple;
    nch = nch < 1 ? (room >= 2 * nch_multiple ? nch_multiple : 1) : nch > 8 ? 8 : nch;
    while (nch > nch_multiple && nch * q.n_inst > 8 * waves) nch -= nch_multiple;
    q.nch = nch;
    q.ipw = (nch * q.n_inst + waves - 1) / waves;
    q.depth = room / nch;
    while (q.depth > 3 && (q.depth - 2) * q.ipw > 32) --q.depth;  // counted waits are built up to 32
    if (q.depth > 8) q.depth = 8;
    return q;
}

// Zero columns >= n_c of the last chunk (`cols` of them from its column `first`) for rows < M.
template <int MODE>
__device__ __forceinline__ void zero_columns(const XArgs& a, char* buf, int first, int cols, int tid, int nthr) {
    for (int id = tid; id < a.M * cols; id += nthr) {
        const int row = id / cols, c = first + id % cols;
        if constexpr (MODE == XM_FP32) {
            *(uint2*)(buf + lds_off(row, c >> 1) + (c & 1) * 8) = make_uint2(0u, 0u);
        } else if constexpr (MODE == XM_FP16_SPLIT) {
            *(unsigned*)(buf + lds_off(row, c >> 2) + (c & 3) * 4) = 0u;        // hi
            *(unsigned*)(buf + lds_off(row, 8 + (c >> 2)) + (c & 3) * 4) = 0u;  // lo
        } else {
            *(unsigned short*)(buf + lds_off(row, c >> 3) + (c & 7) * 2) = 0;
        }
    }
}

// The ring's loop over a channel: body(stage buffer, chunks in the stage, stage index) runs with
// every chunk of the stage in LDS.
template <int MODE, int NWV, class F>
__device__ __forceinline__ void ring_loop(const XArgs& a, const XRing& q, const char* __restrict__ chan, char* lds, int tid, F&& body) {
    constexpr int kc = MODE == XM_INT8 ? 128 : 32;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6), lane = tid & 63;
    const int n_stage = (q.n_chunk + q.nch - 1) / q.nch, n_full = q.n_chunk / q.nch;
    for (int s = 0; s < min(q.depth - 1, n_stage); ++s) ring_issue<MODE, NWV>(a, q, chan, lds, s, wave, lane);
    for (int s = 0; s < n_stage; ++s) {
        // stages s + 1 .. s + depth - 2 may still be in flight (counted where all of them are full)
        wait_transfers(s + q.depth - 2 < n_full ? q.ipw * (q.depth - 2) : 0);
        lds_barrier();                        // ... for every wave; the slot of stage s - 1 is free
        if (s + q.depth - 1 < n_stage) ring_issue<MODE, NWV>(a, q, chan, lds, s + q.depth - 1, wave, lane);
        char* buf = lds + (s % q.depth) * (q.nch * q.chunk_b);
        const int nch = min(q.nch, q.n_chunk - s * q.nch);
        if (s == n_stage - 1 && a.n_c % kc != 0) {
            const int first = a.n_c % kc;
            zero_columns<MODE>(a, buf + (nch - 1) * q.chunk_b, first, kc - first, tid, 64 * NWV);
            lds_barrier();
        }
        body(buf, nch);
    }
    lds_barrier();                            // every wave is done with the chunks
}

// ------------------------------------------------------------------ plain FP32 form ---
// FP32 samples and FP32 products on v_mfma_f32_16x16x4_f32 (one FP32 multiply-add per element, as
// the vector units do, at twice their rate without packed FP32).  The lower triangle of 16 x 16
// tiles (re and im accumulators) is dealt out as tile lists: `groups` workgroups per channel,
// n_tg wave groups in each and TPW tiles per wave; the 8 / n_tg waves of a group split the k-steps
// among them (8 samples each) and add their sums through LDS at the end, in a fixed order.  A
// 16-byte fragment of lane i (row i % 16, samples 2 (i / 16) and 2 (i / 16) + 1 of a k-step) is
// four k values of an A and of a B operand; Im takes (-im, re) as B.
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
constexpr int kF32Waves = 8;
constexpr int kF32LdsB = 147456;
constexpr int kF32Fold = 16;                  // k-steps of 8 samples
constexpr int kF32MaxTpw = 9;                 // 144 accumulator registers, two waves per SIMD

struct XF32 {
    int n_tiles, nb, groups, n_tg;
};

template <int TPW>
__global__ __launch_bounds__(64 * kF32Waves, 2) void xstage_f32_kernel(XArgs a, XRing q, XF32 f) {
    __shared__ __attribute__((aligned(1024))) char lds[kF32LdsB];
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
#pragma unroll
                for (int t = 0; t < TPW; ++t) {
                    const floatx4 A = *(const floatx4*)(base + ti[t] * (16 * kRowB));
                    const floatx4 B = *(const floatx4*)(base + tj[t] * (16 * kRowB));
                    re[t] = __builtin_amdgcn_mfma_f32_16x16x4f32(A[0], B[0], re[t], 0, 0, 0);
                    im[t] = __builtin_amdgcn_mfma_f32_16x16x4f32(A[0], -B[1], im[t], 0, 0, 0);
                    re[t] = __builtin_amdgcn_mfma_f32_16x16x4f32(A[1], B[1], re[t], 0, 0, 0);
                    im[t] = __builtin_amdgcn_mfma_f32_16x16x4f32(A[1], B[0], im[t], 0, 0, 0);
                    re[t] = __builtin_amdgcn_mfma_f32_16x16x4f32(A[2], B[2], re[t], 0, 0, 0);
                    im[t] = __builtin_amdgcn_mfma_f32_16x16x4f32(A[2], -B[3], im[t], 0, 0, 0);
                    re[t] = __builtin_amdgcn_mfma_f32_16x16x4f32(A[3], B[3], re[t], 0, 0, 0);
                    im[t] = __builtin_amdgcn_mfma_f32_16x16x4f32(A[3], B[2], im[t], 0, 0, 0);
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
#pragma unroll
    for (int t = 0; t < TPW; ++t) {
        const int b = 16 * tj[t] + (lane & 15);
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
    XF32 f{};
    f.nb = (a.M + 15) / 16;
    f.n_tiles = f.nb * (f.nb + 1) / 2;
    // Split with the least time per CU: rounds of workgroups x tile slots per channel share.  A
    // smaller number of workgroups per channel reads the channel fewer times; fewer wave groups
    // waste fewer slots but need the k-split sums, so ties go to more groups of waves.
    int best = 0x7fffffff, tpw = 1;
    for (int groups = 1; groups <= 4; ++groups)
        for (int n_tg = kF32Waves; n_tg >= 1; n_tg /= 2) {
            const int per = (f.n_tiles + groups * n_tg - 1) / (groups * n_tg);
            if (per > kF32MaxTpw) continue;
            const int64_t rounds = ((int64_t)a.n_chan * groups + kCUs - 1) / kCUs;
            const int64_t cost = rounds * per * n_tg;
            if (cost < best) { best = (int)cost; tpw = per; f.groups = groups; f.n_tg = n_tg; }
        }
    const int n_kp = kF32Waves / f.n_tg;
    const XRing q = make_ring(XM_FP32, a, kF32Waves, kF32LdsB, (16 * f.nb - (a.M + 3) / 4 * 4) * kRowB, n_kp == 8 ? 2 : 1);
    const dim3 grid((unsigned)((int64_t)a.n_chan * f.groups)), block(64 * kF32Waves);
    switch (tpw) {
        case 1: hipLaunchKernelGGL(xstage_f32_kernel<1>, grid, block, 0, st, a, q, f); break;
        case 2: hipLaunchKernelGGL(xstage_f32_kernel<2>, grid, block, 0, st, a, q, f); break;
        case 3: hipLaunchKernelGGL(xstage_f32_kernel<3>, grid, block, 0, st, a, q, f); break;
        case 4: hipLaunchKernelGGL(xstage_f32_kernel<4>, grid, block, 0, st, a, q, f); break;
        case 5: hipLaunchKernelGGL(xstage_f32_kernel<5>, grid, block, 0, st, a, q, f); break;
        case 6: hipLaunchKernelGGL(xstage_f32_kernel<6>, grid, block, 0, st, a, q, f); break;
        case 7: hipLaunchKernelGGL(xstage_f32_kernel<7>, grid, block, 0, st, a, q, f); break;
        case 8: hipLaunchKernelGGL(xstage_f32_kernel<8>, grid, block, 0, st, a, q, f); break;
        case 9: hipLaunchKernelGGL(xstage_f32_kernel<9>, grid, block, 0, st, a, q, f); break;
        default: return hipErrorInvalidValue;
    }
    return hipGetLastError();
}

}  // namespace cobalt
