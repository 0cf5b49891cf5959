// Plan of the X stage's LDS ring: which work split a form takes, how much LDS it has and how the
// ring is cut into stages.  Plain C++ (no HIP), so that the plan and the order of transfers, waits
// and reads can be checked on the host for every number of inputs.
#pragma once

namespace cobalt {

constexpr int kRowB = 256;                    // LDS bytes per row and chunk (16 granules of 16 B)

constexpr int tile_count(int R) { return R * (R + 1) / 2; }

// Chunks (one K block in FP32 and FP16-split mode, four in int8 mode; 256 bytes per row) stream
// global -> LDS through a ring of `depth` >= 2 stages of `nch` chunks: while a stage is read, the
// next depth - 1 are in flight.  Only ceil(M/4)*4 rows are kept per chunk.  The padding rows of the
// last row block (their results are never stored):
//   FP32: fragment reads fall on whatever follows inside the LDS array, which the ring leaves room for;
//   FP16-split and int8: a zero operand spares the matrix pipes' power, so their reads go to a row of
//   zeros behind the ring; where the chunk itself holds all of the last row block (M = 16 NB - 2 or
//   16 NB) there is no such row, and rows M and M + 1 of every slot are zeroed once instead.  The
//   row is not reserved without need: at 79 and 80 stations two chunks fill the 80 KB to the last byte.
struct XRing {
    int nch, depth;          // chunks per stage, stages
    int n_inst, ipw;         // 1 KB transfers per chunk, transfers per wave and (full) stage
    int chunk_b;             // bytes per chunk
    int n_chunk;             // chunks of a channel
};

// Stages of a channel; stages issued before the first one is read; transfers of a wave that may be
// in flight while stage s is read (those of stages s + 1 .. s + depth - 2, counted where all of them
// are full).
constexpr int ring_stages(const XRing& q) { return (q.n_chunk + q.nch - 1) / q.nch; }
constexpr int ring_ahead(const XRing& q) { return q.depth - 1 < ring_stages(q) ? q.depth - 1 : ring_stages(q); }
constexpr int ring_may_fly(const XRing& q, int s) { return s + q.depth - 2 < q.n_chunk / q.nch ? q.ipw * (q.depth - 2) : 0; }

// Ring of at most lds_b bytes.  Stages of about 8 KB per wave keep the barriers few; three stages or
// more where they fit (a chunk of more than a third of the LDS leaves two), the depth takes the rest.
constexpr XRing make_ring(int kc, int M, int n_c, int waves, int lds_b, int nch_multiple) {
    XRing q{};
    q.n_chunk = (n_c + kc - 1) / kc;
    q.n_inst = (M + 3) / 4;
    q.chunk_b = q.n_inst * 1024;
    const int room = lds_b / q.chunk_b;                            // chunks that fit
    int nch = room / 3;
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

// What the ring's loop takes for granted: a second stage for the transfers in flight, and a share of
// every full stage's k-steps for each of the `parts` waves that split them.
constexpr bool ring_ok(const XRing& q, int steps, int parts) { return q.nch >= 1 && q.depth >= 2 && q.nch * steps % parts == 0; }

// ---- FP16-split and int8: nwv waves per channel, nb row blocks of 16 ----
constexpr int ks_kc(bool int8) { return int8 ? 128 : 32; }         // channel samples per chunk
constexpr int ks_steps(bool int8) { return int8 ? 4 : 2; }         // k-steps per chunk (of 32 / 16 samples)
constexpr int ks_groups(bool int8, int nb, int nwv) {
    if (nb <= 3) return 1;
    if (nb <= 5) return nwv == 8 ? 2 : 1;
    if (nb <= 7) return 2;
    return nb == 8 && int8 ? 2 : 4;
}
constexpr int ks_lds(int nb, int nwv) { return nwv == 8 ? 163840 : nb <= 2 ? 40960 : nb == 3 ? 53248 : 81920; }

constexpr int ks_parts(bool int8, int nb, int nwv) { return nwv / ks_groups(int8, nb, nwv); }   // waves that split the k-steps

// bytes of the row of zeros behind the ring
constexpr int ks_zero_b(int nb, int M) { return (M + 3) / 4 * 4 < 16 * nb ? kRowB : 0; }

constexpr XRing ks_ring(bool int8, int nb, int nwv, int M, int n_c) {
    // a stage holds a multiple of the k-steps that the waves of a group share
    const int parts = ks_parts(int8, nb, nwv), mult = parts > ks_steps(int8) ? parts / ks_steps(int8) : 1;
    return make_ring(ks_kc(int8), M, n_c, nwv, ks_lds(nb, nwv) - ks_zero_b(nb, M), mult);
}

// ---- plain FP32 form ----
constexpr int kF32Waves = 8;
constexpr int kF32LdsB = 147456;
constexpr int kF32MaxTpw = 9;                 // 144 accumulator registers, two waves per SIMD
constexpr int kF32Steps = 4;                  // k-steps of 8 samples per chunk

struct XF32 {
    int n_tiles, nb, groups, n_tg, tpw;       // workgroups per channel, wave groups, tiles per wave
};

// Split with the least time per CU: rounds of workgroups x tile slots per channel share.  Every
// workgroup of a channel reads all of it, so there are several only where their tiles need them
// (more than 8 x 9 tiles) or CUs would idle otherwise (40 stations, 512 channels: three workgroups
// waste no slot and take 690 us, one takes 480); ties go to fewer groups of waves, whose waves
// hold more tiles per barrier (40 stations: 478 us with two groups, 517 with eight).
constexpr XF32 f32_split(int M, long n_chan, int cus) {
    XF32 f{};
    f.nb = (M + 15) / 16;
    f.n_tiles = tile_count(f.nb);
    long best = -1;
    const int least = (f.n_tiles + kF32Waves * kF32MaxTpw - 1) / (kF32Waves * kF32MaxTpw);
    for (int groups = least; groups <= 4 && (groups == least || n_chan * groups <= cus); ++groups)
        for (int n_tg = 1; n_tg <= kF32Waves; n_tg *= 2) {
            const int per = (f.n_tiles + groups * n_tg - 1) / (groups * n_tg);
            if (per > kF32MaxTpw) continue;
            const long cost = (n_chan * groups + cus - 1) / cus * per * n_tg;
            if (best < 0 || cost < best) {
                best = cost;
                f.tpw = per;
                f.groups = groups;
                f.n_tg = n_tg;
            }
        }
    return f;
}
constexpr XRing f32_ring(const XF32& f, int M, int n_c) {
    // reads of the last row block run past the last chunk by its missing rows
    return make_ring(32, M, n_c, kF32Waves, kF32LdsB - (16 * f.nb - (M + 3) / 4 * 4) * kRowB, kF32Waves / f.n_tg == 8 ? 2 : 1);
}

}  // namespace cobalt
