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
    int n_stage, n_full;     // stages of a channel, full ones (divided once, here: a division per stage
                             // costs a wave about as much as the stage's matrix products)
    int parts;               // waves that split the k-steps of a stage
    int lds_b;               // LDS bytes of a workgroup
};

// Stages issued before the first one is read; transfers of a wave that may be in flight while stage s
// is read (those of stages s + 1 .. s + depth - 2, counted where all of them are full); chunks that the
// slots hold in the end.
constexpr int ring_ahead(const XRing& q) { return q.depth - 1 < q.n_stage ? q.depth - 1 : q.n_stage; }
constexpr int ring_may_fly(const XRing& q, int s) { return s + q.depth - 2 < q.n_full ? q.ipw * (q.depth - 2) : 0; }
constexpr int ring_slots(const XRing& q) { return q.depth * q.nch < q.n_chunk ? q.depth * q.nch : q.n_chunk; }

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
    if (q.depth < 2) return q;                                     // refused by ring_ok
    q.n_stage = (q.n_chunk + nch - 1) / nch;
    q.n_full = q.n_chunk / nch;
    return q;
}

// What the ring's loop takes for granted: a second stage for the transfers in flight, and a share of
// every full stage's k-steps for each of the `parts` waves that split them.
constexpr bool ring_ok(const XRing& q, int steps) {
    return q.nch >= 1 && q.depth >= 2 && q.parts >= 1 && q.nch * steps % q.parts == 0;
}

// ---- FP16-split and int8: nwv waves per channel, nb row blocks of 16 ----
constexpr int ks_kc(bool int8) { return int8 ? 128 : 32; }         // channel samples per chunk
constexpr int ks_steps(bool int8) { return int8 ? 4 : 2; }         // k-steps per chunk (of 32 / 16 samples)
// Blocks of one chunk at up to 2 row blocks take one wave per channel (its few products are done before
// several waves could have added theirs up, and a CU holds up to 32 channels: 16384 channels, us with four
// waves and one: FP16-split 32 samples, 1 station 39 and 9, 12 stations 55 and 26; int8 128 samples, 1
// station 37 and 9, 12 stations 51 and 24; 16 stations FP16-split 47 and 35).  At most one channel per CU
// takes eight waves, the rest four.
constexpr int ks_waves(bool int8, int nb, int n_c, long n_chan, int cus) {
    return nb <= 2 && n_c <= ks_kc(int8) ? 1 : n_chan <= cus ? 8 : 4;
}
constexpr int ks_groups(bool int8, int nb, int nwv) {
    if (nb <= 3) return 1;
    if (nb <= 5) return nwv == 8 ? 2 : 1;
    if (nb <= 7) return 2;
    return nb == 8 && int8 ? 2 : 4;
}
constexpr int ks_parts(bool int8, int nb, int nwv) { return nwv / ks_groups(int8, nb, nwv); }   // waves that split the k-steps

// LDS at most; a workgroup takes what its ring and its sums need, so that short blocks leave room for
// more workgroups per CU (16384 channels of 32 samples with the whole of it, us: 28 stations int8 177,
// FP16-split 153; as needed 129 and 118; with the two 32 KB buffers of an earlier form 150 and 155).
// At 9 and 10 row blocks a third workgroup only scatters the stores (76 stations int8, 16384 channels
// of 128 samples: 473 us with two per CU, 508 with three).
// Int8 chunks at 3 and 4 row blocks pass fast: four workgroups per CU beat a deeper ring (16 subbands,
// 3072 samples: 20 stations 53 -> 48, 28 stations 74 -> 61).
constexpr int ks_lds(bool int8, int nb, int nwv) {
    return nwv == 8 ? 163840 : nb <= 2 || (int8 && nb <= 4) ? 40960 : nb == 3 ? 53248 : 81920;
}
// LDS of the sums over the k parts (each wave sends half of its group's tiles) and of the transposes
constexpr int ks_sums(bool int8, int nb, int nwv) {
    const int g = ks_groups(int8, nb, nwv), per = (tile_count(nb) + g - 1) / g;
    const int sums = nwv > g ? nwv * ((per + 1) / 2) * 2 * 64 * 16 : 0, tr = nwv * 2 * 16 * 17 * 4;
    return sums > tr ? sums : tr;
}

// bytes of the row of zeros behind the ring
constexpr int ks_zero_b(int nb, int M) { return (M + 3) / 4 * 4 < 16 * nb ? kRowB : 0; }

constexpr XRing ks_ring(bool int8, int nb, int nwv, int M, int n_c) {
    // a stage holds a multiple of the k-steps that the waves of a group share
    const int parts = ks_parts(int8, nb, nwv);
    int mult = parts > ks_steps(int8) ? parts / ks_steps(int8) : 1;
    // a single chunk of int8 at 2 row blocks is one k-step per wave and barrier (16 stations x 16
    // subbands 42.6 us, with two chunks per stage 38.4)
    if (int8 && nb == 2 && nwv == 4) mult = 2;
    XRing q = make_ring(ks_kc(int8), M, n_c, nwv, ks_lds(int8, nb, nwv) - ks_zero_b(nb, M), mult);
    q.parts = parts;
    const int ring = ring_slots(q) * q.chunk_b + ks_zero_b(nb, M), sums = ks_sums(int8, nb, nwv);
    q.lds_b = nb > 8 ? ks_lds(int8, nb, nwv) : ring > sums ? ring : sums;
    return q;
}

// ---- plain FP32 form ----
constexpr int kF32Waves = 8;
constexpr int kF32LdsB = 147456;              // at most
constexpr int kF32MaxTpw = 9;                 // 144 accumulator registers, two waves per SIMD
constexpr int kF32Steps = 4;                  // k-steps of 8 samples per chunk
constexpr int kF32Short = 64;                 // channel samples of a block whose k-steps are not split

struct XF32 {
    int n_tiles, nb, groups, n_tg, tpw;       // workgroups per channel, wave groups, tiles per wave
};

// Split with the least time per CU: rounds of workgroups x tile slots per channel share.  Every
// workgroup of a channel reads all of it, so there are several only where their tiles need them
// (more than 8 x 9 tiles) or CUs would idle otherwise (40 stations, 512 channels: three workgroups
// waste no slot and take 690 us, one takes 480); ties go to fewer groups of waves, whose waves
// hold more tiles per barrier (40 stations: 478 us with two groups, 517 with eight).  In blocks of one
// or two chunks the sums over k parts cost more than the products: the tiles go to all eight waves
// (16384 channels of 32 samples, us: 20 stations 300 -> 102, 40 stations 402 -> 217; 2048 of 64: 20
// stations 47 -> 23, 28 stations 42 -> 38, 8 stations unchanged; of 128, 28 stations 475 -> 540).
constexpr XF32 f32_split(int M, int n_c, long n_chan, int cus) {
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
    if (n_c <= kF32Short) {
        f.n_tg = kF32Waves;
        f.tpw = (f.n_tiles + f.groups * f.n_tg - 1) / (f.groups * f.n_tg);
    }
    return f;
}
constexpr XRing f32_ring(const XF32& f, int M, int n_c) {
    // reads of the last row block run past the last chunk by its missing rows
    const int past = (16 * f.nb - (M + 3) / 4 * 4) * kRowB, parts = kF32Waves / f.n_tg;
    XRing q = make_ring(32, M, n_c, kF32Waves, kF32LdsB - past, parts == 8 ? 2 : 1);
    q.parts = parts;
    // half of the k parts send their sums at a time; transposes of the diagonal tiles
    const int ring = ring_slots(q) * q.chunk_b + past, sums = parts / 2 * f.n_tg * f.tpw * 2 * 64 * 16, tr = f.n_tg * 16 * 17 * 4;
    q.lds_b = ring > sums ? ring : sums;
    if (q.lds_b < tr) q.lds_b = tr;
    return q;
}

}  // namespace cobalt
