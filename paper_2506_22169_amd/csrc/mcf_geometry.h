// Tile geometry shared by the kernels and the host-side budget checks: tile byte sizes, the
// XOR swizzles of the LDS layouts and the LDS total.  Plain constexpr C++, no HIP.
#pragma once

namespace mcf {

// All LDS tiles keep their natural row pitch (row bytes RB, a multiple of 64) and are
// filled by direct global->LDS loads in units of 16-byte chunks; bank conflicts are avoided
// by XOR-ing the chunk index within a row with a function of the row.  The XOR stays within the
// largest power of two that divides RB (256 bytes, the LDS line, at most), so that rows need not be powers of two.
//
// Bytes within which the swizzles permute the chunks of a row: a lane's address of a later chunk of its row is an XOR
// within a span and a constant beyond it.
constexpr int swz_span(int row_bytes) { return row_bytes % 256 == 0 ? 256 : row_bytes & -row_bytes; }
// Tiles read with plain 128-bit reads (A tile; B tile when K is contiguous): 16 consecutive
// rows are read at the same logical chunk, so consecutive rows must land on distinct 16-byte
// bank groups of the 256-byte LDS line.  Rows of 192 and 320 bytes step through four 64-byte groups of the line by
// themselves, of 384 through two of 128.
constexpr int swz_b128(int row_bytes, int row) {
    switch (swz_span(row_bytes)) {
    case 64: return (row >> 2) & 3;
    case 128: return (row >> 1) & 7;
    default: return row & 15;
    }
}
// Tiles read with the transposing 64-bit read (D tile; B tile when N is contiguous): half a
// wave reads 4 consecutive rows x 64 bytes, so the four rows must land on distinct 64-byte
// groups.  Returned as a chunk mask (multiple of 4 chunks = 64 bytes).
constexpr int swz_tr(int row_bytes, int row) {
    switch (swz_span(row_bytes)) {
    case 64: return 0;
    case 128: return 4 * ((row >> 1) & 1);
    default: return 4 * (row & 3);
    }
}
// Address of 64-byte block `block` of a row from that of the row's block 0: an XOR within a span, an addition beyond it.
constexpr int tr_block_xor(int row_bytes, int block) { return 64 * (block % (swz_span(row_bytes) / 64)); }
constexpr int tr_block_add(int row_bytes, int block) { return block / (swz_span(row_bytes) / 64) * swz_span(row_bytes); }

// Pitch of the LDS rows in elements (K a multiple of 16, L of 8): rows of whole 64-byte groups lie as they are; others (80)
// take the next power of two, and the chunks beyond K or L in a row are loaded from valid memory and never reach a
// result that is stored.  (96, 160 and 192 took the next power of two before: a quarter to three eighths more LDS and loads, which
// left most of their kernels a ring of two and 160 and 192 no softmax pipeline of 8 waves.  us a call, before and after:
// softmax 20 x 2048 x 2048, K = L = 160: 120 and 63, 192: 150 and 134; causal 11 x 2852 x 3733, 160: 104 and 82; plain
// 14 x 1088 x 3840, 160: 58 and 51, 40 x 1024 x 1024, 192: 59 and 53.)
constexpr int pitch_elems(int x) { return x % 32 == 0 && x <= 256 ? x : x <= 32 ? 32 : x <= 64 ? 64 : x <= 128 ? 128 : x <= 256 ? 256 : 512; }
constexpr int pow2_pitch_elems(int x) { return x <= 32 ? 32 : x <= 64 ? 64 : x <= 128 ? 128 : x <= 256 ? 256 : 512; }
constexpr int h_blocks(int L) { return (L + 31) / 32; } // 32-wide column blocks of E (the last may be partial)

constexpr int a_tile_bytes(int K, int mb, int rg) { return 32 * mb * rg * pitch_elems(K) * 2; }
constexpr int b_tile_bytes(int K, int tn) { return pitch_elems(K) * tn * 2; }
constexpr int d_tile_bytes(int L, int tn) { return tn * pitch_elems(L) * 2; }
constexpr int stage_bytes(int K, int L, int tn) { return b_tile_bytes(K, tn) + d_tile_bytes(L, tn); }
// Cross-wave combine when ns > 1: the mb * ceil(L/32) accumulator blocks (32 x 32 of E, 16 fp32
// per lane) of a row-group are dealt out to its ns waves, BPW in a row; every wave parks the
// blocks it does not own and its softmax state in LDS.
constexpr int blocks_per_wave(int L, int mb, int ns) { return (mb * h_blocks(L) + ns - 1) / ns; }
// Most blocks any wave parks: all but the run it owns; the last wave's run is the shortest
// (empty when there are fewer blocks than waves).
constexpr int parked_blocks(int L, int mb, int ns) {
    const int n = mb * h_blocks(L), bpw = blocks_per_wave(L, mb, ns);
    const int last = n - (ns - 1) * bpw;
    return n - (last < 0 ? 0 : last);
}
// A wave's run of blocks must lie within one row set of 32 rows or cover whole row sets.
constexpr bool combine_runs_ok(int L, int mb, int ns) {
    const int hb = h_blocks(L), bpw = blocks_per_wave(L, mb, ns);
    return bpw >= hb ? bpw % hb == 0 : (mb == 1 || hb % bpw == 0);
}
constexpr int combine_bytes(int L, int mb, int rg, int ns) {
    return ns > 1 ? rg * ns * (parked_blocks(L, mb, ns) * 16 + 2 * mb) * 64 * 4 : 0;
}
// Staging tile of the E store, per wave: the rows of the row sets it owns (32 each) times the
// bytes of the h blocks it owns in a row, that pitch rounded up to a power of two; at least what an
// fp32 store stages at a time.
constexpr int estage_row_bytes(int L, int mb, int ns) {
    const int hb = h_blocks(L), bpw = blocks_per_wave(L, mb, ns);
    const int hpw = bpw < hb ? bpw : hb;
    return 2 * pow2_pitch_elems(32 * hpw);
}
constexpr int estage_wave_bytes(int L, int mb, int ns) {
    const int hb = h_blocks(L), bpw = blocks_per_wave(L, mb, ns);
    const int mpw = bpw < hb ? 1 : bpw / hb;
    const int b16 = mpw * 32 * estage_row_bytes(L, mb, ns);
    return b16 > 4096 ? b16 : 4096; // (one 32 x 32 block of fp32 at a time)
}
// Waves of a row-group that own a run of blocks (there may be fewer blocks than waves).
constexpr int owning_waves(int L, int mb, int ns) {
    return (mb * h_blocks(L) + blocks_per_wave(L, mb, ns) - 1) / blocks_per_wave(L, mb, ns);
}
constexpr int estage_bytes(int L, int mb, int rg, int ns) { return rg * owning_waves(L, mb, ns) * estage_wave_bytes(L, mb, ns); }
// Kernels with a k loop inside the block (T_K < K; `K` below is then the chunk T_K): the ring
// carries two kinds of items, an A chunk + B chunk (tm x T_K, T_K x tn) per k step and the D
// tile once per n-tile; a slot is as large as the larger of the two.
constexpr int ksplit_slot_bytes(int TK, int L, int mb, int rg, int tn) {
    const int ab = a_tile_bytes(TK, mb, rg) + b_tile_bytes(TK, tn), d = d_tile_bytes(L, tn);
    return ab > d ? ab : d;
}
// `stages` ring buffers of one B + D tile each; the A tile is staged in the last ring slot
// (it is consumed before that slot is first filled); after the loop the ring space is reused
// by the combine scratch followed by the staging tiles of the E store.
constexpr int total_lds_bytes(int K, int L, int mb, int rg, int ns, int nj, int stages, bool ksplit = false) {
    const int st = stage_bytes(K, L, 32 * ns * nj);
    const int a = a_tile_bytes(K, mb, rg);
    int s = ksplit ? stages * ksplit_slot_bytes(K, L, mb, rg, 32 * ns * nj) : (stages - 1) * st + (a > st ? a : st);
    const int c = combine_bytes(L, mb, rg, ns) + estage_bytes(L, mb, rg, ns);
    return s > c ? s : c;
}
// Largest ring depth (2..4) that keeps a block within `budget` bytes of LDS.
constexpr int pick_stages(int K, int L, int mb, int rg, int ns, int nj, int budget, bool ksplit = false) {
    int s = 4;
    while (s > 2 && total_lds_bytes(K, L, mb, rg, ns, nj, s, ksplit) > budget) --s;
    return s;
}

// Ring depth every kernel variant is built with: as deep (up to 4) as fits 80 KiB, so that two
// blocks can share the 160 KiB LDS of a compute unit (measured: a deeper ring that costs the
// second resident block loses more than it gains).
constexpr int kLdsRingBudget = 80 * 1024;
// Softmax chains (and the plain chains named below) run a software pipeline over three consecutive n-tiles: in iteration i a wave
// issues the MFMAs of GEMM 2 of tile i-1 and of GEMM 1 of tile i+1 with the softmax arithmetic of
// tile i spread between them.  It reads B two tiles ahead of D, so the two have rings of their own: D of tiles i-1 and i
// (landing), B of tiles i+1 and i+2 (landing) and, for a softmax that may have to form the scores of tile i again, of tile i.
// That is two to two and a half tiles where one ring of B + D tiles took four, at the same distance between a request and
// its use; what it leaves is a second block per compute unit, a wider n-tile, the F tile of a three-GEMM chain, rows
// of 160 and 192, or one more tile of each in flight (`ahead`).  The first tiles are requested before the loop, with the A tile
// behind them.
struct PipeRing {
    int ahead;   // tiles of B and of D in flight beyond those an iteration waits for
    int d_first; // D tiles requested before the loop
    int b_slots, d_slots;
    int d_rest, b_offset, a_offset; // offsets of D slots d_first .. (less that of slot d_first in a plain row of slots), the B ring, the A tile
    int bytes;
};
constexpr PipeRing pipe_ring_with(int K, int L, int mb, int rg, int ns, int nj, bool stands, int ahead, int d_first) {
    const int b = b_tile_bytes(K, 32 * ns * nj), d = d_tile_bytes(L, 32 * ns * nj);
    PipeRing r = {};
    r.ahead = ahead;
    r.d_first = d_first;
    r.b_slots = ahead + (stands ? 3 : 2);
    r.d_slots = ahead + 2;
    r.b_offset = d_first * d;
    r.d_rest = r.b_slots * b;
    r.a_offset = r.b_offset + (2 + ahead) * b;
    const int ring = r.b_slots * b + r.d_slots * d, first = r.a_offset + a_tile_bytes(K, mb, rg);
    const int c = combine_bytes(L, mb, rg, ns) + estage_bytes(L, mb, rg, ns);
    r.bytes = ring > first ? ring : first;
    r.bytes = r.bytes > c ? r.bytes : c;
    return r;
}
// Three-GEMM chain (E . F with F[L x P] after the loop): the F tile sits behind everything else
// (`below` bytes and the combined and staged output tile) for the whole life of the block.
constexpr int chain3_f_bytes(int L, int P) { return P > 0 ? L * pitch_elems(P) * 2 : 0; }
constexpr int chain3_f_offset(int below, int P, int mb, int rg, int ns) {
    const int e = combine_bytes(P, mb, rg, ns) + estage_bytes(P, mb, rg, ns);
    return ((below > e ? below : e) + 1023) / 1024 * 1024;
}
constexpr int with_f_tile(int below, int L, int P, int mb, int rg, int ns) {
    return P > 0 ? chain3_f_offset(below, P, mb, rg, ns) + chain3_f_bytes(L, P) : below;
}
// Waves per SIMD a pipelined softmax kernel is compiled for.  A block brings rg*ns/4 of them; a
// second resident block hides the block's barriers and the ends of its pipeline (measured: a
// third to a half faster on the short attention shapes), but the compiler only keeps to the
// registers that leaves a wave (512 / waves) when told so, otherwise it drifts a few registers
// over.  Asked for when two blocks fit the LDS and the registers hold what a lane must: the E
// accumulators, two C^T tiles, P packed to 16 bit, the A operands, and 40 for the LDS operands in flight, addresses and the
// softmax state, more with a second row set (16) or slice (20).  (Asked for with fewer, they spill: K = 128, L = 64, (1,8,1,1).)
// K and L of 32, whose operands are few, need 56 beside the E, C^T and P tiles, however many those are: with two blocks (1,4,1,4)
// takes 10.8 us for 96 x 512 x 512 and 32.6 for 32 x 2048 x 2048, with one 16.8 and 47.6; (2,2,2,2) 11.4 and 31.7, 17.4 and 45.6.
constexpr int pipe_needs(int K, int L, int mb, int nj) {
    if (K <= 32 && L <= 32) return mb * 16 + 2 * nj * mb * 16 + nj * mb * 8 + 56;
    return mb * h_blocks(L) * 16 + 2 * nj * mb * 16 + nj * mb * 8 + mb * (K / 16) * 4 + 4 + 16 * mb + 20 * nj;
}
constexpr int pipe_lds_least(int K, int L, int mb, int rg, int ns, int nj, int P, bool stands) {
    return with_f_tile(pipe_ring_with(K, L, mb, rg, ns, nj, stands, 0, 0).bytes, L, P, mb, rg, ns);
}
constexpr int pipe_waves_with(int K, int L, int mb, int rg, int ns, int nj, int P, bool stands) {
    const int per_block = rg * ns >= 4 ? rg * ns / 4 : 1;
    if (mb * rg == 1) return per_block; // m-tiles of 32 rows: calls of few blocks, for which loads in flight count more
    if (2 * pipe_lds_least(K, L, mb, rg, ns, nj, P, stands) > 160 * 1024) return per_block;
    return pipe_needs(K, L, mb, nj) <= 512 / (2 * per_block) ? 2 * per_block : per_block;
}
// Whether a pipelined softmax kernel leaves the reference of its exponentials where it stands between the
// first tile and the last (see the loop): with two waves on a SIMD or more, and 16 registers more,
// which the way back from an outgrown reference needs (without them the 8-wave kernels of K = L = 64 spill in the loop).
constexpr bool reference_stands(int K, int L, int mb, int rg, int ns, int nj, bool softmax, int P) {
    const int waves = pipe_waves_with(K, L, mb, rg, ns, nj, P, true);
    return softmax && waves >= 2 && pipe_needs(K, L, mb, nj) + 16 <= 512 / waves && pipe_lds_least(K, L, mb, rg, ns, nj, P, true) <= 2 * kLdsRingBudget;
}
constexpr int pipe_waves_per_simd(int K, int L, int mb, int rg, int ns, int nj, bool softmax, int P) {
    // (K = L = 32 in blocks of four waves: five blocks; 95 to 97 registers when not told, and 97 cost the fifth)
    if (K <= 32 && L <= 32 && mb == 1 && nj == 1 && rg > 1 && rg * ns == 4) return 5;
    // (plain chains, (1,4,2,2): two blocks of eight waves; 125 to 134 registers when not told, and more than 128 cost the second: 96 x
    // [512,32].[32,512].[512,32] 7.4 us with it, 9.1 without)
    if (!softmax && mb == 1 && nj == 2 && rg == 4 && ns == 2) return 4;
    return pipe_waves_with(K, L, mb, rg, ns, nj, P, reference_stands(K, L, mb, rg, ns, nj, softmax, P));
}
// The rings of a pipelined kernel, where they cost none of the blocks that the registers let a compute unit hold.  The first D tile
// is requested before the loop: a block of a few n-tiles otherwise waits for a load latency more than it has tiles (9 x 640 x
// 128, K = L = 64: 5.8 -> 6.6 us).  With one wave on a SIMD, whose blocks are few and wait for their loads, so is the second
// (17 x 163 x 167, K = L = 80: 7.6 -> 9.4 us without), and one more tile of B and D is in flight throughout (25 x 1 x 515, K = L =
// 128: 10.2 -> 8.7 us; with two waves 1 % slower, 96 x 512 x 512, K = L = 64: 12.8 -> 13.0).
constexpr PipeRing pipe_ring(int K, int L, int mb, int rg, int ns, int nj, bool softmax, int P) {
    const bool stands = reference_stands(K, L, mb, rg, ns, nj, softmax, P);
    const int waves = rg * ns, by_registers = 512 / pipe_needs(K, L, mb, nj) * 4 / waves;
    int blocks = 160 * 1024 / pipe_lds_least(K, L, mb, rg, ns, nj, P, stands);
    blocks = blocks < by_registers ? blocks : by_registers > 1 ? by_registers : 1;
    const bool one_wave = pipe_waves_per_simd(K, L, mb, rg, ns, nj, softmax, P) == 1;
    if (mb * rg == 1) blocks = 1;
    // (one more in flight is counted in loads of a wave, which must then be as many for every wave)
    const bool counted = stage_bytes(K, L, 32 * ns * nj) / 1024 % waves == 0;
    for (int q = one_wave ? (counted ? 0 : 1) : 2; q < 3; ++q) { // (ahead, d_first): (1, 2), (0, 2), (0, 1)
        const PipeRing r = pipe_ring_with(K, L, mb, rg, ns, nj, stands, q == 0 ? 1 : 0, q < 2 ? 2 : 1);
        if (blocks * with_f_tile(r.bytes, L, P, mb, rg, ns) <= 160 * 1024) return r;
    }
    return pipe_ring_with(K, L, mb, rg, ns, nj, stands, 0, 0);
}
// Whether an arrangement is pipelined (P: columns of F, 0 without a third GEMM): where it fits the LDS of a compute unit and its
// registers (blocks of four waves: the half of the file that vector instructions reach, and a little of the other; beyond that
// they spill, but for L of 64 and fewer, which stay within the file: 32 x 2048 x 2048, K = L = 64, (2,4,1,2) 53.6 us pipelined, 57.9 not,
// (2,2,2,2) 59.7 and 64.2; K = 128, L = 64, (2,4,1,2) 67 - 70 and 71.4).  The softmax loop of the others runs the phases one after the other, see skewed_groups.
constexpr bool pipelined(int K, int L, int mb, int rg, int ns, int nj, bool softmax, bool ksplit, int P) {
    if (ksplit) return false;
    // plain chains: only where K and L are 32, in blocks of 8 waves that own at most two row sets
    // each (measured on 16 x [4096,32].[32,1024].[1024,32]: 3-4 % faster for (1,8,1,2) and (2,4,2,2),
    // no change for (1,4,2,2), a third slower for (4,2,4,1); with K = L = 64 slower throughout)
    if (!softmax && !(K <= 32 && L <= 32 && mb <= 2 && rg * ns == 8)) return false;
    if (softmax && pipe_needs(K, L, mb, nj) > (rg * ns > 4 ? 256 : L <= 64 ? 364 : 320)) return false;
    return pipe_lds_least(K, L, mb, rg, ns, nj, P, reference_stands(K, L, mb, rg, ns, nj, softmax, P)) <= 2 * kLdsRingBudget;
}
// Softmax chains that cannot be pipelined, in blocks of 8 waves, run their two wave groups a
// phase apart, which keeps two n-tiles live: their ring is at least 3 deep.
constexpr bool skewed_groups(int rg, int ns, bool softmax, bool ksplit = false) { return softmax && rg * ns == 8 && !ksplit; }
// Depth of the ring of B + D tiles (k loop: of its items); a pipelined kernel holds two tiles whole.
constexpr int ring_stages(int K, int L, int mb, int rg, int ns, int nj, bool softmax, bool ksplit, int P) {
    // the items of a k loop are small and many, and the shapes that need one rarely fill the
    // machine: as deep as the whole LDS allows, to keep as many loads in flight as possible
    if (ksplit) return pick_stages(K, L, mb, rg, ns, nj, 2 * kLdsRingBudget, true);
    if (pipelined(K, L, mb, rg, ns, nj, softmax, ksplit, P)) return 2;
    const int s = pick_stages(K, L, mb, rg, ns, nj, kLdsRingBudget);
    return (skewed_groups(rg, ns, softmax) && s < 3) ? 3 : s;
}
// LDS bytes of a kernel without the F tile of a three-GEMM chain, offset of that tile, and all of them.
constexpr int ring_lds_bytes(int K, int L, int mb, int rg, int ns, int nj, bool softmax, bool ksplit, int P) {
    if (pipelined(K, L, mb, rg, ns, nj, softmax, ksplit, P)) return pipe_ring(K, L, mb, rg, ns, nj, softmax, P).bytes;
    return total_lds_bytes(K, L, mb, rg, ns, nj, ring_stages(K, L, mb, rg, ns, nj, softmax, ksplit, P), ksplit);
}
constexpr int f_lds_offset(int K, int L, int mb, int rg, int ns, int nj, bool softmax, int P) {
    return chain3_f_offset(ring_lds_bytes(K, L, mb, rg, ns, nj, softmax, false, P), P, mb, rg, ns);
}
constexpr int block_lds_bytes(int K, int L, int mb, int rg, int ns, int nj, bool softmax, bool ksplit, int P) {
    if (P > 0) return f_lds_offset(K, L, mb, rg, ns, nj, softmax, P) + chain3_f_bytes(L, P);
    return ring_lds_bytes(K, L, mb, rg, ns, nj, softmax, ksplit, P);
}

} // namespace mcf
