// Block-factorised int8-MFMA form of the ground-state search (internal
// templates; instantiated per product depth in gemm_blk_kb*.hip).
//
// A block is 256 sequences that differ only in 8 "varying" monomers: the low
// 8 for plain ranges (256 consecutive sequences), the middle 8 for the
// reversal-canonical blocks (reversal then maps blocks onto blocks).
// Splitting each pair (i, j) by whether i and j vary, the quantity
// maximised, F = A sum_k C_k(c) h_i h_j (the negated energy of Eq. 1 up to a
// constant), becomes
//   F(s, c) = base(c) + sum_{v varying} h_v w_v(c) + sum_{varying pairs} A C_vv'(c) h_v h_v'
// with base(c) = A sum over contacts of two outer monomers of h_i h_j and
// w_v(c) = A sum over contacts of v with an outer monomer j of h_j: numbers
// that depend on the block and the conformation but not on the varying
// monomers.  Two products:
//
//   stage one  D1 = V x C1, per 32-conformation tile: V holds 32 block-
//              dependent "virtual rows" (weights -m2 A on outer-outer pairs
//              for base, -m2 A h_j on the pairs of v for w_v, unit rows
//              picking the varying pairs and the 2 window index rows) and C1
//              is the 0/1 contact matrix with the index rows.  D1[m][c] is,
//              for each conformation, the int8 byte of quantity m: -m2 base,
//              -m2 w_v, -m2 A C_vv', u & 127 and -(u >> 7).
//   stage two  key = A2 x S2: A2 = D1 packed to bytes (a lane of the stage-one
//              result holds one conformation and 16 of its virtual rows,
//              exactly the 16 bytes it supplies as the A operand of the next
//              product, so no data moves between lanes), S2 = per-sequence
//              indicators -128 (1, h_v, h_v h_v') and (1, -128) for the index
//              bytes, precomputed on the host per block geometry.  The
//              accumulator is the window key 128 m2 F + u.
//
// Per 32 x 32 (conformation x sequence) tile this issues one MFMA of depth
// 32 instead of K_pad/32 of them; stage one adds K_pad/32 MFMAs per
// conformation tile per 256 sequences.  Blocks of 256 reduce each product's 16
// keys to their largest and update the top-2 where it counts (stage_two); the
// wide blocks below, which run wherever they apply, scan for thresholds.
#pragma once

#include <algorithm>
#include <type_traits>

#include "gemm_body.h"

namespace hpmap {

namespace {

constexpr int kBlkTiles = (1 << kBlkBits) / 32;   // sequence tiles per block (8)

// The 8 varying monomers of a block sit at positions pos(x) (x = 0 .. 7,
// packed 8 bits each in j.blk_pos); j.blk_vmask has their bits.  Virtual
// rows: m = 0 base; 1 .. 8 w_v for v = pos(m - 1); then one row per pair of
// varying monomers with odd separation >= 3 (j.blk_npp pairs, x-indices a | b << 4
// packed a byte each in j.blk_pp[]); then j.blk_ngroups rows of unary terms
// (two-letter tables: B c_i h_i summed over a group of outer monomers); then
// the two index bytes; zero beyond.
// Plain ranges (CANON false) use the low 8 monomers, a geometry known at
// compile time: pos(x) = x and the pairs kLow8Pairs, the same list the host
// lays the second product's operand out by.
constexpr int kRowW = 1, kRowVV = 9;

template <bool CANON>
__device__ __forceinline__ int blk_pos(const EnumJob &j, int x)
{
    return CANON ? int((j.blk_pos >> (8 * x)) & 0xffu) : x;
}

template <bool CANON>
__device__ __forceinline__ int blk_pair(const EnumJob &j, int p)
{
    if (!CANON)
        return p < 8 ? int((kLow8Pairs >> (8 * p)) & 0xffu) : kLow8Pair8;
    const uint64_t w = p < 8 ? j.blk_pp[0] : (p < 16 ? j.blk_pp[1] : j.blk_pp[2]);
    return int((w >> (8 * (p & 7))) & 0xffu);
}

template <bool CANON>
__device__ __forceinline__ int blk_npp(const EnumJob &j) { return CANON ? j.blk_npp : kLow8NumPairs; }

template <bool CANON>
__device__ __forceinline__ uint64_t blk_vmask(const EnumJob &j) { return CANON ? j.blk_vmask : 0xffull; }

// Unary group of monomer i (15: none).  Selects, not an indexed read: a
// runtime index into the job's array would place the job in scratch memory.
__device__ __forceinline__ int blk_group(const EnumJob &j, int i)
{
    const uint64_t w = i < 16 ? j.blk_grp[0] : (i < 32 ? j.blk_grp[1] : j.blk_grp[2]);
    return int((w >> (4 * (i & 15))) & 15u);
}

// Stage-one A operand: this lane's virtual row m = lane & 31 over product
// rows k = 32 kb + 16 half + q of C1, for the block whose outer monomers are
// the bits of `outer`.
// UNARY: the job has unary-group rows (two-letter tables); compiled apart so
// that the pure-pair instances keep this fully unrolled loop small enough to
// stay in registers at every depth.
template <int KB, bool CANON, bool UNARY>
__device__ __forceinline__ void blk_v_fragments(const EnumJob &j, uint64_t outer, int m, int half,
                                                v4i (&vf)[KB])
{
    const int N = j.N;
    const int coef = j.blk_coef;
    const int coefB = UNARY ? j.blk_coefB : 0;
    const uint64_t vmask = blk_vmask<CANON>(j);
    const int row_un = kRowVV + blk_npp<CANON>(j);
    const int row_idx = row_un + (UNARY ? j.blk_ngroups : 0);
    // unary-group rows (two-letter tables): the outer H monomers of this
    // lane's group, as a bit mask over monomer positions
    uint64_t gmask = 0;
    if (UNARY && m >= row_un && m < row_idx)
        for (int i = 0; i < N; ++i)
            if (blk_group(j, i) == m - row_un && ((outer >> i) & 1u) && !((vmask >> i) & 1u))
                gmask |= uint64_t(1) << i;
    const int wv = m >= kRowW && m < kRowVV ? blk_pos<CANON>(j, m - kRowW) : -1;
    int va = -1, vb = -1;
    if (m >= kRowVV && m < row_un) {
        const int pr = blk_pair<CANON>(j, m - kRowVV);
        va = blk_pos<CANON>(j, pr & 15);
        vb = blk_pos<CANON>(j, pr >> 4);
    }
#pragma unroll
    for (int kb = 0; kb < KB; ++kb) {
        // product row k < K is the pair (i, i + d) of the k-th odd separation
        // d >= 3 in (d, i) order: find the first row's pair by skipping whole
        // runs of length N - d, then advance row by row
        const int kbase = kb * 32 + half * 16;
        int d = 3, i = kbase;
        while (d < N && i >= N - d) {
            i -= N - d;
            d += 2;
        }
        uint32_t w[4];
#pragma unroll
        for (int q4 = 0; q4 < 4; ++q4) {
            uint32_t word = 0;
#pragma unroll
            for (int bb = 0; bb < 4; ++bb) {
                const int k = kbase + q4 * 4 + bb;
                int v = 0;
                if (k == j.K) {
                    v = m == row_idx ? 1 : 0;
                } else if (k == j.K + 1) {
                    v = m == row_idx + 1 ? -1 : 0;
                } else if (d < N) {
                    const int jj = i + d;
                    const bool out_i = !((vmask >> i) & 1u), out_j = !((vmask >> jj) & 1u);
                    const bool h_i = (outer >> i) & 1u, h_j = (outer >> jj) & 1u;
                    if (m == 0) {
                        v = out_i && out_j && h_i && h_j ? -coef : 0;
                    } else if (m < kRowVV) {
                        v = (i == wv && out_j && h_j) || (jj == wv && out_i && h_i) ? -coef : 0;
                        v -= i == wv || jj == wv ? coefB : 0;   // B c_v: every contact of v
                    } else if (m < row_un) {
                        v = i == va && jj == vb ? -coef : 0;
                    } else if (UNARY && m < row_idx) {
                        v = -coefB * int(((gmask >> i) & 1u) + ((gmask >> jj) & 1u));
                    }
                }
                word |= (uint32_t(v) & 0xffu) << (8 * bb);
                ++i;   // next row: next i, or the next run
                if (d < N && i + d >= N) {
                    i = 0;
                    d += 2;
                }
            }
            w[q4] = word;
        }
        vf[kb] = v4i{int(w[0]), int(w[1]), int(w[2]), int(w[3])};
    }
}

// Sequence of block sequence x: the outer bits plus x's bits deposited at the
// varying positions.
__device__ __forceinline__ uint64_t blk_sequence(const EnumJob &j, uint64_t outer, int x)
{
    uint64_t s = outer;
#pragma unroll
    for (int b = 0; b < 8; ++b)
        s |= uint64_t((x >> b) & 1) << blk_pos<true>(j, b);
    return s;
}

// Canonical block index t -> outer bits.  With h = j.half_bits outer bits on
// each side (low: b, high: a) and, for odd N, the middle monomer m as an
// outer bit, reversal maps the block (a, m, b) onto (rev b, m, rev a); the
// canonical blocks are a <= b' = rev(b).  The index runs over m, then row
// pairs p < 2^(h-1) of the (a, b') triangle, each holding row b' = p
// (a = 0 .. p) and row b' = 2^h - 1 - p (a = 0 .. 2^h - 1 - p).  *diag is
// set when a == b', i.e. the block is its own reverse.
// (Block counts stay below 2^28 for N <= 36, so 32-bit arithmetic suffices.)
__device__ __forceinline__ uint64_t blk_canonical_outer(const EnumJob &j, uint64_t t64, bool *diag)
{
    const int h = j.half_bits;
    const int odd = j.N & 1;
    const uint32_t t = uint32_t(t64);
    const uint32_t side = 1u << h;
    const uint32_t span = side + 1;
    const uint32_t per_m = h ? (side >> 1) * span : 1;
    const uint32_t m = t / per_m;
    const uint32_t r = t - m * per_m;
    const uint32_t p = h ? r / span : 0;
    const uint32_t o = r - p * span;
    const bool first = o <= p;
    const uint32_t bp = first ? p : side - 1 - p;
    const uint32_t a = first ? o : o - p - 1;
    *diag = a == bp;
    const uint32_t b = h ? (__builtin_bitreverse32(bp) >> (32 - h)) : 0;
    return (uint64_t(a) << (h + 8 + odd)) | (uint64_t(m) << (h + 4)) | b;
}

// Low bytes of four int32 values (each in [-128, 127]) packed little-endian,
// three byte permutes: v_perm_b32(x, y, sel) picks result byte i as byte
// sel_i of the 8-byte value {x (bytes 4..7), y (bytes 0..3)}; 0x0c gives 0.
__device__ __forceinline__ int pack4(int a, int b, int c, int d)
{
    const uint32_t ab = __builtin_amdgcn_perm(uint32_t(b), uint32_t(a), 0x0c0c0400u);
    const uint32_t cd = __builtin_amdgcn_perm(uint32_t(d), uint32_t(c), 0x0c0c0400u);
    return int(__builtin_amdgcn_perm(cd, ab, 0x05040100u));
}

template <int KB>
__device__ __forceinline__ v16i stage_one(const v4i (&vf)[KB], const v4i *tile, int lane)
{
    v16i d1;
#pragma unroll
    for (int kb = 0; kb < KB; ++kb) {
        const v16i zero = {};
        d1 = __builtin_amdgcn_mfma_i32_32x32x32_i8(vf[kb], tile[kb * 64 + lane],
                                                   kb == 0 ? zero : d1, 0, 0, 0);
    }
    return d1;
}

__device__ __forceinline__ v4i pack_d1(const v16i &d1)
{
    return v4i{pack4(d1[0], d1[1], d1[2], d1[3]), pack4(d1[4], d1[5], d1[6], d1[7]),
               pack4(d1[8], d1[9], d1[10], d1[11]), pack4(d1[12], d1[13], d1[14], d1[15])};
}

// Largest of a lane's 16 keys of one product (a v_max3 chain).
__device__ __forceinline__ int max16(const v16i &a)
{
    int m = max(max(a[0], a[1]), a[2]);
#pragma unroll
    for (int r = 3; r < 15; r += 2)
        m = max(max(m, a[r]), a[r + 1]);
    return max(m, a[15]);
}

// Smallest window key S F + u whose F exceeds the F of the global key gs,
// i.e. (F(gs) + 1) S; 0 while gs is "no conformation", so that every real key
// is absorbed until a lane holds two.
__device__ __forceinline__ int absorb_threshold(int gs, int win_shift)
{
    return int((unsigned(gs) + kMaxConf) >> kKeyConfBits) << win_shift;
}

// Stage two of one conformation tile for the wave's 8 sequence tiles.
//
// The running state of a lane (one sequence, half of each tile's 32
// conformations) is the top-2 of global keys (gb, gs) and thr, the window
// key threshold of absorb_threshold(gs).  A product whose 16 keys in every
// lane all have F <= F(gs) is skipped: such a conformation can neither beat
// the lowest energy nor tie it unless the second already does, nor raise the
// second-lowest energy, so the lowest energy, its conformation when unique,
// the uniqueness decision and the gap come out exactly as if every key had
// been absorbed.  Which conformation the second key names may differ; it is
// never reported.  Absorbing is rare once a lane has seen a few windows, so
// the vector ALU spends 9 instructions per product on the test (max3 chain
// and compare) instead of 20 on the key update.  The product of sequence
// tile t+1 is issued before tile t's test (two accumulators), so the wave
// does not wait on each product's latency.
template <bool S2_LDS>
__device__ __forceinline__ void stage_two(const v4i &a2, const v4i (&sf)[S2_LDS ? 1 : kBlkTiles],
                                          const v4i *s2, int lane, int (&gb)[kBlkTiles],
                                          int (&gs)[kBlkTiles], int (&thr)[kBlkTiles],
                                          int conf_base, int win_shift)
{
    const v16i zero = {};
    v16i acc[2];
    acc[0] = __builtin_amdgcn_mfma_i32_32x32x32_i8(a2, S2_LDS ? s2[lane] : sf[0], zero, 0, 0, 0);
#pragma unroll
    for (int t = 0; t < kBlkTiles; ++t) {
        if (t + 1 < kBlkTiles)
            acc[(t + 1) & 1] = __builtin_amdgcn_mfma_i32_32x32x32_i8(
                a2, S2_LDS ? s2[(t + 1) * 64 + lane] : sf[S2_LDS ? 0 : t + 1], zero, 0, 0, 0);
        const v16i &a = acc[t & 1];
        if (__builtin_expect(__any(max16(a) >= thr[t]), 0)) {
            // top-2 of the 16 window keys (one window, so their order is the
            // global keys' order), then only those two become global keys
            int b = 0, sc = 0;
#pragma unroll
            for (int r = 0; r < 16; r += 2)
                top2_add2(b, sc, a[r], a[r + 1]);
            top2_merge(gb[t], gs[t], window_to_global(b, conf_base, win_shift),
                       window_to_global(sc, conf_base, win_shift));
            thr[t] = absorb_threshold(gs[t], win_shift);
        }
    }
}

// Staging of the C1 tiles:
//   kBlkLds  : double-buffered LDS, one barrier per tile; stage one of a tile
//              runs right before its stage two.
//   kBlkPipe : triple-buffered LDS; the stage-one products of tile t+1 are
//              issued during iteration t, so the matrix pipe works on them
//              while the vector ALU runs tile t's key updates.
//   kBlkLdsS2: as kBlkLds, with the per-sequence operand of stage two held in
//              LDS (shared by the workgroup) instead of registers.
enum { kBlkLds = kBlkStageLds, kBlkPipe = kBlkStagePipe, kBlkLdsS2 = kBlkStageS2Lds };

// One wave scores one block of 256 sequences against every conformation
// tile; the NW waves of a workgroup take consecutive blocks and share the
// C1 tiles through LDS.
// The work of one workgroup: wave w scores block blk0 + w (plain jobs: the
// 256 sequences sharing the bits above the low 8, block index = sequence >> 8;
// canonical jobs: canonical block index).  lds holds the staged C1 tiles,
// s2lds the stage-two operand (mode kBlkLdsS2).  Starts and ends at a
// workgroup barrier, so consecutive calls may reuse the LDS.
template <int KB, int NW, int MODE, bool CANON, bool UNARY>
__device__ __forceinline__ void blk_body(const EnumJob &j, uint64_t blk0, v4i *lds, v4i *s2lds)
{
    const int lane = threadIdx.x & 63;
    const int wave = threadIdx.x >> 6;
    const int col = lane & 31;
    const int half = lane >> 5;
    const uint64_t blk = blk0 + wave;
    bool diag = false;
    const uint64_t outer = CANON ? blk_canonical_outer(j, blk, &diag) : blk << kBlkBits;
    const v4i *__restrict__ B1 = reinterpret_cast<const v4i *>(j.gemm_b);

    v4i vf[KB];
    blk_v_fragments<KB, CANON, UNARY>(j, outer, col, half, vf);
    // stage-two B operand: per-sequence indicators, precomputed per geometry
    v4i sf[MODE == kBlkLdsS2 ? 1 : kBlkTiles];
    const v4i *__restrict__ S2 = reinterpret_cast<const v4i *>(j.blk_s2);
    if constexpr (MODE == kBlkLdsS2) {
        for (int i = threadIdx.x; i < kBlkTiles * 64; i += NW * 64)
            s2lds[i] = S2[i];   // made visible by the barrier before the tile loop
    } else {
#pragma unroll
        for (int t = 0; t < kBlkTiles; ++t)
            sf[t] = S2[t * 64 + lane];
    }

    int gb[kBlkTiles], gs[kBlkTiles], thr[kBlkTiles];
#pragma unroll
    for (int t = 0; t < kBlkTiles; ++t)
        gb[t] = gs[t] = thr[t] = 0;

    const int n_tiles = j.n_tiles;
    const int win_tiles = j.blk_win_tiles;
    const int win_shift = j.blk_shift;
    int wend = min(win_tiles, n_tiles);
    int conf_base = 0;

    TileStage<KB, NW> stg;
    constexpr int TV = KB * 64;   // vectors per staged tile
    if constexpr (MODE == kBlkLds || MODE == kBlkLdsS2) {
        stg.load(B1, 0);
        stg.store(lds);
        __syncthreads();
        for (int tile = 0; tile < n_tiles; ++tile) {
            const bool more = tile + 1 < n_tiles;
            if (more)
                stg.load(B1, tile + 1);
            const v16i d1 = stage_one<KB>(vf, lds + (tile & 1) * TV, lane);
            stage_two<MODE == kBlkLdsS2>(pack_d1(d1), sf, s2lds, lane, gb, gs, thr, conf_base,
                                         win_shift);
            if (tile + 1 == wend) {
                conf_base += win_tiles * kTileConf;
                wend = min(wend + win_tiles, n_tiles);
            }
            if (more)
                stg.store(lds + ((tile + 1) & 1) * TV);
            __syncthreads();
        }
    } else {
        // Buffer t % 3 holds tile t.  Iteration t: prefetch tile t+2 from
        // global memory, pack tile t's stage-one result, issue stage one of
        // tile t+1 (buffer (t+1) % 3) and stage two of tile t, store tile t+2
        // into buffer (t+2) % 3 = (t-1) % 3 -- last read by stage one of tile
        // t-1 in iteration t-2, two barriers back -- then one barrier.
        stg.load(B1, 0);
        stg.store(lds);
        if (n_tiles > 1) {
            stg.load(B1, 1);
            stg.store(lds + TV);
        }
        __syncthreads();
        v16i d1 = stage_one<KB>(vf, lds, lane);
        int cur = 0;   // buffer of tile `tile`
        for (int tile = 0; tile < n_tiles; ++tile) {
            const bool has1 = tile + 1 < n_tiles;
            const bool has2 = tile + 2 < n_tiles;
            if (has2)
                stg.load(B1, tile + 2);
            const v4i a2 = pack_d1(d1);
            const int nxt = cur == 2 ? 0 : cur + 1;
            const int nn = nxt == 2 ? 0 : nxt + 1;
            if (has1)
                d1 = stage_one<KB>(vf, lds + nxt * TV, lane);
            stage_two<false>(a2, sf, s2lds, lane, gb, gs, thr, conf_base, win_shift);
            if (tile + 1 == wend) {
                conf_base += win_tiles * kTileConf;
                wend = min(wend + win_tiles, n_tiles);
            }
            if (has2)
                stg.store(lds + nn * TV);
            __syncthreads();
            cur = nxt;
        }
    }

    unsigned del = 0;
#pragma unroll
    for (int t = 0; t < kBlkTiles; ++t) {
        const int ob = __shfl_xor(gb[t], 32);
        const int os = __shfl_xor(gs[t], 32);
        top2_merge(gb[t], gs[t], ob, os);
        if constexpr (CANON) {
            // off the diagonal the block's reverse is never scored: write both;
            // a diagonal block holds each sequence and its reverse itself
            const uint64_t sq = blk_sequence(j, outer, t * 32 + col);
            const uint64_t rs = diag ? sq : __builtin_bitreverse64(sq) >> (64 - j.N);
            del += finish_sequence(j, j.scan_c2q, sq, sq, rs, half == 0 && blk < j.hi, gb[t], gs[t], 1);
        } else {
            const uint64_t idx = outer + uint64_t(t * 32 + col);
            del += finish_sequence(j, j.scan_c2q, idx, idx, idx,
                                   half == 0 && idx >= j.lo && idx < j.hi, gb[t], gs[t], 1);
        }
    }
    count_deleterious(j, del, lane == 0);
}

template <int KB, int NW, int MODE, bool CANON, bool UNARY>
__global__ __launch_bounds__(NW * 64) void k_gemm_blk(EnumJob j)
{
    __shared__ v4i lds[(MODE == kBlkPipe ? 3 : 2) * KB * 64];
    __shared__ v4i s2lds[MODE == kBlkLdsS2 ? kBlkTiles * 64 : 1];
    const uint64_t blk0 = (CANON ? j.lo : j.lo >> kBlkBits) + uint64_t(blockIdx.x) * NW;
    blk_body<KB, NW, MODE, CANON, UNARY>(j, blk0, lds, s2lds);
}

// Batched form for jobs of one product depth: workgroup b scores item
// item_lo + b, NW consecutive blocks of the job whose item range holds it.
template <int KB, int NW, int MODE, bool UNARY>
__global__ __launch_bounds__(NW * 64) void k_gemm_blk_batch(BatchHeader *hdr, int item_lo)
{
    __shared__ v4i lds[2 * KB * 64];
    __shared__ v4i s2lds[MODE == kBlkLdsS2 ? kBlkTiles * 64 : 1];
    const EnumJob *jobs = reinterpret_cast<const EnumJob *>(hdr + 1);
    const int njobs = hdr->njobs;
    const int64_t *start = reinterpret_cast<const int64_t *>(jobs + njobs);
    {
        // uniform indices let the job be read with scalar loads instead of
        // occupying vector registers
        const int it = item_lo + int(blockIdx.x);
        int lo = 0, hi = njobs - 1;   // job with start[job] <= it < start[job+1]
        while (lo < hi) {
            const int mid = (lo + hi + 1) / 2;
            if (start[mid] <= it)
                lo = mid;
            else
                hi = mid - 1;
        }
        lo = __builtin_amdgcn_readfirstlane(lo);
        const EnumJob &j = jobs[lo];
        const uint64_t blk0 = (j.lo >> kBlkBits) + uint64_t(it - start[lo]) * NW;
        blk_body<KB, NW, MODE, false, UNARY>(j, blk0, lds, s2lds);
    }
}

// ---------------------------------------------------------------------------
// Wide blocks (pure pair energies): one block of sequences sharing every
// outer monomer per workgroup.  The block term, the weights w_v of the varying
// monomers and their 16 pair terms are at most 29 virtual rows, so ONE first
// product per 32-conformation tile serves every wave of the workgroup: each
// wave computes it for every NW-th tile (one group of NW tiles ahead) and
// hands the packed result to the others through LDS.  Four geometries (G):
//   0  plain ranges, 1024 sequences (the low 10 monomers), 2 waves;
//   1  reversal-canonical blocks, 1024 sequences (the 10 around the middle),
//      2 waves;
//   2  whole chunks of 2^17 of a plain range, 2048 sequences (monomers 0 .. 4
//      and the even ones 6 .. 16: equal parity never touches, so 11 varying
//      monomers have only 14 pairs), 4 waves;
//   3  whole chunks of 2^19, 4096 sequences (monomers 0 .. 4 and the even ones
//      6 .. 18: 16 pairs), 8 waves.
//
// The second product is a threshold scan.  Counts of H-H contacts are at most 31
// (kScanMaxContacts), so 6 bits hold 32 + n - T, T being the smallest count that
// can still change a sequence's two best (one more than its second best), and
// the top one of them says whether n reaches T.  One float accumulator holds
// four such fields: two sequences, x = 64 t + col and x + 32, times two
// conformation tiles.  The product has depth 64; its two halves carry the same 32
// virtual rows of a conformation (FP6: weights to 15, the block term as a digit
// of 8s and one of 1s, rows 29 and 0) against the indicators of x and of x + 32
// (FP4), with block scales 2^6 apart, and V = 32 - T of each as 9 a + b, two FP4
// digits beside the constants 9 and 1 (rows 30 and 31).  The second tile's
// product adds at scales 2^12 higher.  Starting from 4.0 with units of 2^-21,
// the accumulator's bits hold the fields from bit 0 on: bits 5, 11 and 17 are the
// guards of three, and the fourth's carries into the exponent (bit 24; it then
// displaces the others, so both tiles are looked at).  All of it is exact below
// the carry.  A lane ORs its 16 accumulators: 8 v_or3 per two products, for 64
// conformations x 64 sequences, and only a tile in which some bit is set is
// absorbed.  A
// conformation below T can change neither the lowest energy, nor its
// conformation when unique, nor whether it is unique, nor the gap to the
// second-lowest energy, so every output is that of updating every key (which
// conformation the second key names may differ; it is never reported).
// Simulated on sampled 3x3x3 blocks, 8 % of a wave's tiles hold a hit.  In int8
// (two fields, 8 v_or3 per product) the vector instructions took longer than the
// products: alone, 2 tiles x 64 sequences 98 SIMD cycles against 88; a step of
// the 3x3x3 map 43.3 ms against 38.6.
//
// The first product runs in FP4 (0/1 weights times 0/1 contacts,
// depth 64 per MFMA in the time an int8 product of depth 32 takes, exact in
// the float accumulator), which halves its matrix time and the bytes of the
// contact matrix that every workgroup reads.
//
// Two-letter tables (G 4: plain ranges, 1024 sequences, 4 waves) have one
// sequence per accumulator: F = A n + B sum_i c_i h_i reaches hundreds.  The weights
// A h + B and the block term's A h h' + B (h + h') are bytes, so the first
// product is the int8 one; the block term takes two digits of 64, in rows 0
// and 29, and so does T - 1 in the operand's constants.  With indicator bytes
// -h the accumulator is T - 1 - F, whose sign bit says that F reaches T; the
// OR of 16 accumulators takes the same 8 instructions.  A step of the 3x3x3
// map: 21.0 ms (29.9 ms in blocks of 256 whose waves each form the first
// product and test the largest of 16 keys).
// ---------------------------------------------------------------------------

// Guard bits of an accumulator, as the bits of a float in [4, 8): bits 5, 11 and
// 17 are those of the three lower fields; the fourth's carries into the
// exponent and sets bit 24.
constexpr int kScanHit = (1 << 5) | (1 << 11) | (1 << 17) | (1 << 24);
// scales of the four fields (E8M0; a unit product is 2^-4, a field's unit 2^-21
// 2^6 f), the two of one conformation tile in the lane halves
constexpr int kScanScale = 110, kScanField = 6;

template <int G>
constexpr int wide_bits() { return G == 3 ? kWide12Bits : G == 2 ? kWide11Bits : kWideBits; }
template <int G>
constexpr bool wide_table() { return G == 4; }
template <int G>
constexpr int wide_waves() { return G == 4 ? 4 : 1 << (wide_bits<G>() - kWideWaveBits); }
// sequences of a wave's tile
template <int G>
constexpr int wide_cols() { return G == 4 ? 32 : 64; }
// virtual rows: 0 and 29 block term, 1 .. nb weights, then 16 pairs; 30 and 31
// constants
template <int G>
constexpr int wide_row_vv() { return 1 + wide_bits<G>(); }
// first-product steps for pair depth KB * 32: of depth 64, or 32 with tables
template <int KB, int G>
constexpr int wide_steps() { return wide_table<G>() ? KB : (KB + 1) / 2; }
// waves of the second-product table before those of geometry G
template <int G>
constexpr int wide_s2_slot() { return G == 0 ? 0 : G == 1 ? 2 : G == 2 ? 4 : 8; }

// Varying monomer x of a wide block: G 0 the low 10; G 1 the 10 around the
// middle, h = j.half_bits outer monomers on each side (and, for odd N, the
// middle monomer h + 5 outer as well); G 2, 3 monomers 0 .. 4, 6, 8, ...
template <int G>
__device__ __forceinline__ int wide_pos(const EnumJob &j, int x)
{
    if constexpr (G == 1)
        return j.half_bits + x + (x >= 5 ? (j.N & 1) : 0);
    else if constexpr (G >= 2)
        return x < 5 ? x : 2 * x - 4;
    else
        return x;
}

// Pair p (0 .. 15) of the block's varying monomers as x-indices a | b << 4.
template <int G>
__device__ __forceinline__ int wide_pair(const EnumJob &j, int p)
{
    const uint64_t w = G == 3                     ? (p < 8 ? kW12Pairs0 : kW12Pairs1)
                       : G == 2                   ? (p < 8 ? kW11Pairs0 : kW11Pairs1)
                       : (G == 1 && (j.N & 1)) ? (p < 8 ? kMid10OddPairs0 : kMid10OddPairs1)
                                                 : (p < 8 ? kLow10Pairs0 : kLow10Pairs1);
    return int((w >> (8 * (p & 7))) & 0xffu);
}

// First-product A operand of a wide block, step `st` of this lane: virtual
// row m over product rows k = 64 st + 32 half + n, n < 32.  Every row is a
// symmetric function of two monomer sets, bit (i, j) = X_i Y_j or Y_i X_j: the
// block term has X = Y = the outer H monomers, a weight X = its monomer and Y
// = the outer H monomers, a varying pair one monomer each.
template <int G>
__device__ __forceinline__ v4i wide_v_fragment(const EnumJob &j, uint64_t outer, int m, int half,
                                               int st)
{
    constexpr int kRowVV = wide_row_vv<G>();
    uint64_t X = 0, Y = 0;
    if (m == 0 || m == 29) {
        X = Y = outer;
    } else if (m < kRowVV) {
        X = uint64_t(1) << wide_pos<G>(j, m - 1);
        Y = outer;
    } else if (m < kRowVV + 16) {
        const int pr = wide_pair<G>(j, m - kRowVV);
        X = uint64_t(1) << wide_pos<G>(j, pr & 15);
        Y = uint64_t(1) << wide_pos<G>(j, pr >> 4);
    }
    const uint32_t bits = pair_bits(X, Y, j.N, 64 * st + 32 * half);
    // twice the spread: weights 2.0 (the contact matrix holds 0.5)
    return v4i{int(fp4_spread(bits & 0xffu) << 2), int(fp4_spread((bits >> 8) & 0xffu) << 2),
               int(fp4_spread((bits >> 16) & 0xffu) << 2), int(fp4_spread(bits >> 24) << 2)};
}

// The same for two-letter tables: step `st` covers rows k = 32 st + 16 half + n, n <
// 16, as int8 A X_i Y_j (or Y_i X_j) + B (X_i + X_j); the pair rows have no B.
__device__ __forceinline__ v4i wide_un_fragment(const EnumJob &j, uint64_t outer, int m, int half,
                                                int st)
{
    constexpr int kRowVV = wide_row_vv<4>();
    const uint64_t all = (uint64_t(1) << j.N) - 1;
    uint64_t X = 0, Y = 0, U = 0;
    if (m == 0 || m == 29) {
        X = Y = U = outer;
    } else if (m < kRowVV) {
        X = U = uint64_t(1) << (m - 1);
        Y = outer;
    } else if (m < kRowVV + 16) {
        const int pr = wide_pair<4>(j, m - kRowVV);
        X = uint64_t(1) << (pr & 15);
        Y = uint64_t(1) << (pr >> 4);
    }
    const uint32_t ab = pair_bits(X, Y, j.N, 32 * st) >> (16 * half);
    const uint32_t one = pair_bits(U, all, j.N, 32 * st) >> (16 * half);
    const uint32_t two = pair_bits(U, U, j.N, 32 * st) >> (16 * half);
    v4i w;
#pragma unroll
    for (int q4 = 0; q4 < 4; ++q4) {
        uint32_t word = 0;
#pragma unroll
        for (int b = 0; b < 4; ++b) {
            const int n = 4 * q4 + b;
            const uint32_t v = uint32_t(j.A) * ((ab >> n) & 1u) +
                               uint32_t(j.B) * (((one >> n) & 1u) + ((two >> n) & 1u));
            word |= v << (8 * b);
        }
        w[q4] = int(word);
    }
    return w;
}

// Second operand of a table's sequences x = 32 tile + (lane & 31): byte q of this
// lane is minus the indicator of x for row 8 (q / 4) + 4 half + q % 4, -64 for
// the block term's upper digit; the constants hold T - 1 = -1 (no threshold yet).
__device__ __forceinline__ v4i wide_un_operand(const EnumJob &j, int x, int half)
{
    constexpr int kRowVV = wide_row_vv<4>();
    v4i w;
#pragma unroll
    for (int q4 = 0; q4 < 4; ++q4) {
        uint32_t word = 0;
#pragma unroll
        for (int b = 0; b < 4; ++b) {
            const int m = 8 * q4 + 4 * half + b;
            const int pr = wide_pair<4>(j, (m - kRowVV) & 15);
            const bool pair = m >= kRowVV && m < kRowVV + 16;
            const int first = pair ? pr & 15 : m - 1, second = pair ? pr >> 4 : m - 1;
            int v = -((x >> (first & 15)) & (x >> (second & 15)) & 1);
            v = m == 0 ? -1 : m == 29 ? -64 : m == 30 ? 63 : m == 31 ? -1 : v;
            v = m == 27 || m == 28 ? 0 : v;
            word |= uint32_t(v & 0xff) << (8 * b);
        }
        w[q4] = int(word);
    }
    return w;
}

// Canonical wide block index t -> outer bits, as blk_canonical_outer with 10
// varying monomers: (a, m, b) = high h, middle (odd N), low h bits; the
// canonical blocks are a <= b' = reverse_h(b), indexed over m, then row pairs
// p < 2^(h-1) holding row b' = p (a = 0 .. p) and row b' = 2^h - 1 - p
// (a = 0 .. 2^h - 1 - p).  *diag: a == b', the block is its own reverse.
__device__ __forceinline__ uint64_t wide_canonical_outer(const EnumJob &j, uint64_t t64, bool *diag)
{
    const int h = j.half_bits;
    const int odd = j.N & 1;
    const uint32_t t = uint32_t(t64);
    const uint32_t side = 1u << h;
    const uint32_t span = side + 1;
    const uint32_t per_m = h ? (side >> 1) * span : 1;
    const uint32_t m = t / per_m;
    const uint32_t r = t - m * per_m;
    const uint32_t p = h ? r / span : 0;
    const uint32_t o = r - p * span;
    const bool first = o <= p;
    const uint32_t bp = first ? p : side - 1 - p;
    const uint32_t a = first ? o : o - p - 1;
    *diag = a == bp;
    const uint32_t b = h ? (__builtin_bitreverse32(bp) >> (32 - h)) : 0;
    return (uint64_t(a) << (h + kWideBits + odd)) | (uint64_t(m) << (h + 5)) | b;
}

// Block index of a chunked geometry (G 2: 2^17 sequences in 64 blocks, G 3:
// 2^19 in 128) -> outer bits: the chunk, and within it the low bits of t on
// the outer monomers 5, 7, ...
template <int G>
__device__ __forceinline__ uint64_t wide_chunk_outer(uint64_t t)
{
    constexpr int kOuter = G == 3 ? 7 : 6;
    uint64_t o = (t >> kOuter) << (2 * kOuter + 5);
#pragma unroll
    for (int k = 0; k < kOuter; ++k)
        o |= ((t >> k) & 1u) << (5 + 2 * k);
    return o;
}

// V = 32 - T of a sequence whose second-best scan key is gs: T is one more
// than that key's count, 0 while it is "no conformation".
__device__ __forceinline__ int scan_bias(unsigned gs)
{
    return 32 - int((gs + kMaxConf) >> kKeyConfBits);
}

// V = 9 a + b, a = 0 .. 4, b = -4 .. 4, as the lane's two FP4 digits (codes of
// half units) beside the rows 9 and 1.
__device__ __forceinline__ void scan_set_v(v4i &sf, int v)
{
    const int a = (v + 4) / 9, b = v - 9 * a;
    sf[3] = int((unsigned(sf[3]) & 0x0f0fffffu) | unsigned(a << 20) |
                (unsigned(b < 0 ? 8 - b : b) << 28));
}

__device__ __forceinline__ int scan_get_v(unsigned word)
{
    const int b = int(word >> 28);
    return 9 * int((word >> 20) & 15u) + (b & 8 ? 8 - b : b);
}

// The two V bytes of a table tile's sequence in the last word of the second
// operand of its half-1 lane.
__device__ __forceinline__ void scan_set_bias(v4i &sf, int lower, int upper, int half)
{
    sf[3] = half ? (sf[3] & 0xffff) | (lower << 16) | (upper << 24) : sf[3];
}

__device__ __forceinline__ v16f scan_product(const v6i &a2, const v4i &sf, const v16f &c, int scale)
{
    const v8i a = {a2[0], a2[1], a2[2], a2[3], a2[4], a2[5], 0, 0};
    const v8i b = {sf[0], sf[1], sf[2], sf[3], 0, 0, 0, 0};
    return __builtin_amdgcn_mfma_scale_f32_32x32x64_f8f6f4(a, b, c, 2, 4, 0, scale, 0, 127);
}

__device__ __forceinline__ v16f scan_four()
{
    v16f c;
#pragma unroll
    for (int r = 0; r < 16; ++r)
        c[r] = 4.0f;
    return c;
}

// Absorbs the 32 conformations of tile `tile` into the two best of a tile's
// sequences, top[col] and top[col + 32]: the scan's product of this tile alone
// and, for each field that has a hit, the two best of the lane's 16 rows as
// keys, pushed with LDS atomics (both lane halves, and in split blocks other
// waves, score the same sequences).  The V that the product was formed with
// are the operands' own digits.  A candidate below T is pushed for nothing, one
// of an empty column is none.
__device__ __forceinline__ void scan_absorb(const v6i &a2, v4i &sf, ScanTop2 *top, int tile, int lane)
{
    const int half = lane >> 5, col = lane & 31;
    const v16i a = __builtin_bit_cast(
        v16i, scan_product(a2, sf, scan_four(), kScanScale + kScanField * half));
    const int hit = or16(a);
    if (!__any((hit & (32 | 2048)) != 0))
        return;
    const auto w = __builtin_amdgcn_permlane32_swap(sf[3], sf[3], false, false);
    const int at = tile + 1 + (half << 14);
    auto push = [&](unsigned b, unsigned s, int bias, ScanTop2 *g) {
        const int base = at - (bias << kKeyConfBits);
        auto key = [&](unsigned k) {
            return unsigned(max(0, int(((k >> 26) << kKeyConfBits) + ((k & 31) << 12)) + base));
        };
        scan_push(g, key(b), key(s));
    };
    unsigned b, s;
    if (__any((hit & 32) != 0)) {
        scan_best<26>(a, b, s);
        push(b, s, scan_get_v(w[0]), top + col);
    }
    if (__any((hit & 2048) != 0)) {
        scan_best<20>(a, b, s);
        push(b, s, scan_get_v(w[1]), top + col + 32);
    }
    scan_set_v(sf, scan_bias(top[lane].s));
}

// The same for two-letter tables: T - 1 of a sequence whose second-best key is
// gs, its digits as the operand's bytes, and the absorption of a tile into
// top[col].  Only the accumulators below 0 are candidates, as (T - 1) + e with
// e = -accumulator.
__device__ __forceinline__ int scan_un_threshold(unsigned gs)
{
    return int((gs + kMaxConf) >> kKeyConfBits) - 1;
}

__device__ __forceinline__ void scan_un_set(v4i &sf, unsigned gs, int half)
{
    const int t = scan_un_threshold(gs);
    scan_set_bias(sf, t & 63, (t >> 6) & 0xff, half);
}

__device__ __forceinline__ void scan_un_absorb(const v4i &a2, v4i &sf, ScanTop2 *top, int tile,
                                               int lane)
{
    const int half = lane >> 5, col = lane & 31;
    const v16i zero = {};
    const v16i a = __builtin_amdgcn_mfma_i32_32x32x32_i8(a2, sf, zero, 0, 0, 0);
    const auto w = __builtin_amdgcn_permlane32_swap(sf[3], sf[3], false, false);
    const int word = int(w[1]);   // of the half-1 lane: the T - 1 this product had
    const int t = 64 * (word >> 24) + ((word >> 16) & 63);
    int b = 0, s = 0;   // the two smallest below 0, as 32 accumulator + row
#pragma unroll
    for (int q = 0; q < 16; q += 4) {
        int m[2];
#pragma unroll
        for (int p = 0; p < 2; ++p) {
            const int k0 = int(unsigned(a[q + 2 * p]) << 5 | unsigned(2 * q + 2 * p));
            const int k1 = int(unsigned(a[q + 2 * p + 1]) << 5 | unsigned(2 * q + 2 * p + 1));
            m[p] = med3_i32(b, k0, k1);
            b = min(min(b, k0), k1);
        }
        s = min(min(s, m[0]), m[1]);
    }
    auto key = [&](int k) {
        const unsigned at = unsigned((t - (k >> 5)) << kKeyConfBits) + unsigned((k & 31) << 12);
        return k < 0 ? at + unsigned(tile + 1 + (half << 14)) : 0u;
    };
    scan_push(top + col, key(b), key(s));
    scan_un_set(sf, top[col].s, half);
}

// Second product of two conformation tiles: the threshold scan of the wave's 512
// sequences.  One accumulator beside the constant (the compiler keeps the 4.0 of
// the first product's input in registers, which leaves no room for more at
// four waves per SIMD): the other waves fill the matrix pipe meanwhile.
__device__ __forceinline__ void scan_pair(const v6i (&a2)[2], v4i (&sf)[kBlkTiles], ScanTop2 *top,
                                          int tile, int lane)
{
    const int scale = kScanScale + (lane >> 5) * kScanField;
    const v16f four = scan_four();
    v16f acc[2];
    int hit[kBlkTiles];
    auto product = [&](int t) {
        return scan_product(a2[1], sf[t], scan_product(a2[0], sf[t], four, scale),
                            scale + 2 * kScanField);
    };
    acc[0] = product(0);
#pragma unroll
    for (int t = 0; t < kBlkTiles; ++t) {
        if (t + 1 < kBlkTiles)
            acc[(t + 1) & 1] = product(t + 1);
        hit[t] = or16(__builtin_bit_cast(v16i, acc[t & 1]));
        if (t + 1 < kBlkTiles) {
            __builtin_amdgcn_sched_group_barrier(0x002, 8, 0);
            __builtin_amdgcn_sched_group_barrier(0x008, 2, 0);
        }
    }
    const int any = (hit[0] | hit[1] | hit[2]) | (hit[3] | hit[4]) | (hit[5] | hit[6] | hit[7]);
    if (__builtin_expect(__any((any & kScanHit) != 0), 0)) {
        // ahead of the other waves, which will wait for this one at the group's
        // barrier (with int8 products, 2^24 sequences of 5x5: 1.10 ms, 1.17 without)
        __builtin_amdgcn_s_setprio(2);
#pragma unroll
        for (int t = 0; t < kBlkTiles; ++t) {
            // a carry displaces the lower fields: both tiles are looked at
            if (__any((hit[t] & ((1 << 5) | (1 << 11) | (1 << 24))) != 0))
                scan_absorb(a2[0], sf[t], top + t * 64, tile, lane);
            if (__any((hit[t] & ((1 << 17) | (1 << 24))) != 0))
                scan_absorb(a2[1], sf[t], top + t * 64, tile + 1, lane);
        }
        __builtin_amdgcn_s_setprio(0);
    }
}

// The same for two-letter tables, one conformation tile and 256 sequences.
// Measured alone, an int8 product takes 34 SIMD cycles, and with n vector
// instructions beside it 12 + 4.2 n where that is more: 44 for the 8 v_or3.
__device__ __forceinline__ void scan_un_tile(const v4i &a2, v4i (&sf)[kBlkTiles], ScanTop2 *top,
                                             int tile, int lane)
{
    const v16i zero = {};
    v16i acc[2];
    int hit[kBlkTiles];
    acc[0] = __builtin_amdgcn_mfma_i32_32x32x32_i8(a2, sf[0], zero, 0, 0, 0);
#pragma unroll
    for (int t = 0; t < kBlkTiles; ++t) {
        if (t + 1 < kBlkTiles)
            acc[(t + 1) & 1] = __builtin_amdgcn_mfma_i32_32x32x32_i8(a2, sf[t + 1], zero, 0, 0, 0);
        hit[t] = or16(acc[t & 1]);
        if (t + 1 < kBlkTiles) {
            __builtin_amdgcn_sched_group_barrier(0x002, 8, 0);
            __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
        }
    }
    const int any = (hit[0] | hit[1] | hit[2]) | (hit[3] | hit[4]) | (hit[5] | hit[6] | hit[7]);
    if (__builtin_expect(__any(any < 0), 0)) {
#pragma unroll
        for (int t = 0; t < kBlkTiles; ++t)
            if (__any(hit[t] < 0))
                scan_un_absorb(a2, sf[t], top + t * 32, tile, lane);
    }
}

// The work of one workgroup: B blocks from `blk` on (plain 10: sequence >> 10;
// canonical: canonical block index; chunked: chunk and the outer bits within
// it), each scored by S groups of NW = wide_waves<G>() waves.  Wave w of a
// group scores the 512 sequences x = 512 w + 64 t + lane (t = 0 .. 7) of its
// block against every S-th group of NW conformation tiles.  vlds holds each
// block's first-product fragments, a2s each group's packed first products of
// two groups of tiles, gbs every sequence's two best keys.
template <int KB, int G, int S = 1, int B = 1>
struct WideShared {
    static constexpr int NW = wide_waves<G>();
    v4i vlds[B][wide_steps<KB, G>() * 64];
    v4i a2s[B * S][2][NW][64];   // pure: 6 words of 32 conformations
    ScanTop2 gbs[B][NW][kBlkTiles * wide_cols<G>()];
    unsigned del;
};

// LOOP: called in a loop over blocks, which costs registers.
template <int KB, int G, int S, int B, bool LOOP = false>
__device__ __forceinline__ void wide_body(const EnumJob &j, uint64_t blk, WideShared<KB, G, S, B> &sh,
                                          unsigned *hist = nullptr)
{
    constexpr int NW = wide_waves<G>();
    constexpr int KS = wide_steps<KB, G>();
    constexpr bool UN = wide_table<G>();
    constexpr int kCols = wide_cols<G>();
    // in a loop, nothing that depends on the lane is kept over the blocks
    unsigned tid = threadIdx.x;
    if constexpr (LOOP)
        asm volatile("" : "+v"(tid));
    const int lane = tid & 63;
    const int half = lane >> 5;
    const int w = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int wave = w % NW, sp = w / NW % S, bk = w / (NW * S);
    blk += bk;
    v4i *const vlds = sh.vlds[bk];
    auto &a2s = sh.a2s[bk * S + sp];
    bool diag = false;
    const uint64_t outer = G == 1   ? wide_canonical_outer(j, blk, &diag)
                           : G == 2 || G == 3 ? wide_chunk_outer<G>(blk)
                                              : blk << kWideBits;
    const v4i *__restrict__ C1 = reinterpret_cast<const v4i *>(UN ? j.gemm_b : j.scan_c1);

    if (threadIdx.x == 0)
        sh.del = 0;
    // the waves build the block's fragments, one step at a time
    for (int st = w % (NW * S); st < KS; st += NW * S)
        vlds[st * 64 + lane] = UN ? wide_un_fragment(j, outer, lane & 31, half, st)
                                  : wide_v_fragment<G>(j, outer, lane & 31, half, st);
    v4i sf[kBlkTiles];
    if constexpr (UN) {
#pragma unroll
        for (int t = 0; t < kBlkTiles; ++t)
            sf[t] = wide_un_operand(j, wave * 256 + t * 32 + (lane & 31), half);
    } else {
        const v4i *__restrict__ S2 = reinterpret_cast<const v4i *>(j.wide_s2) +
                                     (wide_s2_slot<G>() + wave) * (kBlkTiles * 64);
#pragma unroll
        for (int t = 0; t < kBlkTiles; ++t)
            sf[t] = S2[t * 64 + lane];
    }
    // Wait for these loads here (s_waitcnt vmcnt(0)): the compiler's wait
    // counts are the same for every pass of the tile loop, so loads of the
    // second operand still counted as in flight there would make each pass
    // also wait for the contact-tile loads issued one group ahead.
    __builtin_amdgcn_s_waitcnt(0x0f70);

    // the two best keys of this wave's sequences, 64 per tile, in LDS
    ScanTop2 *const top2 = sh.gbs[bk][wave];
    if (sp == 0) {
#pragma unroll
        for (int i = lane; i < kBlkTiles * kCols; i += 64)
            top2[i] = ScanTop2{0, 0};
    }

    const int n_tiles = j.n_tiles;
    const int n_conf = j.n_conf;

    // contact tile `tile` of the first product (this lane's fragments); every
    // wave reads only its own tiles, straight from global memory (L2-resident)
    auto load_c1 = [&](int tile, v4i (&c1)[KS]) {
        const v4i *__restrict__ src = C1 + size_t(tile) * (KS * 64) + lane;
#pragma unroll
        for (int st = 0; st < KS; ++st)
            c1[st] = src[st * 64];
    };
    // first product of a tile into this wave's slot of buffer `buf`.  Tables: row
    // 8 (q / 4) + 4 half + q % 4 of the result is byte q of this lane's second
    // operand, and the two constant rows are bytes 14 and 15 of half 1 (0 in
    // columns beyond the last conformation, whose accumulators stay 0)
    auto first_un = [&](const v4i (&c1)[KS], int tile, int buf) {
        v16i d1;
#pragma unroll
        for (int st = 0; st < KS; ++st) {
            const v16i zero = {};
            d1 = __builtin_amdgcn_mfma_i32_32x32x32_i8(vlds[st * 64 + lane], c1[st],
                                                       st == 0 ? zero : d1, 0, 0, 0);
        }
        // the block term's digits: row 0 is byte 0 of half 0, row 29 byte 13 of half 1
        d1[0] = half ? d1[0] : d1[0] & 63;
        d1[13] = half ? d1[13] >> 6 : d1[13];
        const int ones = half && tile * kTileConf + (lane & 31) < n_conf ? 0x40010000 : 0;
        v4i p = pack_d1(d1);
        p[3] |= ones;   // rows 30 and 31 of the product are 0
        a2s[buf][wave][lane] = p;
    };
    auto first = [&](const v4i (&c1)[KS], int tile, int buf) {
        if constexpr (UN) {
            first_un(c1, tile, buf);
            return;
        }
        v16f d1;
#pragma unroll
        for (int st = 0; st < KS; ++st) {
            const v16f zero = {};
            const v4i v = vlds[st * 64 + lane];
            const v8i a = {v[0], v[1], v[2], v[3], 0, 0, 0, 0};
            const v8i b = {c1[st][0], c1[st][1], c1[st][2], c1[st][3], 0, 0, 0, 0};
            d1 = __builtin_amdgcn_mfma_scale_f32_32x32x64_f8f6f4(a, b, st == 0 ? zero : d1, 4, 4,
                                                                 0, 0, 0, 0);
        }
        // the block term's digits, and the constants 9 and 1 of real columns
        const float f0 = 8.0f * __builtin_floorf(0.125f * d1[0]);
        const float f13 = 8.0f * __builtin_floorf(0.125f * d1[13]);
        const bool real = tile * kTileConf + (lane & 31) < n_conf;
        d1[0] = half ? d1[0] : d1[0] - f0;
        d1[13] = half ? f13 : d1[13];
        d1[14] = half ? (real ? 9.0f : 0.0f) : d1[14];
        d1[15] = half ? (real ? 1.0f : 0.0f) : d1[15];
        // 16 values as FP6, d1[i] and d1[8 + i] in turn, in eighths; the other
        // 16 of the conversion are not used
        const v16f up = __builtin_shufflevector(d1, d1, 8, 9, 10, 11, 12, 13, 14, 15, 8, 9, 10, 11,
                                                12, 13, 14, 15);
        const auto p = __builtin_amdgcn_cvt_scalef32_2xpk16_fp6_f32(d1, up, 8.0f);
        // words 0 .. 3 of the 32 conformations, then words 4 and 5
        int *const dst = reinterpret_cast<int *>(a2s[buf][wave]);
        const int conf = lane & 31;
        dst[half ? 4 * conf + 3 : 4 * conf] = int(p[0]);
        dst[half ? 128 + 2 * conf : 4 * conf + 1] = int(p[1]);
        dst[half ? 129 + 2 * conf : 4 * conf + 2] = int(p[2]);
    };

    // first tile of this group's g-th group of tiles
    auto tile0 = [&](int g) { return (g * S + sp) * NW; };
    const int n_groups = (n_tiles + NW * S - 1) / (NW * S);
    v4i c1[KS];
    __syncthreads();   // vlds
    // first product of tile `tile`, loaded; zeros beyond the last, which may be
    // the second of a pair
    auto next_first = [&](int tile, int buf) {
        if (tile < n_tiles)
            first(c1, tile, buf);
        else
            a2s[buf][wave][lane] = v4i{0, 0, 0, 0};
    };
    if (tile0(0) + wave < n_tiles)
        load_c1(tile0(0) + wave, c1);
    next_first(tile0(0) + wave, 0);
    if (tile0(1) + wave < n_tiles)
        load_c1(tile0(1) + wave, c1);
    __syncthreads();
    // The group's barrier sits before its last products: by then every wave has
    // read all of this group's buffer and written its first product of the next
    // group.  Tables read each packed first product one tile ahead of its use;
    // pairs leave no registers for that.
    constexpr int kStep = UN ? 1 : 2;   // conformation tiles at a time
    std::conditional_t<UN, v4i, v6i> a2[kStep];
    auto read = [&](int buf, int tt) {
#pragma unroll
        for (int i = 0; i < kStep; ++i) {
            const v4i *src = a2s[buf][tt + i];
            if constexpr (UN) {
                a2[i] = src[lane];
            } else {
                const v4i q = src[lane & 31];
                const int2 r = reinterpret_cast<const int2 *>(src + 32)[lane & 31];
                a2[i] = v6i{q[0], q[1], q[2], q[3], r.x, r.y};
            }
        }
    };
    if constexpr (UN)
        read(0, 0);
    for (int g = 0; g < n_groups; ++g) {
        const int buf = g & 1;
        const int nt = tile0(g + 1) + wave;   // this wave's tile of the next group
        if constexpr (S > 1) {
            // thresholds raised by the waves that share the sequences: after
            // every group while they rise fast, then every 8 tiles
            constexpr int kEvery = NW >= 8 ? 1 : 8 / NW;
            if (g > 0 && (g <= 8 || g % kEvery == 0)) {
#pragma unroll
                for (int t = 0; t < kBlkTiles; ++t) {
                    if constexpr (UN)
                        scan_un_set(sf[t], top2[t * 32 + (lane & 31)].s, half);
                    else
                        scan_set_v(sf[t], scan_bias(top2[t * 64 + lane].s));
                }
            }
        }
#pragma unroll 1
        for (int tt = 0; tt < NW; tt += kStep) {
            const int tile = tile0(g) + tt;
            [[maybe_unused]] const auto now = a2[0];
            if (tt == 0) {
                next_first(nt, buf ^ 1);
                const int n2 = tile0(g + 2) + wave;
                if (n2 < n_tiles)
                    load_c1(n2, c1);
            }
            if constexpr (UN) {
                if (tt + kStep < NW) {
                    read(buf, tt + kStep);
                } else {
                    // the next group's first products are visible, and this
                    // group's buffer is free for the group after it
                    __syncthreads();
                    read(buf ^ 1, 0);
                }
            } else {
                read(buf, tt);
                if (tt + kStep >= NW)
                    __syncthreads();
            }
            if (tile < n_tiles) {
                if constexpr (UN)
                    scan_un_tile(now, sf, top2, tile, lane);
                else
                    scan_pair(a2, sf, top2, tile, lane);
            }
        }
    }
    if constexpr (S > 1)
        __syncthreads();   // every group's keys

    unsigned del = 0;
#pragma unroll 1
    for (int t = sp; t < kBlkTiles * kCols / 64; t += S) {
        const ScanTop2 k = top2[t * 64 + lane];
        const int2 v = {scan_global(int(k.b)), scan_global(int(k.s))};
        const int x = wave * (kBlkTiles * kCols) + t * 64 + lane;
        if constexpr (G == 1) {
            // off the diagonal the block's reverse is never scored: write both;
            // a diagonal block holds each sequence and its reverse itself
            uint64_t sq = outer;
#pragma unroll
            for (int b = 0; b < kWideBits; ++b)
                sq |= uint64_t((x >> b) & 1) << wide_pos<1>(j, b);
            const uint64_t rs = diag ? sq : __builtin_bitreverse64(sq) >> (64 - j.N);
            del += finish_sequence(j, j.scan_c2q, sq, sq, rs, blk < j.hi, v.x, v.y, j.A);
        } else if constexpr (G == 2 || G == 3) {
            uint64_t sq = outer | uint64_t(x & 31);
#pragma unroll
            for (int b = 5; b < wide_bits<G>(); ++b)
                sq |= uint64_t((x >> b) & 1) << wide_pos<G>(j, b);
            del += finish_sequence(j, j.scan_c2q, sq, sq, sq, sq >= j.lo && sq < j.hi, v.x, v.y,
                                   j.A, hist);
        } else {
            const uint64_t idx = outer + uint64_t(x);
            del += finish_sequence(j, j.scan_c2q, idx, idx, idx, idx >= j.lo && idx < j.hi, v.x,
                                   v.y, UN ? 1 : j.A, hist);
        }
    }
    count_deleterious_wg(j, del, &sh.del);
}

// Blocks of 1024, S groups of 2 waves on each: canonical blocks, and plain
// ranges of few blocks, whose workgroups split the conformations so that they
// still fill the compute units.
template <int KB, bool CANON, int S>
__global__ __launch_bounds__(128 * S, 4) void k_gemm_wide(EnumJob j)
{
    constexpr int G = CANON ? 1 : 0;
    __shared__ WideShared<KB, G, S> sh;
    wide_body<KB, G, S, 1>(j, (CANON ? j.lo : j.lo >> kWideBits) + blockIdx.x, sh);
}

template <int KB>
union WidePlainShared {
    WideShared<KB, 3> b4096;
    WideShared<KB, 2, 1, 2> b2048;
    WideShared<KB, 0, 1, 4> b1024;
};

// A plain range in the largest blocks it holds: workgroups of 8 waves score
// one block of 4096 (the first c.n3), two of 2048 (the next c.n2 / 2) or four
// of 1024 sequences.  Smaller blocks lie on both sides of larger ones: block i
// of a size is block lo + i before the gap, and after it i continues at hi.
template <int KB, bool LOOP>
__device__ __forceinline__ void wide_plain(const EnumJob &j, const WideCut &c, unsigned wg,
                                           WidePlainShared<KB> &sh, unsigned *hist)
{
    if (wg < c.n3) {
        wide_body<KB, 3, 1, 1, LOOP>(j, c.lo3 + wg, sh.b4096, hist);
    } else if (wg < c.n3 + c.n2 / 2) {
        const unsigned i = 2 * (wg - c.n3);
        wide_body<KB, 2, 1, 2, LOOP>(j, i < c.n2_lo ? c.lo2 + i : c.hi2 + (i - c.n2_lo), sh.b2048,
                                     hist);
    } else {
        // four consecutive blocks may reach over the gap: their waves differ
        const unsigned i = 4 * (wg - c.n3 - c.n2 / 2);
        const unsigned bk = __builtin_amdgcn_readfirstlane(threadIdx.x >> 7), b = i + bk;
        const uint64_t blk = b < c.n1_lo ? c.lo1 + b : c.hi1 + (b - c.n1_lo);
        wide_body<KB, 0, 1, 4, LOOP>(j, blk - bk, sh.b1024, hist);
    }
}

template <int KB>
__global__ __launch_bounds__(512, 4) void k_gemm_wide_w8(EnumJob j, WideCut c)
{
    __shared__ WidePlainShared<KB> sh;
    wide_plain<KB, false>(j, c, blockIdx.x, sh, nullptr);
}

// The same for boxes of few classes (and conformations): n_wg workgroups' work
// by two workgroups per compute unit, which count the designability of all
// their blocks in LDS (2^24 sequences of 5x5 with all outputs 1.25 ms, 2.26 ms
// with an atomic per designing sequence).
template <int KB>
__global__ __launch_bounds__(512, 4) void k_gemm_wide_few(EnumJob j, WideCut c, unsigned n_wg)
{
    __shared__ WidePlainShared<KB> sh;
    __shared__ unsigned counts[kHistClasses];
    zero_hist(j, counts);
#pragma unroll 1
    for (unsigned wg = blockIdx.x; wg < n_wg; wg += gridDim.x) {
        wide_plain<KB, true>(j, c, wg, sh, counts);
        __syncthreads();   // the next block's state, or the counts
    }
    flush_hist(j, counts);
}

// Batched wide blocks for jobs of one product depth and geometry G (0, 2 or
// 3): workgroup b scores the wide block of item item_lo + b, in the job whose
// item range holds it, S groups of waves splitting the conformations.
template <int KB, int G, int S>
__global__ __launch_bounds__(64 * S * wide_waves<G>(), 4) void k_gemm_wide_batch(BatchHeader *hdr,
                                                                                 int item_lo)
{
    __shared__ WideShared<KB, G, S> sh;
    const EnumJob *jobs = reinterpret_cast<const EnumJob *>(hdr + 1);
    const int njobs = hdr->njobs;
    const int64_t *start = reinterpret_cast<const int64_t *>(jobs + njobs);
    const int it = item_lo + int(blockIdx.x);
    int lo = 0, hi = njobs - 1;   // job with start[job] <= it < start[job+1]
    while (lo < hi) {
        const int mid = (lo + hi + 1) / 2;
        if (start[mid] <= it)
            lo = mid;
        else
            hi = mid - 1;
    }
    lo = __builtin_amdgcn_readfirstlane(lo);
    const EnumJob &j = jobs[lo];
    const uint64_t blk0 = G == 3   ? (j.lo >> kWide12ChunkBits) << 7
                          : G == 2 ? (j.lo >> kWide11ChunkBits) << 6
                                   : j.lo >> kWideBits;
    wide_body<KB, G, S, 1>(j, blk0 + uint64_t(it - start[lo]), sh);
}

// Two-letter tables: blocks of 1024, S groups of 4 waves on each.
template <int KB, int S>
__global__ __launch_bounds__(256 * S, 4) void k_gemm_wide_un(EnumJob j)
{
    __shared__ WideShared<KB, 4, S> sh;
    wide_body<KB, 4, S, 1>(j, (j.lo >> kWideBits) + blockIdx.x, sh);
}

// The same for boxes of few classes, as k_gemm_wide_few (5x5 with all outputs, 98
// blocks 57 us against 85, 2^20 sequences 0.14 ms; from 64 blocks on).
template <int KB>
__global__ __launch_bounds__(256, 4) void k_gemm_wide_un_few(EnumJob j, unsigned n_blocks)
{
    __shared__ WideShared<KB, 4> sh;
    __shared__ unsigned counts[kHistClasses];
    zero_hist(j, counts);
#pragma unroll 1
    for (unsigned b = blockIdx.x; b < n_blocks; b += gridDim.x) {
        wide_body<KB, 4, 1, 1, true>(j, (j.lo >> kWideBits) + b, sh, counts);
        __syncthreads();   // the next block's state, or the counts
    }
    flush_hist(j, counts);
}

// Groups of waves per block for a launch of n blocks of `waves` waves each: as
// many as bring it to 4096 waves (16 per compute unit), at most 16 waves per
// workgroup.  A sweep over all conformations takes a wave 1.8 ms on 3x3x3
// however few they are; 2^17 sequences take 0.49 ms split eight ways.
inline int wide_split(uint64_t n, int waves)
{
    int s = 1;
    while (2 * s * waves <= 16 && 2 * s * waves * n <= 4096)
        s *= 2;
    return s;
}

template <int KB, int G>
hipError_t launch_wide_batch_g(BatchHeader *hdr, int item_lo, unsigned grid, hipStream_t st)
{
    constexpr int NW = wide_waves<G>();
    const int s = wide_split(grid, NW);
    auto go = [&](auto split) {
        constexpr int S = decltype(split)::value;
        if constexpr (S * NW <= 16)
            hipLaunchKernelGGL((k_gemm_wide_batch<KB, G, S>), dim3(grid), dim3(64 * S * NW), 0, st,
                               hdr, item_lo);
    };
    if (s == 8)
        go(std::integral_constant<int, 8>{});
    else if (s == 4)
        go(std::integral_constant<int, 4>{});
    else if (s == 2)
        go(std::integral_constant<int, 2>{});
    else
        go(std::integral_constant<int, 1>{});
    return hipGetLastError();
}

// wide: 1 blocks of 1024, 2 blocks of 2048, 3 blocks of 4096
template <int KB>
hipError_t launch_wide_batch(BatchHeader *hdr, int item_lo, unsigned grid, int wide,
                             hipStream_t st)
{
    return wide == 3   ? launch_wide_batch_g<KB, 3>(hdr, item_lo, grid, st)
           : wide == 2 ? launch_wide_batch_g<KB, 2>(hdr, item_lo, grid, st)
                       : launch_wide_batch_g<KB, 0>(hdr, item_lo, grid, st);
}

template <int KB, bool CANON>
hipError_t launch_wide_small(const EnumJob &j, uint64_t n, hipStream_t st)
{
    const dim3 grid = dim3(unsigned(n));
    switch (wide_split(n, wide_waves<0>())) {
    case 8: hipLaunchKernelGGL((k_gemm_wide<KB, CANON, 8>), grid, dim3(1024), 0, st, j); break;
    case 4: hipLaunchKernelGGL((k_gemm_wide<KB, CANON, 4>), grid, dim3(512), 0, st, j); break;
    case 2: hipLaunchKernelGGL((k_gemm_wide<KB, CANON, 2>), grid, dim3(256), 0, st, j); break;
    default: hipLaunchKernelGGL((k_gemm_wide<KB, CANON, 1>), grid, dim3(128), 0, st, j); break;
    }
    return hipGetLastError();
}

// Plain ranges: with `chunked`, launches of more than 2048 blocks of 1024 (4096
// waves, 16 per compute unit) take the largest blocks the range holds; fewer
// (or without) take blocks of 1024, which spread more evenly: 2^20 sequences of
// 3x3x3 1.8 ms (3.5 ms in the largest blocks, one workgroup per compute unit);
// 2^22 5.0 ms in the largest, 6.1 ms in blocks of 1024.
// Boxes of few classes take k_gemm_wide_few from 384 blocks on, where its LDS
// counts gain more than its larger workgroups lose: 5x5 with all outputs, 196
// blocks 109 us against 69, 489 blocks 121 against 137, 977 120 against 239.
template <int KB>
hipError_t launch_wide(const EnumJob &j, bool chunked, hipStream_t st)
{
    if (j.mode == kSeqCanonical)
        return launch_wide_small<KB, true>(j, j.hi - j.lo, st);
    const uint64_t n = wide_blocks(1, j.lo, j.hi);
    const bool few = KB <= 5 && j.n_class <= kHistClasses;   // up to 27 monomers, but for 2 x n
    if (!chunked || n <= (few ? 384 : 2048))
        return launch_wide_small<KB, false>(j, n, st);
    const WideCut c = wide_cut(j.N, j.lo, j.hi);
    const unsigned n_wg = c.n3 + c.n2 / 2 + (c.n1 + 3) / 4;
    if constexpr (KB <= 5) {
        if (few) {
            hipLaunchKernelGGL((k_gemm_wide_few<KB>), dim3(std::min(n_wg, 512u)), dim3(512), 0, st, j,
                               c, n_wg);
            return hipGetLastError();
        }
    }
    hipLaunchKernelGGL((k_gemm_wide_w8<KB>), dim3(n_wg), dim3(512), 0, st, j, c);
    return hipGetLastError();
}

template <int KB>
hipError_t launch_blk_batch_kb(BatchHeader *hdr, int item_lo, unsigned grid, bool unary, int wide,
                               hipStream_t st)
{
    if (wide)
        return unary ? hipErrorInvalidValue : launch_wide_batch<KB>(hdr, item_lo, grid, wide, st);
    constexpr int MODE = KB <= 6 ? kBlkLdsS2 : kBlkLds;
    if constexpr (KB <= kBlkUnaryMaxKB) {
        if (unary) {
            hipLaunchKernelGGL((k_gemm_blk_batch<KB, 4, MODE, true>), dim3(grid), dim3(256), 0,
                               st, hdr, item_lo);
            return hipGetLastError();
        }
    }
    if (unary)
        return hipErrorInvalidValue;
    hipLaunchKernelGGL((k_gemm_blk_batch<KB, 4, MODE, false>), dim3(grid), dim3(256), 0, st, hdr,
                       item_lo);
    return hipGetLastError();
}

template <int KB, int NW, int MODE>
hipError_t launch_blk_shape(const EnumJob &j, hipStream_t st)
{
    const bool canon = j.mode == kSeqCanonical;
    const uint64_t n_blocks =
        canon ? j.hi - j.lo : ((j.hi - 1) >> kBlkBits) - (j.lo >> kBlkBits) + 1;
    const dim3 grid(unsigned((n_blocks + NW - 1) / NW));
    if (canon)
        hipLaunchKernelGGL((k_gemm_blk<KB, NW, MODE, true, false>), grid, dim3(NW * 64), 0, st, j);
    else
        hipLaunchKernelGGL((k_gemm_blk<KB, NW, MODE, false, false>), grid, dim3(NW * 64), 0, st, j);
    return hipGetLastError();
}

// Two-letter tables: one launch shape (4 waves, staging by depth).
template <int KB>
hipError_t launch_blk_unary(const EnumJob &j, hipStream_t st)
{
    if constexpr (KB > kBlkUnaryMaxKB) {
        return hipErrorInvalidValue;
    } else {
        constexpr int MODE = KB <= 6 ? kBlkLdsS2 : kBlkLds;
        const bool canon = j.mode == kSeqCanonical;
        const uint64_t n_blocks =
            canon ? j.hi - j.lo : ((j.hi - 1) >> kBlkBits) - (j.lo >> kBlkBits) + 1;
        const dim3 grid(unsigned((n_blocks + 3) / 4));
        if (canon)
            hipLaunchKernelGGL((k_gemm_blk<KB, 4, MODE, true, true>), grid, dim3(256), 0, st, j);
        else
            hipLaunchKernelGGL((k_gemm_blk<KB, 4, MODE, false, true>), grid, dim3(256), 0, st, j);
        return hipGetLastError();
    }
}

template <int KB>
hipError_t launch_wide_un(const EnumJob &j, hipStream_t st)
{
    if constexpr (KB > kBlkUnaryMaxKB) {
        return hipErrorInvalidValue;
    } else {
        const uint64_t n = wide_blocks(1, j.lo, j.hi);
        if (n >= 64 && j.n_class <= kHistClasses) {
            hipLaunchKernelGGL((k_gemm_wide_un_few<KB>), dim3(unsigned(std::min<uint64_t>(n, 1024))), dim3(256), 0, st, j,
                               unsigned(n));
            return hipGetLastError();
        }
        const dim3 grid = dim3(unsigned(n));
        switch (wide_split(n, wide_waves<4>())) {
        case 4: hipLaunchKernelGGL((k_gemm_wide_un<KB, 4>), grid, dim3(1024), 0, st, j); break;
        case 2: hipLaunchKernelGGL((k_gemm_wide_un<KB, 2>), grid, dim3(512), 0, st, j); break;
        default: hipLaunchKernelGGL((k_gemm_wide_un<KB, 1>), grid, dim3(256), 0, st, j); break;
        }
        return hipGetLastError();
    }
}

template <int KB>
hipError_t launch_blk(const EnumJob &j, int nw, int mode, hipStream_t st)
{
    if (mode == kBlkStageWide && j.wide_un)
        return launch_wide_un<KB>(j, st);
    if (j.blk_ngroups > 0 || j.blk_coefB != 0)
        return launch_blk_unary<KB>(j, st);
    if (mode == kBlkStageWide)
        return launch_wide<KB>(j, nw == 8, st);
    if (mode == kBlkLdsS2) {
        switch (nw) {
        case 2: return launch_blk_shape<KB, 2, kBlkLdsS2>(j, st);
        case 8: return launch_blk_shape<KB, 8, kBlkLdsS2>(j, st);
        default: return launch_blk_shape<KB, 4, kBlkLdsS2>(j, st);
        }
    }
    if (mode == kBlkPipe) {
        switch (nw) {
        case 2: return launch_blk_shape<KB, 2, kBlkPipe>(j, st);
        case 8: return launch_blk_shape<KB, 8, kBlkPipe>(j, st);
        default: return launch_blk_shape<KB, 4, kBlkPipe>(j, st);
        }
    }
    switch (nw) {
    case 2: return launch_blk_shape<KB, 2, kBlkLds>(j, st);
    case 8: return launch_blk_shape<KB, 8, kBlkLds>(j, st);
    default: return launch_blk_shape<KB, 4, kBlkLds>(j, st);
    }
}

}  // namespace

// One product depth's launchers, defined by the gemm_blk_kb*.hip units
// (each instantiates the kernels of its depths, so they compile in parallel).
#define HP_BLK_DEPTH(KB)                                                                  \
    hipError_t launch_gemm_blocked_kb##KB(const EnumJob &j, int nw, int mode, hipStream_t st) \
    {                                                                                     \
        return launch_blk<KB>(j, nw, mode, st);                                           \
    }                                                                                     \
    hipError_t launch_gemm_blk_batch_kb##KB(BatchHeader *hdr, int item_lo, unsigned grid,  \
                                            bool unary, int wide, hipStream_t st)         \
    {                                                                                     \
        return launch_blk_batch_kb<KB>(hdr, item_lo, grid, unary, wide, st);              \
    }                                                                                     \
    hipError_t launch_gemm_wide_kb##KB(const EnumJob &j, hipStream_t st)                  \
    {                                                                                     \
        return launch_wide<KB>(j, false, st);                                             \
    }

}  // namespace hpmap
