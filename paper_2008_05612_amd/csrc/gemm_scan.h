// Threshold scan of the dense form (internal templates; instantiated in
// gemm_scan_*.hip): any sequences (plain ranges, random draws, canonical
// sequences) against every conformation, each as its own column of the
// product.
//
// The contact count (pure pair energies) or F = A n + B sum_i h_i c_i
// (two-letter tables) of 32 columns comes from one chain of FP4 / FP6 products
// of depth 64, which the matrix cores run in the time of an int8 product of
// depth 32, exact in the float accumulator.  Further product rows, constant
// on the conformation side, carry T per column, the smallest value that can
// still change that sequence's two best (one more than its second best): a
// bit of the accumulator says whether the threshold is reached, a lane ORs
// its 16 accumulators, and only a tile with a hit is absorbed (what lies below
// T changes no output, as in the wide kernel).
//
//   PURE: counts are at most 31 (kScanMaxContacts), so an accumulator holds
//     two conformations of a column, 16 bits apart: the 32-row blocks of the
//     two lane halves belong to conformation tiles 2 p and 2 p + 1, and the
//     second half's operand carries the block scale 2^16.  One contact is one
//     unit; each field holds 32 + n - T (6 bits, bit 5: n reaches T) and the
//     upper one 128 more, which is 2^23 in all and fixes the exponent, so the
//     float's bits are the two fields.  KB products per 64 conformations.
//   UN: one conformation per accumulator, T - 1/2 - F, negative iff F reaches
//     T; pair rows carry A (FP6) times 0/1, unary rows B times the contact
//     count c_i (at most 4, exact in FP4), in units of 1/8.
//
// A workgroup of Q S waves: wave q + Q s scores TT tiles of 32 columns
// (group q of the workgroup's Q) against every S-th conformation tile.  The
// S waves of a group share each column's two best in LDS, so a launch of few
// sequences still fills the compute units: it is split over conformations,
// not sequences, and the threshold that one wave raises serves the others.
#pragma once

#include "device_common.h"

namespace hpmap {

constexpr int kScanPureHit = (1 << 5) | (1 << 21);

__device__ __forceinline__ unsigned scan_threshold(unsigned s) { return (s + kMaxConf) >> kKeyConfBits; }

// 32 product rows of a column from row `start`: bits h_i h_j of the pairs,
// then (UN) the unary rows h_i, 0 beyond.
template <bool UN>
__device__ __forceinline__ uint32_t scan_rows(const EnumJob &j, uint64_t s, int start)
{
    uint32_t bits = pair_bits(s, s, j.N, start);
    if (UN) {
        const int at = j.K - start;   // where the unary rows start in the word
        if (at < 32 && at + j.N > 0)
            bits |= at >= 0 ? uint32_t(s) << at : uint32_t(s >> -at);
    }
    return bits;
}

// Signed digit -4 .. 4 as an FP4 code (codes 0 .. 4 are multiples of 1/2).
__device__ __forceinline__ uint32_t fp4_digit(int x) { return uint32_t(x < 0 ? 8 - x : x); }

// PURE threshold digits, the top two nibbles of the last word: with V = 32 -
// T, half 0 adds 12 (constant row) + 4 b + d = V, half 1 144 + 4 b + d = V +
// 128.
__device__ __forceinline__ uint32_t scan_pure_digits(int T, int half)
{
    const int r = 32 - T - (half ? 16 : 12);
    const int b = min((r + 2) >> 2, 4);
    return (fp4_digit(b) << 24) | (fp4_digit(r - 4 * b) << 28);
}

// UN threshold digits, the last word of the half-1 lanes: T = 360 a + 24 e +
// 6 f + g on the constant rows 6.0 (twice 360), 6.0, 6.0 and 1.0, as FP6 codes
// in units of 1/8 (0 .. 15 are their own codes).
__device__ __forceinline__ uint32_t scan_un_digits(int T)
{
    const int a = T / 360, r = T - 360 * a;
    const int e = r / 24, q = r - 24 * e;
    const int f = q / 6, g = q - 6 * f;
    const uint32_t ec = e < 4 ? 4 * e : e < 8 ? 8 + 2 * e : 16 + e;   // code of 4 e
    const uint32_t ac = a == 0 ? 0u : a == 1 ? 31u << 2 : (31u << 2) | (31u << 8);
    return ac | (ec << 14) | (uint32_t(f) << 20) | (uint32_t(g) << 26);
}

template <bool UN>
struct ScanFrag {
    int w[UN ? 6 : 4];
};

// Second operand of one column tile, step st: PURE rows 32 st .. 32 st + 31
// (the same pairs in both halves, whose conformation tiles differ); UN rows
// 64 st + 32 half + n.  The last step's last rows are the constant and
// threshold rows, with T = 0.
template <bool UN>
__device__ __forceinline__ ScanFrag<UN> scan_fragment(const EnumJob &j, uint64_t s, int st, int half,
                                                      bool last)
{
    ScanFrag<UN> f;
    if constexpr (!UN) {
        const uint32_t bits = scan_rows<false>(j, s, 32 * st);
#pragma unroll
        for (int w = 0; w < 4; ++w)
            f.w[w] = int(fp4_spread((bits >> (8 * w)) & 0xffu));
        if (last)
            f.w[3] |= ((half ? 7 : 1) << 20) | scan_pure_digits(0, half);
    } else {
        const int start = 64 * st + 32 * half;
        const uint32_t bits = scan_rows<true>(j, s, start);
        // pair rows carry -A, unary rows -B, 6 bits each (sign bit 5)
        const int npair = min(max(j.K - start, 0), 32);
#pragma unroll
        for (int w = 0; w < 6; ++w)
            f.w[w] = 0;
#pragma unroll
        for (int n = 0; n < 32; ++n) {
            const uint32_t code = 32u | uint32_t(n < npair ? j.A : j.B);
            const uint32_t c = (bits >> n) & 1u ? code : 0u;
            f.w[6 * n / 32] |= int(c << (6 * n % 32));
            if (6 * n % 32 > 26)
                f.w[6 * n / 32 + 1] |= int(c >> (32 - 6 * n % 32));
        }
        if (last && half) {
            // row 26: the constant 0.5 (conformation side) times 1/8 below
            // the threshold; rows 27 .. 31 the digits
            f.w[4] |= int((32u | 1u) << 28);
            f.w[5] |= int((32u | 1u) >> 4) | int(scan_un_digits(0));
        }
    }
    return f;
}

template <bool UN>
__device__ __forceinline__ v16f scan_mfma(const v4i &a, const ScanFrag<UN> &b, const v16f &c,
                                          int scale)
{
    const v8i av = {a[0], a[1], a[2], a[3], 0, 0, 0, 0};
    if constexpr (!UN) {
        const v8i bv = {b.w[0], b.w[1], b.w[2], b.w[3], 0, 0, 0, 0};
        return __builtin_amdgcn_mfma_scale_f32_32x32x64_f8f6f4(av, bv, c, 4, 4, 0, scale, 0, 127);
    } else {
        const v8i bv = {b.w[0], b.w[1], b.w[2], b.w[3], b.w[4], b.w[5], 0, 0};
        return __builtin_amdgcn_mfma_scale_f32_32x32x64_f8f6f4(av, bv, c, 4, 2, 0, 0, 0, 0);
    }
}

// Absorbs a tile's accumulators into the column's two best.  PURE: tiles
// `tile` (lower field) and tile + 1 (upper); UN: `tile`.  T: the threshold the
// product was formed with.
template <bool UN>
__device__ __forceinline__ void scan_absorb_dense(const v16i &a, int T, ScanTop2 *g, int tile,
                                                  int half)
{
    if constexpr (!UN) {
        unsigned k[4];
        scan_best<26>(a, k[0], k[1]);
        scan_best<10>(a, k[2], k[3]);
        unsigned key[4];
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const int n = int(k[i] >> 26) - 32 + T;   // below T (no candidate): not negative only by chance
            const unsigned low = ((k[i] & 31) << 12) + unsigned(4 * half << 12) +
                                 unsigned(tile + (i >> 1) + 1);
            key[i] = n >= T ? (unsigned(n) << kKeyConfBits) + low : 0;
        }
        int b = int(key[0]), s = int(key[1]);
        top2_merge(b, s, int(key[2]), int(key[3]));
        scan_push(g, unsigned(b), unsigned(s));
    } else {
        // T - 1/2 - F in eighths: negative where F reaches T, and the more so
        // the larger F, which unsigned order of the bits keeps; the low bits
        // of the mantissa are 0 (F < 2^10) and take the row, plus one: each key
        // is then the result of an OR, which med3_u32 needs
        unsigned b = 0, s = 0;
#pragma unroll
        for (int q = 0; q < 16; q += 2) {
            const unsigned r = 8 * (q / 4) + q % 4 + 1;
            const unsigned k0 = unsigned(a[q]) | r, k1 = unsigned(a[q + 1]) | (r + 1);
            const unsigned m = med3_u32(b, k0, k1);
            b = max(max(b, k0), k1);
            s = max(s, m);
        }
        auto key = [&](unsigned k) {
            const float v = __uint_as_float(k & ~31u);   // -(F - T + 1/2) / 8
            const int F = T + int(-8.0f * v);
            return int(k) < 0 ? (unsigned(F) << kKeyConfBits) + (((k & 31) - 1) << 12) +
                                    unsigned(4 * half << 12) + unsigned(tile + 1)
                              : 0u;
        };
        scan_push(g, key(b), key(s));
    }
}

// KB steps; TT column tiles per wave; Q groups of columns, S waves each.
template <int KB, bool UN, int TT, int Q, int S>
__device__ __forceinline__ void scan_dense_body(const EnumJob &j, uint64_t seq0, ScanFrag<UN> *frag,
                                                ScanTop2 *top, unsigned *del_sum,
                                                unsigned *hist)
{
    constexpr int kCols = Q * TT * 32;
    const int lane = threadIdx.x & 63;
    const int wave = threadIdx.x >> 6;
    const int half = lane >> 5, col = lane & 31;
    const int q = wave % Q, sp = wave / Q;

    for (int i = threadIdx.x; i < kCols; i += 64 * Q * S)
        top[i] = ScanTop2{0, 0};
    if (threadIdx.x == 0)
        *del_sum = 0;
    if (hist)
        zero_hist(j, hist);
    // second operands, through LDS: waves that share them form them together,
    // [Q TT][KB][64]; a wave of its own one tile at a time, [Q][KB][64] (kept
    // out of registers until whole, which an unrolled loop would not)
    ScanFrag<UN> pf[TT][KB];
    if constexpr (S > 1) {
        for (int i = wave; i < Q * TT * KB; i += Q * S) {
            const int st = i % KB, t = i / KB;
            uint64_t rs;
            const uint64_t s = sequence_at(j, seq0 + t * 32 + col, &rs);
            frag[i * 64 + lane] = scan_fragment<UN>(j, s, st, half, st == KB - 1);
        }
        __syncthreads();
    }
#pragma unroll
    for (int t = 0; t < TT; ++t) {
        if constexpr (S == 1) {
            uint64_t rs;
            const uint64_t s = sequence_at(j, seq0 + (q * TT + t) * 32 + col, &rs);
#pragma unroll 1
            for (int st = 0; st < KB; ++st)
                frag[(q * KB + st) * 64 + lane] = scan_fragment<UN>(j, s, st, half, st == KB - 1);
        }
        const ScanFrag<UN> *const src = frag + (S > 1 ? q * TT + t : q) * KB * 64 + lane;
#pragma unroll
        for (int st = 0; st < KB; ++st)
            pf[t][st] = src[st * 64];
    }
    __syncthreads();
    ScanTop2 *const mine = top + q * TT * 32 + col;
    int T[TT];
#pragma unroll
    for (int t = 0; t < TT; ++t)
        T[t] = 0;

    // PURE: lane l reads conformation l & 31 of tile 2 p + half, block st, in
    // the layout of the wide first product ([tile][steps of 64][64 lanes]); UN
    // its own layout, [tile][KB][64 lanes].
    const int n_steps = UN ? j.n_tiles : (j.n_tiles + 1) / 2;
    const int c1_steps = (KB + 1) / 2;
    const v4i *A = reinterpret_cast<const v4i *>(UN ? j.scan_un : j.scan_c1);
    auto load = [&](int p, v4i (&a)[KB]) {
        const v4i *src =
            UN ? A + size_t(p) * (KB * 64) + lane : A + size_t(2 * p + half) * (c1_steps * 64) + col;
#pragma unroll
        for (int st = 0; st < KB; ++st)
            a[st] = UN ? src[st * 64] : src[st * 32];
    };
    const int scale = half ? 127 + 2 + 16 : 127 + 2;   // unit 1/4, upper field 2^16
    // Tile t's threshold in the second operand, T[t], is that of half 0's key: the
    // two lanes of a column have to hold the same one, since scan_absorb_dense
    // decodes fields that either half's digits went into with the lane's own T.
    // Other waves push to the key meanwhile, and nothing says that a read of it
    // serves both halves at once.
    auto raise = [&](int t, unsigned second) {
        const auto both = __builtin_amdgcn_permlane32_swap(second, second, false, false);
        const int now = max(int(scan_threshold(both[0])), T[t]);
        T[t] = now;
        int &w = pf[t][KB - 1].w[UN ? 5 : 3];
        if constexpr (!UN)
            w = int((unsigned(w) & 0xffffffu) | scan_pure_digits(now, half));
        else
            w = half ? int(2u | scan_un_digits(now)) : w;
    };
    // One step: the products of a[], with the next step's tile loaded
    // meanwhile (the empty assembly keeps the compiler from moving the loads
    // down to their use) and the shared second-best keys read before the
    // products, so that neither is waited for.
    auto step = [&](int p, const v4i (&a)[KB], v4i (&next)[KB]) {
        unsigned second[TT];
#pragma unroll
        for (int t = 0; t < TT; ++t)
            second[t] = mine[t * 32].s;
        if (p + S < n_steps)
            load(p + S, next);
        asm volatile("" ::: "memory");
        v16f acc[TT];
#pragma unroll
        for (int st = 0; st < KB; ++st)
#pragma unroll
            for (int t = 0; t < TT; ++t) {
                const v16f zero = {};
                acc[t] = scan_mfma<UN>(a[st], pf[t][st], st == 0 ? zero : acc[t], scale);
            }
#pragma unroll
        for (int t = 0; t < TT; ++t) {
            const v16i bits = __builtin_bit_cast(v16i, acc[t]);
            const int o = or16(bits);
            if (__any(UN ? o < 0 : (o & kScanPureHit) != 0)) {
                scan_absorb_dense<UN>(bits, T[t], &mine[t * 32], UN ? p : 2 * p, half);
                raise(t, mine[t * 32].s);
            } else if (S > 1) {
                // what the waves that share these columns raised
                if (__any(int(scan_threshold(second[t])) > T[t]))
                    raise(t, second[t]);
            }
        }
    };
    v4i a0[KB], a1[KB];
    if (sp < n_steps)
        load(sp, a0);
    for (int p = sp; p < n_steps; p += 2 * S) {
        step(p, a0, a1);
        if (p + S < n_steps)
            step(p + S, a1, a0);
    }
    __syncthreads();
    unsigned del = 0;
    for (int i0 = wave * 64; i0 < kCols; i0 += 64 * Q * S) {
        const int i = i0 + lane;
        const uint64_t idx = seq0 + i;
        const bool in = i < kCols && idx < j.hi;
        uint64_t rs = 0, sq = 0;
        ScanTop2 v = {0, 0};
        if (in) {
            sq = sequence_at(j, idx, &rs);
            v = top[i];
        }
        del += finish_sequence(j, j.scan_c2q, idx, sq, rs, in, scan_global(int(v.b)),
                               scan_global(int(v.s)), UN ? 1 : j.A, hist);
    }
    count_deleterious_wg(j, del, del_sum);
    if (hist)
        flush_hist(j, hist);
}

template <int KB, bool UN, int TT, int Q, int S, int WPE>
__global__ __launch_bounds__(64 * Q * S, WPE) void k_scan(EnumJob j)
{
    __shared__ ScanFrag<UN> frag[(S > 1 ? Q * TT : Q) * KB * 64];
    __shared__ ScanTop2 top[Q * TT * 32];
    __shared__ unsigned del_sum;
    // classes in LDS where the workgroup's sequences are several per class
    constexpr int kHist = Q * TT * 32 / 4;
    __shared__ unsigned counts[kHist];
    scan_dense_body<KB, UN, TT, Q, S>(j, j.lo + uint64_t(blockIdx.x) * (Q * TT * 32), frag, top,
                                      &del_sum, j.n_class <= kHist ? counts : nullptr);
}

template <int KB, bool UN, int TT, int Q, int S, int WPE>
hipError_t launch_scan_shape(const EnumJob &j, hipStream_t st)
{
    constexpr uint64_t per = Q * TT * 32;
    hipLaunchKernelGGL((k_scan<KB, UN, TT, Q, S, WPE>), dim3(unsigned((j.hi - j.lo + per - 1) / per)),
                       dim3(64 * Q * S), 0, st, j);
    return hipGetLastError();
}

// Launch shape by size.  Many columns: 4 groups of TT tiles per workgroup, a
// wave each, two workgroups per compute unit (2^20 draws on 3x3x3: 4.99 ms; 5.80
// and 5.96 ms with TT = 2 and with conformations split).  Fewer: as many
// columns per workgroup as leave one workgroup per compute unit, its waves
// splitting the conformations (2^14 draws on 3x3x3: 0.114 ms with 64 columns,
// 0.154 with 32; 2^13: 0.106 and 0.084).  Waves per SIMD follow the registers of
// the second operands (4 KB TT words, FP6 6 KB TT).  Boxes of few conformations
// have none to split: there up to 2^17 sequences take a tile per wave (4x4, Table
// 1, 4000 sequences 8.9 us, with TT columns 18.8; 5x4, 2^17 draws 33 and 50 us),
// more take TT again, whose class counts in LDS cover more sequences (4x4, 2^18
// draws 28 and 19 us).
template <int KB, bool UN>
hipError_t launch_scan_kb(const EnumJob &j, hipStream_t st)
{
    constexpr int kWords = (UN ? 6 : 4) * KB;   // of one column tile
    constexpr int kBig = kWords * 4 <= 96 ? 4 : UN ? 3 : 2;
    const uint64_t n = j.hi - j.lo;
    const int steps = UN ? j.n_tiles : (j.n_tiles + 1) / 2;
    if (steps < 16 && n <= 1 << 17)
        return launch_scan_shape<KB, UN, 1, 8, 1, 2>(j, st);
    if (steps < 16)
        return launch_scan_shape<KB, UN, kBig, 8, 1, 2>(j, st);
    if (n >= uint64_t(256) * 8 * kBig * 32)
        return launch_scan_shape<KB, UN, kBig, 4, 1, 2>(j, st);
    constexpr bool kFour = kWords <= (UN ? 18 : 20);   // two tiles fit four waves per SIMD
    constexpr bool kOne = kWords <= 36 && (UN || KB <= 5);   // one tile does
    if (n <= 256 * 32)
        return launch_scan_shape<KB, UN, 1, 1, kOne ? 16 : 8, kOne ? 4 : 2>(j, st);
    if (kFour && n <= 256 * 64)
        return launch_scan_shape<KB, UN, 2, 1, kFour ? 16 : 8, kFour ? 4 : 2>(j, st);
    return launch_scan_shape<KB, UN, 2, 1, 8, 2>(j, st);
}

}  // namespace hpmap
