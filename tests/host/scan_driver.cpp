// Workgroups of the threshold scans (dense columns, and wide blocks split over
// groups of waves) on emulated lanes, against a count of every conformation's
// contacts: prints the number of sequences whose phenotype, energy or gap
// differ.  Built by tests/test_scan_lanes_host.py.
#include <cstdio>
#include <string>
#include <vector>

#include "gemm_blk.h"
#include "gemm_scan.h"
#include "hp_internal.h"

using namespace hpmap;

namespace {

struct Run {
    std::vector<uint16_t> out;
    std::vector<int32_t> emin;
    std::vector<uint8_t> gap;
    std::vector<unsigned long long> desig;
    unsigned long long nondesign = 0;
    EnumJob j{};

    Run(const hp_structs &s, uint64_t lo, int n) : out(n), emin(n), gap(n), desig(s.n_class, 0)
    {
        j.scan_c2q = s.scan_c2q.data();
        j.scan_c1 = s.scan_c1.data();
        j.scan_un = s.scan_un.data();
        j.gemm_b = s.gemm_b.data();
        j.wide_s2 = s.wide_s2.data();
        j.out = out.data();
        j.emin = emin.data();
        j.gap = gap.data();
        j.desig = desig.data();
        j.nondesign = &nondesign;
        j.lo = lo;
        j.hi = lo + uint64_t(n);
        j.N = s.N;
        j.K = int32_t(s.K);
        j.U = int32_t(s.U);
        j.n_conf = int32_t(s.n_conf);
        j.n_class = int32_t(s.n_class);
        j.n_tiles = int32_t((s.n_conf + kTileConf - 1) / kTileConf);
        j.A = s.A;
        j.B = s.B;
        j.e0 = s.e0;
        j.mode = kSeqPlain;
        j.threshold = 1;
    }

    int wrong(const hp_structs &s) const
    {
        int bad = 0;
        unsigned long long none = 0;
        for (size_t i = 0; i < out.size(); ++i) {
            const uint64_t q = j.lo + i;
            int best = -1, second = -1;
            uint32_t at = 0;
            for (uint32_t c = 0; c < s.n_conf; ++c) {
                int F = 0;
                for (uint32_t k = 0; k < s.nbp; ++k) {
                    const uint8_t *p = &s.contacts[(size_t(c) * s.nbp + k) * 2];
                    const int a = int(q >> p[0]) & 1, b = int(q >> p[1]) & 1;
                    F += s.A * a * b + s.B * (a + b);
                }
                if (F > best) {
                    second = best;
                    best = F;
                    at = c;
                } else if (F > second) {
                    second = F;
                }
            }
            const bool folds = best > second;
            none += !folds;
            const uint16_t phen = folds ? s.c2q[at] : uint16_t(HP_NONE);
            bad += out[i] != phen || emin[i] != s.e0 - best ||
                   gap[i] != uint8_t(best - second < 255 ? best - second : 255);
        }
        return bad + (none != nondesign);
    }
};

// a dense workgroup of Q TT 32 columns, with a ragged end
template <int KB, bool UN, int TT, int Q, int S>
int dense(const hp_structs &s, uint64_t lo, uint64_t seed)
{
    constexpr int kCols = Q * TT * 32;
    Run r(s, lo, kCols - 5);
    static ScanFrag<UN> frag[(S > 1 ? Q * TT : Q) * KB * 64];
    static ScanTop2 top[kCols];
    static unsigned del_sum;
    emu::run(64 * Q * S, seed, [&]() {
        scan_dense_body<KB, UN, TT, Q, S>(r.j, lo, frag, top, &del_sum, nullptr);
    });
    return r.wrong(s);
}

// a block of 1024 sequences, all but the first three
template <int KB, int G, int S>
int wide(const hp_structs &s, uint64_t blk, uint64_t seed)
{
    Run r(s, blk * 1024 + 3, 1021);
    static WideShared<KB, G, S> sh;
    emu::run(64 * wide_waves<G>() * S, seed, [&]() { wide_body<KB, G, S, 1>(r.j, blk, sh); });
    return r.wrong(s);
}

}  // namespace

int main()
{
    const int32_t pure[4] = {0, 0, 0, -1}, table[4] = {0, -1, -1, -3};
    hp_structs sp, st;
    std::string msg;
    if (build_structures(2, 3, 3, pure, &sp, &msg) != HP_OK ||
        build_structures(2, 3, 3, table, &st, &msg) != HP_OK || sp.scan_kb != 3 ||
        st.scan_kb != 2 || !sp.wide_ok || !st.wide_un) {
        std::printf("no structures: %s\n", msg.c_str());
        return 2;
    }
    int bad[7] = {};
    for (uint64_t r = 0; r < 40; ++r) {
        const uint64_t lo = (r * 104729 + 777) % ((1u << 18) - 64);
        bad[0] += dense<3, false, 1, 1, 16>(sp, lo, 4 * r);
        bad[1] += dense<3, false, 2, 1, 8>(sp, lo, 4 * r + 1);
        bad[2] += dense<2, true, 1, 1, 16>(st, lo, 4 * r + 2);
        bad[3] += dense<2, true, 2, 1, 8>(st, lo, 4 * r + 3);
    }
    for (uint64_t r = 0; r < 3; ++r) {
        const uint64_t blk = 71 * r + 29;
        bad[4] += wide<3, 0, 8>(sp, blk, 3 * r);
        bad[5] += wide<3, 0, 1>(sp, blk, 3 * r + 1);
        bad[6] += wide<3, 4, 4>(st, blk, 3 * r + 2);
    }
    std::printf("dense %d %d tables %d %d wide %d %d tables %d\n", bad[0], bad[1], bad[2], bad[3],
                bad[4], bad[5], bad[6]);
    return 0;
}
