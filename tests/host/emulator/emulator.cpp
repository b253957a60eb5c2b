// Lanes as coroutines (see hip/hip_runtime.h beside this file).
#include <hip/hip_runtime.h>
#undef asm

#include <cmath>
#include <cstdio>
#include <random>
#include <ucontext.h>
#include <vector>

namespace emu {

unsigned lane_id;
dim3 block_dim, block_idx, grid_dim;

namespace {

constexpr size_t kStack = 128 << 10;
enum State { kReady, kAtWave, kAtBarrier, kDone };

struct Fiber {
    ucontext_t ctx;
    State state;
    int op;   // which wave operation it waits in
    // its operands and result
    uint64_t word, result;
    unsigned from;
    v8i a, b;
    v16f c;
    v4i ai, bi;
    v16i ci;
    int fmt_a, fmt_b, scale_a, scale_b;
};

std::vector<Fiber> fibers;
std::vector<char> stacks;
ucontext_t scheduler;
const std::function<void()> *work;

void entry()
{
    (*work)();
    fibers[lane_id].state = kDone;
    swapcontext(&fibers[lane_id].ctx, &scheduler);
}

Fiber &wait(State s, int op)
{
    Fiber &f = fibers[lane_id];
    f.state = s;
    f.op = op;
    swapcontext(&f.ctx, &scheduler);
    return f;   // fibers do not move while they run
}

float value(const v8i &v, int n, int fmt)
{
    if (fmt == 4) {   // E2M1
        static const float mag[8] = {0.f, 0.5f, 1.f, 1.5f, 2.f, 3.f, 4.f, 6.f};
        const unsigned code = (unsigned(v[n / 8]) >> (4 * (n % 8))) & 15u;
        return code & 8 ? -mag[code & 7] : mag[code & 7];
    }
    const int bit = 6 * n;   // E2M3
    uint64_t w = uint32_t(v[bit / 32]);
    if (bit / 32 < 7)
        w |= uint64_t(uint32_t(v[bit / 32 + 1])) << 32;
    const unsigned code = unsigned(w >> (bit % 32)) & 63u;
    const unsigned e = (code >> 3) & 3u, m = code & 7u;
    const float mag = e ? std::ldexp(1.f + m / 8.f, int(e) - 1) : m / 8.f;
    return code & 32 ? -mag : mag;
}

float scale(int s) { return std::ldexp(1.f, (s & 255) - 127); }

void product(Fiber *w)
{
    static float A[32][64], B[64][32];
    const bool scaled = w[0].scale_a != 0 || w[0].scale_b != 0;   // both 0: the unscaled form
    for (int l = 0; l < 64; ++l)
        for (int n = 0; n < 32; ++n) {
            const int k = 32 * (l / 32) + n;
            A[l % 32][k] = value(w[l].a, n, w[l].fmt_a) * (scaled ? scale(w[l].scale_a) : 1.f);
            B[k][l % 32] = value(w[l].b, n, w[l].fmt_b) * (scaled ? scale(w[l].scale_b) : 1.f);
        }
    for (int l = 0; l < 64; ++l)
        for (int q = 0; q < 16; ++q) {
            const int row = 8 * (q / 4) + 4 * (l / 32) + q % 4;
            double sum = w[l].c[q];
            for (int k = 0; k < 64; ++k)
                sum += double(A[row][k]) * B[k][l % 32];
            w[l].c[q] = float(sum);
        }
}

void product_i8(Fiber *w)
{
    static int A[32][32], B[32][32];
    for (int l = 0; l < 64; ++l)
        for (int n = 0; n < 16; ++n) {
            A[l % 32][16 * (l / 32) + n] = int8_t(uint32_t(w[l].ai[n / 4]) >> (8 * (n % 4)));
            B[16 * (l / 32) + n][l % 32] = int8_t(uint32_t(w[l].bi[n / 4]) >> (8 * (n % 4)));
        }
    for (int l = 0; l < 64; ++l)
        for (int q = 0; q < 16; ++q) {
            const int row = 8 * (q / 4) + 4 * (l / 32) + q % 4;
            int sum = w[l].ci[q];
            for (int k = 0; k < 32; ++k)
                sum += A[row][k] * B[k][l % 32];
            w[l].ci[q] = sum;
        }
}

void finish(Fiber *w)
{
    if (w[0].op == 0) {
        uint64_t m = 0;
        for (int l = 0; l < 64; ++l)
            m |= (w[l].word & 1) << l;
        for (int l = 0; l < 64; ++l)
            w[l].result = m;
    } else if (w[0].op == 1) {
        for (int l = 0; l < 64; ++l)
            w[l].result = w[w[l].from].word;
    } else if (w[0].op == 2) {
        product(w);
    } else {
        product_i8(w);
    }
}

}  // namespace

void workgroup_barrier() { wait(kAtBarrier, 0); }

uint64_t ballot(bool on)
{
    fibers[lane_id].word = on;
    return wait(kAtWave, 0).result;
}

uint64_t exchange(uint64_t own, unsigned from)
{
    fibers[lane_id].word = own;
    fibers[lane_id].from = from;
    return wait(kAtWave, 1).result;
}

v16f mfma_scale(const v8i &a, const v8i &b, const v16f &c, int fmt_a, int fmt_b, int scale_a,
                int scale_b)
{
    Fiber &f = fibers[lane_id];
    f.a = a, f.b = b, f.c = c;
    f.fmt_a = fmt_a, f.fmt_b = fmt_b, f.scale_a = scale_a, f.scale_b = scale_b;
    return wait(kAtWave, 2).c;
}

v16i mfma_i8(const v4i &a, const v4i &b, const v16i &c)
{
    Fiber &f = fibers[lane_id];
    f.ai = a, f.bi = b, f.ci = c;
    return wait(kAtWave, 3).ci;
}

unsigned byte_permute(unsigned upper, unsigned lower, unsigned select)
{
    const uint64_t bytes = uint64_t(upper) << 32 | lower;
    unsigned r = 0;
    for (int i = 0; i < 4; ++i) {
        const unsigned s = (select >> (8 * i)) & 255u;
        r |= (s < 8 ? unsigned(bytes >> (8 * s)) & 255u : 0u) << (8 * i);
    }
    return r;
}

v6u to_fp6(const v16f &even, const v16f &odd, float scale)
{
    v6u r = {};
    for (int n = 0; n < 32; ++n) {
        const float x = (n % 2 ? odd : even)[n / 2] / scale;
        const float m = std::fabs(x);
        unsigned code = m < 2.f   ? unsigned(std::nearbyint(m * 8.f))
                        : m < 4.f ? 16u + unsigned(std::nearbyint((m - 2.f) * 4.f))
                                  : 24u + unsigned(std::nearbyint((m - 4.f) * 2.f));
        code = std::min(code, 31u) | (x < 0 ? 32u : 0u);
        const int bit = 6 * n;
        r[bit / 32] |= code << (bit % 32);
        if (bit % 32 > 26)
            r[bit / 32 + 1] |= code >> (32 - bit % 32);
    }
    return r;
}

void run(unsigned threads, uint64_t seed, const std::function<void()> &body)
{
    block_dim = dim3(threads);
    work = &body;
    fibers.resize(threads);
    stacks.resize(threads * kStack);
    for (unsigned i = 0; i < threads; ++i) {
        Fiber &f = fibers[i];
        f.state = kReady;
        getcontext(&f.ctx);
        f.ctx.uc_stack.ss_sp = stacks.data() + i * kStack;
        f.ctx.uc_stack.ss_size = kStack;
        f.ctx.uc_link = &scheduler;
        makecontext(&f.ctx, entry, 0);
    }
    std::mt19937_64 rng(seed);
    std::vector<unsigned> ready(threads);
    for (unsigned i = 0; i < threads; ++i)
        ready[i] = i;
    std::vector<unsigned> waiting(threads / 64, 0);
    unsigned at_barrier = 0, done = 0;
    while (done < threads) {
        if (ready.empty()) {
            if (at_barrier + done != threads) {
                std::fprintf(stderr, "lanes of a wave part at an operation\n");
                std::abort();
            }
            for (unsigned i = 0; i < threads; ++i)
                if (fibers[i].state == kAtBarrier) {
                    fibers[i].state = kReady;
                    ready.push_back(i);
                }
            at_barrier = 0;
        }
        const size_t pick = rng() % ready.size();
        lane_id = ready[pick];
        ready[pick] = ready.back();
        ready.pop_back();
        Fiber &f = fibers[lane_id];
        const unsigned wave = lane_id / 64;
        swapcontext(&scheduler, &f.ctx);
        if (f.state == kDone) {
            ++done;
        } else if (f.state == kAtBarrier) {
            ++at_barrier;
        } else if (++waiting[wave] == 64) {
            waiting[wave] = 0;
            Fiber *w = &fibers[wave * 64];
            for (int l = 1; l < 64; ++l)
                if (w[l].op != w[0].op) {
                    std::fprintf(stderr, "lanes of a wave in different operations\n");
                    std::abort();
                }
            finish(w);
            for (int l = 0; l < 64; ++l) {
                w[l].state = kReady;
                ready.push_back(wave * 64 + unsigned(l));
            }
        }
    }
}

}  // namespace emu
