// The general FIR on split bf16 products, run on the CPU: a workgroup's outputs against the sums in 64 bits, whichever wave
// runs ahead; small magnitudes; values that are not finite.
#include <math.h>
#include <stdio.h>

#include "split_kernels.hip"

// Round to nearest even.  (Not optimised: the compiler knows the idiom and would call its own conversion, which is this one.)
__attribute__((optnone)) static uint16_t to_bf16(float x) {
    const uint32_t u = __builtin_bit_cast(uint32_t, x);
    return (uint16_t)(x != x ? 0x7fc0 : (u + 0x7fff + ((u >> 16) & 1)) >> 16);
}
extern "C" __bf16 __truncsfbf2(float x) { return __builtin_bit_cast(__bf16, to_bf16(x)); }  // the compiler's conversion

namespace hy {
static bool g_general;  // a call came to the general kernel
hy_status launch_fir(const FirProblem*, int, int64_t, int64_t, int64_t, int32_t, int32_t, hy_dtype, hipStream_t) {
    g_general = true;
    return HY_OK;
}
}  // namespace hy

using namespace hy;

namespace {

uint32_t g_state = 1;
float draw() {
    g_state = g_state * 1664525u + 1013904223u;
    return (float)(int32_t)g_state * 4.6566129e-10f;
}

struct Tensor {  // [L, D]
    int64_t L, D;
    bool bf16;
    void* p;
    Tensor(int64_t L_, int64_t D_, bool bf) : L(L_), D(D_), bf16(bf), p(nullptr) {
        if (posix_memalign(&p, 64, (size_t)(L * D * (bf ? 2 : 4)))) abort();
        memset(p, 0xff, (size_t)(L * D * (bf ? 2 : 4)));  // NaN where a test leaves it
    }
    ~Tensor() { free(p); }
    float get(int64_t t, int64_t c) const {
        return bf16 ? __builtin_bit_cast(float, (uint32_t)static_cast<uint16_t*>(p)[t * D + c] << 16) : static_cast<float*>(p)[t * D + c];
    }
    void set(int64_t t, int64_t c, float x) {
        if (bf16) static_cast<uint16_t*>(p)[t * D + c] = to_bf16(x);
        else static_cast<float*>(p)[t * D + c] = x;
    }
};

struct Case {
    int64_t L, D;
    int lh, group;
    bool bf16, rev;
    float size = 1.0f;        // of a and b
    float tap = 1.0f;         // of the taps
    int64_t infinite = -1;    // the step of a sample that is (-1: none)
    int64_t huge = -1;        // the step of a finite one whose bf16 head is not
    bool two = false;         // a second gate and output
    int order = 0;            // the first wave to run: the first, the last, in between
};

// Every channel block and tile of a launch.
int check(const Case& k) {
    Tensor a(k.L, k.D, k.bf16), b(k.L, k.D, k.bf16), gate(k.L, k.D, k.bf16), gate2(k.L, k.D, k.bf16), out(k.L, k.D, k.bf16), out2(k.L, k.D, k.bf16);
    float* h = static_cast<float*>(malloc((size_t)(k.D / k.group * k.lh * 4)));
    for (int64_t i = 0; i < k.D / k.group * k.lh; ++i) h[i] = draw() * k.tap;
    for (int64_t t = 0; t < k.L; ++t)
        for (int64_t c = 0; c < k.D; ++c) {
            a.set(t, c, draw() * k.size);
            b.set(t, c, draw() * k.size);
            gate.set(t, c, draw());
            gate2.set(t, c, draw());
        }
    if (k.lh > k.L) h[k.lh - 1] = NAN;  // (meets no data)
    const int64_t bad_c = k.D - 3, huge_c = k.D / 2;
    if (k.infinite >= 0) a.set(k.infinite, bad_c, INFINITY);
    if (k.huge >= 0) {
        a.set(k.huge, huge_c, k.bf16 ? 1.8e19f : 3.4e38f);  // (bf16: the product of the two)
        b.set(k.huge, huge_c, k.bf16 ? 1.8875e19f : 1.0f);
        for (int j = 0; j < k.lh; ++j) h[huge_c / k.group * k.lh + j] *= 1e-3f;
    }
    FirProblem p;
    p.a = a.p; p.b = b.p; p.h = h; p.gate = gate.p; p.out = out.p;
    if (k.two) { p.gate2 = gate2.p; p.out2 = out2.p; }
    p.stride_ab = p.stride_gate = p.stride_out = k.L * k.D;
    p.lo = 0; p.hi = k.L; p.rev = k.rev;
    emu::wave_order = [&](int i, int n) { return k.order == 0 ? i : k.order == 1 ? n - 1 - i : (i + n / 2) % n; };
    if (launch_split_fir(&p, 1, 1, k.L, k.D, k.lh, k.group, k.bf16 ? HY_BF16 : HY_F32, nullptr) != HY_OK) return printf("launch\n"), 1;
    int64_t wrong = 0, count = 0, unlike = 0;  // unlike: bf16 outputs that are not the rounded sum
    double err = 0, all = 0;
    for (int64_t t = 0; t < k.L; ++t)
        for (int64_t c = 0; c < k.D; ++c) {
            double s = 0;
            for (int j = 0; j < k.lh; ++j) {
                const int64_t src = k.rev ? t + j : t - j;
                if (src >= 0 && src < k.L) s += (double)h[c / k.group * k.lh + j] * (double)(a.get(src, c) * b.get(src, c));
            }
            for (int o = 0; o <= k.two; ++o) {
                const float g = (o ? gate2 : gate).get(t, c), got = (o ? out2 : out).get(t, c);
                const double want = s * g;
                if (!isfinite(want) || !isfinite(got)) {
                    wrong += isfinite(want) != isfinite(got);
                    continue;
                }
                if (c / k.group == huge_c / k.group && k.huge >= 0) {
                    wrong += !(fabs(got - want) <= (k.bf16 ? 0x1p-7 : 1e-5) * fabs(want) + 1e-6);
                    continue;
                }
                if (k.bf16) {
                    unlike += __builtin_bit_cast(uint32_t, got) != (uint32_t)to_bf16((float)want) << 16;
                    wrong += !(fabs(got - want) <= 0x1.1p-8 * fabs(want) + 1e-6 * k.size * k.size * k.tap + 0x1p-134);  // (the last: half of the smallest bf16 step)
                }
                err += (got - want) * (got - want);
                all += want * want;
                ++count;
            }
        }
    free(h);
    // fp32: the gate's product and the sums' last addition round (4e-8 in the 2-norm together); the pieces not multiplied add
    // up to 2^-24 of a product at most, far less over many.  Such an error takes a bf16 output over the middle between two
    // values about once in 2^-8 / 7e-8 / 2, some 30 000.
    const double rel = sqrt(err / all);
    const bool bad = wrong || (k.bf16 ? unlike > 1 + count / 2000 : !(rel <= 7e-8));
    printf("L=%lld D=%lld lh=%d group=%d %s %s size %g, taps %g%s%s%s, order %d: error %.1e, %lld unlike, %lld wrong%s\n", (long long)k.L, (long long)k.D, k.lh,
           k.group, k.bf16 ? "bf16" : "f32", k.rev ? "transposed" : "causal", k.size, k.tap, k.infinite >= 0 ? ", infinite" : "",
           k.huge >= 0 ? ", huge" : "", k.two ? ", two" : "", k.order, rel, (long long)unlike, (long long)wrong, bad ? " <-" : "");
    return bad;
}

// The kernel that the dispatch takes for a forward call.
int check_route(int64_t B, int64_t L, int64_t D, int lh, int group, bool bf16, bool general) {
    ConvShape s;
    s.B = B; s.L = L; s.D = D; s.lh = lh; s.group = group; s.gated = true; s.dtype = bf16 ? HY_BF16 : HY_F32;
    float x = 0;
    const ConvPtrs p{&x, &x, &x, &x, &x};
    emu::wanted = [](dim3) { return false; };
    g_general = false;
    const hy_status rc = launch_direct(&p, 1, s, nullptr);
    emu::wanted = [](dim3) { return true; };
    const bool bad = rc != HY_OK || g_general != general;
    printf("B=%lld L=%lld D=%lld lh=%d group=%d %s: status %d, %s kernel%s\n", (long long)B, (long long)L, (long long)D, lh, group,
           bf16 ? "bf16" : "f32", (int)rc, g_general ? "general" : "this", bad ? " <-" : "");
    return bad;
}

}  // namespace

int main() {
    int bad = 0, i = 0;
    for (int group : {8, 16})
        for (bool bf16 : {false, true})
            for (int lh : {9, 34, 65, 98, 129}) {  // two source blocks to five
                Case k{i % 3 == 0 ? 300 : i % 3 == 1 ? 129 : 200, group == 8 ? 72 : 80, lh, group, bf16, i % 2 == 1};
                k.order = i % 3;
                k.two = i % 4 == 1;
                bad += check(k);
                k.infinite = k.L / 2 + 1;
                k.huge = 63;
                k.rev = !k.rev;
                bad += check(k);
                ++i;
            }
    // what is far below 1 keeps its bits (x = a*b down to 1e-36, sums that are normal numbers all the same)
    for (int group : {8, 16})
        for (bool bf16 : {false, true}) {
            bad += check({130, 16 + 2 * group, 128, group, bf16, false, 1e-17f});
            bad += check({130, 16 + 2 * group, 128, group, bf16, true, 2e-18f});
            bad += check({130, 16 + 2 * group, 40, group, bf16, false, 1.0f, 1e-35f});
            bad += check({130, 16 + 2 * group, 9, group, bf16, true, 1e-9f, 1e-17f});
        }
    // filters longer than their sequence
    bad += check({100, 72, 400, 8, false, false});
    bad += check({40, 80, 150, 16, true, true});
    bad += check({9, 72, 33, 8, false, true});
    bad += check_route(1, 128, 8, 9, 8, false, false);
    // as many workgroups as HIP takes threads for (fewer than 2^32), and more, which the general kernel's smaller ones may fit
    bad += check_route((1 << 23) - 1, 65, 8, 129, 8, false, false);
    bad += check_route(1 << 23, 65, 8, 129, 8, false, true);
    bad += check_route(10000000, 100, 8, 128, 8, true, true);
    // short sequences in several rounds of workgroups, by taps that meet data; one round
    for (bool bf16 : {false, true}) {
        bad += check_route(4096, 4, 1000, 128, 8, bf16, true);
        bad += check_route(1, 8, 64, 128, 8, bf16, true);
        bad += check_route(1, 9, 64, 128, 8, bf16, false);
        bad += check_route(512, 33, 1000, 128, 8, bf16, true);
        bad += check_route(17, 64, 1000, 129, 8, bf16, true);
        bad += check_route(16, 64, 1000, 129, 8, bf16, false);
        bad += check_route(17, 65, 1000, 129, 8, bf16, false);
        bad += check_route(17, 96, 1000, 64, 8, bf16, !bf16);
        bad += check_route(17, 97, 1000, 33, 8, bf16, false);
        // (up to 32 taps: few columns, long sequences, tiles that fill 78%, 67%, 64%, 52%, 36% of the chip's
        // time)
        bad += check_route(16, 320, 1000, 9, 8, bf16, false);
        bad += check_route(9, 400, 1000, 16, 8, bf16, true);
        bad += check_route(9, 400, 1000, 17, 8, bf16, false);
        bad += check_route(8, 400, 1000, 16, 8, bf16, false);
        bad += check_route(17, 256, 1000, 32, 8, bf16, true);
        bad += check_route(16, 600, 1000, 9, 8, bf16, false);
        bad += check_route(12, 1200, 1000, 9, 8, bf16, true);
        bad += check_route(17, 1535, 1000, 9, 8, bf16, false);
        bad += check_route(24, 400, 1000, 16, 8, bf16, true);
        bad += check_route(24, 400, 1000, 32, 8, bf16, false);
        bad += check_route(17, 300, 1000, 32, 8, bf16, true);
        bad += check_route(64, 128, 1000, 9, 8, bf16, !bf16);
        bad += check_route(64, 96, 1000, 9, 8, bf16, true);
        bad += check_route(12, 1536, 1000, 9, 8, bf16, false);
    }
    printf("split emulation: %d problem(s)\n", bad);
    return bad != 0;
}
