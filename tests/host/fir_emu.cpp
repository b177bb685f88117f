// The general FIR kernel, run on the CPU: values and barriers of walks over several tiles.  Every output has to be the
// bits of a plain loop over its terms (the order the kernel states), whichever wave of a workgroup runs ahead.
#include <math.h>
#include <stdio.h>

#include "direct_kernels.hip"

static uint16_t to_bf16(float x) {  // round to nearest even, finite values
    const uint32_t u = __builtin_bit_cast(uint32_t, x);
    return (uint16_t)((u + 0x7fff + ((u >> 16) & 1)) >> 16);
}
extern "C" __bf16 __truncsfbf2(float x) { return __builtin_bit_cast(__bf16, to_bf16(x)); }  // the compiler's conversion

using namespace hy;

namespace {

uint32_t g_state = 1;
float draw() {
    g_state = g_state * 1664525u + 1013904223u;
    return (float)(int32_t)g_state * 4.6566129e-10f;
}
float bf16_value(float x) { return __builtin_bit_cast(float, (uint32_t)to_bf16(x) << 16); }

struct Tensor {  // [B, L, D]
    int64_t L, D;
    bool bf16;
    void* p;
    Tensor(int64_t B, int64_t L_, int64_t D_, bool bf) : L(L_), D(D_), bf16(bf), p(nullptr) {
        if (posix_memalign(&p, 64, (size_t)(B * L * D * (bf ? 2 : 4)))) abort();
        memset(p, 0xff, (size_t)(B * L * D * (bf ? 2 : 4)));  // NaN where a test leaves it
    }
    ~Tensor() { free(p); }
    float get(int64_t t, int64_t c) const {
        return bf16 ? __builtin_bit_cast(float, (uint32_t)static_cast<uint16_t*>(p)[t * D + c] << 16)
                    : static_cast<float*>(p)[t * D + c];
    }
    void set(int64_t t, int64_t c, float x) {
        if (bf16) static_cast<uint16_t*>(p)[t * D + c] = to_bf16(x);
        else static_cast<float*>(p)[t * D + c] = x;
    }
};

// All outputs of one workgroup of the second walk (the last, possibly ragged channel block), against the plain loop.
// `infinite`: the step, counted from the walk's first one in its direction, of a sample that is (kFinite: none).
constexpr int kFinite = 1 << 20;
int check(int64_t L, int64_t D, int lh, int group, bool bf16, bool rev, bool descending, int infinite) {
    FirProblem p;
    p.stride_ab = p.stride_gate = p.stride_out = L * D;
    p.lo = 0; p.hi = L; p.rev = rev;
    auto launch = [&] { return launch_fir(&p, 1, 1, L, D, lh, group, bf16 ? HY_BF16 : HY_F32, nullptr); };
    emu::wanted = [](dim3) { return false; };  // only the launch's grid
    if (launch() != HY_OK) return printf("launch\n"), 1;
    const bool pieces = bf16 && D % 8 == 0;  // rows of 16-byte bf16 pieces
    const int tile = lh <= 32 || (bf16 && !pieces && lh <= 128) ? 32 : pieces && lh <= 128 ? 64 : 128;
    const int64_t ncb = (D + 63) / 64, tiles = (L + tile - 1) / tile, walks = emu::grid_dim.x / ncb;
    const int64_t steps = (tiles + walks - 1) / walks;
    const int64_t c0 = (ncb - 1) * 64, t0 = steps * tile, t1 = 2 * steps * tile < L ? 2 * steps * tile : L;
    if ((steps < 3 && lh <= 128) || t1 - t0 != steps * tile) return printf("not the walk this is meant for\n"), 1;
    Tensor a(1, L, D, bf16), b(1, L, D, bf16), gate(1, L, D, bf16), out(1, L, D, bf16);
    float* h = static_cast<float*>(malloc((size_t)(D / group * lh * 4)));
    for (int64_t i = 0; i < D / group * lh; ++i) h[i] = draw();
    for (int64_t t = t0 > lh ? t0 - lh : 0; t < (t1 + lh < L ? t1 + lh : L); ++t)
        for (int64_t c = c0; c < D; ++c) {
            a.set(t, c, draw());
            b.set(t, c, draw());
            gate.set(t, c, draw());
        }
    if (infinite != kFinite) a.set(rev ? t1 - 1 - infinite : t0 + infinite, c0 + 5, INFINITY);
    p.a = a.p; p.b = b.p; p.h = h; p.gate = gate.p; p.out = out.p;
    const uint32_t n = emu::grid_dim.x, block = (uint32_t)(ncb + (ncb - 1));  // (in whichever order the launch has them)
    emu::wanted = [&](dim3 i) { return i.x == block || xcd_contiguous(i.x, n) == block; };
    emu::wave_order = [&](int i, int n) { return descending ? n - 1 - i : i; };
    if (launch() != HY_OK) return printf("launch\n"), 1;
    int64_t wrong = 0;
    for (int64_t t = t0; t < t1; ++t)
        for (int64_t c = c0; c < D; ++c) {
            float s = 0.0f;
            for (int i = 0; i < lh; ++i) {  // ascending tap (transposed) or source (causal) order
                const int j = rev ? i : lh - 1 - i;
                const int64_t src = rev ? t + j : t - j;
                if (src >= 0 && src < L) s = fmaf(h[c / group * lh + j], a.get(src, c) * b.get(src, c), s);
            }
            s *= gate.get(t, c);
            const float want = bf16 && isfinite(s) ? bf16_value(s) : s, got = out.get(t, c);
            wrong += isnan(want) ? !isnan(got) : !(want == got);
        }
    free(h);
    printf("L=%lld D=%lld lh=%d group=%d %s %s%s, %s wave first, %lld tiles: %lld of %lld outputs wrong\n", (long long)L,
           (long long)D, lh, group, bf16 ? "bf16" : "f32", rev ? "transposed" : "causal", infinite != kFinite ? ", one sample infinite" : "",
           descending ? "last" : "first", (long long)steps, (long long)wrong, (long long)((t1 - t0) * (D - c0)));
    return wrong != 0;
}

// Rows of a tile, by the launch's workgroups.
int check_rows(int64_t B, int64_t L, int64_t D, int lh, int rows) {
    Tensor a(1, 8, 8, true);
    FirProblem p;
    p.a = p.b = p.gate = p.out = a.p;
    p.h = static_cast<float*>(a.p);
    p.stride_ab = p.stride_gate = p.stride_out = L * D;
    p.lo = 0; p.hi = L; p.rev = false;
    emu::wanted = [](dim3) { return false; };
    if (launch_fir(&p, 1, B, L, D, lh, 1, HY_BF16, nullptr) != HY_OK) return printf("launch\n"), 1;
    const int64_t want = B * ((L + rows - 1) / rows) * ((D + 63) / 64), got = emu::grid_dim.x;
    printf("B=%lld L=%lld D=%lld lh=%d: %lld workgroups\n", (long long)B, (long long)L, (long long)D, lh, (long long)got);
    return got != want;
}

}  // namespace

int main() {
    int lost = 0;  // every tile once, whatever their number
    for (uint32_t n = 1; n < 700; ++n) {
        std::vector<int> seen(n, 0);
        for (uint32_t i = 0; i < n; ++i) {
            const uint32_t x = xcd_contiguous(i, n);
            if (x < n) ++seen[x];
        }
        for (uint32_t i = 0; i < n; ++i) lost += seen[i] != 1;
    }
    if (lost) printf("order of workgroups: %d tiles not once\n", lost);
    const int64_t L = 128 * 3 * 64 - 50;  // three tiles of 128 rows or more of 32 to a walk
    int bad = lost != 0;
    for (int lh : {12, 20, 40, 65, 128})  // one segment of 16, 32, 64, 128 taps
        for (int i = 0; i < 4; ++i) {
            const int64_t D = i / 2 ? 509 : 512;  // rows of single elements, of 16-byte pieces
            const int group = i / 2 ? 1 : 8;
            bad += check(L, D, lh, group, i % 2, lh == 40 || lh == 65, false, kFinite);
            bad += check(L, D, lh, group, i % 2, lh == 20 || lh == 128, true, kFinite);
        }
    bad += check(L, 512, 150, 8, true, false, false, kFinite);  // three segments of 64
    bad += check(L, 512, 200, 8, true, true, false, kFinite);   // two segments of 128
    bad += check(L, 509, 129, 1, false, true, true, kFinite);
    bad += check(L, 512, 128, 8, true, false, true, -3);
    bad += check(L, 512, 40, 1, false, true, false, -4);
    bad += check(L, 512, 150, 8, false, false, true, -3);
    // inside the walk's first 64-row tile, in reach of the third
    bad += check(L, 512, 128, 8, true, false, false, 60);
    bad += check(L, 512, 128, 8, true, true, true, 60);
    bad += check(L, 512, 64, 8, true, false, true, 63);
    // bf16 rows of whole pieces: 64-row tiles, 32-row ones where the compute units take no more turns for them
    bad += check_rows(1, 65, 1000, 33, 32);
    bad += check_rows(6, 158, 1000, 65, 32);
    bad += check_rows(2, 256, 1024, 64, 32);
    bad += check_rows(2, 288, 1024, 64, 64);
    bad += check_rows(6, 84, 2056, 50, 64);
    printf("fir emulation: %d problem(s)\n", bad);
    return bad != 0;
}
