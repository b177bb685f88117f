// The grouped Hyena-MR backward, run on the CPU: gradients of batches whose tiles run on from one item into the next, and rows
// of 2^24 bytes and more, whose tensors lie between pages that may not be touched.
#include <math.h>
#include <stdio.h>
#include <sys/mman.h>

#include "mr_bwd_kernels.hip"

// Round to nearest even, finite values.  (Not optimised: the compiler knows the idiom and would call its own conversion.)
__attribute__((optnone)) static uint16_t to_bf16(float x) {
    const uint32_t u = __builtin_bit_cast(uint32_t, x);
    return (uint16_t)((u + 0x7fff + ((u >> 16) & 1)) >> 16);
}
extern "C" __bf16 __truncsfbf2(float x) { return __builtin_bit_cast(__bf16, to_bf16(x)); }  // the compiler's conversion

namespace hy {
static DhReduce g_reduce;
const Tuning& tuning() {
    static const Tuning t;
    return t;
}
hy_status launch_dh_reduce(const DhReduce* items, int, hipStream_t) {
    g_reduce = items[0];
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
float value(uint16_t x) { return __builtin_bit_cast(float, (uint32_t)x << 16); }
float bf16_value(float x) { return value(to_bf16(x)); }

// n bytes (only what is touched takes memory) that begin behind one guard of `guard` bytes and end before another
struct Guarded {
    char* base;
    size_t size, guard;
    char* p;
    Guarded(size_t n, size_t guard_) : size((n + 4095) / 4096 * 4096), guard((guard_ + 4095) / 4096 * 4096) {
        base = static_cast<char*>(mmap(nullptr, size + 2 * guard, PROT_NONE, MAP_PRIVATE | MAP_ANONYMOUS | MAP_NORESERVE, -1, 0));
        if (base == MAP_FAILED) abort();
        p = base + guard;
        if (size && mprotect(p, size, PROT_READ | PROT_WRITE)) abort();
    }
    ~Guarded() { munmap(base, size + 2 * guard); }
};

// One block of 64 channels, every tile, against the sums in 64 bits of the operands as the kernel rounds them.
int check(int64_t B, int64_t L, int64_t D, int lh, int64_t block, bool across = false) {
    printf("B=%lld L=%lld D=%lld lh=%d, channels %lld on: ", (long long)B, (long long)L, (long long)D, lh, (long long)(64 * block));
    fflush(stdout);  // (a read out of range ends the program)
    const int group = 16;
    const size_t bytes = (size_t)(B * L * D * 2), guard = (size_t)D * 2 * 32;  // (a chunk of rows)
    Guarded in[4] = {{bytes, guard}, {bytes, guard}, {bytes, guard}, {bytes, guard}}, out[3] = {{bytes, guard}, {bytes, guard}, {bytes, guard}};
    BwdShape s;
    s.B = B; s.L = L; s.D = D; s.lh = lh; s.group = group; s.dtype = HY_BF16;
    Guarded table((size_t)(D / group * lh * 4), 4096), ws((size_t)mr_bwd_workspace_bytes(s), 4096);
    const int64_t c0 = 64 * block, n = 64;
    float* h = reinterpret_cast<float*>(table.p);
    for (int64_t g = c0 / group; g < (c0 + n) / group; ++g)
        for (int j = 0; j < lh; ++j) h[g * lh + j] = bf16_value(draw());
    auto at = [&](const Guarded& x, int64_t r, int64_t c) -> uint16_t& { return reinterpret_cast<uint16_t*>(x.p)[r * D + c]; };
    for (auto& x : in)
        for (int64_t r = 0; r < B * L; ++r)
            for (int64_t c = c0; c < c0 + n; ++c) at(x, r, c) = to_bf16(draw());
    BwdPtrs p{in[0].p, in[1].p, in[2].p, in[3].p, h, out[0].p, out[1].p, out[2].p, nullptr};
    const int64_t ncb = D / 64;
    emu::wanted = [&](dim3 i) { return i.x % ncb == block; };
    if (tiling(s).across != across) return printf("not the tiles this is meant for\n"), 1;
    if (launch_mr_bwd(p, s, ws.p, nullptr) != HY_OK) return printf("launch\n"), 1;
    auto product = [&](int a, int b, int64_t r, int64_t c) { return (double)bf16_value(value(at(in[a], r, c)) * value(at(in[b], r, c))); };
    int64_t wrong = 0;
    auto compare = [&](double got, double want, double size, double rel) { wrong += !(fabs(got - want) <= rel * fabs(want) + 1e-5 * size); };
    for (int64_t c = c0; c < c0 + n; ++c)
        for (int64_t b = 0; b < B; ++b)
            for (int64_t t = 0; t < L; ++t) {
                double z = 0, du = 0;
                for (int64_t j = 0; j < lh; ++j) {
                    const double tap = h[c / group * lh + j];
                    if (t >= j) z += tap * product(2, 3, b * L + t - j, c);
                    if (t + j < L) du += tap * product(0, 1, b * L + t + j, c);
                }
                const int64_t r = b * L + t;
                compare(value(at(out[0], r, c)), z * value(at(in[0], r, c)), 1, 0x1p-8);
                compare(value(at(out[1], r, c)), du * value(at(in[3], r, c)), 1, 0x1p-8);
                compare(value(at(out[2], r, c)), du * value(at(in[2], r, c)), 1, 0x1p-8);
            }
    for (int64_t x = c0 / 16; x < (c0 + n) / 16; ++x)  // (a group is one row of partial sums)
        for (int64_t j = 0; j < lh; ++j) {
            double got = 0, want = 0;
            for (int64_t i = 0; i < g_reduce.nsets; ++i) got += g_reduce.partial[(i * g_reduce.rows + x) * lh + j];
            for (int64_t c = 16 * x; c < 16 * x + 16; ++c)
                for (int64_t b = 0; b < B; ++b)
                    for (int64_t t = j; t < L; ++t) want += product(2, 3, b * L + t - j, c) * product(0, 1, b * L + t, c);
            compare(got, want, sqrt((double)(B * L)), 1e-5);
        }
    printf("%lld sets, %lld values wrong\n", (long long)g_reduce.nsets, (long long)wrong);
    return wrong != 0;
}

}  // namespace

int main() {
    int bad = 0;
    bad += check(1, 45, 64, 33, 0);
    bad += check(3, 300, 2048, 128, 31);
    bad += check(3, 250, 8192, 128, 127, true);  // tiles across items: one that begins inside an item,
    bad += check(5, 70, 4096, 33, 0, true);      // ... between two items,
    bad += check(3, 129, 8192, 129, 5, true);    // ... items of four chunks and a step
    // rows of 2^24 bytes and more: a last chunk that is not whole, in front of which no row lies
    for (int64_t D : {(1 << 23) - 64, 1 << 23, (1 << 23) + 64, (1 << 24) + 64}) {
        bad += check(1, 33, D, 9, 0);
        bad += check(1, 33, D, 9, D / 64 - 1);
    }
    bad += check(2, 5, 1 << 23, 40, 1);
    printf("MR backward emulation: %d problem(s)\n", bad);
    return bad != 0;
}
