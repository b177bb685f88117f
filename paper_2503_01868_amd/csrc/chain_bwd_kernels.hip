// Backward of the whole operator chain, q' = hq * q, k' = hk * k, v' = hv * v, y = q' (.) (h * (k' (.) v')) (Eq. 1), for
// medium grouped bf16 filters on the gfx950 matrix cores, ONE pass over the tensors: dy, q, k, v are read once and dq, dk, dv
// written once, where the composition featurizers - inner backward - featurizer gradients makes 22 tensor passes.
//
// With u = k'v', g = dy q':
//     z = h * u, dq' = dy z;  du[s] = sum_j h[j] g[s+j], dk' = du v', dv' = du k';  dh[j] = sum g[t] u[t-j]
//     dx[s] = sum_j hx[j] dx'[s+j],  dhx[j] = sum_t dx'[t] x[t-j]                     for x = q, k, v
// The kernel walks the sequence from its end, tau = L-1-t, in chunks of 32 steps.  There du and the dx are causal, z and the
// featurizers anti-causal: the featurizers look 8 steps ahead, z of a chunk is complete LAG = NKB - 1 chunks later
// (mr_bwd_kernels.hip), and dx of a chunk needs the dx' of the 8 steps before it, so a tile computes du and z from one chunk
// before its first one on.
//
// A workgroup owns 64 channels with 12 waves, three per SIMD and of three kinds:
//  * four move all data and run the featurizers: per channel and 16 steps, X'[i][j] = sum_m sum_k B_m[i][k] x[tau0+4j+4m+k],
//    B_m[i][k] = hx[4m+k-i], as batched 4 x 4 x 4 products (v_mfma_f32_4x4x4_16B_bf16, one channel per block), a tap as a bf16
//    head plus a bf16 remainder;
//  * four run du of 16 channels each as block-Toeplitz products (v_mfma_f32_16x16x32_bf16, operands and source window in
//    registers, steps x channels) and then, per channel again, dk and dv, DX[i][j] = sum_m sum_k A_m[i][k]
//    dx'[tau0+4j-4m+k], A_m[i][k] = hx[4m+i-k], and the featurizers' filter gradients, D[i][j] += sum_k H[i][k]
//    dx'[T+k-4(3-j)], H[i][k] = x[T+i+k]: entry (i, j) collects the lag 4(3-j)+i;
//  * four run z in the same way, then dq, and the inner filter gradient as products over channels
//    (v_mfma_f32_16x16x16_bf16, operands read transposed).
// The intermediates enter products rounded to bf16 (u, g, dx', and k', v' as gates) and are otherwise fp32 on chip.  A product
// also multiplies its structural zeros, so a value that is not finite would reach 3 steps to the wrong side of a featurizer and up
// to 11 to the other; a lane whose featurizer products gave such a value takes its steps term by term instead (1 to 2% of the
// time, most of it the test for it; doing the same for the inner filter, whose blocks are 32 steps, would not fit the registers).
//
// Everything lies in one 2400-byte LDS record per channel, time contiguous.  Results take the place of what is dead: dk, dv
// that of the raw k, v of their chunk, dq that of the raw q (rings of 8 chunks for q and dy, which wait for z, and of 4 for k
// and v).  In iteration j the first kind stores dk, dv of chunk j-1 and dq of chunk j-1-LAG, writes the raw chunk j+3 into the
// same places and runs the featurizers of chunk j+1; the second runs chunk j and the third z, dq of chunk j-LAG; one barrier.
//
// What bounds it: 7 tensor passes through 128-byte row pieces (98 us at the rate of a large copy), and the LDS, whose pipe is
// the busiest unit on chip (42% of the time at 1 x 8192 x 4096, 55% at 4 x 32768 x 4096; vector ALUs 37 and 47%, matrix cores 25
// and 35%): every value crosses it several times.  128 and 7 taps, whole call: 1 x 8192 x 4096 301 us as a composition, 140 here;
// 4 x 32768 x 4096 4448 -> 1953.  On the way there, before values that are not finite had a path of their own: 8 waves of two
// kinds 162 us (too few waves to cover LDS latency between dependent products), twelve 156, record skews that keep the three
// ways of reading apart 143, whole quads instead of each row's own dwords for H 139, transposed instead of 2-byte reads for the
// filter gradient 135.
#include <type_traits>

#include "hy_common.hpp"
#include "hy_launch.hpp"

namespace hy {
namespace {

typedef short s16x4_t __attribute__((ext_vector_type(4)));
// LDS is read and written in several widths by the same lane
typedef uint32_t __attribute__((may_alias)) lds1_t;
typedef uint32_t lds2_t __attribute__((ext_vector_type(2), may_alias));
typedef uint32_t lds4_t __attribute__((ext_vector_type(4), may_alias));
typedef uint16_t __attribute__((may_alias)) lds16_t;

struct ChainBwdArgs {
    const uint16_t* in[4];    // q, k, v, dy
    const float* hx[3];       // hq, hk, hv
    const float* h;
    uint16_t* out[3];         // dq, dk, dv
    float* partial;           // dh: [B * tiles_per_seq][D / 16][lh]
    float* partial_x[3];      // dhq, dhk, dhv: [B * tiles_per_seq][D][lf]
    int64_t L, D;
    int32_t lf, feat_group, lh, group;
    int32_t rows;           // time steps per workgroup, multiple of 32
    int32_t tiles_per_seq;  // ceil(L / rows)
    int32_t ncb;            // channel blocks = D / 64
};

constexpr int kT = 32;        // steps per chunk
constexpr int kNW = 4;        // waves of each kind per workgroup
constexpr int kKinds = 3;
constexpr int kC = 16 * kNW;  // channels per workgroup
constexpr int kSlot = 2 * kT;  // bytes of a chunk
constexpr int kMaxLf = 8;

// A channel's record: rings of raw chunks (each with a copy of its first 8 steps behind it, for reads across its end),
// g, u, k', v' of two chunks, and dx' of one chunk with the 16 steps before it in front.  The stride is an odd multiple of 32
// bytes: 8 neighbouring channels' pieces of 32 bytes meet every bank.  Every 8 records start 48 bytes further, so that one
// piece of 8 bytes of 16 neighbouring channels does too (with 32 they met half of the banks twice, 13 us).
constexpr int kBack = 16;
constexpr int kQ = 0, kK = kQ + 8 * kSlot + kBack, kV = kK + 4 * kSlot + kBack, kY = kV + 4 * kSlot + kBack;
constexpr int kG = kY + 8 * kSlot, kU = kG + 2 * kSlot, kKf = kU + 2 * kSlot, kVf = kKf + 2 * kSlot;
constexpr int kFront = 32;
constexpr int kDx = kVf + 2 * kSlot, kDxSize = kFront + kSlot;  // q, k, v
constexpr int kRec = 2400;
static_assert(kDx + 3 * kDxSize <= kRec && kRec % 16 == 0 && kRec % 64 == 32, "record layout");
__device__ __forceinline__ int rec(int c) { return c * kRec + (c >> 3) * 48; }
constexpr int kRecs = kC * kRec + kC / 8 * 48;

struct Quad {  // 4 steps of a channel: two dwords, step 0 in the low half of the first
    uint32_t w[2];
};
__device__ __forceinline__ s16x4_t operand(const Quad& x) { return __builtin_bit_cast(s16x4_t, x); }
__device__ __forceinline__ Quad quad_at(const char* p) { return __builtin_bit_cast(Quad, *reinterpret_cast<const lds2_t*>(p)); }
__device__ __forceinline__ void put_quad(char* p, const Quad& x) { *reinterpret_cast<lds2_t*>(p) = __builtin_bit_cast(lds2_t, x); }
__device__ __forceinline__ Quad pack_quad(const f32x4_t& x) { return Quad{{pack_bf16x2(x[0], x[1]), pack_bf16x2(x[2], x[3])}}; }
__device__ __forceinline__ f32x4_t unpack_quad(const Quad& x) {
    return f32x4_t{bf16_lo(x.w[0]), bf16_hi(x.w[0]), bf16_lo(x.w[1]), bf16_hi(x.w[1])};
}
// z, or not zero any more if one of the four steps is not finite
__device__ __forceinline__ float probe(float z, const Quad& x) {
    typedef __bf16 bf16x2_t __attribute__((ext_vector_type(2)));
#pragma unroll
    for (int i = 0; i < 2; ++i)
        z = __builtin_amdgcn_fdot2_f32_bf16(__builtin_bit_cast(bf16x2_t, x.w[i]), __builtin_bit_cast(bf16x2_t, 0u), z, false);
    return z;
}
// four taps as bf16 heads and remainders
__device__ __forceinline__ void split_taps(const float (&t)[4], s16x4_t (&o)[2]) {
    const Quad head = pack_quad(f32x4_t{t[0], t[1], t[2], t[3]});
    const f32x4_t h = unpack_quad(head);
    o[0] = operand(head);
    o[1] = operand(pack_quad(f32x4_t{t[0] - h[0], t[1] - h[1], t[2] - h[2], t[3] - h[3]}));
}

template <int NKB>
__global__ __launch_bounds__(kKinds * kNW * 64, kKinds) void chain_bwd_kernel(ChainBwdArgs a) {
    constexpr int LAG = NKB - 1;     // chunks between a chunk's arrival and its complete z
    constexpr int ND = 2 * NKB - 1;  // 16-step offsets x with a tap 16 x + i - n inside [0, lh)
    constexpr int kTaps = 32 * NKB;
    constexpr int NF = 3;            // quads a featurizer spans
    constexpr int PF = 2;            // chunks of loads in flight
    static_assert(LAG >= 1 && LAG <= 4, "the rings of q and dy hold 8 chunks: j - LAG .. j + 3");
    __shared__ __attribute__((aligned(16))) char lds[kRecs];
    __shared__ float hs[kNW][kTapPad + kTaps];
    __shared__ float fold[kNW][16 * 17];

    const int tid = threadIdx.x;
    const int wave = __builtin_amdgcn_readfirstlane(tid / 64), lane = tid % 64;
    const int w = wave % kNW;  // channels 16 w .. 16 w + 15 of the block
    const uint32_t lb = blockIdx.x;
    const int cb = lb % (uint32_t)a.ncb;
    const uint32_t tile = lb / (uint32_t)a.ncb;
    const int64_t b = tile / (uint32_t)a.tiles_per_seq;
    // everything below is in reversed time tau = L - 1 - t
    const int L = (int)a.L;
    const int t_start = (int)(tile % (uint32_t)a.tiles_per_seq) * a.rows;
    const int t_end = ((int64_t)t_start + a.rows < a.L) ? t_start + a.rows : L;
    const int t_ext = t_start - kT > 0 ? t_start - kT : 0;                    // dx' from here on
    const int t_begin = t_ext - kT * LAG > 0 ? t_ext - kT * LAG : 0;          // g from here on
    const int ntot = (t_end - t_begin + kT - 1) / kT + LAG;
    const int64_t D = a.D;
    const int64_t cblock0 = (int64_t)cb * kC;
    const int64_t seq0 = b * a.L * D + cblock0;
    auto chunk_start = [&](int j) { return t_begin + j * kT; };
    auto in_tile = [&](int j) { return chunk_start(j) >= t_start && chunk_start(j) < t_end; };
    auto in_ext = [&](int j) { return chunk_start(j) >= t_ext && chunk_start(j) < t_end; };
    using std::integral_constant;

    const int blk = lane >> 2, l4 = lane & 3;  // 4 x 4 x 4 products: block = channel, row i / column j
    auto tap_at = [&](const float* hp, int j) { return (uint32_t)j < (uint32_t)a.lf ? hp[j] : 0.0f; };
    auto feat_row = [&](int x) {
        return a.hx[x] + (int64_t)(((uint32_t)cblock0 + 16 * w + blk) / (uint32_t)a.feat_group) * a.lf;
    };

    char* const rc4 = lds + rec(16 * w + blk) + 8 * l4;
    const int li = lane % 16, lq = lane / 16;  // 16 x 16 products
    char* const rc16 = lds + rec(16 * w + li);  // steps x channels: column = channel

    // operands of the featurizers' gradients
    auto grad_taps = [&](int x, s16x4_t (&fa)[NF][2]) {
        const float* hp = feat_row(x);
#pragma unroll
        for (int m = 0; m < NF; ++m) {
            float t4[4];
#pragma unroll
            for (int k = 0; k < 4; ++k) t4[k] = tap_at(hp, 4 * m + l4 - k);
            split_taps(t4, fa[m]);
        }
    };
    // the last 16 steps of dx' move in front of the next chunk's
    auto keep_last = [&](int x) { put_quad(rc4 + kDx + x * kDxSize, quad_at(rc4 + kDx + x * kDxSize + kSlot)); };
    // 20 steps of the raw x from byte `at` of the record on, for H: the same quads in all lanes of a channel (a read of
    // each row's own dwords instead takes twice the LDS cycles), of which rows 2 and 3 start one dword later and odd rows
    // one step
    struct Steps {
        Quad q[5];
    };
    auto read_steps = [&](int at) {
        Steps r;
#pragma unroll
        for (int i = 0; i < 5; ++i) r.q[i] = quad_at(rc4 - 8 * l4 + at + 8 * i);
        return r;
    };
    struct Shifts {
        s16x4_t w[4];  // quads of dx', shift i: column j holds quad j - i
    };
    auto read_shifts = [&](int x, int n) {
        Shifts r;
#pragma unroll
        for (int i = 0; i < 4; ++i) r.w[i] = operand(quad_at(rc4 + kDx + x * kDxSize + kFront + 32 * n - 8 * i));
        return r;
    };
    // dx of 16 steps and their share of its filter gradient.  `first`: the walk's first steps, where the quad before them, column
    // 2 of the first product, is no steps of the sequence: its zeros are not multiplied with x
    auto unit = [&](const s16x4_t (&fa)[NF][2], const Steps& x, const Shifts& r, bool first, f32x4_t& facc) {
        const uint32_t sh = (l4 & 1) * 16;
        f32x4_t dx = {0.0f, 0.0f, 0.0f, 0.0f};
        uint32_t d[9];
#pragma unroll
        for (int i = 0; i < 9; ++i) d[i] = l4 < 2 ? x.q[i >> 1].w[i & 1] : x.q[(i + 1) >> 1].w[(i + 1) & 1];
        auto dh_product = [&](int kq) {
            const Quad hk{{__builtin_amdgcn_alignbit(d[2 * kq + 1], d[2 * kq], sh),
                           __builtin_amdgcn_alignbit(d[2 * kq + 2], d[2 * kq + 1], sh)}};
            const f32x4_t sum = __builtin_amdgcn_mfma_f32_4x4x4bf16_1k(operand(hk), r.w[3 - kq], facc, 0, 0, 0);
            if (kq > 0 || !first || l4 == 3) facc = sum;
        };
        auto dx_product = [&](int m, int part) { dx = __builtin_amdgcn_mfma_f32_4x4x4bf16_1k(fa[m][part], r.w[m], dx, 0, 0, 0); };
        dx_product(2, 1); dh_product(0);
        dx_product(1, 1); dh_product(1);
        dx_product(0, 1); dh_product(2);
        dx_product(2, 0); dh_product(3);
        dx_product(1, 0);
        dx_product(0, 0);
        return pack_quad(dx);
    };
    // the lane holds dhx[c][4 (3 - l4) + i], i = 0..3
    auto store_featurizer_dh = [&](int x, const f32x4_t& facc) {
        float* out = a.partial_x[x] + ((int64_t)tile * D + cblock0 + 16 * w + blk) * a.lf;
#pragma unroll
        for (int i = 0; i < 4; ++i)
            if (4 * (3 - l4) + i < a.lf) out[4 * (3 - l4) + i] = facc[i];
    };
    // ---- the definition's terms alone, one by one with fp32 taps, for a lane whose products gave something that is not finite:
    // a product also multiplies its structural zeros, and the remainder of an infinite tap is none.  (What this needs beside
    // its arguments is formed from a value that the compiler cannot move out of the rare branch.)
    auto taps_of = [&](int x) {
        int c = 16 * w + blk;
        asm volatile("" : "+v"(c));
        return a.hx[x] + (int64_t)(((uint32_t)cblock0 + c) / (uint32_t)a.feat_group) * a.lf;
    };
    auto step_at = [&](int at) { return bf16_lo(*reinterpret_cast<const lds16_t*>(rc4 + at)); };
    auto put_step = [&](int at, float x) { *reinterpret_cast<lds16_t*>(rc4 + at) = (uint16_t)pack_bf16x2(x, 0.0f); };
    auto exact_dx = [&](int x, int at) {  // of the lane's steps of a chunk
        const float* const hp = taps_of(x);
#pragma unroll 1
        for (int o = 0; o < kSlot; o = (o & 7) == 6 ? o + 26 : o + 2) {
            float sum = 0.0f;
#pragma unroll 1
            for (int j = 0; j < a.lf; ++j) sum = __builtin_fmaf(hp[j], step_at(kDx + x * kDxSize + kFront + o - 2 * j), sum);
            put_step(at + o, sum);
        }
    };
    // body(slot, j) for the chunks j = 0 .. ntot - 1, slot = j % 8; then last(slot, ntot)
    auto walk = [&](auto&& body, auto&& last) {
#define HY_STEP(S)                                                  \
    body(integral_constant<int, S>{}, j + S);                       \
    if (j + S + 1 >= ntot) {                                        \
        last(integral_constant<int, (S + 1) & 7>{}, j + S + 1);     \
        break;                                                      \
    }
        for (int j = 0;; j += 8) {
            HY_STEP(0) HY_STEP(1) HY_STEP(2) HY_STEP(3) HY_STEP(4) HY_STEP(5) HY_STEP(6) HY_STEP(7)
        }
#undef HY_STEP
    };
    auto nothing = [](auto, int) {};
    const f32x4_t zero4 = {0.0f, 0.0f, 0.0f, 0.0f};

    if (wave < kNW) {
        // ================= du, dk, dv
        s16x4_t fa[2][NF][2];
#pragma unroll
        for (int x = 0; x < 2; ++x) {
            grad_taps(1 + x, fa[x]);
            put_quad(rc4 + kDx + (1 + x) * kDxSize + kSlot, Quad{{0u, 0u}});  // the chunk before the first: no steps
        }
        stage_filter<kTaps>(hs[w], a.h + (int64_t)(((uint32_t)cblock0 + 16 * w) / (uint32_t)a.group) * a.lh, a.lh, lane);
        __syncthreads();
        bf16x8_t tz[2 * NKB];
        toeplitz_operands(tz, hs[w], li, lq);
        bf16x8_t gw[8];  // g of chunk c in gw[c % 8]: steps 8 lq .. of channel li
#pragma unroll
        for (int x = 0; x < 8; ++x) gw[x] = __builtin_bit_cast(bf16x8_t, zero_words<4>());
        f32x4_t facc[2] = {zero4, zero4};

        __syncthreads();  // the featurizers' results of chunk 0 are there
        walk([&](auto slot_c, int j) {
            constexpr int SL = decltype(slot_c)::value;
            constexpr int two = (SL & 1) * kSlot;  // g, u, k', v'
            constexpr int at[2] = {kK + (SL & 3) * kSlot, kV + (SL & 3) * kSlot};
            gw[SL] = __builtin_bit_cast(bf16x8_t, *reinterpret_cast<const lds4_t*>(rc16 + kG + two + 16 * lq));
            if (in_ext(j)) {
                Quad kf[2], vf[2];
#pragma unroll
                for (int p = 0; p < 2; ++p) {
                    kf[p] = quad_at(rc16 + kKf + two + 32 * p + 8 * lq);
                    vf[p] = quad_at(rc16 + kVf + two + 32 * p + 8 * lq);
                }
                keep_last(1);
                keep_last(2);
                Steps steps[2];
                steps[0] = read_steps(at[0]);
                __builtin_amdgcn_sched_barrier(0);
                f32x4_t acc[2] = {zero4, zero4};
#pragma unroll
                for (int m = NKB - 1; m >= 0; --m)
#pragma unroll
                    for (int p = 0; p < 2; ++p)
                        acc[p] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(tz[2 * m + p], gw[(SL - m) & 7], acc[p], 0, 0, 0);
#pragma unroll
                for (int p = 0; p < 2; ++p) {
                    put_quad(rc16 + kDx + kDxSize + kFront + 32 * p + 8 * lq, pack_quad(acc[p] * unpack_quad(vf[p])));
                    put_quad(rc16 + kDx + 2 * kDxSize + kFront + 32 * p + 8 * lq, pack_quad(acc[p] * unpack_quad(kf[p])));
                }
                if (in_tile(j)) {
                    // four units of 16 steps of a tensor, the next one's reads under way during one's products
                    Shifts sh[2];
                    float z[2] = {0.0f, 0.0f};
                    sh[0] = read_shifts(1, 0);
#pragma unroll
                    for (int un = 0; un < 4; ++un) {
                        const int x = un >> 1, n = un & 1;
                        __builtin_amdgcn_sched_barrier(0);
                        if (un < 3) {
                            steps[(un + 1) & 1] = read_steps(at[(un + 1) >> 1] + 32 * ((un + 1) & 1));
                            sh[(un + 1) & 1] = read_shifts(1 + ((un + 1) >> 1), (un + 1) & 1);
                        }
                        const Quad dx = unit(fa[x], steps[un & 1], sh[un & 1], n == 0 && chunk_start(j) == 0, facc[x]);
                        put_quad(rc4 + at[x] + 32 * n, dx);
                        z[x] = probe(z[x], dx);
                    }
#pragma unroll
                    for (int x = 0; x < 2; ++x)
                        if (__builtin_expect(!(z[x] == 0.0f), 0)) exact_dx(1 + x, at[x]);
                }
            }
            __syncthreads();
        }, nothing);
        store_featurizer_dh(1, facc[0]);
        store_featurizer_dh(2, facc[1]);
    } else if (wave < 2 * kNW) {
        // ================= z, dq, dh
        // 16 steps of the 16 channels, read transposed: this lane gets step li of the channels 4 lq .. 4 lq + 3 (each lane
        // addresses 4 steps of channel lane / 4)
        auto across = [&](int at) {
            typedef __attribute__((address_space(3))) s16x4_t lds_quad_t;
            return __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_quad_t*)(rc4 + at));
        };
        s16x4_t fa[NF][2];
        grad_taps(0, fa);
        put_quad(rc4 + kDx + kSlot, Quad{{0u, 0u}});  // the chunk before the first: no steps
        __syncthreads();
        bf16x8_t tz[2 * NKB];
        toeplitz_operands(tz, hs[w], li, lq);
        // u of chunk c in uw[c % 8] (steps 31 - 8 lq down, of channel li); g of the steps 16 x .. in gt[x % 16] (step li,
        // channels 4 lq ..)
        bf16x8_t uw[8];
        s16x4_t gt[16];
#pragma unroll
        for (int x = 0; x < 8; ++x) uw[x] = __builtin_bit_cast(bf16x8_t, zero_words<4>());
#pragma unroll
        for (int x = 0; x < 16; ++x) gt[x] = s16x4_t{0, 0, 0, 0};
        f32x4_t cacc[ND], facc = zero4;
#pragma unroll
        for (int x = 0; x < ND; ++x) cacc[x] = zero4;

        __syncthreads();
        walk([&](auto slot_c, int j) {
            constexpr int SL = decltype(slot_c)::value;
            constexpr int SZ = (SL + 8 - LAG) & 7;  // (j - LAG) % 8
            constexpr int two = (SL & 1) * kSlot;
            const lds4_t uo = *reinterpret_cast<const lds4_t*>(rc16 + kU + two + 16 * (3 - lq));
            s16x4_t ut[2];
#pragma unroll
            for (int p = 0; p < 2; ++p) {
                gt[2 * SL + p] = across(kG + two + 32 * p);
                ut[p] = across(kU + two + 32 * p);
            }
            {
                Words<4> r;
#pragma unroll
                for (int e = 0; e < 4; ++e) r.w[e] = __builtin_amdgcn_alignbit(uo[3 - e], uo[3 - e], 16);
                uw[SL] = __builtin_bit_cast(bf16x8_t, r);
            }
            // filter gradient: u of steps 16 p + i of this chunk against g of steps 16 p - 16 x + n
            auto products_dh = [&](int p) {
#pragma unroll
                for (int x = 0; x < ND; ++x)
                    cacc[x] = __builtin_amdgcn_mfma_f32_16x16x16bf16_1k(ut[p], gt[(2 * SL + p - x) & 15], cacc[x], 0, 0, 0);
            };
            const bool own = in_tile(j);
            if (j >= LAG && in_ext(j - LAG)) {
                Quad y4[2];
#pragma unroll
                for (int p = 0; p < 2; ++p) y4[p] = quad_at(rc16 + kY + SZ * kSlot + 32 * p + 8 * (3 - lq));
                keep_last(0);
                // z of chunk j - LAG, sources and outputs in reversed order with du's operands: row n is step 15 - n
                f32x4_t acc[2] = {zero4, zero4};
#pragma unroll
                for (int s = 0; s < NKB; ++s)
#pragma unroll
                    for (int p = 0; p < 2; ++p)
                        acc[p] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(tz[2 * s + 1 - p], uw[(SL - LAG + s) & 7], acc[p], 0, 0, 0);
#pragma unroll
                for (int p = 0; p < 2; ++p)
                    put_quad(rc16 + kDx + kFront + 32 * p + 8 * (3 - lq),
                             pack_quad(__builtin_shufflevector(acc[p], acc[p], 3, 2, 1, 0) * unpack_quad(y4[p])));
                if (in_tile(j - LAG)) {
                    float z = 0.0f;
#pragma unroll
                    for (int n = 0; n < 2; ++n) {
                        const Steps steps = read_steps(kQ + SZ * kSlot + 32 * n);
                        const Shifts sh = read_shifts(0, n);
                        __builtin_amdgcn_sched_barrier(0);
                        if (own) products_dh(n);  // while the reads are under way
                        const Quad dx = unit(fa, steps, sh, n == 0 && chunk_start(j - LAG) == 0, facc);
                        put_quad(rc4 + kQ + SZ * kSlot + 32 * n, dx);
                        z = probe(z, dx);
                    }
                    if (__builtin_expect(!(z == 0.0f), 0)) exact_dx(0, kQ + SZ * kSlot);
                }
            }
            if (own && !(j >= LAG && in_tile(j - LAG))) {
                products_dh(0);
                products_dh(1);
            }
            __syncthreads();
        }, nothing);
        store_featurizer_dh(0, facc);
        // ---- fold the diagonals: dh[16 x + i - n] += C_x[i][n]; the lane holds C_x[4 lq + r][li], r = 0..3
        float* const tilebuf = fold[w];  // this wave's 16 x 16 tile, row stride 17
        float* const dhw = hs[w];        // reuse: this wave's partial dh
        for (int j = lane; j < kTaps; j += 64) dhw[j] = 0.0f;
#pragma unroll
        for (int x = 0; x < ND; ++x) {
            __builtin_amdgcn_wave_barrier();
#pragma unroll
            for (int r = 0; r < 4; ++r) tilebuf[(4 * lq + r) * 17 + li] = cacc[x][r];
            __builtin_amdgcn_wave_barrier();
            if (lane < 31) {
                const int delta = lane - 15;  // i - n
                const int j = 16 * x + delta;
                if (j >= 0 && j < a.lh) {
                    float v[16], s = 0.0f;  // all reads in flight, then the diagonal in order
#pragma unroll
                    for (int i = 0; i < 16; ++i) v[i] = tilebuf[i * 17 + ((i - delta) & 15)];
#pragma unroll
                    for (int i = 0; i < 16; ++i) s += (i - delta >= 0 && i - delta < 16) ? v[i] : 0.0f;
                    dhw[j] += s;
                }
            }
        }
        __builtin_amdgcn_wave_barrier();
        float* out = a.partial + ((int64_t)tile * (D / 16) + (cblock0 / 16 + w)) * a.lh;
        for (int j = lane; j < a.lh; j += 64) out[j] = dhw[j];
    } else {
        // ================= data movement (rows 2 rp, 2 rp + 1 of a chunk, channels 4 lp .. 4 lp + 3) and featurizers
        // Ahead of the multipliers on its SIMD, which wait for its rows at every barrier (priority 0 / 1 / 2 / 3, 128 taps, us: 1 x
        // 8192 x 4096 145 / 135 / 135 / 136, 4 x 32768 x 4096 2028 / 1899 / 1899 / 1897, 2 x 500 x 1024 28 / 27 / 28 / 28).
        __builtin_amdgcn_s_setprio(1);
        const int mt = tid - 2 * kNW * 64;
        const int lp = mt % 16, rp = mt / 16;
        const uint32_t row_bytes = (uint32_t)D * 2;
        // addresses: a uniform base, the first row of a chunk in memory, and a 32-bit byte offset per lane; rows outside
        // [lo, hi] become the nearest one
        struct Rows {
            int64_t base;     // elements from the batch item's start
            uint32_t off[2];  // bytes
        };
        const Rows inside{0, {(uint32_t)(__umul24(kT - 1 - 2 * rp, row_bytes) + 8 * lp), (uint32_t)(__umul24(kT - 2 - 2 * rp, row_bytes) + 8 * lp)}};
        auto rows_at = [&](int T, int lo, int hi) {
            Rows r = inside;
            const int t0 = L - kT - T;
            if (t0 >= lo && t0 + kT - 1 <= hi) {
                r.base = (int64_t)t0 * D;
            } else {
                int first = t0 > lo ? t0 : lo;
                first = first < hi ? first : hi;
                r.base = (int64_t)first * D;
#pragma unroll
                for (int i = 0; i < 2; ++i) {
                    int t = L - 1 - T - 2 * rp - i;
                    t = t > first ? t : first;
                    t = t < hi ? t : hi;
                    r.off[i] = __umul24((uint32_t)(t - first), row_bytes) + 8 * lp;
                }
            }
            return r;
        };
        auto ld = [](const uint16_t* p, uint32_t off) { return load_words_nt<2>(reinterpret_cast<const char*>(p) + off); };
        auto st = [](uint16_t* p, uint32_t off, const Words<2>& x) { store_words_nt<2>(reinterpret_cast<char*>(p) + off, x); };

        Words<2> raw[PF][4][2];  // chunk c of q, k, v, dy in stage c % PF
        const int g_end = t_end + kT < L ? t_end + kT : L;                                      // q and dy needed below this
        const int u_end = t_begin + (ntot + 1) * kT < L ? t_begin + (ntot + 1) * kT : L;        // k and v
        auto load_chunk = [&](auto st_c, int c) {
            constexpr int ST = decltype(st_c)::value % PF;
            const Rows rg = rows_at(chunk_start(c), L - g_end, L - 1 - t_begin);
            const Rows ru = rows_at(chunk_start(c), L - u_end, L - 1 - t_ext);
#pragma unroll
            for (int x = 0; x < 4; ++x) {
                const Rows& r = (x == 1 || x == 2) ? ru : rg;
                const uint16_t* p = a.in[x] + seq0 + r.base;
#pragma unroll
                for (int i = 0; i < 2; ++i) raw[ST][x][i] = ld(p, r.off[i]);
            }
        };
        load_chunk(integral_constant<int, 0>{}, 0);
        load_chunk(integral_constant<int, 1>{}, 1);

        s16x4_t fb[3][NF][2];
#pragma unroll
        for (int x = 0; x < 3; ++x) {
            const float* hp = feat_row(x);
#pragma unroll
            for (int m = 0; m < NF; ++m) {
                float t4[4];
#pragma unroll
                for (int k = 0; k < 4; ++k) t4[k] = tap_at(hp, 4 * m + k - l4);
                split_taps(t4, fb[x][m]);
            }
        }
        char* const rw = lds + rec(4 * lp) + 4 * rp;

        auto write_chunk = [&](auto slot_c, int c) {
            constexpr int SL = decltype(slot_c)::value, ST = SL % PF;  // SL = c % 8
            if (chunk_start(c) + kT > L) {  // zeros before the sequence's first row
                const int tau = chunk_start(c) + 2 * rp;
#pragma unroll
                for (int x = 0; x < 4; ++x)
#pragma unroll
                    for (int i = 0; i < 2; ++i)
                        if (tau + i >= L) raw[ST][x][i] = zero_words<2>();
            }
#pragma unroll
            for (int x = 0; x < 4; ++x) {
                uint32_t o[4];
#pragma unroll
                for (int p = 0; p < 2; ++p) {
                    o[2 * p] = __builtin_amdgcn_perm(raw[ST][x][1].w[p], raw[ST][x][0].w[p], 0x05040100u);
                    o[2 * p + 1] = __builtin_amdgcn_perm(raw[ST][x][1].w[p], raw[ST][x][0].w[p], 0x07060302u);
                }
                constexpr int S4 = SL & 3;
                const int at = x == 0 ? kQ + SL * kSlot : x == 1 ? kK + S4 * kSlot : x == 2 ? kV + S4 * kSlot : kY + SL * kSlot;
#pragma unroll
                for (int e = 0; e < 4; ++e) *reinterpret_cast<lds1_t*>(rw + at + e * kRec) = o[e];
                if ((x == 0 && SL == 0) || ((x == 1 || x == 2) && S4 == 0)) {
                    if (rp < kBack / 4) {  // the first steps once more behind the ring
                        const int back = at + (x == 0 ? 8 : 4) * kSlot;
#pragma unroll
                        for (int e = 0; e < 4; ++e) *reinterpret_cast<lds1_t*>(rw + back + e * kRec) = o[e];
                    }
                }
            }
        };
        auto store_rows = [&](int at, uint16_t* out, int c) {
            const int T = chunk_start(c);
            const Rows ro = rows_at(T, L - t_end, L - 1);
            uint32_t o[4];
#pragma unroll
            for (int e = 0; e < 4; ++e) o[e] = *reinterpret_cast<const lds1_t*>(rw + at + e * kRec);
#pragma unroll
            for (int i = 0; i < 2; ++i) {
                const uint32_t sel = i == 0 ? 0x05040100u : 0x07060302u;
                Words<2> x;
                x.w[0] = __builtin_amdgcn_perm(o[1], o[0], sel);
                x.w[1] = __builtin_amdgcn_perm(o[3], o[2], sel);
                if (T + 2 * rp + i < t_end) st(out + seq0 + ro.base, ro.off[i], x);
            }
        };
        // dk, dv of the chunk before j, dq of the one LAG older
        auto store_chunk = [&](auto slot_c, int j) {
            constexpr int PV = (decltype(slot_c)::value + 7) & 7, DQ = (PV + 8 - LAG) & 7;
            if (j > 0 && in_tile(j - 1)) {
                store_rows(kK + (PV & 3) * kSlot, a.out[1], j - 1);
                store_rows(kV + (PV & 3) * kSlot, a.out[2], j - 1);
            }
            if (j > LAG && in_tile(j - 1 - LAG)) store_rows(kQ + DQ * kSlot, a.out[0], j - 1 - LAG);
        };
        // q', k', v' of chunk c, and from them g and u
        auto featurize = [&](auto slot_c, int c) {
            constexpr int SL = decltype(slot_c)::value, S4 = SL & 3, two = (SL & 1) * kSlot;  // SL = c % 8
            constexpr int at[3] = {kQ + SL * kSlot, kK + S4 * kSlot, kV + S4 * kSlot};
            float z = 0.0f;
#pragma unroll
            for (int n = 0; n < 2; ++n) {
                s16x4_t xq[3][NF];
#pragma unroll
                for (int x = 0; x < 3; ++x)
#pragma unroll
                    for (int m = 0; m < NF; ++m) xq[x][m] = operand(quad_at(rc4 + at[x] + 32 * n + 8 * m));
                const f32x4_t y4 = unpack_quad(quad_at(rc4 + kY + SL * kSlot + 32 * n));
                f32x4_t f[3] = {zero4, zero4, zero4};
#pragma unroll
                for (int m = NF - 1; m >= 0; --m)
#pragma unroll
                    for (int part = 1; part >= 0; --part)
#pragma unroll
                        for (int x = 0; x < 3; ++x)
                            f[x] = __builtin_amdgcn_mfma_f32_4x4x4bf16_1k(fb[x][m][part], xq[x][m], f[x], 0, 0, 0);
                const Quad g4 = pack_quad(y4 * f[0]), u4 = pack_quad(f[1] * f[2]);
                put_quad(rc4 + kG + two + 32 * n, g4);
                put_quad(rc4 + kU + two + 32 * n, u4);
                put_quad(rc4 + kKf + two + 32 * n, pack_quad(f[1]));
                put_quad(rc4 + kVf + two + 32 * n, pack_quad(f[2]));
                z = probe(probe(z, g4), u4);
            }
            if (__builtin_expect(!(z == 0.0f), 0)) {
                const float *const h0 = taps_of(0), *const h1 = taps_of(1), *const h2 = taps_of(2);
                const int T = chunk_start(c) + 4 * l4;
#pragma unroll 1
                for (int o = 0; o < kSlot; o = (o & 7) == 6 ? o + 26 : o + 2) {
                    float s0 = 0.0f, s1 = 0.0f, s2 = 0.0f;
#pragma unroll 1
                    for (int j = 0; j < a.lf && T + (o >> 1) + j < L; ++j) {
                        s0 = __builtin_fmaf(h0[j], step_at(at[0] + o + 2 * j), s0);
                        s1 = __builtin_fmaf(h1[j], step_at(at[1] + o + 2 * j), s1);
                        s2 = __builtin_fmaf(h2[j], step_at(at[2] + o + 2 * j), s2);
                    }
                    put_step(kG + two + o, step_at(kY + SL * kSlot + o) * s0);
                    put_step(kU + two + o, s1 * s2);
                    put_step(kKf + two + o, s1);
                    put_step(kVf + two + o, s2);
                }
            }
        };
        auto step = [&](auto slot_c, int j) {
            constexpr int SL = decltype(slot_c)::value;  // j % 8
            store_chunk(slot_c, j);
            if (j + 3 <= ntot) {
                write_chunk(integral_constant<int, (SL + 3) & 7>{}, j + 3);
                load_chunk(integral_constant<int, (SL + 3) & 7>{}, j + 3 + PF);
            }
            if (j + 1 < ntot) featurize(integral_constant<int, (SL + 1) & 7>{}, j + 1);
            __syncthreads();
        };
        write_chunk(integral_constant<int, 0>{}, 0);
        load_chunk(integral_constant<int, 0>{}, PF);
        write_chunk(integral_constant<int, 1>{}, 1);
        load_chunk(integral_constant<int, 1>{}, 1 + PF);
        write_chunk(integral_constant<int, 2>{}, 2);
        load_chunk(integral_constant<int, 2>{}, 2 + PF);
        __syncthreads();
        featurize(integral_constant<int, 0>{}, 0);
        __syncthreads();
        walk(step, store_chunk);
    }
}

int64_t chain_rows(const ChainShape& s) {
    const int64_t ncb = s.D / kC;
    int64_t rows = tuning().mr_rows;
    if (rows <= 0) {
        // one workgroup per compute unit, down to the length of the halo (each tile also leaves partial filter gradients)
        const int64_t halo = s.lh <= 65 ? 2 * kT : 4 * kT;
        rows = one_round_rows(s.B * ncb, s.L, 4 * halo, kT);
        if (rows < halo) rows = halo;
    }
    rows = (rows + kT - 1) / kT * kT;
    const int64_t cap = (s.L + kT - 1) / kT * kT;
    return rows > cap ? cap : rows;
}

}  // namespace

bool chain_bwd_supported(const ChainShape& s) {
    return s.dtype == HY_BF16 && s.group % 16 == 0 && s.D % kC == 0 && s.D < (1 << 23) && s.L <= 0x7fff0000LL && s.lh > 8 &&
           s.lh <= 129 && s.lf >= 1 && s.lf <= kMaxLf;
}

int64_t chain_bwd_workspace_bytes(const ChainShape& s) {
    const int64_t rows = chain_rows(s);
    const int64_t nsets = s.B * ((s.L + rows - 1) / rows);
    return nsets * (s.D / 16 * s.lh + 3 * s.D * s.lf) * (int64_t)sizeof(float);
}

hy_status launch_chain_bwd(const ChainBwdPtrs& p, const ChainShape& s, void* ws, hipStream_t st) {
    if (!chain_bwd_supported(s)) return HY_ERR_UNSUPPORTED;
    ChainBwdArgs a;
    const void* const in[4] = {p.q, p.k, p.v, p.dy};
    void* const out[3] = {p.dq, p.dk, p.dv};
    const float* const hx[3] = {p.hq, p.hk, p.hv};
    float* const dhx[3] = {p.dhq, p.dhk, p.dhv};
    a.rows = (int32_t)chain_rows(s);
    a.tiles_per_seq = (int32_t)((s.L + a.rows - 1) / a.rows);
    const int64_t nsets = s.B * a.tiles_per_seq;
    a.partial = static_cast<float*>(ws);
    for (int x = 0; x < 4; ++x) a.in[x] = static_cast<const uint16_t*>(in[x]);
    for (int x = 0; x < 3; ++x) {
        a.hx[x] = hx[x];
        a.out[x] = static_cast<uint16_t*>(out[x]);
        a.partial_x[x] = a.partial + nsets * (s.D / 16) * s.lh + x * nsets * s.D * s.lf;
    }
    a.h = p.h;
    a.L = s.L;
    a.D = s.D;
    a.lf = s.lf;
    a.feat_group = s.feat_group;
    a.lh = s.lh;
    a.group = s.group;
    a.ncb = (int32_t)(s.D / kC);
    const int64_t nb = nsets * a.ncb;
    if (nb > 0x7fffffffLL) return HY_ERR_UNSUPPORTED;
    const dim3 grid((uint32_t)nb), block(kKinds * kNW * 64);
    // the window and z's delay are as many chunks as the filter reaches back (mr_bwd_kernels.hip's, and so is the reach of a
    // value that is not finite)
    hy_status rc;
    switch ((s.lh + 30) / 32 + 1) {
        case 2: rc = launch_kernel((chain_bwd_kernel<2>), grid, block, st, a); break;
        case 3: rc = launch_kernel((chain_bwd_kernel<3>), grid, block, st, a); break;
        case 4: rc = launch_kernel((chain_bwd_kernel<4>), grid, block, st, a); break;
        default: rc = launch_kernel((chain_bwd_kernel<5>), grid, block, st, a);
    }
    if (rc != HY_OK) return rc;
    // partial rows of dh are per 16-channel slice, those of dhq, dhk, dhv per channel
    DhReduce r[4] = {{a.partial, p.dh, nsets, s.D / 16, s.lh, s.group / 16}};
    for (int i = 0; i < 3; ++i) r[1 + i] = DhReduce{a.partial_x[i], dhx[i], nsets, s.D, s.lf, s.feat_group};
    return launch_dh_reduce(r, 4, st);
}

}  // namespace hy
