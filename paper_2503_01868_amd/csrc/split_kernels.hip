// General gated FIR in fp32 precision on the bf16 matrix cores, for filters that 8 or 16 adjacent channels share: fp32
// medium filters, and bf16 shapes whose width does not tile the bf16 kernels' workgroups, forward and backward.
//
//     out[t] = gate[t] * sum_j h[j] x[t -+ j],  x = a*b
//
// Every factor is split into bf16 pieces that add up to it: head, then what rounding left times 2^8, twice, so that a piece
// is as large as its factor may be and keeps its bits down to the smallest normal numbers.  A tap and an fp32 x are three
// pieces, the product x of two bf16 values has 16 bits and is two.  A product of two pieces is exact in fp32.  The sums of the
// piece products of one weight (1, 2^-8, 2^-16; 6 of 9 for fp32, 5 of 6 for bf16) are kept apart and joined at the end; the
// products left out are two of 2^-25 of theirs at most (bf16: one) and one far below.  What else rounds is the additions, and of
// those the matrix instruction makes one per 32 terms and output where a chain of FMAs makes one per term.  At 16 times the rate
// of the fp32 products that is 2.7 to 3.2 times their rate.
//
// A workgroup owns 64 channels and walks a tile of the sequence in chunks of 64 steps (towards the past for the transposed
// sum, which is then causal) like mr_kernels.hip: rows of a and b are loaded two chunks ahead, x goes as bf16 planes
// [piece][step][channel] into LDS and comes back transposed into a register window of the last NKB source blocks of 32
// steps, the sums go back through LDS to be gated and stored as row pieces.  A product is 16 rows x 32 source steps x 16
// output steps, and a wave makes one of the two that 16 channels x 32 steps take per source block, so that operands and
// window of a wave fit 256 registers and two waves per SIMD overlap products with conversions (one wave with both, 32-step
// chunks, the SIMD to itself: 47 us where this took 38, 3 x 5003 x 1000 bf16, 128 taps, inputs changing from call to call; four
// chunks ahead instead of two gained that form nothing):
//   kGroup = 16: rows are 16 channels; the two waves of a slice have a 16-step half of every 32 steps each;
//   kGroup = 8:  rows are the 8 channels of a filter x the two halves; a source block begins 16 steps before its half.
//
// The products multiply structural zeros (taps outside the filter, rows that hold no data), which is only harmless for
// finite values: sums that come out not finite are formed again term by term from global memory in the general kernel's
// order, without the terms the definition does not have.  (A value that is not finite, or rounds to infinity as a head,
// makes every sum not finite that it is multiplied into, by zero or not.)
//
// Bound: long sequences the row pieces (fp32 256 bytes of every row, 1 x 8192 x 4096 108 us = 5.0 TB/s; bf16 128 bytes),
// short ones the start of a tile (operands, two chunks of warm-up).  General kernel / this one, 128 taps, us: 3 x 5003 x 1000
// bf16, groups of 8 70 / 31 (33 taps 51 / 27), fp32 95 / 51; 2 x 2048 x 1024 fp32, groups of 16 27 / 17; 1 x 8192 x 4096 fp32
// 169 / 108; 1 x 300 x 512 fp32 10.3 / 7.9.  Error against 64 bits of 2 x 2048 x 1024 fp32, forward and gradients: 2.6e-7 / 6e-8.
#include <type_traits>

#include "hy_common.hpp"
#include "hy_launch.hpp"

namespace hy {
namespace {

typedef short s16x4_t __attribute__((ext_vector_type(4)));

constexpr int kChan = 64;   // channels per workgroup
constexpr int kWaves = 8;
constexpr int kThreads = kWaves * kWave;
constexpr int kBlock = 32;  // source steps per product
constexpr int kChunk = 64;  // steps between barriers
constexpr int kAhead = 2;   // chunks of a, b and the gates in flight (the loops and register stages below are written for two)
constexpr int kRowBytes = kChan * 2;    // a staged row of one plane
constexpr int kPlane = kChunk * kRowBytes;
constexpr int kZRow = kChan * 4 + 16;   // a row of sums

struct SplitArgs {
    FirProblem p[2];
    int64_t L, D;
    int32_t lh, group;  // lh: the taps that can meet data
    int32_t row_taps;   // taps per filter in memory
    int32_t rows, tiles_per_seq, ncb;
    int32_t together;  // neighbouring channel blocks on one XCD
};

// Staged rows are permuted by 16-byte pieces so that the transposed reads of a wave (for every octet of steps, 4 rows x 16
// channels, or 2 x 4 rows x 8 channels) meet every bank twice, which is what 512 bytes take.
template <int kGroup>
__device__ __forceinline__ int skew(int row) {
    return kGroup == 16 ? ((row >> 1) & 1) * 2 + ((row >> 3) & 1) * 4 : ((row >> 1) & 1) + ((row >> 3) & 3) * 2;
}

template <typename T, int kGroup, int NKB, bool kTwo>
__global__ __launch_bounds__(kThreads, 2) void split_fir_kernel(SplitArgs a) {
    constexpr int VEC = 16 / T::kBytes;      // channels per 16-byte piece
    constexpr int PPR = kChan / VEC;         // pieces per row
    constexpr int RPP = kThreads / PPR;      // rows per pass over the workgroup's lanes
    constexpr int NP = kChunk / RPP;         // passes per chunk
    constexpr int P = T::kBytes == 4 ? 3 : 2;   // pieces of x
    constexpr int kBuf = kGroup == 16 ? 2 : 3;  // staged chunks (a block of 8 channels reaches back into the one before)
    constexpr int kTaps = kBlock * NKB;
    using PV = Pack<T, VEC>;
    using Raw = typename PV::Raw;
    __shared__ uint4 planes[kBuf][P * kPlane / 16];
    __shared__ __attribute__((aligned(16))) char zst[2][kChunk * kZRow];
    // the pieces of a wave's filter: word kTapPad + j holds those of taps j (low half) and j - 1, zero outside the filter
    __shared__ uint32_t hs[kWaves][3][kTapPad + kTaps + 1];

    uint32_t order = blockIdx.y * gridDim.x + blockIdx.x;
    if (a.together) order = xcd_contiguous(order, gridDim.x * gridDim.y);
    const FirProblem pr = a.p[order / gridDim.x];
    const uint32_t lb = order % gridDim.x;
    const int tid = threadIdx.x, lane = tid % kWave, w = __builtin_amdgcn_readfirstlane(tid / kWave);
    const int li = lane % 16, lq = lane / 16;
    const int64_t cblock = (int64_t)(lb % (uint32_t)a.ncb) * kChan;
    const uint32_t tile = lb / (uint32_t)a.ncb;
    const int64_t b = tile / (uint32_t)a.tiles_per_seq;
    const int64_t L = a.L, D = a.D;
    const int lh = a.lh;
    const bool rev = pr.rev != 0;
    // steps of the walk: tau = t, or L - 1 - t for the transposed sum; chunk c begins at t_start + 64 c
    const int t_start = (int)(tile % (uint32_t)a.tiles_per_seq) * a.rows;
    const int t_end = t_start + a.rows < L ? t_start + a.rows : (int)L;
    const int t_data = (int)(rev ? L - pr.hi : pr.lo);  // first step of the walk at which a and b hold data
    // chunks before the tile that its first sums reach into; two are left out where they hold no data
    constexpr int kWarm = ((NKB - 1) * kBlock + kChunk - 1) / kChunk, kOdd = kWarm & 1;
    const int warm = kWarm == 2 && t_start <= t_data ? 0 : kWarm;
    const int nchunks = (t_end - t_start + kChunk - 1) / kChunk;
    const int64_t row_bytes = D * T::kBytes;

    // this lane's piece of the rows it loads and stores (a piece past the last channel reads the block's first one)
    const int pc = tid % PPR, lr = tid / PPR;
    const bool own = cblock + (int64_t)pc * VEC < D;
    const int64_t col = own ? cblock + (int64_t)pc * VEC : cblock;
    auto item = [&](const void* p, int64_t stride) __attribute__((always_inline)) { return static_cast<const char*>(p) + (b * stride + col) * T::kBytes; };
    const char* const ap = item(pr.a, pr.stride_ab);
    const char* const bp = item(pr.b, pr.stride_ab);
    const char* const gp = item(pr.gate, pr.stride_gate);
    const char* const gp2 = kTwo && pr.out2 ? item(pr.gate2, pr.stride_gate) : gp;
    char* const op = const_cast<char*>(item(pr.out, pr.stride_out));
    char* const op2 = kTwo && pr.out2 ? const_cast<char*>(item(pr.out2, pr.stride_out)) : nullptr;
    auto at = [&](int tau) { return (rev ? L - 1 - tau : (int64_t)tau) * row_bytes; };

    // every lane issues the same loads for every chunk; rows past the tile's end repeat its last one
    Raw ar[kAhead][NP], br[kAhead][NP], gr[kAhead][NP], gr2[kAhead][NP];
    auto load_ab = [&](int c, Raw (&x)[NP], Raw (&y)[NP]) __attribute__((always_inline)) {
#pragma unroll
        for (int i = 0; i < NP; ++i) {
            int tau = t_start + c * kChunk + i * RPP + lr;
            tau = tau < t_end ? tau : t_end - 1;
            tau = tau > t_data ? tau : t_data;
            const int64_t off = at(tau);
            x[i] = PV::load(ap + off);
            y[i] = PV::load(bp + off);
        }
    };
    auto load_gate = [&](int c, Raw (&x)[NP], Raw (&y)[NP]) __attribute__((always_inline)) {
#pragma unroll
        for (int i = 0; i < NP; ++i) {
            int tau = t_start + c * kChunk + i * RPP + lr;
            tau = tau < t_end ? tau : t_end - 1;
            const int64_t off = at(tau);
            x[i] = PV::load_nt(gp + off);
            if constexpr (kTwo) y[i] = PV::load_nt(gp2 + (op2 ? off : 0));
        }
    };
    load_ab(-warm, ar[0], br[0]);  // chunk c waits in stage (c + kOdd) % 2
    load_ab(-warm + 1, ar[1], br[1]);
    load_gate(0, gr[0], gr2[0]);

    // a source block of 8 channels begins 16 steps before its chunk: no steps before the first one
    if constexpr (kGroup == 8)
        for (int i = tid; i < P * kPlane / 16; i += kThreads) planes[kBuf - 1][i] = make_uint4(0u, 0u, 0u, 0u);

    // ---- operands: pieces of h[d + li - 8 lq - e], d = 32 m, + 16 for the second half (kGroup = 16) or always (8)
    bf16x8_t tz[NKB][3];
    {
        int64_t c0 = cblock + (kGroup == 16 ? 16 * (w >> 1) : 8 * w);
        c0 = c0 < D ? c0 : D - 1;  // past the last channel: any filter
        const float* hp = pr.h + (uint32_t)c0 / (uint32_t)a.group * (int64_t)a.row_taps;
        constexpr int kEach = (kTapPad + kTaps + kWave - 1) / kWave;
        float f[kEach];
#pragma unroll
        for (int i = 0; i < kEach; ++i) {
            const int j = i * kWave + lane - kTapPad;
            f[i] = hp[j >= 0 && j < lh ? j : 0];
        }
#pragma unroll
        for (int i = 0; i < kEach; ++i) {
            const int word = i * kWave + lane, j = word - kTapPad;
            float x = j >= 0 && j < lh ? f[i] : 0.0f;
#pragma unroll
            for (int s = 0; s < 3; ++s) {
                const uint32_t piece = pack_bf16x2(x, 0.0f);
                x = (x - bf16_lo(piece)) * 256.0f;
                uint16_t* half = reinterpret_cast<uint16_t*>(&hs[w][s][word]);
                if (word < kTapPad + kTaps) {
                    half[0] = (uint16_t)piece;
                    half[3] = (uint16_t)piece;
                }
            }
        }
        __syncthreads();
        // (no lane reads word 0, whose high half is not written)
        const int p = kTapPad + (kGroup == 16 ? 16 * (w & 1) : 16) + li - 8 * lq;
#pragma unroll
        for (int m = 0; m < NKB; ++m)
#pragma unroll
            for (int s = 0; s < 3; ++s) {
                Words<4> x;
#pragma unroll
                for (int e = 0; e < 4; ++e) x.w[e] = hs[w][s][p + kBlock * m - 2 * e];
                tz[m][s] = __builtin_bit_cast(bf16x8_t, x);
            }
    }

    // ---- window: source block m, piece s
    bf16x8_t win[NKB][P];
#pragma unroll
    for (int m = 0; m < NKB; ++m)
#pragma unroll
        for (int s = 0; s < P; ++s) win[m][s] = __builtin_bit_cast(bf16x8_t, zero_words<4>());

    // Transposed reads: 16 lanes with one lq address 4 rows x 4 quads of channels and get 4 steps of one channel each.
    // Byte offsets into the chunk's planes; for 8 channels the rows of the first half lie 16 steps earlier, in the first
    // block of a chunk partly in the chunk before.
    int rd[2];
    bool rd_before = false;
    {
        const int r4 = 8 * lq + (li >> 2), quad = li & 3;
#pragma unroll
        for (int sub = 0; sub < 2; ++sub) {
            if constexpr (kGroup == 16) {
                const int r = r4 + kBlock * sub;
                rd[sub] = r * kRowBytes + ((2 * (w >> 1) + (quad >> 1)) ^ skew<16>(r)) * 16 + (quad & 1) * 8;
            } else {
                const int row = r4 + kBlock * sub + 16 * (quad >> 1) - 16, r = row & (kChunk - 1);
                if (sub == 0) rd_before = row < 0;
                rd[sub] = r * kRowBytes + (w ^ skew<8>(r)) * 16 + (quad & 1) * 8;
            }
        }
    }
    // Sums: this lane holds channels 4 lq .. 4 lq + 3 (of 8: half lq / 2, channels 4 (lq % 2) ..) at step li of a half
    const int zw = kGroup == 16 ? (16 * (w & 1) + li) * kZRow + (16 * (w >> 1) + 4 * lq) * 4
                                : (16 * (lq >> 1) + li) * kZRow + (8 * w + 4 * (lq & 1)) * 4;

    // chunk c's sums where this lane reads them, term by term from global memory, in ascending source order (causal) or tap
    // order; the channels of a piece share their filter
    auto exact_sums = [&](int c) __attribute__((always_inline)) {
        const float* hp = pr.h + (uint32_t)col / (uint32_t)a.group * (int64_t)a.row_taps;
#pragma unroll 1
        for (int row = lr; row < kChunk; row += RPP) {
            const int tau = t_start + c * kChunk + row;
            const int reach = tau - t_data < lh - 1 ? tau - t_data : lh - 1;  // the last tap that meets data
            float z[VEC];
#pragma unroll
            for (int e = 0; e < VEC; ++e) z[e] = 0.0f;
#pragma unroll 1
            for (int i = tau < t_end ? 0 : lh; i <= reach; ++i) {
                const int j = rev ? i : reach - i;
                float x[VEC], y[VEC];
                PV::unpack(PV::load(ap + at(tau - j)), x);
                PV::unpack(PV::load(bp + at(tau - j)), y);
#pragma unroll
                for (int e = 0; e < VEC; ++e) z[e] = __builtin_fmaf(hp[j], x[e] * y[e], z[e]);
            }
            float* zp = reinterpret_cast<float*>(zst[c & 1] + row * kZRow) + pc * VEC;
#pragma unroll
            for (int e = 0; e < VEC; ++e) zp[e] = z[e];
        }
    };
    auto read_sums = [&](int c, float (&z)[NP][VEC]) __attribute__((always_inline)) {
        float chk = 0.0f;  // stays zero over finite sums
#pragma unroll
        for (int i = 0; i < NP; ++i) {
            const float* zp = reinterpret_cast<const float*>(zst[c & 1] + (i * RPP + lr) * kZRow) + pc * VEC;
#pragma unroll
            for (int e = 0; e < VEC; e += 4) {
                const float4 x = *reinterpret_cast<const float4*>(zp + e);
                z[i][e] = x.x; z[i][e + 1] = x.y; z[i][e + 2] = x.z; z[i][e + 3] = x.w;
            }
#pragma unroll
            for (int e = 0; e < VEC; ++e) chk = __builtin_fmaf(z[i][e], 0.0f, chk);
        }
        return chk;
    };
    // gate and store chunk c, whose sums were staged one iteration earlier
    auto finish = [&](int c, const Raw (&ga)[NP], const Raw (&gb)[NP]) __attribute__((always_inline)) {
        float z[NP][VEC];
        if (__builtin_expect(!(read_sums(c, z) == 0.0f), 0)) {
            exact_sums(c);
            read_sums(c, z);
        }
#pragma unroll
        for (int i = 0; i < NP; ++i) {
            const int tau = t_start + c * kChunk + i * RPP + lr;
            float g[VEC], o[VEC];
            PV::unpack(ga[i], g);
#pragma unroll
            for (int e = 0; e < VEC; ++e) o[e] = z[i][e] * g[e];
            const Raw y = PV::pack(o);
            Raw y2;
            if constexpr (kTwo) {
                PV::unpack(gb[i], g);
#pragma unroll
                for (int e = 0; e < VEC; ++e) o[e] = z[i][e] * g[e];
                y2 = PV::pack(o);
            }
            if (own && tau < t_end) {
                const int64_t off = at(tau);
                PV::store_nt(op + off, y);
                if constexpr (kTwo)
                    if (op2) PV::store_nt(op2 + off, y2);
            }
        }
    };

    // x of chunk c, from a register stage, into its planes; the stage is refilled with the chunk kAhead later.  Only chunks of
    // the warm-up can hold steps without data (t_data <= 0).
    auto stage = [&](int c, int buf, Raw (&xr)[NP], Raw (&yr)[NP], auto warming) __attribute__((always_inline)) {
#pragma unroll
        for (int i = 0; i < NP; ++i) {
            const int row = i * RPP + lr;
            const bool data = !decltype(warming)::value || t_start + c * kChunk + row >= t_data;
            float x[VEC], y[VEC];
            PV::unpack(xr[i], x);
            PV::unpack(yr[i], y);
#pragma unroll
            for (int e = 0; e < VEC; ++e) x[e] = data ? x[e] * y[e] : 0.0f;
            const int piece = VEC == 8 ? pc : pc >> 1;
            char* dst = reinterpret_cast<char*>(planes[buf]) + row * kRowBytes + (piece ^ skew<kGroup>(row)) * 16 +
                        (VEC == 8 ? 0 : (pc & 1) * 8);
#pragma unroll
            for (int s = 0; s < P; ++s) {
                Words<VEC / 2> wd;
#pragma unroll
                for (int e = 0; e < VEC / 2; ++e) {
                    wd.w[e] = pack_bf16x2(x[2 * e], x[2 * e + 1]);
                    x[2 * e] = (x[2 * e] - bf16_lo(wd.w[e])) * 256.0f;
                    x[2 * e + 1] = (x[2 * e + 1] - bf16_hi(wd.w[e])) * 256.0f;
                }
                store_words<VEC / 2>(dst + s * kPlane, wd);
            }
        }
        load_ab(c + kAhead, xr, yr);
    };
    // the window moves on by block `sub` of the chunk staged in `buf`
    auto advance = [&](int buf, int sub) __attribute__((always_inline)) {
#pragma unroll
        for (int m = NKB - 1; m > 0; --m)
#pragma unroll
            for (int s = 0; s < P; ++s) win[m][s] = win[m - 1][s];
        typedef __attribute__((address_space(3))) s16x4_t lds_quad_t;
        int off = rd[sub] + buf * (P * kPlane);
        if (kGroup == 8 && sub == 0) off += rd_before ? (buf == 0 ? kBuf - 1 : -1) * (P * kPlane) : 0;
        const char* src = reinterpret_cast<const char*>(planes[0]) + off;
#pragma unroll
        for (int s = 0; s < P; ++s) {
            struct { s16x4_t lo, hi; } x;
            x.lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_quad_t*)(src + s * kPlane));
            x.hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_quad_t*)(src + s * kPlane + 4 * kRowBytes));
            win[0][s] = __builtin_bit_cast(bf16x8_t, x);
        }
    };
    // the sums of block `sub` of chunk c, each weight apart: the roundings of all but the heads' then do not count
    auto products = [&](int c, int sub) __attribute__((always_inline)) {
        f32x4_t hi = {0.0f, 0.0f, 0.0f, 0.0f}, lo[2] = {hi, hi};
#pragma unroll
        for (int m = NKB - 1; m >= 0; --m)
#pragma unroll
            for (int s = P - 1; s >= 0; --s)
#pragma unroll
                for (int r = 2 - s; r >= 0; --r) {
                    f32x4_t& acc = s + r == 0 ? hi : lo[s + r - 1];
                    acc = __builtin_amdgcn_mfma_f32_16x16x32_bf16(win[m][s], tz[m][r], acc, 0, 0, 0);
                }
        auto joined = [&](int i) { return __builtin_fmaf(__builtin_fmaf(lo[1][i], 0x1p-8f, lo[0][i]), 0x1p-8f, hi[i]); };
        const float4 z = make_float4(joined(0), joined(1), joined(2), joined(3));
        *reinterpret_cast<float4*>(zst[c & 1] + sub * kBlock * kZRow + zw) = z;
    };
    auto next = [&](int buf) __attribute__((always_inline)) { return buf == kBuf - 1 ? 0 : buf + 1; };

    int buf = 0;
    stage(-warm, 0, ar[0], br[0], std::true_type{});
#pragma unroll
    for (int g = 0; g < kWarm; ++g) {
        if (warm > 0) {
            __syncthreads();  // this chunk's rows
            advance(buf, 0);
            advance(buf, 1);
            stage(g - kWarm + 1, next(buf), ar[(g + 1) % 2], br[(g + 1) % 2], std::true_type{});
            buf = next(buf);
        }
    }
    for (int base = 0; base < nchunks; base += kAhead) {
#pragma unroll
        for (int g = 0; g < kAhead; ++g) {
            const int c = base + g;
            if (c < nchunks) {
                __syncthreads();  // this chunk's rows and the previous chunk's sums
                advance(buf, 0);
                if (c > 0) finish(c - 1, gr[g ^ 1], gr2[g ^ 1]);
                load_gate(c + 1, gr[g ^ 1], gr2[g ^ 1]);
                stage(c + 1, next(buf), ar[(g + 1 + kOdd) % 2], br[(g + 1 + kOdd) % 2], std::false_type{});
                products(c, 0);
                advance(buf, 1);
                products(c, 1);
                buf = next(buf);
            }
        }
    }
    __syncthreads();
    if ((nchunks - 1) & 1) finish(nchunks - 1, gr[1], gr2[1]);
    else finish(nchunks - 1, gr[0], gr2[0]);
}

// As many tiles per sequence as make the fewest chunks in a row, a tile's start and its warm-up (by the source blocks of a
// window) priced as chunks; `cost`: those chunks.
int64_t tiles_per_sequence(int64_t columns, int64_t chunks, int nkb, int64_t* cost) {
    constexpr int64_t resident = 256;
    const int64_t start = nkb > 3 ? 3 : 2, least = (columns + resident - 1) / resident;
    auto chunks_in_a_row = [&](int64_t n) { return (columns * n + resident - 1) / resident * ((chunks + n - 1) / n + start); };
    int64_t tiles = 1;
    for (int64_t rounds = least; rounds < least + 4; ++rounds) {
        int64_t n = rounds * resident / columns;
        n = n < chunks ? n : chunks;
        if (n > 0 && chunks_in_a_row(n) < chunks_in_a_row(tiles)) tiles = n;
    }
    *cost = chunks_in_a_row(tiles);
    return tiles;
}

template <typename T, int kGroup, int NKB, bool kTwo>
hy_status launch_as(SplitArgs& a, int nprob, int64_t B, hipStream_t st) {
    const int64_t chunks = (a.L + kChunk - 1) / kChunk;
    int64_t cost, tiles = tiles_per_sequence(B * a.ncb * nprob, chunks, NKB, &cost);
    const int64_t rows = (chunks + tiles - 1) / tiles * kChunk;
    tiles = (a.L + rows - 1) / rows;
    // (HIP takes fewer than 2^32 threads: the general kernel's workgroups are half the size)
    if (B > 0x7fffffffLL || B * tiles > 0xffffffffLL / kThreads / a.ncb) return HY_ERR_UNSUPPORTED;
    a.rows = (int32_t)rows;
    a.tiles_per_seq = (int32_t)tiles;
    return launch_kernel((split_fir_kernel<T, kGroup, NKB, kTwo>), dim3((uint32_t)(B * tiles * a.ncb), (uint32_t)nprob),
                         dim3(kThreads), st, a);
}

template <typename T, int kGroup, bool kTwo>
hy_status launch_nkb(SplitArgs& a, int nprob, int64_t B, hipStream_t st) {
    switch ((a.lh - 1 + 31) / 32 + 1) {
        case 2: return launch_as<T, kGroup, 2, kTwo>(a, nprob, B, st);
        case 3: return launch_as<T, kGroup, 3, kTwo>(a, nprob, B, st);
        case 4: return launch_as<T, kGroup, 4, kTwo>(a, nprob, B, st);
        case 5: return launch_as<T, kGroup, 5, kTwo>(a, nprob, B, st);
        default: return HY_ERR_UNSUPPORTED;
    }
}

template <typename T>
hy_status launch_t(SplitArgs& a, int nprob, int64_t B, bool two, hipStream_t st) {
    if (a.group % 16 == 0)
        return two ? launch_nkb<T, 16, true>(a, nprob, B, st) : launch_nkb<T, 16, false>(a, nprob, B, st);
    return two ? launch_nkb<T, 8, true>(a, nprob, B, st) : launch_nkb<T, 8, false>(a, nprob, B, st);
}

}  // namespace

hy_status launch_split_fir(const FirProblem* p, int nprob, int64_t B, int64_t L, int64_t D, int32_t lh, int32_t group,
                           hy_dtype dtype, hipStream_t st) {
    const int32_t row_taps = lh;
    // taps beyond the first row with data (causal) or the last (transposed) meet none
    int64_t reach = 1;
    for (int i = 0; i < nprob; ++i) {
        const int64_t r = p[i].rev ? p[i].hi : L - p[i].lo;
        if (r > reach) reach = r;
    }
    if (lh > reach) lh = (int32_t)reach;
    if (nprob < 1 || nprob > 2 || group % 8 != 0 || lh < 9 || lh > 129 || L > 0x3fff0000LL || D > 0x7fff0000LL) return HY_ERR_UNSUPPORTED;
    // A workgroup has a compute unit to itself and works in chunks of 64 steps, so where sequences come in several rounds of
    // workgroups the short ones pay for padding and for starts that nothing hides, which the general kernel's smaller workgroups
    // hide among themselves; and up to 32 taps its segments of 16 and 32 are about as fast as blocks of 32 source steps.  This
    // kernel's share of the general one's time, by columns of 64 channels:
    // - more than 32 taps: 128 columns, 128 taps, bf16 33 steps 0.80, 80 0.59, fp32 0.82, 0.57; 1344 and more, 40 taps 33 steps 0.93,
    //   fp32 1.10, 64 1.03, 1.11, 80 0.81, 0.99, 97 0.83, 0.90; 128 taps 80 steps 0.58, 0.67; 17 x 300 x 1000, 40 and 128 taps 0.61,
    //   0.52, fp32 0.68, 0.50;
    // - up to 32 taps, 9 and 32: 3 x 5003 x 1000 bf16 0.87, 0.78 (31 us), fp32 0.90, 0.87 (49 us); 128 columns 8 x 400 x 1000 0.95, 0.88,
    //   8 x 1300 0.88, 0.80; 256 columns 16 x 300 0.80, 0.71, fp32 0.87, 0.81; 1024 and more of 4 to 80 steps 1.3 to 3, 64 x 128 x 4088
    //   0.89, 0.90, fp32 1.13, 1.15 (1600 x 97 x 1000 bf16 0.97, 0.97), 64 x 160 x 1000 1.32, 1.16;
    //   longer ones by the share of the chip's time that the tiles fill (`filled`): 17 x 300 x 1000, 36%, 1.16, 1.03, fp32 1.18, 1.11,
    //   40 x 257, 48%, 1.07, 0.96, 24 x 400, 52%, 1.04, 0.94, fp32 1.06, 1.02, 17 x 300 x 4088, 57%, 1.04, 0.87, fp32 0.99, 0.88,
    //   17 x 300 x 6008, 59%, 0.91, 0.89, fp32 0.86, 0.87, 5 x 1000 x 6008, 80%, 0.90, 0.82, fp32 0.84, 0.82; 17 x 1700 x 1000 0.89, 0.89,
    //   fp32 0.87, 0.92; and where tiles come in a round or two, which hide no starts, 9 x 1100 x 1000, 60%, 1.09, 0.97, 12 x 1200, 67%,
    //   1.10, 1.01, fp32 1.00, 0.96, 16 x 600, 78%, 0.95, 0.85, fp32 1.10, 1.07;
    // - gradients of up to 32 taps: 3 x 300 x 1000 bf16 22.3 / 24.3 us, 9 taps, 25.0 / 25.2, 32 taps, 2 x 2000 x 1000 the same (33
    //   taps 28.7 / 27.6, 62 / 54).
    const int64_t ncb = (D + kChan - 1) / kChan, columns = B * ncb * nprob;
    bool served = lh > 32 ? columns <= 256 || L > (dtype == HY_BF16 || lh > 64 ? 64 : 96)
                          : nprob == 1 && (L >= 1536 || columns <= (lh > 16 || L <= 320 ? 256 : 128));
    if (lh <= 32 && nprob == 1 && dtype == HY_BF16 && L > 96 && L <= 128) served = true;  // (the general kernel's longest tiles)
    if (lh <= 32 && nprob == 1 && !served && L > 256) {
        int64_t cost;
        tiles_per_sequence(columns, (L + kChunk - 1) / kChunk, 2, &cost);
        const int64_t filled = 100 * (columns * L) / (cost * 256 * kChunk);
        served = filled >= (columns <= 256 ? 70 : lh > 16 ? 50 : 59);
    }
    if (!served) return HY_ERR_UNSUPPORTED;
    SplitArgs a;
    bool two = false;
    for (int i = 0; i < 2; ++i) {
        const FirProblem& x = a.p[i] = p[i < nprob ? i : 0];
        if (!x.b || !x.gate || x.lo > 0 || x.hi < L) return HY_ERR_UNSUPPORTED;
        two |= x.out2 != nullptr;
    }
    a.L = L;
    a.D = D;
    a.lh = lh;
    a.row_taps = row_taps;
    a.group = group;
    a.ncb = (int32_t)ncb;
    // rows that are no whole lines: a piece shares its first and last line with its neighbours', so those go to one L2 (3 x
    // 5003 x 1000 bf16: 216 -> 141 MB, 40.4 -> 37.9 us, fp32 59.1 -> 50.8; rows of whole lines run better spread out, general
    // kernel, 2 x 2048 x 1024 fp32, forward and gradients 109 against 118)
    a.together = D * (dtype == HY_BF16 ? 2 : 4) % 128 != 0;
    return dtype == HY_BF16 ? launch_t<BF16>(a, nprob, B, two, st) : launch_t<F32>(a, nprob, B, two, st);
}

hy_status launch_direct(const ConvPtrs* p, int nprob, const ConvShape& s, hipStream_t st) {
    FirProblem f[3];
    for (int i = 0; i < nprob; ++i) {
        f[i].a = p[i].k;
        f[i].b = s.gated ? p[i].v : nullptr;
        f[i].h = p[i].h;
        f[i].gate = s.gated ? p[i].q : nullptr;
        f[i].out = p[i].y;
        f[i].stride_ab = s.stride_kv();
        f[i].stride_gate = f[i].stride_out = s.stride_qy();
        f[i].lo = -(int64_t)s.history;
        f[i].hi = s.L;
    }
    const hy_status rc = launch_split_fir(f, nprob, s.B, s.L, s.D, s.lh, s.group, s.dtype, st);
    return rc == HY_ERR_UNSUPPORTED ? launch_fir(f, nprob, s.B, s.L, s.D, s.lh, s.group, s.dtype, st) : rc;
}

}  // namespace hy
