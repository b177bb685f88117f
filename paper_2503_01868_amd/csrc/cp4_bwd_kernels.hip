// Backward of the gated convolution for filters that are NOT shared by 16 channels (one filter per channel or
// per small group), on the gfx950 matrix cores, ONE pass over the tensors: the chunk-parallel scheme of App. A.1
// applied to the backward structure of App. A.4.  With u = k*v, g = dy*q:
//     dq[t] = dy[t] * z[t],   z[t] = sum_j h[j] u[t-j]
//     du[s] = sum_j h[j] g[s+j],  dk = du (.) v,  dv = du (.) k
//     dh[c, j] = sum_{b, t} g[b,t,c] u[b,t-j,c]
//
// All three contractions run as batched 4 x 4 x 4 products (v_mfma_f32_4x4x4_16B_bf16: 16 independent blocks per
// instruction, one channel per block).  The kernel walks the sequence from its end, tau = L-1-t, where du is causal and z
// anti-causal (mr_bwd_kernels.hip does the same for grouped filters), in groups of 16 steps, tau0 = 16 gamma:
//     du[tau] = sum_j h[j] g[tau-j]     DU[i][j] = sum_m sum_k A_m[i][k] g[tau0 + 4j - 4m + k],  A_m[i][k] = h[4m + i - k]
//     z[tau]  = sum_j h[j] u[tau+j]     Z[i][j]  = sum_m sum_k B_m[i][k] u[tau0 + 4j + 4m + k],  B_m[i][k] = h[4m + k - i]
//     dh[j]   = sum_tau g[tau] u[tau+j] D_a[i][j] += sum_k H[i][k] g[T + k - 4(3 - j) - 16a],    H[i][k] = u[T + i + k - 3],
//                                       entry (i, j) collects the lag 16a + 4(3 - j) + i - 3
// (h is zero outside [0, lh)).  A_m and B_m stay in registers for the whole tile, 2 VGPRs per m.  A column of a right operand
// is one aligned quad (4 steps of a channel): the operand of shift i of group gamma holds quad 4 gamma + j - i in column j.
// du of group gamma takes the operands (gamma - a, i) of g for m = 4a + i, dh the same ones for T = 16 gamma + 4(3 - i), and z
// of group gamma - 4 LAG, which is complete when group gamma is there, those of u at group gamma - 4 LAG + a for m = 4a - i.
// So a group's four operands are read from LDS once (8 bytes per lane each) and stay in a register window of up to 4 LAG + 1
// groups.
//
// What bounds it: 7 tensor passes through 128-byte row pieces (three launches, dq, then dk and dv, then dh, made 13).  A
// workgroup owns 64 channels with 8 waves, two per SIMD and of two kinds: four run du and dh (filter operands 66 registers,
// window 72, accumulators 36), four run z (operands 66, window 72) and move all data; one wave with everything does not
// fit 512 registers.  The pair issues 102 products per group and SIMD, so vector instructions between them count: windows
// formed from one read by selects and rotations inside lane quads, and H from neighbouring quads likewise, took 40
// instructions per group more and 160 us a call against 126 at 1 x 8192 x 4096, 128 taps (three launches: 217); a wave that
// divides once for all its filters saves 3 more (126 on average over a trace of 970 calls, the reduction's 5 among them; matrix
// cores 36%, vector ALUs 39%, LDS 29% busy; traffic 1.05 x).
//
// Time goes in chunks of 64 steps, one barrier each.  In iteration j the first four waves multiply chunk j and gate du with
// the chunk's k and v lines, dk and dv over k and v in place; the other four store dk, dv of chunk j - 1 and dq of chunk
// j - 1 - LAG, run z of chunk j - LAG (dq over dy in place) and write chunk j + 1 into the lines: every lane loads two rows
// x 8 channels of dy, q, k, v and writes g, u, k, v, dy transposed as bf16 [channel][time] lines, in the same places from
// which it read the results of the chunk before.  A tile walks LAG chunks of dy, q before its first step (du) and LAG of k, v
// past its last (z).  The filter gradient's tile owns the steps T + k of H, so it takes u from 3 steps before the tile, and
// the sequence's last tile 3 steps more.  Each tile leaves one partial row per channel (App. A.4); dh_reduce_kernel sums
// them over tiles and the channels of a group.
#include <type_traits>

#include "hy_common.hpp"
#include "hy_launch.hpp"

namespace hy {
namespace {

typedef short s16x4_t __attribute__((ext_vector_type(4)));

struct Cp4BwdArgs {
    const uint16_t* dy;
    const uint16_t* q;
    const uint16_t* k;
    const uint16_t* v;
    const float* h;
    uint16_t* dq;
    uint16_t* dk;
    uint16_t* dv;
    float* partial;  // [B * tiles_per_seq][D][lh]
    int64_t L, D;
    int64_t skv, sgq, sout;  // elements between batch items in k, v / dy, q / dq, dk, dv
    int32_t hist, fut;       // rows of k, v in front of row 0 / of dy, q behind row L - 1 that hold data
    int32_t lh, group;
    int32_t rows;           // time steps per workgroup, multiple of 64
    int32_t tiles_per_seq;  // ceil(L / rows)
    int32_t ncb;            // channel blocks = D / 64
};

constexpr int kT = 64;        // steps per chunk
constexpr int kNW = 4;        // waves of each kind per workgroup
constexpr int kC = 16 * kNW;  // channels per workgroup
// Bytes per channel line and 32 bytes (8 banks) more after every 8 lines: the transposing writes of a wave (8 lines 8
// apart x 8 neighbouring dwords) and its reads (16 neighbouring lines x 4 pieces) then both meet every bank once.
constexpr int kSkew = 32;
constexpr int kLS = 2 * 2 * kT + 32;  // k, v: two slots of 64 bf16 steps
constexpr int kRS = 4 * 2 * kT + 32;  // g, u: four slots and in front of them 16 steps, a copy of the ring's last; dy: four
constexpr int kFront = 32;            // bytes of that copy
constexpr int kLines = kC * kLS + kC / 8 * kSkew;
constexpr int kRing = kC * kRS + kC / 8 * kSkew;
constexpr int kTapStride = 140;  // floats per channel of the staged filters: 3 zeros, 129 taps, 8 zeros

__device__ __forceinline__ int line_off(int c, int stride) { return c * stride + (c >> 3) * kSkew; }

// one 4-step piece of a channel's line: two dwords, step 0 in the low half of the first
struct Quad {
    uint32_t w[2];
};
__device__ __forceinline__ s16x4_t operand(const Quad& x) { return __builtin_bit_cast(s16x4_t, x); }
__device__ __forceinline__ Quad quad_at(const char* p) { return __builtin_bit_cast(Quad, *reinterpret_cast<const uint2*>(p)); }

// NG = groups of 16 steps a filter reaches back; filters of up to 16 NG + 1 taps.  A product with a tap of zero carries a value
// that is not finite as far as NG reaches, so NG follows the filter (calls with 9 to 33 and 66 to 97 taps are also up to 11%
// faster than with the 4 or 8 groups of the window).  PF = chunks of loads in flight.  kShard: the call is one rank's share of
// a sequence (halo rows next to the tensors, batch strides).  kWide: a row is too long for the 24-bit products that place one.
template <int NG, int PF, bool kShard, bool kWide>
__global__ __launch_bounds__(2 * kNW * 64, 2) void cp4_bwd_kernel(Cp4BwdArgs a) {
    constexpr int LAG = (NG + 3) / 4;  // chunks between a chunk's arrival and its complete z
    constexpr int NBK = 4 * NG + 1;    // products per group and convolution
    constexpr int PPR = kC / 8;      // 16-byte pieces per row
    static_assert(kNW * 64 == PPR * (kT / 2), "one lane per (row pair, piece)");
    static_assert(LAG == 1 || LAG == 2, "the window and the dy ring hold up to two chunks");
    static_assert(PF == 1 || PF == 2, "one or two register stages");
    __shared__ __attribute__((aligned(16))) char kvlines[2 * kLines];
    __shared__ __attribute__((aligned(16))) char glines[kRing];
    __shared__ __attribute__((aligned(16))) char ulines[kRing];
    __shared__ __attribute__((aligned(16))) char ylines[kRing];
    static_assert(kC * kTapStride * 4 <= 2 * kLines, "the filters lie in the lines of k and v first");
    char* const klines = kvlines;
    char* const vlines = kvlines + kLines;
    float* const taps = reinterpret_cast<float*>(kvlines);

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
    const int t_floor = kShard ? -((a.fut + kT - 1) / kT) * kT : 0;
    const int t_begin = t_start - kT * LAG > t_floor ? t_start - kT * LAG : t_floor;
    const int tau_lo = kShard ? -a.fut : 0;      // smallest step at which dy and q hold data
    const int tau_hi = kShard ? L + a.hist : L;  // k and v hold data below this step
    const int ntot = (t_end - t_begin + kT - 1) / kT + LAG;

    const int64_t D = a.D;
    using Off = std::conditional_t<kWide, uint64_t, uint32_t>;  // bytes between rows of a chunk
    const Off row_bytes = (Off)D * 2;
    const int64_t cblock0 = (int64_t)cb * kC;
    const int64_t seq0 = (kShard ? b * a.sout : b * a.L * D) + cblock0;
    const int64_t seq0kv = kShard ? b * a.skv + cblock0 : seq0, seq0gq = kShard ? b * a.sgq + cblock0 : seq0;
    auto chunk_start = [&](int it) { return t_begin + it * kT; };
    auto in_tile = [&](int it) { return chunk_start(it) >= t_start && chunk_start(it) < t_end; };

    using std::integral_constant;

    // the steps before the walk's first chunk are zeros to the windows
    for (int i = tid; i < kC * kFront / 4; i += 2 * kNW * 64) {
        const int at = line_off(i / (kFront / 4), kRS) + i % (kFront / 4) * 4;
        *reinterpret_cast<uint32_t*>(glines + at) = 0u;
        *reinterpret_cast<uint32_t*>(ulines + at) = 0u;
    }

    // ---- the filters go through LDS (whole rows, all loads in flight), zeros around the taps instead of tests
    {
        constexpr int N = (kTapStride + 63) / 64, CW = kC / (2 * kNW);
        const uint32_t row = ((uint32_t)cblock0 + CW * wave + lane % CW) / (uint32_t)a.group;  // one division for all
        float f[CW][N];
#pragma unroll
        for (int c = 0; c < CW; ++c) {
            const float* hp = a.h + (int64_t)(uint32_t)__builtin_amdgcn_readlane(row, c) * a.lh;
#pragma unroll
            for (int i = 0; i < N; ++i) {
                const int tap = 64 * i + lane - 3;
                f[c][i] = hp[(uint32_t)tap < (uint32_t)a.lh ? tap : 0];
            }
        }
#pragma unroll
        for (int c = 0; c < CW; ++c)
#pragma unroll
            for (int i = 0; i < N; ++i) {
                const int x = 64 * i + lane;
                if (x < kTapStride) taps[(CW * wave + c) * kTapStride + x] = (uint32_t)(x - 3) < (uint32_t)a.lh ? f[c][i] : 0.0f;
            }
    }
    const int blk = lane >> 2, l4 = lane & 3;  // block = channel 16 w + blk; row i / column j of its products
    const int cw = 16 * w + blk;
    __syncthreads();
    // operand of shift i of group gamma in win[gamma % 16][i]; an entry is dead NG + 1 groups later
    s16x4_t ares[NBK], win[16][4];
#pragma unroll
    for (int x = 0; x < 16; ++x)
#pragma unroll
        for (int i = 0; i < 4; ++i) win[x][i] = s16x4_t{0, 0, 0, 0};
    const int ln = line_off(cw, kLS) + 8 * l4, rn = line_off(cw, kRS) + kFront + 8 * l4;
    auto push_group = [&](int G, const char* p) {  // G and p's offset are constants after unrolling
#pragma unroll
        for (int i = 0; i < 4; ++i) win[G][i] = operand(quad_at(p - 8 * i));
    };
    // 4 steps of a result, gated by the same steps of a line
    auto gated = [](const f32x4_t& x, const Quad& y) {
        return make_uint2(pack_bf16x2(x[0] * bf16_lo(y.w[0]), x[1] * bf16_hi(y.w[0])),
                          pack_bf16x2(x[2] * bf16_lo(y.w[1]), x[3] * bf16_hi(y.w[1])));
    };

    if (wave < kNW) {
        // ================= du and dh
        {
            const float* p = taps + cw * kTapStride + l4;  // h[4m + l4 - 3 ..]
#pragma unroll
            for (int m = 0; m < NBK; ++m)
                ares[m] = operand(Quad{{pack_bf16x2(p[4 * m + 3], p[4 * m + 2]), pack_bf16x2(p[4 * m + 1], p[4 * m])}});
        }
        __syncthreads();
        // H of 4 steps: the dwords from step l4 - 3, rounded down to even, on; rows that start at an odd step shift by one
        const char* const h_lane = ulines + line_off(cw, kRS) + kFront + 4 * ((l4 - 3) >> 1);
        const uint32_t h_shift = (l4 - 3) & 1 ? 16u : 0u;
        const int e_end = t_end == L ? L + 3 : t_end;  // the tile's steps T + k of H
        f32x4_t dacc[NG + 1];
#pragma unroll
        for (int x = 0; x <= NG; ++x) dacc[x] = f32x4_t{0.0f, 0.0f, 0.0f, 0.0f};

        auto step = [&](auto slot_c, int it) {
            constexpr int SL = decltype(slot_c)::value;  // it % 4
            const int T = chunk_start(it);
            auto group = [&](auto n_c) {
                constexpr int n = decltype(n_c)::value, G = 4 * SL + n;
                push_group(G, glines + rn + 32 * G);
                if (T + 16 * n >= t_start && T + 16 * n < e_end) {
                    const int off = ln + (SL & 1) * 2 * kT + 32 * n;
                    const Quad k4 = quad_at(klines + off), v4 = quad_at(vlines + off);
                    uint32_t d[9];
#pragma unroll
                    for (int x = 0; x < 9; ++x) d[x] = *reinterpret_cast<const uint32_t*>(h_lane + 32 * G + 4 * x);
                    s16x4_t hk[4];
#pragma unroll
                    for (int kq = 0; kq < 4; ++kq) {
                        Quad x{{__builtin_amdgcn_alignbit(d[2 * kq + 1], d[2 * kq], h_shift),
                                __builtin_amdgcn_alignbit(d[2 * kq + 2], d[2 * kq + 1], h_shift)}};
                        if constexpr (kShard) {  // steps past the shard's are real data, but not its own
                            const int rem = L - (T + 16 * n + 4 * kq + l4 - 3);
                            x.w[0] &= rem >= 2 ? 0xffffffffu : (rem == 1 ? 0x0000ffffu : 0u);
                            x.w[1] &= rem >= 4 ? 0xffffffffu : (rem == 3 ? 0x0000ffffu : 0u);
                        }
                        hk[kq] = operand(x);
                    }
                    f32x4_t du[2] = {{0.0f, 0.0f, 0.0f, 0.0f}, {0.0f, 0.0f, 0.0f, 0.0f}};
#pragma unroll
                    for (int i = 0; i < 4; ++i)
#pragma unroll
                        for (int x = 0; x <= NG; ++x) {
                            const s16x4_t g4 = win[(G - x) & 15][i];
                            dacc[x] = __builtin_amdgcn_mfma_f32_4x4x4bf16_1k(hk[3 - i], g4, dacc[x], 0, 0, 0);
                            if (x < NG || i == 0)
                                du[x & 1] = __builtin_amdgcn_mfma_f32_4x4x4bf16_1k(ares[x < NG ? 4 * x + i : 4 * NG], g4, du[x & 1], 0, 0, 0);
                        }
                    const f32x4_t d4 = du[0] + du[1];
                    *reinterpret_cast<uint2*>(klines + off) = gated(d4, v4);  // dk
                    *reinterpret_cast<uint2*>(vlines + off) = gated(d4, k4);  // dv
                }
            };
            group(integral_constant<int, 0>{});
            group(integral_constant<int, 1>{});
            group(integral_constant<int, 2>{});
            group(integral_constant<int, 3>{});
            __syncthreads();
        };
        __syncthreads();  // chunk 0 is in the lines
        for (int it = 0;; it += 4) {
            step(integral_constant<int, 0>{}, it);
            if (it + 1 >= ntot) break;
            step(integral_constant<int, 1>{}, it + 1);
            if (it + 2 >= ntot) break;
            step(integral_constant<int, 2>{}, it + 2);
            if (it + 3 >= ntot) break;
            step(integral_constant<int, 3>{}, it + 3);
            if (it + 4 >= ntot) break;
        }
        // ---- the lane holds dh[c][16 x + 4 (3 - l4) + i - 3], i = 0..3
        float* out = a.partial + ((int64_t)tile * D + cblock0 + cw) * a.lh;
#pragma unroll
        for (int x = 0; x <= NG; ++x) {
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                const int j = 16 * x + 9 - 4 * l4 + i;
                if (j >= 0 && j < a.lh) out[j] = dacc[x][i];
            }
        }
    } else {
        // ================= z, and all data movement: rows 2 rp, 2 rp + 1 of a chunk, channels 8 lp .. 8 lp + 7
        const int mt = tid - kNW * 64;
        const int lp = mt % PPR, rp = mt / PPR;
        // Addresses are a uniform base, the first row of a chunk in memory, and a byte offset per lane (of 32 bits, see kWide);
        // rows outside [lo, hi] become the nearest one, so a chunk that lies wholly outside reads one row piece.
        struct Rows {
            int64_t base;  // elements from the batch item's start
            Off off[2];    // bytes
        };
        auto rows_at = [&](int T, int lo, int hi) {
            int first = L - kT - T;
            first = first > lo ? first : lo;
            first = first < hi ? first : hi;
            Rows r;
            r.base = (int64_t)first * D;
#pragma unroll
            for (int i = 0; i < 2; ++i) {
                int t = L - 1 - T - 2 * rp - i;
                t = t > first ? t : first;
                t = t < hi ? t : hi;
                if constexpr (kWide) r.off[i] = (Off)(t - first) * row_bytes + 16 * lp;
                else r.off[i] = __umul24((uint32_t)(t - first), row_bytes) + 16 * lp;
            }
            return r;
        };
        auto ld = [](const uint16_t* p, Off off) { return load_words_nt<4>(reinterpret_cast<const char*>(p) + off); };
        auto st = [](uint16_t* p, Off off, const Words<4>& x) { store_words_nt<4>(reinterpret_cast<char*>(p) + off, x); };

        Words<4> yw[PF][2], qw[PF][2], kw[PF][2], vw[PF][2];  // chunk it in stage it % PF
        const int u_lo = t_start > 4 ? t_start - 4 : 0;
        const int u_end = t_begin + ntot * kT < tau_hi ? t_begin + ntot * kT : tau_hi;  // one past the last step of k, v needed
        auto load_rows = [&](auto st_c, int it) {
            constexpr int ST = decltype(st_c)::value % PF;
            const Rows rg = rows_at(chunk_start(it), L - t_end, L - 1 - tau_lo);
            const Rows ru = rows_at(chunk_start(it), L - u_end, L - 1 - u_lo);
            const uint16_t *py = a.dy + seq0gq + rg.base, *pq = a.q + seq0gq + rg.base;
            const uint16_t *pk = a.k + seq0kv + ru.base, *pv = a.v + seq0kv + ru.base;
#pragma unroll
            for (int r = 0; r < 2; ++r) {
                yw[ST][r] = ld(py, rg.off[r]);
                qw[ST][r] = ld(pq, rg.off[r]);
                kw[ST][r] = ld(pk, ru.off[r]);
                vw[ST][r] = ld(pv, ru.off[r]);
            }
        };
        load_rows(integral_constant<int, 0>{}, 0);
        if constexpr (PF == 2) load_rows(integral_constant<int, 1>{}, 1);
        {
            const float* p = taps + cw * kTapStride + 3 - l4;  // h[4m - l4 ..]
#pragma unroll
            for (int m = 0; m < NBK; ++m)
                ares[m] = operand(Quad{{pack_bf16x2(p[4 * m], p[4 * m + 1]), pack_bf16x2(p[4 * m + 2], p[4 * m + 3])}});
        }
        __syncthreads();

        const int l_wr = line_off(8 * lp, kLS) + 4 * rp, r_wr = line_off(8 * lp, kRS) + 4 * rp;
        // x = a*b of 2 rows x 8 channels, transposed: one dword (2 steps) per channel, steps outside `keep` zero
        auto product = [](const Words<4> (&a2)[2], const Words<4> (&b2)[2], uint32_t keep, uint32_t (&x)[8]) {
#pragma unroll
            for (int p = 0; p < 4; ++p) {
                x[2 * p] = keep & pack_bf16x2(bf16_lo(a2[0].w[p]) * bf16_lo(b2[0].w[p]), bf16_lo(a2[1].w[p]) * bf16_lo(b2[1].w[p]));
                x[2 * p + 1] = keep & pack_bf16x2(bf16_hi(a2[0].w[p]) * bf16_hi(b2[0].w[p]), bf16_hi(a2[1].w[p]) * bf16_hi(b2[1].w[p]));
            }
        };
        auto write8 = [](char* lines, const uint32_t (&x)[8]) {
#pragma unroll
            for (int e = 0; e < 8; ++e) *reinterpret_cast<uint32_t*>(lines + e * kRS) = x[e];
        };
        auto write_raw = [&](char* lines, int stride, const Words<4> (&x)[2]) {
#pragma unroll
            for (int p = 0; p < 4; ++p) {
                *reinterpret_cast<uint32_t*>(lines + (2 * p) * stride) = __builtin_amdgcn_perm(x[1].w[p], x[0].w[p], 0x05040100u);
                *reinterpret_cast<uint32_t*>(lines + (2 * p + 1) * stride) = __builtin_amdgcn_perm(x[1].w[p], x[0].w[p], 0x07060302u);
            }
        };
        auto read_raw = [&](const char* lines, int stride, Words<4> (&x)[2]) {
#pragma unroll
            for (int p = 0; p < 4; ++p) {
                const uint32_t c0 = *reinterpret_cast<const uint32_t*>(lines + (2 * p) * stride);
                const uint32_t c1 = *reinterpret_cast<const uint32_t*>(lines + (2 * p + 1) * stride);
                x[0].w[p] = __builtin_amdgcn_perm(c1, c0, 0x05040100u);
                x[1].w[p] = __builtin_amdgcn_perm(c1, c0, 0x07060302u);
            }
        };
        auto write_chunk = [&](auto slot_c, int it) {
            constexpr int SL = decltype(slot_c)::value, ST = SL % PF;
            const int tau = chunk_start(it) + 2 * rp;
            auto steps = [](bool a0, bool a1) { return (a0 ? 0x0000ffffu : 0u) | (a1 ? 0xffff0000u : 0u); };
            auto has_g = [&](int t) { return t < t_end && (!kShard || t >= tau_lo); };
            auto has_u = [&](int t) { return t >= u_lo && t < tau_hi; };
            uint32_t gx[8], ux[8];
            product(yw[ST], qw[ST], steps(has_g(tau), has_g(tau + 1)), gx);
            product(kw[ST], vw[ST], steps(has_u(tau), has_u(tau + 1)), ux);
            write8(glines + r_wr + kFront + SL * 2 * kT, gx);
            write8(ulines + r_wr + kFront + SL * 2 * kT, ux);
            if constexpr (SL == 3) {
                if (rp >= (2 * kT - kFront) / 4) {  // the copy in front of the ring
                    write8(glines + r_wr + kFront - 2 * kT, gx);
                    write8(ulines + r_wr + kFront - 2 * kT, ux);
                }
            }
            write_raw(klines + l_wr + (SL & 1) * 2 * kT, kLS, kw[ST]);
            write_raw(vlines + l_wr + (SL & 1) * 2 * kT, kLS, vw[ST]);
            write_raw(ylines + r_wr + SL * 2 * kT, kRS, yw[ST]);
        };
        // dk, dv of the chunk before iteration `it`, dq of the one LAG chunks older
        auto store_chunk = [&](auto slot_c, int it) {
            constexpr int PV = (decltype(slot_c)::value + 3) & 3, DQ = (PV + 4 - LAG) & 3;
            if (it > 0 && in_tile(it - 1)) {
                const int T = chunk_start(it - 1);
                const Rows ro = rows_at(T, L - t_end, L - 1);
                Words<4> x[2], y[2];
                read_raw(klines + l_wr + (PV & 1) * 2 * kT, kLS, x);
                read_raw(vlines + l_wr + (PV & 1) * 2 * kT, kLS, y);
#pragma unroll
                for (int r = 0; r < 2; ++r)
                    if (T + 2 * rp + r < t_end) {
                        st(a.dk + seq0 + ro.base, ro.off[r], x[r]);
                        st(a.dv + seq0 + ro.base, ro.off[r], y[r]);
                    }
            }
            if (it > LAG && in_tile(it - 1 - LAG)) {
                const int T = chunk_start(it - 1 - LAG);
                const Rows ro = rows_at(T, L - t_end, L - 1);
                Words<4> x[2];
                read_raw(ylines + r_wr + DQ * 2 * kT, kRS, x);
#pragma unroll
                for (int r = 0; r < 2; ++r)
                    if (T + 2 * rp + r < t_end) st(a.dq + seq0 + ro.base, ro.off[r], x[r]);
            }
        };
        auto step = [&](auto slot_c, int it) {
            constexpr int SL = decltype(slot_c)::value;  // it % 4
            constexpr int DQ = (SL + 4 - LAG) & 3;
            store_chunk(slot_c, it);
            const bool done = it >= LAG && in_tile(it - LAG);
            auto group = [&](auto n_c) {
                constexpr int n = decltype(n_c)::value, G = 4 * SL + n;
                push_group(G, ulines + rn + 32 * G);
                if (done) {
                    char* const yl = ylines + rn - kFront + DQ * 2 * kT + 32 * n;
                    const Quad y4 = quad_at(yl);
                    f32x4_t z[2] = {{0.0f, 0.0f, 0.0f, 0.0f}, {0.0f, 0.0f, 0.0f, 0.0f}};  // two chains: a product's result is late for the next
#pragma unroll
                    for (int x = 0; x <= NG; ++x)
#pragma unroll
                        for (int i = 0; i < 4; ++i)
                            if (x > 0 || i == 0)
                                z[i & 1] = __builtin_amdgcn_mfma_f32_4x4x4bf16_1k(ares[x > 0 ? 4 * x - i : 0], win[(G - 4 * LAG + x) & 15][i], z[i & 1], 0, 0, 0);
                    *reinterpret_cast<uint2*>(yl) = gated(z[0] + z[1], y4);  // dq
                }
            };
            group(integral_constant<int, 0>{});
            group(integral_constant<int, 1>{});
            group(integral_constant<int, 2>{});
            group(integral_constant<int, 3>{});
            if (it + 1 < ntot) {
                write_chunk(integral_constant<int, (SL + 1) & 3>{}, it + 1);
                load_rows(integral_constant<int, SL + 1>{}, it + 1 + PF);
            }
            __syncthreads();
        };
        write_chunk(integral_constant<int, 0>{}, 0);
        load_rows(integral_constant<int, 0>{}, PF);
        __syncthreads();
        for (int it = 0;; it += 4) {
            step(integral_constant<int, 0>{}, it);
            if (it + 1 >= ntot) { store_chunk(integral_constant<int, 1>{}, it + 1); break; }
            step(integral_constant<int, 1>{}, it + 1);
            if (it + 2 >= ntot) { store_chunk(integral_constant<int, 2>{}, it + 2); break; }
            step(integral_constant<int, 2>{}, it + 2);
            if (it + 3 >= ntot) { store_chunk(integral_constant<int, 3>{}, it + 3); break; }
            step(integral_constant<int, 3>{}, it + 3);
            if (it + 4 >= ntot) { store_chunk(integral_constant<int, 0>{}, it + 4); break; }
        }
    }
}

int64_t bwd_rows(const BwdShape& s) {
    const int64_t ncb = s.D / kC;
    int64_t rows = tuning().mr_rows;
    if (rows <= 0) {
        rows = one_round_rows(s.B * ncb, s.L, 8 * kT, kT);
        // as short as the longer halo: each tile also leaves partial rows (half or twice that: the same times within 5%)
        if (rows < 2 * kT) rows = 2 * kT;
    }
    rows = (rows + kT - 1) / kT * kT;
    const int64_t cap = (s.L + kT - 1) / kT * kT;
    return rows > cap ? cap : rows;
}

}  // namespace

bool cp4_bwd_supported(const BwdShape& s) {
    return s.gated && s.dtype == HY_BF16 && s.D % 128 == 0 && s.lh > 8 && s.lh <= 129 && s.L <= 0x7fff0000LL && s.D <= 0x7fff0000LL;
}

int64_t cp4_bwd_workspace_bytes(const BwdShape& s) {
    const int64_t rows = bwd_rows(s);
    const int64_t tiles = (s.L + rows - 1) / rows;
    return s.B * tiles * s.D * s.lh * (int64_t)sizeof(float);
}

// dq, dk, dv and dh in one pass.  `ws` holds the partial filter gradients.
hy_status launch_cp4_bwd(const BwdPtrs& p, const BwdShape& s, void* ws, hipStream_t st) {
    if (!cp4_bwd_supported(s)) return HY_ERR_UNSUPPORTED;
    Cp4BwdArgs a;
    a.dy = static_cast<const uint16_t*>(p.dy);
    a.q = static_cast<const uint16_t*>(p.q);
    a.k = static_cast<const uint16_t*>(p.k);
    a.v = static_cast<const uint16_t*>(p.v);
    a.h = p.h;
    a.dq = static_cast<uint16_t*>(p.dq);
    a.dk = static_cast<uint16_t*>(p.dk);
    a.dv = static_cast<uint16_t*>(p.dv);
    a.partial = static_cast<float*>(ws);
    a.L = s.L;
    a.D = s.D;
    a.skv = s.stride_kv();
    a.sgq = s.stride_gq();
    a.sout = s.stride_out();
    a.hist = s.history;
    a.fut = s.future;
    a.lh = s.lh;
    a.group = s.group;
    a.ncb = (int32_t)(s.D / kC);
    a.rows = (int32_t)bwd_rows(s);
    a.tiles_per_seq = (int32_t)((s.L + a.rows - 1) / a.rows);
    const int64_t nsets = s.B * a.tiles_per_seq;
    const int64_t nb = nsets * a.ncb;
    if (nb > 0x7fffffffLL) return HY_ERR_UNSUPPORTED;
    const dim3 grid((uint32_t)nb), block(2 * kNW * 64);
    // Up to 65 taps one chunk of history instead of two: half the halo, and room for a second chunk of loads in flight
    // (with two chunks of history and 8 groups one chunk in flight already spills 4 registers).  Against the three launches
    // (dq; dk and dv; dh) on 40 shapes of 64 to 8192 channels and up to 2^25 elements: 1.4 to 2.6 times as fast, nothing slower.
    auto launch = [&](auto ng) {
        constexpr int NG = decltype(ng)::value, PF = NG <= 4 ? 2 : 1;
        // rows of 2^24 bytes and more: the shards' kernel (1 x 70 x 2^23, 65 taps 6.4 ms; the general kernel 26.7)
        if (s.D >= 1 << 23) return launch_kernel((cp4_bwd_kernel<NG, PF, true, true>), grid, block, st, a);
        return s.sharded() ? launch_kernel((cp4_bwd_kernel<NG, PF, true, false>), grid, block, st, a)
                           : launch_kernel((cp4_bwd_kernel<NG, PF, false, false>), grid, block, st, a);
    };
    using std::integral_constant;
    const hy_status rc = s.lh <= 17   ? launch(integral_constant<int, 1>{})
                         : s.lh <= 33 ? launch(integral_constant<int, 2>{})
                         : s.lh <= 65 ? launch(integral_constant<int, 4>{})
                         : s.lh <= 97 ? launch(integral_constant<int, 6>{})
                                      : launch(integral_constant<int, 8>{});
    if (rc != HY_OK) return rc;
    const DhReduce r{static_cast<const float*>(ws), p.dh, nsets, s.D, s.lh, s.group};
    return launch_dh_reduce(&r, 1, st);
}

}  // namespace hy
