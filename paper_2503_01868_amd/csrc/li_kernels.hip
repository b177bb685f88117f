// Hyena-LI forward on gfx950: gated causal convolution with the long implicit filter of Sec. 2.1,
//   h[g, j] = sum_{n < order} R[g, n] * lambda[g, n]^j,   j = 0 .. L-1  (as long as the sequence).
// The filter is never materialised.  Because it is a sum of real exponentials, everything older than the
// current 32-step chunk acts through `order` running sums per channel (the recurrent form the paper
// mentions for this operator), and the whole operator becomes three small dense products per chunk:
//   z_chunk = T u_chunk + Q s,        T[t, i] = h[t - i] (lower triangular, 32 x 32: the H_0 of Sec. 3.1),
//                                      Q[t, n] = R_n lambda_n^(t+1),
//   s'      = Lambda^32 s + P u_chunk, P[n, i] = lambda_n^(31-i),   s[n, c] = sum_{i<=end} lambda_n^(end-i) u[i, c].
// With 16 channels of one filter group on a matrix tile (as in mr_kernels.hip) these are v_mfma_f32_16x16x32_bf16,
// two for T, two for P and four for Q; s stays in fp32 accumulators and enters the Q product split into a bf16 head
// and a bf16 remainder, as do the coefficients of P and Q, so carrying the state over 10^5 steps costs no precision
// beyond 16 bits of the coefficients.  The state product comes out with 4 consecutive n of one channel per lane:
// head and remainder of the state, side by side, are the operand of the Q product, and the state never leaves its
// registers.
//
// The recurrence runs along time, and one GPU needs more than B * D / 256 workgroups, so the sequence is cut
// into tiles and scanned in two passes (the classic chunked scan): pass 1 walks every tile but the last of
// each sequence with a zero start and leaves the tile's final state in a workspace (reads k and v only);
// pass 2 rebuilds its start state from the tiles before it, s_in = sum_tau Lambda^(rows * (tile-1-tau)) s_tau
// (a short Horner loop over 1 KiB records), and computes y.  With a single tile per sequence pass 1 is skipped;
// tiles short enough to be kept on chip between the passes are done in one (li_one_pass_kernel).
// Data movement per chunk is that of mr_kernels.hip: whole row pieces, u and z through LDS, one barrier.
#include <type_traits>

#include "hy_common.hpp"
#include "hy_launch.hpp"

namespace hy {
namespace {

struct LiArgs {
    const uint16_t* q;
    const uint16_t* k;
    const uint16_t* v;
    const float* R;
    const float* lam;
    uint16_t* y;
    float* ws;              // [B][tiles_per_seq - 1][D / 16][64 lanes][4] end-of-tile states
    const float* s_in;      // [B][D / 16][64 lanes][4] running sums before the first step (nullptr: zero)
    float* s_out;           // same layout: running sums after the last step (nullptr: not wanted)
    int64_t L, D;
    int32_t order, group;
    int32_t rows;           // time steps per workgroup, multiple of 32
    int32_t tiles_per_seq;  // ceil(L / rows)
    int32_t ncb;            // channel blocks = D / (16 NW)
    int32_t polls;          // li_one_pass_kernel: looks at an earlier tile's state before a wave computes it itself
};

constexpr int kChunk = 32;
constexpr int kMaxOrder = 16;

__device__ __forceinline__ float powi(float x, int e) {  // x^e, e >= 0, by squaring
    float r = 1.0f;
    while (e > 0) {
        if (e & 1) r *= x;
        x *= x;
        e >>= 1;
    }
    return r;
}

// T operands: tile x (steps 16x..16x+15 of the chunk) against the chunk's 32 source steps; lane (li = step,
// lq = source octet), element e = h[16x + li - 8lq - e].  `h` holds the filter's first 32 values.
__device__ __forceinline__ void t_operands(bf16x8_t (&tz)[2], const float* h, int li, int lq) {
#pragma unroll
    for (int x = 0; x < 2; ++x) {
        Words<4> wds;
#pragma unroll
        for (int e2 = 0; e2 < 4; ++e2) {
            const int i0 = 16 * x + li - 8 * lq - 2 * e2;
            const int i1 = i0 - 1;
            const float f0 = (i0 >= 0 && i0 < kChunk) ? h[i0] : 0.0f;
            const float f1 = (i1 >= 0 && i1 < kChunk) ? h[i1] : 0.0f;
            wds.w[e2] = pack_bf16x2(f0, f1);
        }
        tz[x] = __builtin_bit_cast(bf16x8_t, wds);
    }
}

// P operand: lane (li = n, lq = source octet), element e = lambda_n^(31 - 8lq - e), as a bf16 head and a bf16
// remainder.  The exponentials of a filter may nearly cancel (close poles, residues of opposite sign); each
// one's running sum therefore has to be accurate well beyond bf16, or the error of the individual terms shows
// at full size in their small difference.  The same holds for the Q operands below.
__device__ __forceinline__ void p_operands(bf16x8_t& pop, bf16x8_t& pop_lo, const float* lam, int li, int lq) {
    const float ln = lam[li];
    Words<4> wds, wlo;
    float pw = powi(ln, 31 - 8 * lq - 7);  // smallest exponent of the lane (element 7), then multiply up
    float pe[8];
#pragma unroll
    for (int e = 7; e >= 0; --e) {
        pe[e] = pw;
        pw *= ln;
    }
#pragma unroll
    for (int e2 = 0; e2 < 4; ++e2) {
        wds.w[e2] = pack_bf16x2(pe[2 * e2], pe[2 * e2 + 1]);
        wlo.w[e2] = pack_bf16x2(pe[2 * e2] - bf16_lo(wds.w[e2]), pe[2 * e2 + 1] - bf16_hi(wds.w[e2]));
    }
    pop = __builtin_bit_cast(bf16x8_t, wds);
    pop_lo = __builtin_bit_cast(bf16x8_t, wlo);
}

// Q operands: lane (li = step of tile x, lq), R_n lambda_n^(16x + li + 1), n = 4lq + e: remainders in the elements 0..3, heads
// in 4..7
__device__ __forceinline__ void q_operands(bf16x8_t (&qop)[2], const float* res, const float* lam, int li, int lq) {
#pragma unroll
    for (int x = 0; x < 2; ++x) {
        float qe[4];
#pragma unroll
        for (int e = 0; e < 4; ++e) qe[e] = res[4 * lq + e] * powi(lam[4 * lq + e], 16 * x + li + 1);
        Words<4> wds;
        wds.w[2] = pack_bf16x2(qe[0], qe[1]);
        wds.w[3] = pack_bf16x2(qe[2], qe[3]);
        wds.w[0] = pack_bf16x2(qe[0] - bf16_lo(wds.w[2]), qe[1] - bf16_hi(wds.w[2]));
        wds.w[1] = pack_bf16x2(qe[2] - bf16_lo(wds.w[3]), qe[3] - bf16_hi(wds.w[3]));
        qop[x] = __builtin_bit_cast(bf16x8_t, wds);
    }
}

// z of a chunk: steps 16x + li of channels 4 lq .. 4 lq + 3 of the wave in acc[x].
// Head and remainder of the state lie side by side in one operand, remainder and head of Q in the other: one product adds head
// times remainder and remainder times head, a second one, with the state's parts exchanged, the heads and the remainders.
// All products of this file have one shape, 16x16x32, and no 16x16x16 product feeds one of them or takes its sum: on gfx950
// a 16x16x16 product that accumulates onto the result of a 16x16x32 product fewer than 5 wait states old read the register's
// previous contents, and a 16x16x32 product that accumulates onto the result of a 16x16x16 product 4 wait states old, with no
// other product between, left the upper two registers of its result wrong in some waves (both measured).  The compiler does
// not always keep such a distance; tests/test_isa_hazards.py looks for either pair in the generated code.
__device__ __forceinline__ void chunk_outputs(f32x4_t (&acc)[2], const f32x4_t& s, const bf16x8_t& uw, const bf16x8_t (&tz)[2],
                                              const bf16x8_t (&qop)[2]) {
    Words<4> a, b;
    a.w[0] = b.w[2] = pack_bf16x2(s[0], s[1]);
    a.w[1] = b.w[3] = pack_bf16x2(s[2], s[3]);
    a.w[2] = b.w[0] = pack_bf16x2(s[0] - bf16_lo(a.w[0]), s[1] - bf16_hi(a.w[0]));
    a.w[3] = b.w[1] = pack_bf16x2(s[2] - bf16_lo(a.w[1]), s[3] - bf16_hi(a.w[1]));
    const bf16x8_t s1 = __builtin_bit_cast(bf16x8_t, a), s2 = __builtin_bit_cast(bf16x8_t, b);
    acc[0] = acc[1] = f32x4_t{0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
    for (int x = 0; x < 2; ++x) acc[x] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(s1, qop[x], acc[x], 0, 0, 0);
#pragma unroll
    for (int x = 0; x < 2; ++x) acc[x] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(s2, qop[x], acc[x], 0, 0, 0);
#pragma unroll
    for (int x = 0; x < 2; ++x) acc[x] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(uw, tz[x], acc[x], 0, 0, 0);
}

// s' = Lambda^32 s + P u
__device__ __forceinline__ void advance(f32x4_t& s, const float (&lam32)[4], const bf16x8_t& pop, const bf16x8_t& pop_lo,
                                        const bf16x8_t& uw) {
#pragma unroll
    for (int r = 0; r < 4; ++r) s[r] *= lam32[r];
    s = __builtin_amdgcn_mfma_f32_16x16x32_bf16(pop, uw, s, 0, 0, 0);
    s = __builtin_amdgcn_mfma_f32_16x16x32_bf16(pop_lo, uw, s, 0, 0, 0);
}

// k*v of 8 channels of a row, rounded to bf16
__device__ __forceinline__ uint4 products(const Words<4>& kk, const Words<4>& vv) {
    float kf[8], vf[8];
    Pack<BF16, 8>::unpack(kk, kf);
    Pack<BF16, 8>::unpack(vv, vf);
    uint32_t x[4];
#pragma unroll
    for (int e = 0; e < 4; ++e) x[e] = pack_bf16x2(kf[2 * e] * vf[2 * e], kf[2 * e + 1] * vf[2 * e + 1]);
    return make_uint4(x[0], x[1], x[2], x[3]);
}

// element e of a lane = u[row 8 lq + e][channel 16 w + li] of a staged chunk (rd_piece: the lane's piece of a row)
template <int PPR>
__device__ __forceinline__ bf16x8_t transposed(const uint4* stage, int rd_piece, int li, int lq) {
    const uint16_t* s16 = reinterpret_cast<const uint16_t*>(stage);
    Words<4> wds;
#pragma unroll
    for (int e2 = 0; e2 < 4; ++e2) {
        const int r0 = 8 * lq + 2 * e2;
        const uint32_t lo = s16[((r0 * PPR + rd_piece) << 3) + (li & 7)];
        const uint32_t hi = s16[(((r0 + 1) * PPR + rd_piece) << 3) + (li & 7)];
        wds.w[e2] = lo | (hi << 16);
    }
    return __builtin_bit_cast(bf16x8_t, wds);
}

// kStateOnly: pass 1 (no q, no output, the tile's final state goes to the workspace).
template <int NW, int kPrefetch, bool kStateOnly>
__global__ __launch_bounds__(NW * 64, NW == 16 ? 4 : 2) void li_mfma_kernel(LiArgs a) {
    constexpr int PPR = 2 * NW;             // 16-byte pieces per staged row of u (bf16)
    constexpr int ZROW = 16 * NW * 4 + 16;  // bytes per staged row of z (fp32), padded against bank conflicts
    static_assert(NW % 4 == 0, "the LDS swizzle needs 8 pieces per row");
    __shared__ uint4 stage[2][kChunk * PPR];
    __shared__ __attribute__((aligned(16))) char zst[kStateOnly ? 1 : 2][kStateOnly ? 16 : kChunk * ZROW];
    __shared__ float rs[NW][kMaxOrder], ls[NW][kMaxOrder], hs[NW][kChunk];

    const int tid = threadIdx.x;
    const int w = tid / 64, lane = tid % 64;
    const int li = lane % 16, lq = lane / 16;

    const uint32_t lb = blockIdx.x;
    const int cb = lb % a.ncb;
    const int64_t tl = lb / a.ncb;
    const int tiles_run = kStateOnly ? a.tiles_per_seq - 1 : a.tiles_per_seq;  // pass 1 skips the last tile
    const int64_t b = tl / tiles_run;
    const int tile = (int)(tl % tiles_run);
    const int64_t t_start = (int64_t)tile * a.rows;
    const int64_t t_end = (t_start + a.rows < a.L) ? t_start + a.rows : a.L;
    const int nchunks = (int)((t_end - t_start + kChunk - 1) / kChunk);

    const int64_t D = a.D;
    const int64_t cblock0 = (int64_t)cb * 16 * NW;
    const int64_t c0 = cblock0 + 16 * w;
    const int64_t seq0 = b * a.L * D;

    const int lr = tid / PPR, lp = tid % PPR;
    const int64_t ld_off = cblock0 + 8 * lp;
    // unconditional, clamped loads (see mr_kernels.hip): rows past the end of the tile re-read its last row; loads
    // for chunk indices past the last chunk (results unused) all go to one 16-byte location of the tile
    const int64_t idle_off = (t_end - 1) * D + cblock0;
    auto load_kv = [&](int ci, Words<4>& kk, Words<4>& vv) {
        int64_t t = t_start + (int64_t)ci * kChunk + lr;
        t = t < t_end ? t : t_end - 1;
        const int64_t off = ci < nchunks ? t * D + ld_off : idle_off;
        kk = load_words_nt<4>(a.k + seq0 + off);
        vv = load_words_nt<4>(a.v + seq0 + off);
    };
    auto load_q = [&](int ci, Words<4>& qq) {
        int64_t t = t_start + (int64_t)ci * kChunk + lr;
        t = t < t_end ? t : t_end - 1;
        qq = load_words_nt<4>(a.q + seq0 + (ci < nchunks ? t * D + ld_off : idle_off));
    };

    Words<4> kpre[kPrefetch], vpre[kPrefetch], qpre[kPrefetch];
#pragma unroll
    for (int i = 0; i < kPrefetch; ++i) {
        load_kv(i, kpre[i], vpre[i]);
        if constexpr (!kStateOnly)
            if (i + 1 < kPrefetch) load_q(i, qpre[i]);
    }

    // ---- per-wave filter set-up: residues and poles of the wave's group, taps 0..31 of the implicit filter
    {
        const int64_t g = c0 / a.group;
        if (lane < kMaxOrder) {
            rs[w][lane] = lane < a.order ? a.R[g * a.order + lane] : 0.0f;
            ls[w][lane] = lane < a.order ? a.lam[g * a.order + lane] : 0.0f;
        }
    }
    __syncthreads();
    // ---- start state: zero at the start of a sequence, else the Horner sum over the earlier tiles' end states,
    // sixteen records per round (the loads do not depend on the running sum, only the FMAs do; indices past the
    // last record are clamped so that the loads stay unconditional), so that up to sixteen earlier tiles cost one
    // memory latency.  Done before the operands are built, while few registers are live.
    // state layout: lane (li = channel, lq) holds s[n = 4lq + r][channel], r = 0..3
    f32x4_t s = {0.0f, 0.0f, 0.0f, 0.0f};
    const int64_t ws_wave = ((c0 / 16) * 64 + lane) * 4;  // this lane's 4 floats inside one (b, tile) record set
    const int64_t ws_tile = (D / 16) * 256;               // floats per (b, tile)
    if constexpr (!kStateOnly) {
        if (a.s_in) {  // a call that continues a sequence: what the steps before it left behind decays like any state
            const float4 c4 = *reinterpret_cast<const float4*>(a.s_in + b * ws_tile + ws_wave);
            s = f32x4_t{c4.x, c4.y, c4.z, c4.w};
        }
        float lam_rows[4];
#pragma unroll
        for (int r = 0; r < 4; ++r) lam_rows[r] = powi(ls[w][4 * lq + r], a.rows);
        const float* wp = a.ws + b * (a.tiles_per_seq - 1) * ws_tile + ws_wave;
        for (int tau0 = 0; tau0 < tile; tau0 += 16) {
            float4 st[16];
#pragma unroll
            for (int i = 0; i < 16; ++i) {
                const int tau = tau0 + i < tile ? tau0 + i : tile - 1;
                st[i] = *reinterpret_cast<const float4*>(wp + tau * ws_tile);
            }
#pragma unroll
            for (int i = 0; i < 16; ++i) {
                if (tau0 + i < tile) {
                    s[0] = lam_rows[0] * s[0] + st[i].x;
                    s[1] = lam_rows[1] * s[1] + st[i].y;
                    s[2] = lam_rows[2] * s[2] + st[i].z;
                    s[3] = lam_rows[3] * s[3] + st[i].w;
                }
            }
        }
    }

    if (lane < kChunk) {
        float hj = 0.0f;
        for (int n = 0; n < kMaxOrder; ++n) hj += rs[w][n] * powi(ls[w][n], lane);
        hs[w][lane] = hj;
    }
    __syncthreads();

    bf16x8_t tz[2];
    if constexpr (!kStateOnly) t_operands(tz, hs[w], li, lq);
    bf16x8_t pop, pop_lo;
    p_operands(pop, pop_lo, ls[w], li, lq);
    float lam32[4];
#pragma unroll
    for (int r = 0; r < 4; ++r) lam32[r] = powi(ls[w][4 * lq + r], kChunk);
    bf16x8_t qop[2];
    if constexpr (!kStateOnly) q_operands(qop, rs[w], ls[w], li, lq);

    const int swz = ((lr >> 3) & 3) << 1;
    const int st_idx = lr * PPR + (lp ^ swz);
    const int rd_piece = (2 * w + (li >> 3)) ^ (lq << 1);
    const int zwr_off = li * ZROW + (16 * w + 4 * lq) * 4;
    const int zrd_off = lr * ZROW + 8 * lp * 4;

    auto gate_store = [&](int ci, const Words<4>& qq) {
        const int64_t t = t_start + (int64_t)ci * kChunk + lr;
        if (t < t_end) {
            const char* zp = zst[ci & 1] + zrd_off;
            const float4 za = *reinterpret_cast<const float4*>(zp);
            const float4 zb = *reinterpret_cast<const float4*>(zp + 16);
            float qf[8];
            Pack<BF16, 8>::unpack(qq, qf);
            float y8[8] = {za.x * qf[0], za.y * qf[1], za.z * qf[2], za.w * qf[3],
                           zb.x * qf[4], zb.y * qf[5], zb.z * qf[6], zb.w * qf[7]};
            store_words_nt<4>(a.y + seq0 + t * D + ld_off, Pack<BF16, 8>::pack(y8));
        }
    };

    for (int base = 0; base < nchunks; base += kPrefetch) {
#pragma unroll
        for (int sgi = 0; sgi < kPrefetch; ++sgi) {
            const int ci = base + sgi;
            const bool live = ci < nchunks;
            stage[ci & 1][st_idx] = products(kpre[sgi], vpre[sgi]);
            load_kv(ci + kPrefetch, kpre[sgi], vpre[sgi]);

            __syncthreads();

            const bf16x8_t uw = transposed<PPR>(stage[ci & 1], rd_piece, li, lq);

            if (live) {
                if constexpr (!kStateOnly) {
                    f32x4_t acc[2];
                    chunk_outputs(acc, s, uw, tz, qop);
                    char* zp = zst[ci & 1] + zwr_off;
                    *reinterpret_cast<float4*>(zp) = make_float4(acc[0][0], acc[0][1], acc[0][2], acc[0][3]);
                    *reinterpret_cast<float4*>(zp + 16 * ZROW) = make_float4(acc[1][0], acc[1][1], acc[1][2], acc[1][3]);
                }
                advance(s, lam32, pop, pop_lo, uw);
            }
            if constexpr (!kStateOnly) {
                const int prev = (sgi + kPrefetch - 1) % kPrefetch;
                if (ci > 0 && ci <= nchunks) gate_store(ci - 1, qpre[prev]);
                load_q(ci - 1 + kPrefetch, qpre[prev]);
            }
        }
    }
    if constexpr (!kStateOnly) {
        if (nchunks % kPrefetch == 0) {
            __syncthreads();
            gate_store(nchunks - 1, qpre[kPrefetch - 1]);
        }
        if (a.s_out && tile == a.tiles_per_seq - 1)  // (the launcher admits this only for L % 32 == 0: no padded rows)
            *reinterpret_cast<float4*>(a.s_out + b * ws_tile + ws_wave) = make_float4(s[0], s[1], s[2], s[3]);
    } else {
        float* wp = a.ws + (b * (a.tiles_per_seq - 1) + tile) * ws_tile + ws_wave;
        *reinterpret_cast<float4*>(wp) = make_float4(s[0], s[1], s[2], s[3]);
    }
}

// ---------------------------------------------------------------------------------------------------------
// One pass, for tiles of up to kOneTile steps: a workgroup forms u of its whole tile once and keeps it (LDS and registers,
// 4 VGPRs per chunk), walks the tile's state from zero and leaves it in the workspace, waits for the states of the tiles
// before it and only then reads q and computes y, from the u it kept.  k and v are read once: 8 bytes per output instead of
// 12.  The states are those of the two passes above, bit for bit.
//
// What bounds it: the 4-tensor stream through 512-byte strips (44.4 us at 8192 x 4096) in two phases, and between them the
// wait, the operands of the second and the records' launch (4.9): 57 us a call where two passes take 76, in a row of calls that
// share their inputs; 60 with inputs that change from call to call.
//
// The wait is per wave and per record, without flags or fences: li_mark_kernel has filled the records with kUnset, a NaN that
// no state ever is (a producer that holds it stores the plain NaN), every word is stored and loaded as an atomic at device
// scope, and a record counts as there when none of its words is kUnset.  A workgroup waits only for workgroups with a lower
// index, which are dealt out before it; and the wait is bounded all the same (each XCD starts its share on its own, so one
// that is busy with another stream's kernel may start it late): after kPolls looks, about 2 ms, a wave walks the missing tile
// itself, to the same bits.
constexpr int kOneTileChunks = 16;
constexpr uint32_t kUnset = 0xffffdeadu;
constexpr int kPolls = 1024;

constexpr int kMarks = 4;  // 16-byte pieces per lane
__global__ __launch_bounds__(256) void li_mark_kernel(uint4* rec, int64_t n) {
    const int64_t i0 = (int64_t)blockIdx.x * 256 * kMarks + threadIdx.x;
#pragma unroll
    for (int x = 0; x < kMarks; ++x)
        if (i0 + 256 * x < n) store_words_nt<4>(rec + i0 + 256 * x, Words<4>{{kUnset, kUnset, kUnset, kUnset}});
}

__device__ __forceinline__ uint64_t device_load(const float* p) {
    return __hip_atomic_load(reinterpret_cast<const uint64_t*>(p), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ void publish(float* p, const f32x4_t& s) {
    uint32_t x[4];
#pragma unroll
    for (int r = 0; r < 4; ++r) {
        x[r] = __float_as_uint(s[r]);
        if (x[r] == kUnset) x[r] = 0x7fc00000u;
    }
#pragma unroll
    for (int r = 0; r < 2; ++r)
        __hip_atomic_store(reinterpret_cast<uint64_t*>(p) + r, x[2 * r] | (uint64_t)x[2 * r + 1] << 32, __ATOMIC_RELAXED,
                           __HIP_MEMORY_SCOPE_AGENT);
}

// KL: chunks of u kept in LDS (the first ones), the others in registers.  PF, QF: chunks of k, v and of q in flight.
template <int NW, int KL, int PF, int QF>
__global__ __launch_bounds__(NW * 64, NW == 16 ? 4 : 2) void li_one_pass_kernel(LiArgs a) {
    constexpr int PPR = 2 * NW;
    constexpr int ZROW = 16 * NW * 4 + 16;
    constexpr int KR = kOneTileChunks - KL;
    using std::integral_constant;
    __shared__ uint4 keep[KL > 0 ? KL : 1][kChunk * PPR];
    __shared__ __attribute__((aligned(16))) char zst[2][kChunk * ZROW];  // z, fp32 rows; u of the other chunks before that
    __shared__ float rs[NW][kMaxOrder], ls[NW][kMaxOrder], hs[NW][kChunk];
    static_assert(kChunk * ZROW >= kChunk * PPR * 16, "a chunk of u fits a chunk of z");

    const int tid = threadIdx.x;
    const int w = __builtin_amdgcn_readfirstlane(tid / 64), lane = tid % 64;
    const int li = lane % 16, lq = lane / 16;

    const uint32_t lb = blockIdx.x;
    const int cb = lb % (uint32_t)a.ncb;
    const uint32_t tl = lb / (uint32_t)a.ncb;
    const int64_t b = tl / (uint32_t)a.tiles_per_seq;
    const int tile = (int)(tl % (uint32_t)a.tiles_per_seq);
    const int64_t t_start = (int64_t)tile * a.rows;
    const int nrows = (int)((t_start + a.rows < a.L ? t_start + a.rows : a.L) - t_start);
    const int nchunks = (nrows + kChunk - 1) / kChunk;

    const int64_t D = a.D;
    const int64_t cblock0 = (int64_t)cb * 16 * NW;
    const int64_t c0 = cblock0 + 16 * w;
    const int64_t tile0 = (b * a.L + t_start) * D + cblock0;

    // A lane moves 8 channels of one row of a chunk; rows past the tile re-read its last row, chunks past the tile one
    // 16-byte location (their values are not used)
    const int lr = tid / PPR, lp = tid % PPR;
    const uint32_t row_bytes = (uint32_t)D * 2;
    auto offset = [&](int ci) {
        int row = ci * kChunk + lr;
        row = row < nrows ? row : nrows - 1;
        return ci < nchunks ? (uint32_t)row * row_bytes + 16u * lp : 0u;
    };
    auto load = [&](const uint16_t* p, uint32_t off) { return load_words_nt<4>(reinterpret_cast<const char*>(p + tile0) + off); };
    Words<4> kpre[PF], vpre[PF], qpre[QF];
#pragma unroll
    for (int i = 0; i < PF; ++i) {
        const uint32_t off = offset(i);
        kpre[i] = load(a.k, off);
        vpre[i] = load(a.v, off);
    }

    // ---- residues and poles of the wave's group
    {
        const int64_t g = c0 / a.group;
        if (lane < kMaxOrder) {
            rs[w][lane] = lane < a.order ? a.R[g * a.order + lane] : 0.0f;
            ls[w][lane] = lane < a.order ? a.lam[g * a.order + lane] : 0.0f;
        }
    }
    __syncthreads();
    bf16x8_t pop, pop_lo;
    p_operands(pop, pop_lo, ls[w], li, lq);
    float lam32[4];
#pragma unroll
    for (int r = 0; r < 4; ++r) lam32[r] = powi(ls[w][4 * lq + r], kChunk);

    const int st_idx = lr * PPR + (lp ^ (((lr >> 3) & 3) << 1));
    const int rd_piece = (2 * w + (li >> 3)) ^ (lq << 1);

    // ---- phase 1: u of the tile, and its state from zero
    bf16x8_t ukeep[KR];
    f32x4_t s = {0.0f, 0.0f, 0.0f, 0.0f};
    auto staged = [&](int ci) { return ci < KL ? keep[ci] : reinterpret_cast<uint4*>(zst[ci & 1]); };
    auto phase1 = [&](auto self, auto chunk) {
        constexpr int ci = decltype(chunk)::value;
        if constexpr (ci < kOneTileChunks) {
            if (ci >= nchunks) return;
            staged(ci)[st_idx] = products(kpre[ci % PF], vpre[ci % PF]);
            const uint32_t off = offset(ci + PF);
            kpre[ci % PF] = load(a.k, off);
            vpre[ci % PF] = load(a.v, off);
            __syncthreads();
            const bf16x8_t uw = transposed<PPR>(staged(ci), rd_piece, li, lq);
            if constexpr (ci >= KL) ukeep[ci - KL] = uw;
            advance(s, lam32, pop, pop_lo, uw);
            self(self, integral_constant<int, ci + 1>{});
        }
    };
    phase1(phase1, integral_constant<int, 0>{});

    const int64_t ws_wave = (c0 / 16) * 256;  // this wave's 1 KiB inside the records of a (b, tile); a lane's 4 floats
    const int64_t ws_tile = (D / 16) * 256;   // hold s[n = 4lq + r][channel li], r = 0..3
    float* const rec = a.ws + b * (a.tiles_per_seq - 1) * ws_tile + ws_wave;
    if (tile < a.tiles_per_seq - 1) publish(rec + tile * ws_tile + 4 * lane, s);

#pragma unroll
    for (int i = 0; i < QF; ++i) qpre[i] = load(a.q, offset(i));
    if (lane < kChunk) {
        float hj = 0.0f;
        for (int n = 0; n < kMaxOrder; ++n) hj += rs[w][n] * powi(ls[w][n], lane);
        hs[w][lane] = hj;
    }
    __syncthreads();  // hs; and the last chunk of u has been read from where z goes
    // ---- start state: the Horner sum over the earlier tiles' end states (li_mfma_kernel's)
    s = f32x4_t{0.0f, 0.0f, 0.0f, 0.0f};
    if (a.s_in) {
        const float4 c4 = *reinterpret_cast<const float4*>(a.s_in + b * ws_tile + ws_wave + 4 * lane);
        s = f32x4_t{c4.x, c4.y, c4.z, c4.w};
    }
    if (tile > 0) {
        float lam_rows[4];
#pragma unroll
        for (int r = 0; r < 4; ++r) lam_rows[r] = powi(ls[w][4 * lq + r], a.rows);
        int looks = a.polls;
        // one word of every record first, a lane each: most of the waiting costs one load per look
        for (int base = 0; base < tile; base += 64) {
            const int mine = base + lane < tile ? base + lane : tile - 1;
            const uint32_t* p = reinterpret_cast<const uint32_t*>(rec + mine * ws_tile);
            while (looks > 0 && __any(__hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) == kUnset)) {
                --looks;
                __builtin_amdgcn_s_sleep(4);
            }
        }
        auto horner = [&](const f32x4_t& x) {
#pragma unroll
            for (int r = 0; r < 4; ++r) s[r] = lam_rows[r] * s[r] + x[r];
        };
        constexpr int NB = 4;  // records in flight (with 16: 4096 x 4096 33.8 -> 36.7 us)
        for (int tau = 0; tau < tile;) {
            uint64_t x[NB][2];
            bool there = a.polls > 0;
#pragma unroll
            for (int i = 0; i < NB; ++i) {
                const float* p = rec + (tau + i < tile ? tau + i : tile - 1) * ws_tile + 4 * lane;
                x[i][0] = device_load(p);
                x[i][1] = device_load(p + 2);
            }
#pragma unroll
            for (int i = 0; i < NB; ++i)
#pragma unroll
                for (int r = 0; r < 2; ++r) there = there && (uint32_t)x[i][r] != kUnset && (uint32_t)(x[i][r] >> 32) != kUnset;
            if (__all(there)) {
#pragma unroll
                for (int i = 0; i < NB; ++i)
                    if (tau + i < tile)
                        horner(f32x4_t{__uint_as_float((uint32_t)x[i][0]), __uint_as_float((uint32_t)(x[i][0] >> 32)),
                                       __uint_as_float((uint32_t)x[i][1]), __uint_as_float((uint32_t)(x[i][1] >> 32))});
                tau += NB;
            } else if (looks > 0) {
                --looks;
                __builtin_amdgcn_s_sleep(4);
            } else {  // walk tile `tau` (all its rows exist: it is not the sequence's last)
                f32x4_t e = {0.0f, 0.0f, 0.0f, 0.0f};
                const uint32_t at = 8u * lq * row_bytes + 2u * li;
                for (int t0 = 0; t0 < a.rows; t0 += kChunk) {
                    const int64_t chunk0 = (b * a.L + (int64_t)tau * a.rows + t0) * D + c0;
                    auto u_at = [&](int row) {
                        const char *pk = reinterpret_cast<const char*>(a.k + chunk0 + row * D),
                                   *pv = reinterpret_cast<const char*>(a.v + chunk0 + row * D);
                        return bf16_lo(*reinterpret_cast<const uint16_t*>(pk + at)) *
                               bf16_lo(*reinterpret_cast<const uint16_t*>(pv + at));
                    };
                    Words<4> u;
#pragma unroll
                    for (int e2 = 0; e2 < 4; ++e2) {
                        u.w[e2] = pack_bf16x2(u_at(2 * e2), u_at(2 * e2 + 1));
                        __builtin_amdgcn_sched_barrier(0);  // (few registers are free here)
                    }
                    advance(e, lam32, pop, pop_lo, __builtin_bit_cast(bf16x8_t, u));
                }
                horner(e);
                ++tau;
            }
        }
    }

    // ---- phase 2: y of the tile
    bf16x8_t tz[2];
    t_operands(tz, hs[w], li, lq);
    bf16x8_t qop[2];
    q_operands(qop, rs[w], ls[w], li, lq);
    const int zwr_off = li * ZROW + (16 * w + 4 * lq) * 4;
    const int zrd_off = lr * ZROW + 8 * lp * 4;
    auto phase2 = [&](auto self, auto chunk) {
        constexpr int ci = decltype(chunk)::value;
        if constexpr (ci < kOneTileChunks) {
            if (ci >= nchunks) return;
            bf16x8_t uw;
            if constexpr (ci < KL)
                uw = transposed<PPR>(keep[ci], rd_piece, li, lq);
            else
                uw = ukeep[ci - KL];
            f32x4_t acc[2];
            chunk_outputs(acc, s, uw, tz, qop);
            char* zw = zst[ci & 1] + zwr_off;
            *reinterpret_cast<float4*>(zw) = make_float4(acc[0][0], acc[0][1], acc[0][2], acc[0][3]);
            *reinterpret_cast<float4*>(zw + 16 * ZROW) = make_float4(acc[1][0], acc[1][1], acc[1][2], acc[1][3]);
            advance(s, lam32, pop, pop_lo, uw);
            __syncthreads();
            if (ci * kChunk + lr < nrows) {
                const char* zp = zst[ci & 1] + zrd_off;
                const float4 za = *reinterpret_cast<const float4*>(zp);
                const float4 zb = *reinterpret_cast<const float4*>(zp + 16);
                float qf[8];
                Pack<BF16, 8>::unpack(qpre[ci % QF], qf);
                float y8[8] = {za.x * qf[0], za.y * qf[1], za.z * qf[2], za.w * qf[3],
                               zb.x * qf[4], zb.y * qf[5], zb.z * qf[6], zb.w * qf[7]};
                store_words_nt<4>(reinterpret_cast<char*>(a.y + tile0) + offset(ci), Pack<BF16, 8>::pack(y8));
            }
            qpre[ci % QF] = load(a.q, offset(ci + QF));
            self(self, integral_constant<int, ci + 1>{});
        }
    };
    phase2(phase2, integral_constant<int, 0>{});
    if (a.s_out && tile == a.tiles_per_seq - 1)  // (the launcher admits this only for L % 32 == 0: no padded rows)
        *reinterpret_cast<float4*>(a.s_out + b * ws_tile + ws_wave + 4 * lane) = make_float4(s[0], s[1], s[2], s[3]);
}

// ---------------------------------------------------------------------------------------------------------
// Folding states: out = Lambda^(steps of all records) s_in + sum_i Lambda^(steps after record i) rec_i, where every
// record is the end state of a stretch of `steps` steps walked from zero (`last_steps` for the last one).  This is
// the Horner sum of pass 2's start state as a kernel of its own: it turns the tile records of a state-only walk
// into the state after the walk, and the end states of several ranks' stretches into each rank's start state.
// One lane per float4 of a state ([B][D/16][64 lanes][4]: lane (li, lq) of a 16-channel block holds exponentials
// 4 lq .. 4 lq + 3 of channel li); records of one batch item are rec_stride_i floats apart, batch items rec_stride_b.
__device__ __forceinline__ float powi64(float x, int64_t e) {  // x^e, e >= 0, by squaring
    float r = 1.0f;
    while (e > 0) {
        if (e & 1) r *= x;
        x *= x;
        e >>= 1;
    }
    return r;
}

__global__ __launch_bounds__(256) void li_fold_kernel(const float* __restrict__ rec, int64_t n, int64_t rec_stride_b,
                                                      int64_t rec_stride_i, const float* __restrict__ lam,
                                                      const float* __restrict__ s_in, float* __restrict__ s_out, int64_t B,
                                                      int64_t D, int32_t order, int32_t group, int64_t steps,
                                                      int64_t last_steps) {
    const int64_t per_b = (D / 16) * 64;  // float4s of one batch item's state
    const int64_t x = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (x >= B * per_b) return;
    const int64_t b = x / per_b, within = x % per_b;
    const int lane = (int)(within % 64);
    const int64_t channel = (within / 64) * 16 + lane % 16;
    const float* lp = lam + (channel / group) * (int64_t)order;
    float pw[4], pl[4];
#pragma unroll
    for (int r = 0; r < 4; ++r) {
        const int nn = 4 * (lane / 16) + r;
        const float l = nn < order ? lp[nn] : 0.0f;
        pw[r] = powi64(l, steps);
        pl[r] = powi64(l, last_steps);
    }
    float4 s = make_float4(0.0f, 0.0f, 0.0f, 0.0f);
    if (s_in) s = *reinterpret_cast<const float4*>(s_in + x * 4);
    const float* rp = rec + b * rec_stride_b + within * 4;
    for (int64_t i0 = 0; i0 < n; i0 += 8) {
        float4 st[8];
#pragma unroll
        for (int i = 0; i < 8; ++i) {  // the loads do not depend on the running sum; past the end the last record repeats
            const int64_t ii = i0 + i < n ? i0 + i : n - 1;
            st[i] = *reinterpret_cast<const float4*>(rp + ii * rec_stride_i);
        }
#pragma unroll
        for (int i = 0; i < 8; ++i) {
            if (i0 + i < n) {
                const bool last = i0 + i == n - 1;
                s.x = (last ? pl[0] : pw[0]) * s.x + st[i].x;
                s.y = (last ? pl[1] : pw[1]) * s.y + st[i].y;
                s.z = (last ? pl[2] : pw[2]) * s.z + st[i].z;
                s.w = (last ? pl[3] : pw[3]) * s.w + st[i].w;
            }
        }
    }
    *reinterpret_cast<float4*>(s_out + x * 4) = s;
}

// ---------------------------------------------------------------------------------------------------------
// General kernel: the recurrence itself, one lane per (batch item, channel).  Any dtype, any group, up to
// kMaxOrderDirect exponentials; slow (B * D lanes in all), the correctness path for what the matrix-core kernel
// does not take.  The running sums and the output sum are kept in fp64: a slow pole (lambda close to 1) carries
// thousands of steps, and in fp32 one rounding per step and exponential would add up past the 1e-5 that fp32
// storage is held to; in fp64 the only roundings left are the final conversion of z and the gate.  The running
// sums live in registers (MAXO of them); residues and poles of the lane's group sit in LDS.
constexpr int kMaxOrderDirect = 64;

template <typename T, int MAXO>
__global__ __launch_bounds__(64) void li_direct_kernel(const void* qv, const void* kv, const void* vv, const float* R,
                                                       const float* lam, void* yv, int64_t B, int64_t L, int64_t D,
                                                       int32_t order, int32_t group) {
    __shared__ float rtab[MAXO][64], ltab[MAXO][64];  // [exponential][lane]: conflict-free per-lane columns
    const int64_t idx = (int64_t)blockIdx.x * 64 + threadIdx.x;
    const bool live = idx < B * D;
    const int64_t b = live ? idx / D : 0, c = live ? idx % D : 0;
    const int64_t g = c / group;
    double sn[MAXO];
#pragma unroll
    for (int n = 0; n < MAXO; ++n) {
        rtab[n][threadIdx.x] = n < order ? R[g * order + n] : 0.0f;
        ltab[n][threadIdx.x] = n < order ? lam[g * order + n] : 0.0f;
        sn[n] = 0.0;
    }
    if (!live) return;  // (each lane reads only its own column of the tables: no barrier needed)
    const char* qp = static_cast<const char*>(qv);
    const char* kp = static_cast<const char*>(kv);
    const char* vp = static_cast<const char*>(vv);
    char* yp = static_cast<char*>(yv);
    for (int64_t t = 0; t < L; ++t) {
        const int64_t off = ((b * L + t) * D + c) * T::kBytes;
        float qf[1], kf[1], vf[1];
        Pack<T, 1>::unpack(Pack<T, 1>::load(qp + off), qf);
        Pack<T, 1>::unpack(Pack<T, 1>::load(kp + off), kf);
        Pack<T, 1>::unpack(Pack<T, 1>::load(vp + off), vf);
        const double u = (double)kf[0] * (double)vf[0];
        double z = 0.0;
#pragma unroll
        for (int n = 0; n < MAXO; ++n) {
            sn[n] = __builtin_fma((double)ltab[n][threadIdx.x], sn[n], u);
            z = __builtin_fma((double)rtab[n][threadIdx.x], sn[n], z);
        }
        float y1[1] = {(float)((double)qf[0] * z)};
        Pack<T, 1>::store(yp + off, Pack<T, 1>::pack(y1));
    }
}

int64_t li_rows(const LiShape& s, int nw) {
    int64_t rows = tuning().mr_rows;
    const int64_t ncb = s.D / (16 * nw);
    if (rows <= 0) {
        int64_t tiles = 256 / (s.B * ncb);
        if (tiles < 1) tiles = 1;
        rows = (s.L + tiles - 1) / tiles;
        // (up to four chunks stay one tile: a second pass costs more than their chain; 3 x 114 x 1536 11.5 against 15.0 us)
        const int64_t min_rows = (nw == 4 && s.L > 4 * kChunk ? 2 : 4) * kChunk;
        if (rows < min_rows) rows = min_rows;
    }
    rows = (rows + kChunk - 1) / kChunk * kChunk;
    const int64_t cap = (s.L + kChunk - 1) / kChunk * kChunk;
    return rows > cap ? cap : rows;
}

// One pass where a workgroup can keep its tile's u and the tiles are long against their number (a wave adds up the states
// of all earlier tiles while nothing else goes on), the more so the fewer channels a workgroup moves per step.  Us, two
// passes / one: 16 waves 8192 x 4096 (16 tiles of 512 steps) 75.1 / 56.7, 20001 x 1536 (42 of 480) 83.1 / 64.0, 65536 x 512
// (128 of 512) 97 / 84, 131072 x 256 (256 of 512) 98 / 117; 8 waves 4096 x 4096 (8 of 512) 43.8 / 34, 32768 x 512 (64 of
// 512) 54 / 44, 65536 x 256 (128 of 512) 51.8 / 53.7, 4096 x 1024 (32 of 128) 21.4 / 23.0, 16384 x 256 (128 of 128)
// 31 / 43; 4 waves 512 x 256 (4 of 128) 15.4 / 14.4, 3 x 1333 x 1024 (5 of 288) 21.5 / 19.1.
bool li_one_pass(const LiShape& s, int nw) {
    const int64_t rows = li_rows(s, nw), tiles = (s.L + rows - 1) / rows;
    return tiles > 1 && rows <= kOneTileChunks * kChunk && rows * nw >= 64 * tiles && s.D <= (1 << 21) && tuning().li_wait != 2;
}

// `state_only`: no outputs are wanted, one pass over k and v in any case
int li_waves(const LiShape& s, bool state_only = false) {
    const int nw = tuning().mr_waves > 0 ? tuning().mr_waves : 16;
    // One pass with tiles that only fit it with the widest workgroup (narrower ones have half as many, twice as long): us
    // with the choice below / with 16 waves in one pass, 5500 x 4096 54 / 43, 7000 x 4096 69 / 51, 2 x 12000 x 1024
    // 62 / 52, 3 x 2500 x 4096 57 / 52; but not while they are short against their number (27593 x 768, 79 tiles of 352 steps,
    // 57 / 62; 13375 x 1280, 47 of 288, 48 / 51; but 24680 x 1024, 60 of 416, 64 / 57), nor two of them where 128-channel workgroups walk the sequence as one tile
    // (3 x 562 x 8192 29 / 32, 5 x 746 x 5120 37 / 40).  Up to 256 steps 8 waves keep theirs as well: 4096 x 4096 34 against 37.
    if (!state_only && !s.fewest && tuning().mr_waves == 0 && tuning().mr_rows == 0 && s.D % 256 == 0 && li_rows(s, 16) > 8 * kChunk &&
        li_one_pass(s, 16)) {
        const int64_t rows = li_rows(s, 16), tiles = (s.L + rows - 1) / rows;
        if (rows >= 160 + 3 * tiles && (tiles > 2 || li_rows(s, 8) < s.L)) return 16;
    }
    // Left to itself, a problem that gives a 256-channel workgroup fewer than 512 steps takes 128-channel workgroups
    // (half as many tiles per sequence, twice as long): measured at B = 1, D = 4096: L = 2048 23.2 against 28.4 us,
    // L = 4096 34 against 37.
    // Where those would be at their shortest (four chunks) as well, 64-channel workgroups: B = 1, L = 512: D = 256 17.7 ->
    // 15.0 us, D = 4096 20.0 -> 18.4; L = 2048, D = 1024 19.9 -> 18.5, unless their tiles would
    // be much longer (L = 1000, D = 4096: 256 steps 22.2 us, 128 steps of 8 waves 21.4).
    if (tuning().mr_waves == 0 && tuning().mr_rows == 0 && s.D % 256 == 0 && li_rows(s, 16) < 512)
        return li_rows(s, 8) <= 4 * kChunk && li_rows(s, 4) <= 6 * kChunk ? 4 : 8;
    // A batch that fills the chip with narrower workgroups of ONE tile per sequence takes them: a single pass moves
    // 8 bytes per output where the two-pass scan moves 12 (measured at L = 8192, D = 4096: B = 8 400 us with 8
    // waves against 445 with 16, B = 4 197 us with 4 waves against 241; B = 16 fills it with 16 waves: 695 us, 77%).
    // "Fills" means that at least three quarters of the compute units are busy in every round of 256 workgroups
    // (B = 6: 192 workgroups of 8 waves 309 us against 374; B = 3: 192 of 4 waves 165 us against 190).
    if (tuning().mr_waves == 0 && tuning().mr_rows == 0 && s.D % 256 == 0 && li_rows(s, 16) < s.L) {
        auto fills = [](int64_t wg) { return 4 * wg >= 3 * ((wg + 255) / 256) * 256; };
        if (fills(s.B * (s.D / 128))) return 8;
        if (fills(s.B * (s.D / 64))) return 4;
    }
    if (nw == 16 && s.D % 256 == 0) return 16;
    if (nw >= 8 && s.D % 128 == 0) return 8;
    return 4;
}

hy_status launch_fold(const float* rec, int64_t n, int64_t stride_b, int64_t stride_i, const float* lam, const float* s_in,
                      float* s_out, int64_t B, int64_t D, int32_t order, int32_t group, int64_t steps, int64_t last_steps,
                      hipStream_t st) {
    const int64_t items = B * (D / 16) * 64;
    const int64_t nb = (items + 255) / 256;
    if (nb > 0x7fffffffLL) return HY_ERR_UNSUPPORTED;
    return launch_kernel(li_fold_kernel, dim3((uint32_t)nb), dim3(256), st, rec, n, stride_b, stride_i, lam, s_in, s_out, B,
                         D, order, group, steps, last_steps);
}

// State-only walk: pass 1 over EVERY tile (the kernel skips the last of `tiles_per_seq` tiles, so it is told of one
// more than there are), then the fold of the tile records.
template <int NW>
hy_status launch_li_state_nw(const LiPtrs& p, const LiShape& s, void* ws, hipStream_t st) {
    constexpr int PF = 2;
    LiArgs a;
    a.q = nullptr;
    a.k = static_cast<const uint16_t*>(p.k);
    a.v = static_cast<const uint16_t*>(p.v);
    a.R = p.lam;  // the state does not depend on the residues; the kernel's set-up reads the table all the same
    a.lam = p.lam;
    a.y = nullptr;
    a.ws = static_cast<float*>(ws);
    a.s_in = nullptr;
    a.s_out = nullptr;
    a.L = s.L;
    a.D = s.D;
    a.order = s.order;
    a.group = s.group;
    a.polls = 0;
    a.ncb = (int32_t)(s.D / (16 * NW));
    const int64_t rows = li_rows(s, NW);
    a.rows = (int32_t)rows;
    const int64_t tiles = (s.L + rows - 1) / rows;
    a.tiles_per_seq = (int32_t)(tiles + 1);
    const int64_t nb = s.B * tiles * a.ncb;
    if (nb > 0x7fffffffLL) return HY_ERR_UNSUPPORTED;
    const hy_status rc = launch_kernel((li_mfma_kernel<NW, PF, true>), dim3((uint32_t)nb), dim3(NW * 64), st, a);
    if (rc != HY_OK) return rc;
    const int64_t ws_tile = (s.D / 16) * 256;
    return launch_fold(a.ws, tiles, tiles * ws_tile, ws_tile, p.lam, p.state_in, p.state_out, s.B, s.D, s.order, s.group,
                       rows, s.L - (tiles - 1) * rows, st);
}

template <int NW>
hy_status launch_li_nw(const LiPtrs& p, const LiShape& s, void* ws, hipStream_t st) {
    constexpr int PF = 2;
    LiArgs a;
    a.q = static_cast<const uint16_t*>(p.q);
    a.k = static_cast<const uint16_t*>(p.k);
    a.v = static_cast<const uint16_t*>(p.v);
    a.R = p.R;
    a.lam = p.lam;
    a.y = static_cast<uint16_t*>(p.y);
    a.ws = static_cast<float*>(ws);
    a.s_in = p.state_in;
    a.s_out = p.state_out;
    a.L = s.L;
    a.D = s.D;
    a.order = s.order;
    a.group = s.group;
    a.polls = 0;
    a.ncb = (int32_t)(s.D / (16 * NW));
    const int64_t rows = li_rows(s, NW);
    a.rows = (int32_t)rows;
    a.tiles_per_seq = (int32_t)((s.L + rows - 1) / rows);
    const int64_t nb2 = s.B * a.tiles_per_seq * a.ncb;
    const int64_t nb1 = s.B * (a.tiles_per_seq - 1) * a.ncb;
    if (nb2 > 0x7fffffffLL) return HY_ERR_UNSUPPORTED;
    if (nb1 > 0 && li_one_pass(s, NW)) {
        a.polls = tuning().li_wait == 1 ? 0 : kPolls;
        const int64_t n16 = s.B * (a.tiles_per_seq - 1) * (s.D / 16) * 64;
        const int64_t marks = (n16 + 256 * kMarks - 1) / (256 * kMarks);
        const hy_status rc =
            launch_kernel(li_mark_kernel, dim3((uint32_t)marks), dim3(256), st, static_cast<uint4*>(ws), n16);
        if (rc != HY_OK) return rc;
        return launch_kernel((li_one_pass_kernel<NW, NW == 16 ? 5 : 0, 3, 3>), dim3((uint32_t)nb2), dim3(NW * 64), st, a);
    }
    if (nb1 > 0) {
        const hy_status rc = launch_kernel((li_mfma_kernel<NW, PF, true>), dim3((uint32_t)nb1), dim3(NW * 64), st, a);
        if (rc != HY_OK) return rc;
    }
    return launch_kernel((li_mfma_kernel<NW, PF, false>), dim3((uint32_t)nb2), dim3(NW * 64), st, a);
}

}  // namespace

bool li_mfma_supported(const LiShape& s) {
    return s.dtype == HY_BF16 && s.group % 16 == 0 && s.D % 64 == 0 && s.order >= 1 && s.order <= kMaxOrder &&
           s.L <= 0x7fffffffLL - 64;
}

int64_t li_workspace_bytes(const LiShape& s) {
    if (!li_mfma_supported(s) || s.B == 0 || s.L == 0 || s.D == 0) return 0;
    const int64_t rows = li_rows(s, li_waves(s));
    const int64_t tiles = (s.L + rows - 1) / rows;
    return s.B * (tiles - 1) * (s.D / 16) * 256 * (int64_t)sizeof(float);
}

hy_status launch_li_mfma(const LiPtrs& p, const LiShape& s, void* ws, hipStream_t st) {
    if (!li_mfma_supported(s)) return HY_ERR_UNSUPPORTED;
    // a last chunk with rows past the end would carry them into the state it leaves behind
    if (p.state_out && s.L % kChunk != 0) return HY_ERR_UNSUPPORTED;
    switch (li_waves(s)) {
        case 16: return launch_li_nw<16>(p, s, ws, st);
        case 8: return launch_li_nw<8>(p, s, ws, st);
        default: return launch_li_nw<4>(p, s, ws, st);
    }
}

int64_t li_state_workspace_bytes(const LiShape& s) {
    if (!li_mfma_supported(s) || s.B == 0 || s.L == 0 || s.D == 0) return 0;
    const int64_t rows = li_rows(s, li_waves(s, true));
    const int64_t tiles = (s.L + rows - 1) / rows;
    return s.B * tiles * (s.D / 16) * 256 * (int64_t)sizeof(float);
}

hy_status launch_li_state(const LiPtrs& p, const LiShape& s, void* ws, hipStream_t st) {
    if (!li_mfma_supported(s) || s.L % kChunk != 0 || !p.state_out) return HY_ERR_UNSUPPORTED;
    switch (li_waves(s, true)) {
        case 16: return launch_li_state_nw<16>(p, s, ws, st);
        case 8: return launch_li_state_nw<8>(p, s, ws, st);
        default: return launch_li_state_nw<4>(p, s, ws, st);
    }
}

hy_status launch_li_state_fold(const float* states, int64_t n, int64_t steps, const float* lam, const float* state_in,
                               float* state_out, int64_t B, int64_t D, int32_t order, int32_t group, hipStream_t st) {
    if (D % 16 != 0 || order < 1 || order > kMaxOrder) return HY_ERR_UNSUPPORTED;
    const int64_t per = (D / 16) * 256;  // floats of one batch item's state
    return launch_fold(states, n, per, B * per, lam, state_in, state_out, B, D, order, group, steps, steps, st);
}

hy_status launch_li_direct(const LiPtrs& p, const LiShape& s, hipStream_t st) {
    if (s.order < 1 || s.order > kMaxOrderDirect) return HY_ERR_UNSUPPORTED;
    const int64_t n = s.B * s.D;
    const int64_t nb = (n + 63) / 64;
    if (nb > 0x7fffffffLL) return HY_ERR_UNSUPPORTED;
    const dim3 grid((uint32_t)nb), block(64);
    const bool small = s.order <= kMaxOrder;
    if (s.dtype == HY_F32) {
        if (small)
            return launch_kernel((li_direct_kernel<F32, kMaxOrder>), grid, block, st, p.q, p.k, p.v, p.R, p.lam, p.y, s.B,
                                 s.L, s.D, s.order, s.group);
        return launch_kernel((li_direct_kernel<F32, kMaxOrderDirect>), grid, block, st, p.q, p.k, p.v, p.R, p.lam, p.y,
                             s.B, s.L, s.D, s.order, s.group);
    }
    if (small)
        return launch_kernel((li_direct_kernel<BF16, kMaxOrder>), grid, block, st, p.q, p.k, p.v, p.R, p.lam, p.y, s.B,
                             s.L, s.D, s.order, s.group);
    return launch_kernel((li_direct_kernel<BF16, kMaxOrderDirect>), grid, block, st, p.q, p.k, p.v, p.R, p.lam, p.y, s.B,
                         s.L, s.D, s.order, s.group);
}

}  // namespace hy
