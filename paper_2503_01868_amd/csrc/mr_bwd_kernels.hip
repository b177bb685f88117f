// Hyena-MR backward on the gfx950 matrix cores (bf16 operands, fp32 accumulation), ONE pass over the tensors.
//
// With u = k*v and g = dy*q the gradients of y = q (.) (h * u) are (Sec. 2.1 Eq. 1, Sec. 3.1 Eq. 2):
//     dq[t] = dy[t] * z[t],   z[t] = sum_j h[j] u[t-j]
//     du[s] = sum_j h[j] g[s+j],  dk = du (.) v,  dv = du (.) k
//     dh[j] = sum_{b, c in group, s} u[s] g[s+j]
// The kernel walks the sequence from its end, tau = L-1-t.  In tau the transposed convolution is causal,
// du'[tau] = sum_j h[j] g'[tau-j], so du is the forward block-Toeplitz scheme of mr_kernels.hip (Toeplitz operands
// in registers, register window of the last NKB source blocks, LDS transposition) with g in the role of u and two
// post-gates.  The forward sum is anti-causal in tau, z'[tau] = sum_j h[j] u'[tau+j]: the outputs of a chunk are
// complete once the NKB-1 chunks after it have arrived, so z (and dq) come out NKB-1 chunks late, from a second
// register window that holds the u blocks.  No second set of operands is needed: with the 32 source steps of a
// block fed in reversed order and the 16 output steps written in reversed order, the operand of the anti-causal
// product for output tile tau0 and source block sigma0 has the element h[(sigma0 - tau0 + 16) + n - k], which is the
// causal operand for the offset sigma0 - tau0 + 16.  dy waits NKB chunks for its z in a lane-private LDS ring.
// So dy, q, k, v are each read once and dq, dk, dv written once (7 tensor passes; with the forward kernel computing
// dq in a launch of its own it was 10).  A tile needs NKB-1 chunks of dy, q before it (for du) and NKB-1 chunks of
// k, v after it (for z).
// The filter gradient is a second contraction over the 16 channels of a group,
//     C_x[i][n] = sum_c u[tau_s + i, c] * g[tau_s - 16 x + n, c],    dh[16 x + i - n] += C_x[i][n],
// which is what v_mfma_f32_16x16x16_bf16 computes from plain row-major operands (4 adjacent channels of
// one row per lane): 2*(2 NKB - 1) extra MFMAs per chunk into 2 NKB - 1 accumulators that live in registers
// for the whole tile.  At the end of the tile each wave folds the diagonals of its accumulators into one
// partial dh row and writes it to the workspace (App. A.4: partial accumulation by block, written out
// contiguously); dh_reduce_kernel sums the partials.
// Four waves (64 channels) per workgroup, one wave per SIMD: operands, two windows, the filter-gradient
// accumulators and the prefetch need ~280 registers per lane.  With one wave per SIMD the instructions between the products
// are time: the windows' blocks are read transposed (ds_read_b64_tr_b16; 2-byte reads put together by the vector ALUs and
// 64-bit row offsets per lane were 60 instructions per chunk more), and a row's address is a uniform offset plus 32 bits.
// Bound: 128-byte row pieces.  Measured, 128 taps, before / now: 3 x 5000 x 2048 117 / 97 us, 1 x 8192 x 4096 105 / 104,
// 60 taps 111 / 96, 1 x 65536 x 4096 728 / 729.
#include "hy_common.hpp"
#include "hy_launch.hpp"

namespace hy {
namespace {

typedef short s16x4_t __attribute__((ext_vector_type(4)));

struct MrBwdArgs {
    const uint16_t* dy;
    const uint16_t* q;
    const uint16_t* k;
    const uint16_t* v;
    const float* h;
    uint16_t* dq;
    uint16_t* dk;
    uint16_t* dv;
    float* partial;  // [B * tiles_per_seq][D / 16][lh]: one row per (tile, 16-channel slice)
    int64_t L, D;
    int64_t skv, sgq, sout;  // elements between batch items in k, v / dy, q / dq, dk, dv
    int32_t hist, fut;       // rows of k, v in front of row 0 / of dy, q behind row L - 1 that hold data
    int32_t lh, group;
    int32_t ncb;
    // Tile x of a channel block: chunks x % tiles_per_seq * chunks .. of batch item x / tiles_per_seq; with `across`,
    // chunks x * chunks .. of all batch items in a row, kGap chunks without data between two items (plain calls).
    int32_t chunks, tiles_per_seq, across, items;
};

constexpr int kChunk = 32;
constexpr int64_t kWideRows = 1 << 23;  // channels from which on a row's 2 D bytes take more than the 24 bits of __umul24

// kShard: the call is one rank's share of a sequence (halo rows next to the tensors, batch strides), or its rows are of
// kWideRows channels and more; the plain call's instantiation carries none of that arithmetic.
template <int NKB, int NW, int PF, bool kShard>
__global__ __launch_bounds__(NW * 64, 1) void mr_bwd_kernel(MrBwdArgs a) {
    constexpr int PPR = 2 * NW;              // 16-byte pieces per staged row
    constexpr int CPR = 2 * PPR;             // 8-byte chunks per staged row
    constexpr int kTaps = 32 * NKB;
    constexpr int ZROW = 16 * NW * 4 + 16;
    constexpr int ND = 2 * NKB - 1;          // 16-step offsets x with a tap 16 x + i - n inside [0, lh)
    constexpr int NSLOT = NKB + 1;           // chunks of g kept for the filter gradient (+1: no write/read overlap)
    constexpr int NR = NKB + 1;              // chunks of dy waiting for their z
    constexpr int LAG = NKB - 1;             // chunks between a chunk's arrival and its complete z
    static_assert(NW == 4, "the LDS swizzle is for rows of 8 pieces");
    __shared__ uint4 gst[2][kChunk * PPR];             // g of the newest chunk, swizzled for the transposed read
    __shared__ uint4 utr[2][kChunk * PPR];             // u of the newest chunk, same layout (source of z)
    __shared__ uint2 gring[NSLOT][kChunk * CPR];       // g rows, 8-byte chunks XOR-swizzled by row
    __shared__ uint2 ust[2][kChunk * CPR];             // u rows of the current chunk, same layout (filter gradient)
    __shared__ uint4 dyring[NR][kChunk * PPR];         // raw dy pieces, written and read back by the same lane
    __shared__ __attribute__((aligned(16))) char zst[2][kChunk * ZROW];   // du, fp32 rows
    __shared__ __attribute__((aligned(16))) char zst2[2][kChunk * ZROW];  // z, fp32 rows
    __shared__ float hs[NW][kTapPad + kTaps];

    const int tid = threadIdx.x;
    const int w = tid / 64, lane = tid % 64;
    const int li = lane % 16, lq = lane / 16;

    const uint32_t lb = blockIdx.x;
    const int cb = (int)(lb % (uint32_t)a.ncb);
    const uint32_t tile = lb / (uint32_t)a.ncb;
    const int64_t L = a.L, D = a.D;
    // Everything below is in reversed time tau = L - 1 - t, in chunks of 32 steps: chunk r of a batch item.  What lies
    // kGap = LAG chunks past the last one is the first one of the next item, so that neither sum reaches over.
    constexpr int kGap = LAG;
    const int nseq = (int)((L + kChunk - 1) / kChunk);  // chunks of a batch item
    const int period = nseq + kGap;
    int b = kShard || !a.across ? (int)(tile / (uint32_t)a.tiles_per_seq) : 0;
    int r0 = kShard || !a.across ? (int)(tile % (uint32_t)a.tiles_per_seq) * a.chunks : 0;
    int ntile = nseq - r0 < a.chunks ? nseq - r0 : a.chunks;  // chunks of the tile
    if constexpr (!kShard) {
        if (a.across) {
            const uint32_t v0 = tile * (uint32_t)a.chunks;  // (the launcher admits fewer than 2^31 chunks in a row)
            const int left = (int)((uint32_t)a.items * (uint32_t)period - (uint32_t)kGap - v0);
            b = (int)(v0 / (uint32_t)period);
            r0 = (int)(v0 % (uint32_t)period);
            ntile = left < a.chunks ? left : a.chunks;
        }
    }
    const int64_t t_start = (int64_t)r0 * kChunk;                       // (shards)
    const int64_t t_end = kShard && t_start + (int64_t)ntile * kChunk < L ? t_start + (int64_t)ntile * kChunk : L;
    // dy, q of the chunks before the tile feed its du; before tau = 0 lie the `fut` rows behind the sequence's end
    // that hold data (a shard's right halo), down to the first chunk boundary at or below them
    const int back = kShard ? r0 + (a.fut + kChunk - 1) / kChunk : r0;
    const int warm = back < LAG ? back : LAG;
    const int64_t tau_lo = kShard ? -(int64_t)a.fut : 0;     // smallest reversed step at which dy and q hold data
    const int64_t tau_hi = kShard ? L + (int64_t)a.hist : L;  // k and v hold data below this reversed step
    // k, v of the LAG chunks after the tile feed its z; the walk always runs LAG chunks past the tile, also where
    // the sequence ends first (those chunks then hold zeros and load nothing)
    const int ntot = warm + ntile + LAG;
    // Where a walk stands: chunk r of a batch item, and in plain calls the byte offset of the chunk's lowest row in memory
    // (step 31 of its 32).  A walk that runs past the last item does so with chunk indices that nothing uses.
    struct At {
        int r;
        int64_t row0;
    };
    const int64_t step = (int64_t)kChunk * D * 2, jump = L * D * 2 + (int64_t)(period - 1) * step;  // to the next item's first chunk
    auto forward = [&](At& x) {
        ++x.r;
        if constexpr (!kShard) {
            const bool wrap = x.r == period;
            x.row0 += wrap ? jump : -step;
            x.r = wrap ? 0 : x.r;
        }
    };
    auto has_data = [&](const At& x) { return kShard || x.r < nseq; };
    const int rem = (int)(L - 1 - (int64_t)(nseq - 1) * kChunk);  // last step of the chunk that the sequence ends in
    auto last_step = [&](const At& x) { return x.r == nseq - 1 ? rem : 31; };

    const int64_t cblock0 = (int64_t)cb * 16 * NW;
    const int64_t c0 = cblock0 + 16 * w;
    const int64_t item0 = b;
    const int64_t seq0 = kShard ? item0 * a.sout : 0;  // plain calls: in the walk's position
    const int64_t seq0kv = kShard ? item0 * a.skv : 0, seq0gq = kShard ? item0 * a.sgq : 0;

    const int lr = tid / PPR, lp = tid % PPR;
    const int64_t ld_off = cblock0 + 8 * lp;
    // element offset of reversed step tau for this lane, without the batch item's offset
    auto row_off = [&](int64_t tau) { return (L - 1 - tau) * D + ld_off; };
    auto in_tile = [&](int ci, const At& x) { return (uint32_t)(ci - warm) < (uint32_t)ntile && has_data(x); };
    // loads whose result is never used (chunk indices past the last chunk; k and v before the tile, dy and q after
    // it; chunks between batch items) all go to one 16-byte location of the tile, the same for every lane of the workgroup:
    // one cache line per wave
    const int64_t idle_off = kShard ? (L - t_end) * D + cblock0
                                    : item0 * L * D + (L - 1 - (t_start < L ? t_start : L - 1)) * D + cblock0;
    // plain calls (D < kWideRows): a uniform offset and 32 bits per lane
    const uint32_t lane_off = kShard ? 0u : 2u * ((uint32_t)(31 - lr) * (uint32_t)D + (uint32_t)ld_off);
    auto bytes_at = [](const uint16_t* p, int64_t base, uint32_t off) { return reinterpret_cast<const char*>(p) + base + off; };
    auto two_rows = [&](const uint16_t* p1, const uint16_t* p2, const At& x, bool used, Words<4>& r1, Words<4>& r2) {
        // a chunk that the sequence ends in repeats its last row
        const int past = lr - last_step(x);
        const uint32_t off = used ? lane_off + __umul24(past > 0 ? past : 0, (uint32_t)D * 2u) : 0u;
        const int64_t base = used ? x.row0 : idle_off * 2;
        r1 = load_words_nt<4>(bytes_at(p1, base, off));
        r2 = load_words_nt<4>(bytes_at(p2, base, off));
    };
    auto load_g = [&](int ci, const At& x, Words<4>& yy, Words<4>& qq) {
        if constexpr (kShard) {
            int64_t tau = (int64_t)x.r * kChunk + lr;
            tau = tau < t_end ? tau : t_end - 1;
            tau = tau > tau_lo ? tau : tau_lo;  // rows past the data read its last row; their g is zeroed below
            const int64_t off = seq0gq + (ci < warm + ntile ? row_off(tau) : idle_off);
            yy = load_words_nt<4>(a.dy + off);
            qq = load_words_nt<4>(a.q + off);
        } else {
            two_rows(a.dy, a.q, x, ci < warm + ntile && has_data(x), yy, qq);
        }
    };
    auto load_kv = [&](int ci, const At& x, Words<4>& kk, Words<4>& vv) {
        if constexpr (kShard) {
            const int64_t t0 = (int64_t)x.r * kChunk;
            int64_t tau = t0 + lr;
            tau = tau < tau_hi ? tau : tau_hi - 1;
            const int64_t off = seq0kv + ((ci < ntot && ci >= warm && t0 < tau_hi) ? row_off(tau) : idle_off);
            kk = load_words_nt<4>(a.k + off);
            vv = load_words_nt<4>(a.v + off);
        } else {
            two_rows(a.k, a.v, x, ci < ntot && ci >= warm && has_data(x), kk, vv);
        }
    };

    Words<4> ypre[PF], qpre[PF], kpre[PF], vpre[PF];
    At here{r0 - warm, 2 * (item0 * L * D + (L - kChunk - (int64_t)(r0 - warm) * kChunk) * D)};  // the chunk of an iteration, the one before, the one whose dq it stores,
    At before = here, late = here, late_before = here, ahead = here;  // and the one whose dy and q it requests
#pragma unroll
    for (int i = 0; i < PF; ++i) {
        load_g(i, ahead, ypre[i], qpre[i]);
        if (i + 1 < PF) {
            load_kv(i, ahead, kpre[i], vpre[i]);  // the last k, v stage is filled by the first iteration
            forward(ahead);
        }
    }
    At ahead_kv = ahead;  // one behind
    forward(ahead);

    // zero the g ring: slots of chunks before the start of the walk stand for steps past the end of the sequence
    for (int i = tid; i < NSLOT * kChunk * CPR; i += NW * 64) (&gring[0][0])[i] = make_uint2(0u, 0u);

    bf16x8_t tz[2 * NKB];
    {
        const float* hp = a.h + (c0 / a.group) * (int64_t)a.lh;
        stage_filter<kTaps>(hs[w], hp, a.lh, lane);
        __syncthreads();
        toeplitz_operands(tz, hs[w], li, lq);
    }
    // gw[m]: g block of chunk ci - m, source steps in walk order; uw[m]: u block of chunk ci - m, source steps in
    // reversed order (element e of octet lq = step 31 - 8 lq - e of the chunk)
    bf16x8_t gw[NKB], uw[NKB];
    {
        Words<4> z = zero_words<4>();
#pragma unroll
        for (int m = 0; m < NKB; ++m) {
            gw[m] = __builtin_bit_cast(bf16x8_t, z);
            uw[m] = __builtin_bit_cast(bf16x8_t, z);
        }
    }
    f32x4_t cacc[ND];
#pragma unroll
    for (int x = 0; x < ND; ++x) cacc[x] = f32x4_t{0.0f, 0.0f, 0.0f, 0.0f};

    // Rows are permuted by 16-byte pieces so that a wave's transposed reads (for every octet of steps 4 rows x 16 channels)
    // meet every bank twice, which is what their 512 bytes take.
    auto skew = [](int row) { return ((row >> 1) & 1) * 2 + ((row >> 3) & 1) * 4; };
    const int st_idx = lr * PPR + (lp ^ skew(lr));
    // a lane addresses 4 channels of one row and gets 4 steps of channel li: rows 8 lq .. 8 lq + 3 (and 4 rows on), and for
    // the reversed order rows 31 - 8 lq down to 28 - 8 lq (and 4 rows back)
    auto tr_off = [&](int row) { return row * PPR * 16 + ((2 * w + ((li & 3) >> 1)) ^ skew(row)) * 16 + (li & 1) * 8; };
    const int rd_fwd = tr_off(8 * lq + (li >> 2)), rd_rev = tr_off(31 - 8 * lq - (li >> 2));
    const int zwr_off = li * ZROW + (16 * w + 4 * lq) * 4;           // du: step li of a 16-step tile
    const int zwr_off_rev = (15 - li) * ZROW + (16 * w + 4 * lq) * 4;  // z: step 15 - li
    const int zrd_off = lr * ZROW + 8 * lp * 4;
    // 8-byte chunk layout: logical chunk c8 of row r sits at c8 ^ (r & 15)
    const int x8 = lr & 15;
    const int wr8a = lr * CPR + ((2 * lp) ^ x8), wr8b = lr * CPR + ((2 * lp + 1) ^ x8);
    const int rd8 = (4 * w + lq) ^ li;  // this lane's chunk in a row whose index is li (mod 16)

    // dk, dv of chunk ci (du staged one iteration earlier)
    auto out_at = [&](uint16_t* p, const At& x) {
        if constexpr (kShard) return reinterpret_cast<char*>(p + seq0 + row_off((int64_t)x.r * kChunk + lr));
        else return reinterpret_cast<char*>(p) + x.row0 + lane_off;
    };
    auto row_in_tile = [&](int ci, const At& x) {
        return in_tile(ci, x) && (kShard ? (int64_t)x.r * kChunk + lr < t_end : lr <= last_step(x));
    };
    auto gate_store_du = [&](int ci, const At& x, const Words<4>& kk, const Words<4>& vv) {
        if (row_in_tile(ci, x)) {
            const char* zp = zst[ci & 1] + zrd_off;
            const float4 za = *reinterpret_cast<const float4*>(zp);
            const float4 zb = *reinterpret_cast<const float4*>(zp + 16);
            const float du[8] = {za.x, za.y, za.z, za.w, zb.x, zb.y, zb.z, zb.w};
            float kf[8], vf[8], o1[8], o2[8];
            Pack<BF16, 8>::unpack(kk, kf);
            Pack<BF16, 8>::unpack(vv, vf);
#pragma unroll
            for (int e = 0; e < 8; ++e) {
                o1[e] = du[e] * vf[e];
                o2[e] = du[e] * kf[e];
            }
            store_words_nt<4>(out_at(a.dk, x), Pack<BF16, 8>::pack(o1));
            store_words_nt<4>(out_at(a.dv, x), Pack<BF16, 8>::pack(o2));
        }
    };
    // dq of chunk cq, whose z was staged in iteration cq + LAG (buffer parity of that iteration)
    auto gate_store_dq = [&](int cq, const At& x) {
        if (row_in_tile(cq, x)) {
            const char* zp = zst2[(cq + LAG) & 1] + zrd_off;
            const float4 za = *reinterpret_cast<const float4*>(zp);
            const float4 zb = *reinterpret_cast<const float4*>(zp + 16);
            const uint4 raw = dyring[cq % NR][tid];
            Words<4> yy;
            yy.w[0] = raw.x; yy.w[1] = raw.y; yy.w[2] = raw.z; yy.w[3] = raw.w;
            float yf[8];
            Pack<BF16, 8>::unpack(yy, yf);
            float o[8] = {za.x * yf[0], za.y * yf[1], za.z * yf[2], za.w * yf[3],
                          zb.x * yf[4], zb.y * yf[5], zb.z * yf[6], zb.w * yf[7]};
            store_words_nt<4>(out_at(a.dq, x), Pack<BF16, 8>::pack(o));
        }
    };

    // one more iteration than chunks: the last chunk's du and the last finished z are gated one iteration late
    for (int base = 0; base < ntot + 1; base += PF) {
#pragma unroll
        for (int sgi = 0; sgi < PF; ++sgi) {
            const int ci = base + sgi;
            const int64_t t0 = (int64_t)here.r * kChunk;
            const bool main_chunk = in_tile(ci, here);
            const bool in_seq = kShard ? t0 + lr < tau_hi : lr <= (has_data(here) ? last_step(here) : -1);
            const int slot = __builtin_amdgcn_readfirstlane(ci % NSLOT);

            // g = dy*q and u = k*v of this lane's row piece, rounded to bf16, into LDS; dy itself into its ring
            {
                float a8[8], b8[8];
                Pack<BF16, 8>::unpack(ypre[sgi], a8);
                Pack<BF16, 8>::unpack(qpre[sgi], b8);
                Words<4> gg;
#pragma unroll
                for (int e2 = 0; e2 < 4; ++e2) gg.w[e2] = pack_bf16x2(a8[2 * e2] * b8[2 * e2], a8[2 * e2 + 1] * b8[2 * e2 + 1]);
                // past the rows that hold data and between batch items: zeros
                if (kShard ? t0 + lr < tau_lo : !in_seq) gg = zero_words<4>();
                gst[ci & 1][st_idx] = make_uint4(gg.w[0], gg.w[1], gg.w[2], gg.w[3]);
                gring[slot][wr8a] = make_uint2(gg.w[0], gg.w[1]);
                gring[slot][wr8b] = make_uint2(gg.w[2], gg.w[3]);
                dyring[ci % NR][tid] = make_uint4(ypre[sgi].w[0], ypre[sgi].w[1], ypre[sgi].w[2], ypre[sgi].w[3]);
                Pack<BF16, 8>::unpack(kpre[sgi], a8);
                Pack<BF16, 8>::unpack(vpre[sgi], b8);
                Words<4> uu;
#pragma unroll
                for (int e2 = 0; e2 < 4; ++e2) uu.w[e2] = pack_bf16x2(a8[2 * e2] * b8[2 * e2], a8[2 * e2 + 1] * b8[2 * e2 + 1]);
                // z reaches over the end of the tile but not over the end of the sequence; the filter gradient
                // takes u of the tile only
                const bool in_own = kShard ? t0 + lr < t_end : in_seq;
                utr[ci & 1][st_idx] = in_seq ? make_uint4(uu.w[0], uu.w[1], uu.w[2], uu.w[3]) : make_uint4(0u, 0u, 0u, 0u);
                ust[ci & 1][wr8a] = in_own ? make_uint2(uu.w[0], uu.w[1]) : make_uint2(0u, 0u);
                ust[ci & 1][wr8b] = in_own ? make_uint2(uu.w[2], uu.w[3]) : make_uint2(0u, 0u);
            }
            load_g(ci + PF, ahead, ypre[sgi], qpre[sgi]);

            __syncthreads();

#pragma unroll
            for (int m = NKB - 1; m > 0; --m) {
                gw[m] = gw[m - 1];
                uw[m] = uw[m - 1];
            }
            {
                typedef __attribute__((address_space(3))) s16x4_t lds_quad_t;
                auto octet = [&](const uint4* rows, int at, int on) {
                    const char* p = reinterpret_cast<const char*>(rows) + at;
                    struct { s16x4_t lo, hi; } x;
                    x.lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_quad_t*)p);
                    x.hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_quad_t*)(p + on));
                    return __builtin_bit_cast(bf16x8_t, x);
                };
                gw[0] = octet(gst[ci & 1], rd_fwd, 4 * PPR * 16);
                uw[0] = octet(utr[ci & 1], rd_rev, -4 * PPR * 16);
            }

            if (main_chunk) {
                f32x4_t acc0 = {0.0f, 0.0f, 0.0f, 0.0f}, acc1 = {0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
                for (int m = 0; m < NKB; ++m) {
                    acc0 = __builtin_amdgcn_mfma_f32_16x16x32_bf16(gw[m], tz[2 * m], acc0, 0, 0, 0);
                    acc1 = __builtin_amdgcn_mfma_f32_16x16x32_bf16(gw[m], tz[2 * m + 1], acc1, 0, 0, 0);
                }
                char* zp = zst[ci & 1] + zwr_off;
                *reinterpret_cast<float4*>(zp) = make_float4(acc0[0], acc0[1], acc0[2], acc0[3]);
                *reinterpret_cast<float4*>(zp + 16 * ZROW) = make_float4(acc1[0], acc1[1], acc1[2], acc1[3]);

                // filter gradient: u rows 16 p + i of this chunk against g rows 16 p - 16 x + n
#pragma unroll
                for (int p = 0; p < 2; ++p) {
                    const uint2 ua = ust[ci & 1][(16 * p + li) * CPR + rd8];
                    const s16x4_t av = __builtin_bit_cast(s16x4_t, ua);
#pragma unroll
                    for (int x = 0; x < ND; ++x) {
                        const int rel = 16 * p - 16 * x;                  // row of the g tile relative to this chunk
                        const int back = (31 - rel) / 32;                 // chunks back (0 for rel >= 0); rel <= 16
                        const int rin = rel + 32 * back;                  // row inside that chunk
                        int gs = slot - back;
                        if (gs < 0) gs += NSLOT;
                        const uint2 gb = gring[gs][(rin + li) * CPR + rd8];
                        cacc[x] = __builtin_amdgcn_mfma_f32_16x16x16bf16_1k(av, __builtin_bit_cast(s16x4_t, gb), cacc[x], 0, 0, 0);
                    }
                }
            }
            // z of chunk ci - LAG: its source blocks ci - LAG .. ci are all in the window now.  Source block
            // ci - LAG + s sits s chunks after the output chunk: offset 32 s + 16 for the first 16 outputs,
            // 32 s for the second 16.
            // (`late` is chunk ci - LAG here)
            if (ci < ntot && in_tile(ci - LAG, late)) {
                f32x4_t acc0 = {0.0f, 0.0f, 0.0f, 0.0f}, acc1 = {0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
                for (int s = 0; s < NKB; ++s) {
                    acc0 = __builtin_amdgcn_mfma_f32_16x16x32_bf16(uw[LAG - s], tz[2 * s + 1], acc0, 0, 0, 0);
                    acc1 = __builtin_amdgcn_mfma_f32_16x16x32_bf16(uw[LAG - s], tz[2 * s], acc1, 0, 0, 0);
                }
                char* zp = zst2[ci & 1] + zwr_off_rev;
                *reinterpret_cast<float4*>(zp) = make_float4(acc0[0], acc0[1], acc0[2], acc0[3]);
                *reinterpret_cast<float4*>(zp + 16 * ZROW) = make_float4(acc1[0], acc1[1], acc1[2], acc1[3]);
            }
            const int prev = (sgi + PF - 1) % PF;  // static after unrolling
            if (ci > 0 && ci <= ntot) {
                gate_store_du(ci - 1, before, kpre[prev], vpre[prev]);
                gate_store_dq(ci - 1 - LAG, late_before);
            }
            load_kv(ci - 1 + PF, ahead_kv, kpre[prev], vpre[prev]);
            ahead_kv = ahead;
            forward(ahead);
            before = here;
            forward(here);
            late_before = late;
            if (ci >= LAG) forward(late);
        }
    }

    // ---- fold the diagonals: dh[16 x + i - n] += C_x[i][n]; the lane holds C_x[4 lq + r][li], r = 0..3
    __syncthreads();  // every wave is done with zst
    float* tilebuf = reinterpret_cast<float*>(zst[0]) + w * (16 * 17);  // this wave's 16 x 16 tile, row stride 17
    float* dhw = hs[w];                                                 // reuse: this wave's partial dh, kTaps floats
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
    float* out = a.partial + ((int64_t)tile * (D / 16) + (c0 / 16)) * a.lh;
    for (int j = lane; j < a.lh; j += 64) out[j] = dhw[j];
}

constexpr int kBwdWaves = 4;  // waves (16-channel slices) per workgroup

struct Tiling {
    int64_t chunks, tiles_per_seq, ntiles;  // ntiles: per channel block
    bool across;
};

// Tiles of mr_bwd_rows() steps within a batch item, or tiles of all items in a row, as many as make one round of
// workgroups, where that takes fewer chunks (a tile's halo and its start priced as chunks): a batch that does not divide the
// compute units otherwise pays for a round that is partly empty or for two rounds of short tiles (3 x 5000 x 2048, 128 taps:
// 480 tiles of 32 chunks or 256 of 61, 110 and 97 us).
Tiling tiling(const BwdShape& s) {
    const int64_t ncb = s.D / (16 * kBwdWaves), rows = mr_bwd_rows(s);
    Tiling t{rows / kChunk, (s.L + rows - 1) / rows, 0, false};
    t.ntiles = s.B * t.tiles_per_seq;
    if (s.sharded() || s.D >= kWideRows || s.B < 2 || tuning().mr_rows > 0) return t;
    const int64_t lag = (s.lh - 1 + 31) / 32, total = s.B * ((s.L + kChunk - 1) / kChunk + lag) - lag;
    if (total + lag > 0x7fffffffLL) return t;
    const int64_t want = ncb < 256 ? 256 / ncb : 1, chunks = (total + want - 1) / want, n = (total + chunks - 1) / chunks;
    auto cost = [&](int64_t tiles, int64_t each) { return (ncb * tiles + 255) / 256 * (each + lag + 8); };
    if (n <= t.ntiles && 33 * cost(n, chunks) <= 32 * cost(t.ntiles, t.chunks)) t = Tiling{chunks, n, n, true};
    return t;
}

template <int NKB, int NW>
hy_status launch_nw(const BwdPtrs& p, const BwdShape& s, void* ws, hipStream_t st, int64_t* nsets) {
    // Chunks of dy, q, k, v in flight per lane.  A fourth makes long walks at full width slower, not faster: the columns of a
    // row drift apart (2 / 3 / 4 / 5 / 6, 128 taps, us: 1 x 65536 x 4096 968 / 729 / 744 / 759 / 809, 1 x 8192 x 4096 137 / 104 /
    // 101 / 101 / 108, 3 x 5000 x 2048 131 / 99 / 100 / 95 / 99; 60 taps 1 x 8192 x 4096 122 / 96 / 113 / 113 / 117).
    constexpr int PF = 3;
    MrBwdArgs a;
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
    a.ncb = (int32_t)(s.D / (16 * NW));
    const Tiling t = tiling(s);
    a.chunks = (int32_t)t.chunks;
    a.tiles_per_seq = (int32_t)t.tiles_per_seq;
    a.across = t.across;
    a.items = (int32_t)s.B;
    *nsets = t.ntiles;
    const int64_t nb = *nsets * a.ncb;
    if (nb > 0x7fffffffLL) return HY_ERR_UNSUPPORTED;
    if (s.sharded() || s.D >= kWideRows)  // (the shard form has wide row offsets)
        return launch_kernel((mr_bwd_kernel<NKB, NW, PF, true>), dim3((uint32_t)nb), dim3(NW * 64), st, a);
    return launch_kernel((mr_bwd_kernel<NKB, NW, PF, false>), dim3((uint32_t)nb), dim3(NW * 64), st, a);
}

template <int NKB>
hy_status launch_nkb(const BwdPtrs& p, const BwdShape& s, void* ws, hipStream_t st, int64_t* nsets) {
    return launch_nw<NKB, kBwdWaves>(p, s, ws, st, nsets);
}

}  // namespace

bool mr_bwd_supported(const BwdShape& s) {
    return s.gated && s.dtype == HY_BF16 && s.group % 16 == 0 && s.D % 64 == 0 && s.lh > 8 && s.lh <= 129;
}

// time steps per workgroup: one workgroup per CU where the sequence allows it (same rule as the forward kernel)
int64_t mr_bwd_rows(const BwdShape& s) {
    const int64_t ncb = s.D / (16 * kBwdWaves);
    const int nkb = (s.lh - 1 + 31) / 32 + 1;
    int64_t rows = tuning().mr_rows;
    if (rows <= 0) {
        const int64_t halo = (int64_t)kChunk * (nkb > 1 ? nkb - 1 : 1);
        rows = one_round_rows(s.B * ncb, s.L, 4 * halo, kChunk);
        // (a tile as short as its halo: each one also leaves a row of partial filter gradients per slice)
        if (rows < halo) rows = halo;
    }
    rows = (rows + kChunk - 1) / kChunk * kChunk;
    const int64_t cap = (s.L + kChunk - 1) / kChunk * kChunk;
    return rows > cap ? cap : rows;
}

int64_t mr_bwd_workspace_bytes(const BwdShape& s) {
    return tiling(s).ntiles * (s.D / 16) * s.lh * (int64_t)sizeof(float);
}

// dq, dk, dv and dh in one pass.  `ws` holds the partial filter gradients.
hy_status launch_mr_bwd(const BwdPtrs& p, const BwdShape& s, void* ws, hipStream_t st) {
    if (!mr_bwd_supported(s)) return HY_ERR_UNSUPPORTED;
    const int nkb = (s.lh - 1 + 31) / 32 + 1;
    int64_t nsets = 0;
    hy_status rc;
    switch (nkb) {
        case 2: rc = launch_nkb<2>(p, s, ws, st, &nsets); break;
        case 3: rc = launch_nkb<3>(p, s, ws, st, &nsets); break;
        case 4: rc = launch_nkb<4>(p, s, ws, st, &nsets); break;
        case 5: rc = launch_nkb<5>(p, s, ws, st, &nsets); break;
        default: return HY_ERR_UNSUPPORTED;
    }
    if (rc != HY_OK) return rc;
    // partial rows are per 16-channel slice: a group of `group` channels owns group/16 adjacent slices
    const DhReduce r{static_cast<const float*>(ws), p.dh, nsets, s.D / 16, s.lh, s.group / 16};
    return launch_dh_reduce(&r, 1, st);
}

}  // namespace hy
