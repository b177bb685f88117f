// General FIR kernel: causal convolution and its transpose with optional gates, for any filter length, any group size,
// any width and both storage types, in fp32.  It stands behind every entry point, forward and backward, for the shapes
// the bf16 kernels do not cover (fp32 medium filters, widths and groups that do not tile the matrix cores, filters
// longer than the specialised limits).
//
// Bound: 2 lh flop per output (128 taps are 16 flop/B in fp32 against 10 the vector ALUs have per HBM byte and 20 the
// fp32 matrix products have).  So the sums run on v_mfma_f32_4x4x1_16B_f32, twice the rate of vector FMAs and the same
// arithmetic (fp32 products and sums): a block is one channel,
//     D[i][j] += w[m - i] * x[x0 + 4 j],   output row 16 k + 4 j + i, staged row x0 + 4 j = output row + tap (m = x0 - 16 k),
// so one operand of taps per m (lane = channel, i) serves every output block k, and one read of u per lane and x0 serves
// all output blocks whose taps it meets.  The kSeg + 3 tap operands stay in registers; a wave owns 16 channels x 128 rows
// (8 output blocks; small problems and short filters 32 rows, 2 blocks; whole bf16 pieces 64 rows), a workgroup 4 waves = 64
// channels.  The operand product u = a*b is formed once per workgroup into
// LDS as fp32 rows; 255 rows take 68 KiB, so two workgroups share a compute unit.  A workgroup walks several tiles of
// its sequence where there are enough of them, keeping the halo in LDS (bf16: with the next tile's rows and the tile's gate
// in flight while it computes; in fp32 they do not fit the registers beside the operands).  Outputs go back through LDS so that gates
// are read and outputs stored as whole row pieces.  Filters of more than 128 taps go through in segments, the sums staying
// where they are.  Every output adds its terms in ascending source order for the causal direction and ascending
// tap order for the transposed one, as a plain loop over the definition does.
// The products multiply structural zeros (taps outside the segment, rows that hold no data), which is only harmless for
// finite values: a workgroup that stages anything else takes the sums of that tile term by term on the vector ALUs,
// without the terms the definition does not have, so a non-finite tap or sample reaches exactly the outputs it reaches
// in the definition.
// Measured, 128 taps: B = 3, L = 5003, D = 1000 bf16 70 us (79 with 128-row tiles and the gate loaded behind the products),
// B = 2, L = 2048, D = 1024 fp32 25 us, B = 1, L = 8192, D = 4096 fp32 159 us (a filter of 32 taps there: 86); the same walk
// with vector FMAs, a lane one channel and 32 outputs: 100, 30, 198 us; 8 outputs per lane straight from global memory: 259,
// 64, 519 us.
#include <type_traits>
#include <utility>

#include "hy_common.hpp"
#include "hy_launch.hpp"

namespace hy {
namespace {

constexpr int kChan = 64;   // channels per workgroup, 16 per wave
constexpr int kWaves = 4;
constexpr int kThreads = kWaves * kWave;
constexpr int kStride = kChan + 4;  // floats per staged row: the operand reads and the row accesses hit all banks evenly

struct FirArgs {
    FirProblem p[3];
    int64_t L, D;
    int32_t lh, group;       // lh: the taps that can meet data
    int32_t row_taps;        // taps per filter in memory
    int32_t ncb;             // channel blocks
    int32_t steps;           // tiles a workgroup walks
    int32_t walks_per_seq;
    uint32_t together;  // neighbouring channel blocks on one XCD: the workgroups of the launch (0: apart)
};

__device__ __forceinline__ bool not_finite(float x) { return !(__builtin_fabsf(x) <= 3.402823466e+38f); }

// f(0), f(1), ... with the index as a compile-time constant
template <typename F, int... I>
__device__ __forceinline__ void each_index(F&& f, std::integer_sequence<int, I...>) {
    (f(std::integral_constant<int, I>{}), ...);
}

// VEC: elements per row access (16 bytes where the rows allow it, else one element); kSeg: taps per segment;
// NT: 16-row output blocks per tile
constexpr int per_cu(int seg, int nt) { return seg <= 32 && nt <= 2 ? 4 : 2; }  // workgroups a compute unit holds

template <typename T, int VEC, int kSeg, int NT, bool kOne>
__global__ __launch_bounds__(kThreads, per_cu(kSeg, NT)) void fir_kernel(FirArgs a) {
    constexpr int TR = 16 * NT;                    // output rows per tile
    constexpr int kRows = TR + kSeg - 1;           // staged rows
    constexpr int PPR = kChan / VEC;               // pieces per staged row
    constexpr int RPP = kThreads / PPR;            // rows per pass over the workgroup's lanes
    constexpr int kPassAll = (TR + RPP - 1) / RPP;  // passes that cover one tile's rows
    constexpr bool kAhead = kOne && T::kBytes == 2 && VEC > 1;  // the next tile's rows are loaded while this one is computed
    // passes in flight: 16-byte pieces take eight registers per pass, single elements (a quarter of the rows per pass) two
    constexpr int kPassFew = VEC == 1 ? (kSeg == 64 ? 16 : 8) : 4;
    constexpr int kPass = kAhead || kPassAll < kPassFew ? kPassAll : kPassFew;
    constexpr int kBatch = kPass * RPP < TR ? kPass * RPP : TR;  // rows they cover
    static_assert(!kAhead || kPass == kPassAll, "a tile's rows in flight at once");
    constexpr int kPutFew = VEC == 1 ? 8 : 4;
    constexpr int kPut = kPassAll < kPutFew ? kPassAll : kPutFew;  // pieces of a gate in flight
    constexpr bool kGateAhead = kAhead && NT <= 4 && kPut == kPassAll;  // ... loaded before the products
    constexpr int kMove = ((kSeg - 1) * (kChan / 4) + kThreads - 1) / kThreads;  // float4s of halo per lane
    constexpr int kTapStride = kSeg + 8;           // a channel's taps with three zeros on either side
    static_assert(kChan * kTapStride <= kRows * kStride, "the taps pass through the rows' memory");
    using PV = Pack<T, VEC>;
    __shared__ __attribute__((aligned(16))) float us[kRows * kStride];
    __shared__ int flags[2][kWaves];

    const FirProblem pr = a.p[blockIdx.y];
    const int tid = threadIdx.x, lane = tid % kWave, w = __builtin_amdgcn_readfirstlane(tid / kWave);
    const uint32_t lb = a.together ? xcd_contiguous(blockIdx.x, a.together) : blockIdx.x;
    const uint32_t walk = lb / (uint32_t)a.ncb;
    const int64_t c0 = (int64_t)(lb % (uint32_t)a.ncb) * kChan;
    const int64_t b = walk / (uint32_t)a.walks_per_seq;
    const int64_t t_first = (int64_t)(walk % (uint32_t)a.walks_per_seq) * a.steps * TR;
    const int64_t D = a.D, L = a.L;
    const int lh = a.lh;
    // filter of the block's first channel, and how many filters further the wave's channel `lane` % 16 is
    const int64_t g0 = c0 / a.group;
    const int cw = 16 * w + lane % 16;
    const uint32_t gstep = ((uint32_t)(c0 - g0 * a.group) + (uint32_t)(c0 + cw < D ? cw : D - 1 - c0)) / (uint32_t)a.group;
    const float* const h0 = pr.h + g0 * (int64_t)a.row_taps;
    const int64_t row_bytes = D * T::kBytes;

    // ---- rows of 64 channels: this lane's piece of the rows it loads and stores (a piece past the last channel reads
    // the block's first one)
    const int pc = tid % PPR, pr0 = tid / PPR;
    const bool own = c0 + (int64_t)pc * VEC < D;
    const int64_t col = own ? c0 + (int64_t)pc * VEC : c0;
    const char* const ap = static_cast<const char*>(pr.a) + (b * pr.stride_ab + col) * T::kBytes;
    const char* const bp = pr.b ? static_cast<const char*>(pr.b) + (b * pr.stride_ab + col) * T::kBytes : nullptr;
    typename PV::Raw ra[kPass], rb[kPass];
    auto load_rows = [&](int64_t t) {  // kBatch rows from time t on, clamped into the rows that hold data
#pragma unroll
        for (int i = 0; i < kPass; ++i) {
            int64_t tt = t + i * RPP + pr0;
            tt = tt < pr.hi ? tt : pr.hi - 1;
            tt = tt > pr.lo ? tt : pr.lo;
            const int64_t off = tt * row_bytes;
            ra[i] = PV::load(ap + off);
            if (bp) rb[i] = PV::load(bp + off);
        }
    };
    bool bad = false;  // this lane staged a value that is not finite
    // the loaded rows, whose first is time t, to the staged rows row .. min(row + kBatch, end) - 1; zeros where no data is
    auto write_rows = [&](int64_t t, int row, int end) {
#pragma unroll
        for (int i = 0; i < kPass; ++i) {
            const int rr = row + i * RPP + pr0;
            if (rr < end && (kBatch % RPP == 0 || i * RPP + pr0 < kBatch)) {
                const int64_t tt = t + i * RPP + pr0;
                const bool data = tt >= pr.lo && tt < pr.hi;
                float f[VEC], g[VEC];
                PV::unpack(ra[i], f);
                if (bp) PV::unpack(rb[i], g);
#pragma unroll
                for (int e = 0; e < VEC; ++e) {
                    if (bp) f[e] *= g[e];
                    f[e] = data ? f[e] : 0.0f;
                    bad |= not_finite(f[e]);
                }
                float* dst = us + rr * kStride + pc * VEC;
                if constexpr (VEC >= 4) {
#pragma unroll
                    for (int e = 0; e < VEC; e += 4)
                        *reinterpret_cast<float4*>(dst + e) = make_float4(f[e], f[e + 1], f[e + 2], f[e + 3]);
                } else {
#pragma unroll
                    for (int e = 0; e < VEC; ++e) dst[e] = f[e];
                }
            }
        }
    };

    // ---- products: block (channel) ch of the wave, row / column l4 of the 4 x 4 tiles
    const int ch = lane >> 2, l4 = lane & 3;
    const float* const up = us + 4 * l4 * kStride + 16 * w + ch;
    float wt[kSeg + 3];  // wt[m] = tap m - l4 of the segment in staged order, zero outside it
    bool bad_tap = false;

    // Tap j' of segment [ja, jb) is h[jb - 1 - j'] (causal) or h[ja + j'] (transposed); with it output row r meets the
    // staged row r + j', whose time is tb + r + j'
    auto load_taps = [&](int ja, int nt) {  // through the rows' memory
        bad_tap = false;
        constexpr int kX = (kTapStride + kWave - 1) / kWave, kCh = 8;  // channels in flight per wave
        for (int i0 = 0; i0 < 16; i0 += kCh) {  // a wave loads its own channels' taps
            float f[kCh][kX];
#pragma unroll
            for (int c = 0; c < kCh; ++c) {
                const float* hp = h0 + (int64_t)__builtin_amdgcn_readlane(gstep, i0 + c) * a.row_taps;
#pragma unroll
                for (int x = 0; x < kX; ++x) {  // unconditional loads: outside the segment its first tap, not used
                    const int jp = x * kWave + lane - 3;
                    const int j = jp >= 0 && jp < nt ? jp : 0;
                    f[c][x] = hp[pr.rev ? ja + j : ja + nt - 1 - j];
                }
            }
#pragma unroll
            for (int c = 0; c < kCh; ++c)
#pragma unroll
                for (int x = 0; x < kX; ++x) {
                    const int jp = x * kWave + lane - 3;
                    const float v = jp >= 0 && jp < nt ? f[c][x] : 0.0f;
                    bad_tap |= not_finite(v);
                    if (x * kWave + lane < kTapStride) us[(16 * w + i0 + c) * kTapStride + x * kWave + lane] = v;
                }
        }
        __syncthreads();
        const float* tp = us + (16 * w + ch) * kTapStride + 3 - l4;
#pragma unroll
        for (int m = 0; m < kSeg + 3; ++m) wt[m] = tp[m];
        __syncthreads();
    };

    const int nseg = kOne ? 1 : (lh + kSeg - 1) / kSeg;
    if constexpr (kOne) load_taps(0, lh);
    const int64_t t_stop = t_first + (int64_t)a.steps * TR < L ? t_first + (int64_t)a.steps * TR : L;
    int clean = 1 << 30;  // tiles since values that are not finite were staged
    int par = 0;
    for (int64_t t0 = t_first; t0 < t_stop; t0 += TR) {
        typename PV::Raw gahead[kGateAhead ? kPut : 1];
        auto load_gate = [&](typename PV::Raw* gr, const void* gate, int i0) {  // kPut pieces of the tile's rows
            const char* gp = static_cast<const char*>(gate) + (b * pr.stride_gate + col) * T::kBytes;
#pragma unroll
            for (int i = 0; i < kPut; ++i) {
                int64_t t = t0 + (i0 + i) * RPP + pr0;
                t = t < L ? t : L - 1;
                gr[i] = PV::load_nt(gp + t * row_bytes);
            }
        };
        f32x4_t acc[NT];
        if constexpr (!kOne) {
#pragma unroll
            for (int k = 0; k < NT; ++k) acc[k] = f32x4_t{0.0f, 0.0f, 0.0f, 0.0f};
        }
        for (int sg = 0; sg < nseg; ++sg) {
            const int si = pr.rev ? sg : nseg - 1 - sg;
            const int ja = si * kSeg, jb = ja + kSeg < lh ? ja + kSeg : lh;
            const int nt = jb - ja;
            const int64_t tb = pr.rev ? t0 + ja : t0 - (jb - 1);
            const int nrow = TR + nt - 1;
            if constexpr (!kOne) {
                if (tb + nrow <= pr.lo || tb >= pr.hi) continue;  // a filter longer than the sequence: no row holds data
                __syncthreads();  // every wave is done with the previous segment's rows
                load_taps(ja, nt);
            }
            bad = bad_tap;
            if (kOne && t0 > t_first) {
                // one segment: the halo is the end of the rows staged for the previous tile
                f32x4_t mv[kMove];
                const int nmv = (nt - 1) * (kChan / 4);
                auto at = [&](int row0, int x) {
                    return reinterpret_cast<f32x4_t*>(us + (row0 + x / (kChan / 4)) * kStride) + x % (kChan / 4);
                };
                // all of it at once where its old and new places overlap, else in parts (fewer registers).  The rows written
                // after this are among its old places, so parts that are read behind the first barrier need another.
                constexpr int kPart = TR >= kSeg - 1 && kMove > 2 ? 2 : kMove;
#pragma unroll
                for (int i0 = 0; i0 < kMove; i0 += kPart) {
#pragma unroll
                    for (int i = i0; i < i0 + kPart && i < kMove; ++i)
                        mv[i] = *at(TR, tid + i * kThreads < nmv ? tid + i * kThreads : 0);
                    if (i0 == 0) __syncthreads();  // (nobody reads the previous tile's outputs in rows 0 .. TR - 1 any more)
#pragma unroll
                    for (int i = i0; i < i0 + kPart && i < kMove; ++i)
                        if (tid + i * kThreads < nmv) *at(0, tid + i * kThreads) = mv[i];
                }
                if constexpr (kPart < kMove) __syncthreads();
                if constexpr (kAhead) {
                    write_rows(tb + nt - 1, nt - 1, nrow);
                } else {
                    for (int rw = nt - 1; rw < nrow; rw += kBatch) {
                        load_rows(tb + rw);
                        write_rows(tb + rw, rw, nrow);
                    }
                }
            } else {
                for (int rw = 0; rw < nrow; rw += kBatch) {
                    load_rows(tb + rw);
                    write_rows(tb + rw, rw, nrow);
                }
                for (int x = nrow * kStride + tid; x < kRows * kStride; x += kThreads) us[x] = 0.0f;  // meet zero taps
            }
            const bool wave_bad = __builtin_amdgcn_ballot_w64(bad) != 0;
            if (lane == 0) flags[par][w] = wave_bad;
            __syncthreads();
            bool new_bad = false;
#pragma unroll
            for (int i = 0; i < kWaves; ++i) new_bad |= flags[par][i] != 0;
            par ^= 1;
            // rows of this tile's halo were staged up to kBack tiles ago
            constexpr int kBack = kOne ? (kSeg - 1 + TR - 1) / TR : 0;
            clean = new_bad ? 0 : (clean < kBack + 1 ? clean + 1 : clean);
            const bool exact = __builtin_amdgcn_readfirstlane(clean <= kBack);
            if constexpr (kAhead)
                if (t0 + TR < t_stop) load_rows(tb + TR + nt - 1);  // the next tile's rows

            if constexpr (kGateAhead)
                if (pr.gate) load_gate(gahead, pr.gate, 0);
            if constexpr (kOne) {
#pragma unroll
                for (int k = 0; k < NT; ++k) acc[k] = f32x4_t{0.0f, 0.0f, 0.0f, 0.0f};
            }
            if (c0 + 16 * w < D) {
                if (!exact) {
                    // kX rows at a time, the next ones read while these are multiplied; the fences keep the scheduler
                    // from reading them all at once
                    constexpr int kX = 4, kAll = 16 * (NT - 1) + kSeg + 3;
                    float u[2][kX];
#pragma unroll
                    for (int i = 0; i < kX; ++i) u[0][i] = up[i * kStride];
                    auto rows = [&](auto xb_c) {
                        constexpr int XB = decltype(xb_c)::value;
#pragma unroll
                        for (int i = 0; i < kX; ++i)
                            if ((XB + 1) * kX + i < kAll) u[(XB + 1) & 1][i] = up[((XB + 1) * kX + i) * kStride];
#pragma unroll
                        for (int i = 0; i < kX; ++i) {
#pragma unroll
                            for (int k = 0; k < NT; ++k) {
                                const int m = XB * kX + i - 16 * k;
                                if (m >= 0 && m < kSeg + 3)
                                    acc[k] = __builtin_amdgcn_mfma_f32_4x4x1f32(wt[m], u[XB & 1][i], acc[k], 0, 0, 0);
                            }
                        }
                        __builtin_amdgcn_sched_barrier(0);
                    };
                    each_index(rows, std::make_integer_sequence<int, (kAll + kX - 1) / kX>{});
                } else {
                    // not everything is finite: the sums term by term, without the products' structural zeros and
                    // without the rows that hold no data
                    const int64_t vlo = pr.lo - tb, vhi = pr.hi - tb;
                    const float* hp = h0 + (int64_t)__shfl(gstep, ch) * a.row_taps;
                    for (int jp = 0; jp < nt; ++jp) {
                        const float h1 = hp[pr.rev ? ja + jp : jb - 1 - jp];
#pragma unroll
                        for (int k = 0; k < NT; ++k)
#pragma unroll
                            for (int i = 0; i < 4; ++i) {
                                const int row = 16 * k + i + jp;
                                const float x = __builtin_fmaf(h1, up[row * kStride], acc[k][i]);
                                acc[k][i] = (row + 4 * l4 >= vlo && row + 4 * l4 < vhi) ? x : acc[k][i];
                            }
                    }
                }
            }
        }

        // ---- outputs: through rows 0 .. TR - 1 (the halo of the next tile lies behind them), then as whole row pieces
        __syncthreads();
#pragma unroll
        for (int k = 0; k < NT; ++k)
#pragma unroll
            for (int i = 0; i < 4; ++i)
                us[(16 * k + 4 * l4 + i) * kStride + 16 * w + ch] = acc[k][i];
        __syncthreads();
        auto put = [&](const void* gate, void* out, auto ahead) {
            char* op = static_cast<char*>(out) + (b * pr.stride_out + col) * T::kBytes;
#pragma unroll
            for (int i0 = 0; i0 < kPassAll; i0 += kPut) {
                typename PV::Raw gr[kPut];
                if constexpr (decltype(ahead)::value) {
#pragma unroll
                    for (int i = 0; i < kPut; ++i) gr[i] = gahead[i];
                } else {
                    if (gate) load_gate(gr, gate, i0);
                }
#pragma unroll
                for (int i = 0; i < kPut; ++i) {
                    const int row = (i0 + i) * RPP + pr0;
                    float z[VEC], gf[VEC];
                    const float* zp = us + (row < TR ? row : 0) * kStride + pc * VEC;
#pragma unroll
                    for (int e = 0; e < VEC; ++e) z[e] = zp[e];
                    if (gate) {
                        PV::unpack(gr[i], gf);
#pragma unroll
                        for (int e = 0; e < VEC; ++e) z[e] *= gf[e];
                    }
                    if (own && row < TR && t0 + row < L) PV::store_nt(op + (t0 + row) * row_bytes, PV::pack(z));
                }
            }
        };
        put(pr.gate, pr.out, std::bool_constant<kGateAhead>{});
        if (pr.out2) put(pr.gate2, pr.out2, std::false_type{});
        if constexpr (!kOne) __syncthreads();  // before the next tile's taps
    }
}

template <typename T, int VEC, int kSeg, int NT, bool kOne>
hy_status launch_nt(FirArgs& a, int nprob, int64_t B, hipStream_t st) {
    constexpr int TR = 16 * NT;
    const int64_t tiles = (a.L + TR - 1) / TR;
    // Where there are tiles enough a workgroup walks its share of a sequence: as long as lets every workgroup be resident
    // at once, or in whole rounds where one round would be half empty (a walk's start, its halo and taps, is priced as
    // one tile).  With several segments nothing is kept from one tile to the next, so there every tile is a workgroup of
    // its own (3 x 2730 x 1024 fp32, 200 taps: 119 -> 99 us).
    int64_t walks = tiles;
    if (kOne) {
        constexpr int64_t resident = 256 * per_cu(kSeg, NT);
        const int64_t units = B * a.ncb * nprob, least = (units + resident - 1) / resident;
        auto cost = [&](int64_t w) { return (units * w + resident - 1) / resident * ((tiles + w - 1) / w + 1); };
        walks = 1;
        for (int64_t rounds = least; rounds < least + 4; ++rounds) {
            const int64_t w = rounds * resident / units < tiles ? rounds * resident / units : tiles;
            if (cost(w) < cost(walks)) walks = w;
        }
    }
    const int64_t steps = (tiles + walks - 1) / walks;
    walks = (tiles + steps - 1) / steps;
    if (steps > 0x7fffffffLL || B > 0x7fffffffLL || B * walks > 0x7fffffffLL / a.ncb) return HY_ERR_UNSUPPORTED;
    a.steps = (int32_t)steps;
    a.walks_per_seq = (int32_t)walks;
    // Rows that are no whole lines: a row piece shares its first and last line with its neighbours', which one L2 then holds for
    // all.  Us, apart / together: 2 x 1500 x 1000, 9 taps bf16 12.5 / 10.4, fp32 16.1 / 13.8, x 1001 15.9 / 14.5 and 17.7 / 16.3;
    // 1 x 3000 x 1000, 64 taps bf16 17.6 / 15.8, fp32 20.4 / 18.4.  Not
    // - where every workgroup has a compute unit to itself anyway (128 taps fp32 1 x 300 x 1000, 160 of them, 11.3 / 11.9, 1 x 600 x
    //   1000, 304 of them, 14.5 / 13.9);
    // - for rows of whole lines, which run better spread out (2 x 2048 x 1024 fp32, forward and gradients 109 / 118), and two problems
    //   side by side (gradients 2 x 2000 x 1000 120.6 / 122.7);
    // - for wide fp32 rows of short sequences (64 x 128 x 4088, 9 taps 121 / 137, 40 x 100 x 4088 68 / 70, 100 x 40 x 6000 94 / 98;
    //   64 x 128 x 3000 94 / 95, 20 x 200 x 3000 58 / 53, x 6000 95 / 92, 5 x 1000 x 4088 84 / 75, bf16 20 x 200 x 8184 85 / 75);
    // - for several segments of wide rows (1 x 4000 x 4088, 250 taps fp32 172 / 193), or where XCDs would have unequal shares: the
    //   first tiles of a sequence leave segments out (2 x 700 x 1000, 300 taps fp32 47 / 50.5, 1 x 9000 x 1000, 1000 taps 344 / 356;
    //   1 x 4000 x 1000, 250 taps 51 / 46, 8 x 300 x 1000, 250 taps 41.5 / 35.6).
    const int64_t nblocks = B * walks * a.ncb, row = a.D * T::kBytes;
    const bool even = kOne ? T::kBytes == 2 || row <= 12288 || a.L >= 192
                           : row <= 4096 && (B >= 8 || 16 * (int64_t)a.lh <= a.L);
    a.together = row % 128 != 0 && nprob == 1 && nblocks > 256 && even ? (uint32_t)nblocks : 0;
    return launch_kernel((fir_kernel<T, VEC, kSeg, NT, kOne>), dim3((uint32_t)nblocks, (uint32_t)nprob),
                         dim3(kThreads), st, a);
}

// Rows of 16-byte bf16 pieces: 64-row tiles leave the registers to load both the next tile's rows and this tile's gate before
// the products.
template <typename T, int VEC>
constexpr bool half_tiles() { return T::kBytes == 2 && VEC > 1; }

template <typename T, int VEC, int NT>
hy_status launch_seg(FirArgs& a, int nprob, int64_t B, hipStream_t st) {
    if constexpr (NT <= 2)  // (3 x 2730 x 1024 fp32, 9 taps, against a segment of 32: 28.5 -> 26.4 us)
        if (a.lh <= 16) return launch_nt<T, VEC, 16, NT, true>(a, nprob, B, st);
    if (a.lh <= 32) return launch_nt<T, VEC, 32, NT, true>(a, nprob, B, st);
    if constexpr (NT <= 2 || !half_tiles<T, VEC>()) {  // (else launch_vec's)
        if (a.lh <= 64) return launch_nt<T, VEC, 64, NT, true>(a, nprob, B, st);
        if (a.lh <= 128) return launch_nt<T, VEC, 128, NT, true>(a, nprob, B, st);
    }
    // three segments of 64 are 201 products per output block, two of 128 are 262 (3 x 5003 x 1000 fp32, 150 taps: 152
    // against 166 us); beyond 192 taps staging the rows once more costs what the products save (400 taps: 304 / 285)
    if (a.lh <= 192) return launch_nt<T, VEC, 64, NT, false>(a, nprob, B, st);
    return launch_nt<T, VEC, 128, NT, false>(a, nprob, B, st);
}

template <typename T, int VEC>
hy_status launch_vec(FirArgs& a, int nprob, int64_t B, hipStream_t st) {
    // (rows 128 or 32 by the rules below / 64, bf16, 128 taps, us: 3 x 5003 x 1000 84.0 / 68.4, 4 x 4096 x 2056 189 / 153,
    // 6 x 690 x 1000 42.3 / 29.3, 1 x 700 x 1000 13.5 / 11.1, gradients 3 x 1300 x 1000 103 / 89; 50 taps 3 x 5003 x 1000
    // 51.3 / 51.1, 40 taps 1 x 4000 x 1000 17.8 / 16.4; but 30 taps 3 x 5003 x 1000 39.7 / 40.6.)  fp32 rows are twice as
    // many registers: they do not fit.  A problem for whose 32-row tiles the compute units take no more turns than for 64-row
    // ones has the shorter turns (32 / 64: 1 x 65 x 1000, 33 taps 6.9 / 8.1, 6 x 158 x 1000, 65 taps 12.4 / 14.4; with
    // twice the turns 6 x 84 x 2056, 50 taps 13.0 / 10.7).
    if constexpr (half_tiles<T, VEC>()) {
        if (a.lh > 32 && a.lh <= 128) {
            auto turns = [&](int64_t rows) { return (B * a.ncb * nprob * ((a.L + rows - 1) / rows) + 255) / 256; };
            if (turns(32) == turns(64)) return launch_seg<T, VEC, 2>(a, nprob, B, st);
            if (a.lh > 64) return launch_nt<T, VEC, 128, 4, true>(a, nprob, B, st);
            return launch_nt<T, VEC, 64, 4, true>(a, nprob, B, st);
        }
    }
    // 128-row tiles amortise the 127 halo rows of a 128-tap filter; a problem that leaves compute units without a
    // workgroup that way is cut into 32-row tiles instead, and so is one whose last tile would be mostly padding.  (Eight
    // waves over 128 channels, one workgroup per compute unit, measured the same on long sequences and 13% slower at
    // 2 x 2048 x 1024.)  Up to 32 taps the halo is small and short tiles, four workgroups to a compute unit, hide more
    // of each other's loads, unless one long tile holds the whole sequence and there is no halo at all; rows of single
    // bf16 elements, which take the most load instructions per byte, gain from that at any length.  Rows 128 / 32, us:
    // 57 x 30 x 2048 fp32 34.4 / 17.8, 8 x 60 x 2048, 128 taps 11.1 / 9.0; 9 taps: 2 x 1500 x 1001 fp32 23.5 / 16.4,
    // 3 x 2730 x 1024 fp32 34.1 / 26.4, 3 x 5003 x 1000 bf16 44.8 / 44.1, but 40 x 102 x 2048 fp32 32.2 / 36; 33 and 128
    // taps: 2 x 1500 x 1001 bf16 28 / 21 and 35 / 30, 4 x 8000 x 1001 bf16 161 / 151 and 216 / 202, fp32 152 / 162 and
    // 212 / 210.  Several segments: 3 x 5003 x 1000 bf16, 200 taps 154 / 319.
    const int64_t rows = (a.L + 127) / 128 * 128;
    const bool full = B * (rows / 128) * a.ncb * nprob >= 256;
    const bool padded = 4 * rows > 5 * ((a.L + 31) / 32 * 32);
    const bool short_tiles = a.lh <= 32 ? a.L > 128 : VEC == 1 && T::kBytes == 2;
    const bool wide = full && (a.lh > 128 || !(padded || short_tiles));
    return wide ? launch_seg<T, VEC, 8>(a, nprob, B, st) : launch_seg<T, VEC, 2>(a, nprob, B, st);
}

template <typename T>
hy_status launch_t(FirArgs& a, int nprob, int64_t B, hipStream_t st) {
    constexpr int V = 16 / T::kBytes;
    // rows are 16-byte aligned when D is a multiple of V (base pointers and batch strides always are)
    return a.D % V == 0 ? launch_vec<T, V>(a, nprob, B, st) : launch_vec<T, 1>(a, nprob, B, st);
}

}  // namespace

hy_status launch_fir(const FirProblem* p, int nprob, int64_t B, int64_t L, int64_t D, int32_t lh, int32_t group,
                     hy_dtype dtype, hipStream_t st) {
    FirArgs a;
    for (int i = 0; i < 3; ++i) a.p[i] = p[i < nprob ? i : 0];
    a.L = L;
    a.D = D;
    // taps beyond the first row with data (causal) or the last (transposed) meet none: a filter longer than its sequence
    // is one of its length (15 x 31 x 333 fp32 featurizers, 800 taps: 28 -> 12 us)
    int64_t reach = 1;
    for (int i = 0; i < nprob; ++i) {
        const int64_t r = p[i].rev ? p[i].hi : L - p[i].lo;
        if (r > reach) reach = r;
    }
    a.lh = lh < reach ? lh : (int32_t)reach;
    a.row_taps = lh;
    a.group = group;
    const int64_t ncb = (D + kChan - 1) / kChan;
    if (ncb > 0x7fffffffLL) return HY_ERR_UNSUPPORTED;
    a.ncb = (int32_t)ncb;
    return dtype == HY_BF16 ? launch_t<BF16>(a, nprob, B, st) : launch_t<F32>(a, nprob, B, st);
}

}  // namespace hy
