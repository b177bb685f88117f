// General FIR kernel: causal convolution and its transpose with optional gates, for any filter length, any group size,
// any width and both storage types, fp32 arithmetic on the vector ALUs.  It stands behind every entry point, forward
// and backward, for the shapes the specialised kernels do not cover (fp32 medium filters, widths and groups that do not
// tile the matrix cores, filters longer than the specialised limits).
//
// Bound: vector FMA issue (2 lh flop per output; 128 taps are 16 flop/B in fp32 against 10 the ALUs have per HBM byte).
// So the kernel is laid out around the FMAs: a lane owns one channel and kR consecutive outputs, whose sums stay in
// registers; the operand product u = a*b is formed once per workgroup into LDS as fp32 rows of 64 channels (a lane's
// column: conflict-free), and a block of 16 taps then costs kR + 15 reads of u and 16 of taps per 16 kR FMAs.  One
// workgroup is 4 waves x kR rows x 64 channels.  u (255 rows) and one stage of 64 taps take 80 KiB, so two workgroups
// share a compute unit; a workgroup walks several tiles of its sequence where there are enough of them, keeping the
// halo in LDS and loading the next tile's rows while it computes.  Filters of more than 128 taps go through in segments
// of 128, the sums staying where they are.  Every output adds its terms in ascending source order for the causal
// direction and ascending tap order for the transposed one, as a plain loop over the definition does.
// Terms the definition does not have (sources before the first or behind the last row that holds data) are left out and
// not multiplied by zeros, so a non-finite tap or sample reaches exactly the outputs it reaches in the definition; only
// the blocks of taps that cross such an end pay for the test.
// Measured, 128 taps, against a kernel with 8 outputs per lane and every sample and tap loaded from global memory:
// B = 3, L = 5003, D = 1000 bf16 245 -> 106 us; B = 2, L = 2048, D = 1024 fp32 67 -> 30 us forward and 126 -> 64 us for
// dq, dk, dv (the FMAs alone take 51, 14 and 28 us at their peak rate).
#include <type_traits>

#include "hy_common.hpp"
#include "hy_launch.hpp"

namespace hy {
namespace {

constexpr int kChan = 64;   // channels per workgroup, one per lane
constexpr int kWaves = 4;
constexpr int kThreads = kWaves * kWave;
constexpr int kSeg = 128;   // taps per segment
constexpr int kStage = 64;  // taps staged in LDS at a time
constexpr int kBlk = 16;    // taps per register block
constexpr int kTapStride = kChan + 1;  // floats per staged tap: the transposing writes hit 64 different banks

struct FirArgs {
    FirProblem p[3];
    int64_t L, D;
    int32_t lh, group;
    int32_t ncb;             // channel blocks of 64
    int32_t steps;           // tiles of kWaves * kR rows a workgroup walks
    int32_t walks_per_seq;
};

// VEC: elements per staging load (16 bytes where the rows allow it, else one element)
template <typename T, int VEC, int kR>
__global__ __launch_bounds__(kThreads, 2) void fir_kernel(FirArgs a) {
    constexpr int TR = kWaves * kR;                // output rows per tile
    constexpr int kRows = TR + kSeg - 1;           // staged rows
    constexpr int PPR = kChan / VEC;               // pieces per staged row
    constexpr int RPP = kThreads / PPR;            // rows per pass over the workgroup's lanes
    constexpr bool kAhead = VEC > 1;               // the next tile's rows are loaded while this one is computed
    constexpr int kPassAll = (TR + RPP - 1) / RPP;  // passes that load one tile's rows
    constexpr int kPass = kAhead || kPassAll < 8 ? kPassAll : 8;  // passes in flight
    constexpr int kBatch = kPass * RPP < TR ? kPass * RPP : TR;   // rows they load
    constexpr int kTapsPer = kStage * kChan / kThreads;
    constexpr int kMove = (kSeg - 1) * (kChan / 4) / kThreads + 1;  // float4s of halo per lane
    using PV = Pack<T, VEC>;
    using P1 = Pack<T, 1>;
    // taps first: their offsets and those of a register block's rows then fit the LDS instructions
    __shared__ __attribute__((aligned(256))) float lds[kStage * kTapStride + kRows * kChan];
    float* const ts = lds;
    float* const us = lds + kStage * kTapStride;
    static_assert(kStage * kTapStride % kChan == 0, "rows start on a multiple of 256 bytes");

    const FirProblem pr = a.p[blockIdx.y];
    const int tid = threadIdx.x, lane = tid % kWave, w = __builtin_amdgcn_readfirstlane(tid / kWave);
    const uint32_t lb = blockIdx.x;
    const uint32_t walk = lb / (uint32_t)a.ncb;
    const int64_t c0 = (int64_t)(lb % (uint32_t)a.ncb) * kChan;
    const int64_t b = walk / (uint32_t)a.walks_per_seq;
    const int64_t t_first = (int64_t)(walk % (uint32_t)a.walks_per_seq) * a.steps * TR;
    const int64_t D = a.D, L = a.L;
    const int lh = a.lh;
    const bool own = c0 + lane < D;
    const int r0 = w * kR;  // first row of this wave in a tile
    // filter of the block's first channel, and how many filters further this lane's channel is
    const int64_t g0 = c0 / a.group;
    const uint32_t gstep = ((uint32_t)(c0 - g0 * a.group) + (uint32_t)(own ? lane : D - 1 - c0)) / (uint32_t)a.group;
    const float* const h0 = pr.h + g0 * (int64_t)lh;
    const int64_t row_bytes = D * T::kBytes;

    // ---- staging: this lane's piece of the rows it loads (a piece past the last channel re-reads the block's first)
    const int pc = tid % PPR, pr0 = tid / PPR;
    const int64_t piece = (b * pr.stride_ab + (c0 + (int64_t)pc * VEC < D ? c0 + (int64_t)pc * VEC : c0)) * T::kBytes;
    const char* const ap = static_cast<const char*>(pr.a) + piece;
    const char* const bp = pr.b ? static_cast<const char*>(pr.b) + piece : nullptr;
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
    auto write_rows = [&](int row, int end) {  // the loaded rows to the staged rows row .. min(row + kBatch, end) - 1
#pragma unroll
        for (int i = 0; i < kPass; ++i) {
            const int rr = row + i * RPP + pr0;
            if (rr < end && (kBatch % RPP == 0 || i * RPP + pr0 < kBatch)) {
                float f[VEC], g[VEC];
                PV::unpack(ra[i], f);
                if (bp) {
                    PV::unpack(rb[i], g);
#pragma unroll
                    for (int e = 0; e < VEC; ++e) f[e] *= g[e];
                }
                float* dst = us + rr * kChan + pc * VEC;
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

    // ---- outputs: one channel per lane, a wave stores 64 channels of a row
    constexpr int kPut = kR < 16 ? kR : 16;  // gate rows in flight
    const uint32_t own_off = (uint32_t)(own ? lane : 0) * T::kBytes;
    auto put = [&](int64_t t, const float (&acc)[kR], const void* gate, void* out) {  // rows t .. t + kR - 1
        if (t >= L) return;
        const char* gp = static_cast<const char*>(gate) + (b * pr.stride_gate + c0) * T::kBytes + t * row_bytes;
        char* op = static_cast<char*>(out) + (b * pr.stride_out + c0) * T::kBytes + t * row_bytes;
        const int n = L - t < kR ? (int)(L - t) : kR;
#pragma unroll
        for (int rb = 0; rb < kR; rb += kPut) {
            typename P1::Raw gr[kPut];
            if (gate) {
#pragma unroll
                for (int r = 0; r < kPut; ++r) {
                    gr[r] = P1::load(gp + own_off);
                    gp += rb + r + 1 < n ? row_bytes : 0;  // behind the last row it repeats
                }
            }
#pragma unroll
            for (int r = 0; r < kPut; ++r) {
                float z[1] = {acc[rb + r]}, gf[1];
                if (gate) {
                    P1::unpack(gr[r], gf);
                    z[0] *= gf[0];
                }
                if (own && rb + r < n) P1::store(op + own_off, P1::pack(z));
                op += row_bytes;
            }
        }
    };

    // tap j' of segment [ja, jb) is h[jb - 1 - j'] (causal) or h[ja + j'] (transposed); with it output row r meets the
    // staged row r + j', whose time is tb + r + j'
    const int nseg = (lh + kSeg - 1) / kSeg;
    const int64_t t_stop = t_first + (int64_t)a.steps * TR < L ? t_first + (int64_t)a.steps * TR : L;
    bool staged = false;
    for (int64_t t0 = t_first; t0 < t_stop; t0 += TR) {
        float acc[kR];
#pragma unroll
        for (int r = 0; r < kR; ++r) acc[r] = 0.0f;

        for (int sg = 0; sg < nseg; ++sg) {
            const int si = pr.rev ? sg : nseg - 1 - sg;
            const int ja = si * kSeg, jb = ja + kSeg < lh ? ja + kSeg : lh;
            const int nt = jb - ja;
            const int64_t tb = pr.rev ? t0 + ja : t0 - (jb - 1);
            const int nrow = TR + nt - 1;

            auto load_taps = [&](int first, float (&f)[kTapsPer]) {
                const int jt = first + lane;  // a wave reads 64 consecutive taps of one filter per step
#pragma unroll
                for (int i = 0; i < kTapsPer; ++i) {
                    const uint32_t gs = __builtin_amdgcn_readlane(gstep, w + kWaves * i);
                    f[i] = 0.0f;
                    if (jt < nt) f[i] = h0[(int64_t)gs * lh + (pr.rev ? ja + jt : jb - 1 - jt)];
                }
            };
            auto write_taps = [&](const float (&f)[kTapsPer]) {
#pragma unroll
                for (int i = 0; i < kTapsPer; ++i) ts[lane * kTapStride + w + kWaves * i] = f[i];
            };

            float tp[kTapsPer];
            load_taps(0, tp);
            if (staged) {
                // one segment: the halo is the end of the rows staged for the previous tile, the new rows were loaded
                // while that tile was computed
                f32x4_t mv[kMove];
                const int nmv = (nt - 1) * (kChan / 4);
                const f32x4_t* src = reinterpret_cast<const f32x4_t*>(us + TR * kChan);
                __syncthreads();  // every wave is done with the previous tile
#pragma unroll
                for (int i = 0; i < kMove; ++i) mv[i] = src[tid + i * kThreads < nmv ? tid + i * kThreads : 0];
                __syncthreads();
#pragma unroll
                for (int i = 0; i < kMove; ++i)
                    if (tid + i * kThreads < nmv) reinterpret_cast<f32x4_t*>(us)[tid + i * kThreads] = mv[i];
                if constexpr (kAhead) {
                    write_rows(nt - 1, nrow);
                } else {
                    for (int rw = nt - 1; rw < nrow; rw += kBatch) {
                        load_rows(tb + rw);
                        write_rows(rw, nrow);
                    }
                }
            } else {
                if (t0 > t_first || sg > 0) __syncthreads();
                for (int rw = 0; rw < nrow; rw += kBatch) {
                    load_rows(tb + rw);
                    write_rows(rw, nrow);
                }
            }
            write_taps(tp);
            __syncthreads();
            staged = nseg == 1 && t0 + TR < t_stop;
            if constexpr (kAhead)
                if (staged) load_rows(tb + TR + nt - 1);  // the next tile's rows

            // staged rows [vlo, vhi) hold data
            const int64_t vlo64 = pr.lo - tb, vhi64 = pr.hi - tb;
            const int vlo = vlo64 > 0 ? (vlo64 < nrow ? (int)vlo64 : nrow) : 0;
            const int vhi = vhi64 < nrow ? (vhi64 > 0 ? (int)vhi64 : 0) : nrow;
            for (int st = 0; st < nt; st += kStage) {
                const int n = nt - st < kStage ? nt - st : kStage;
                const bool more = st + kStage < nt;
                if (more) load_taps(st + kStage, tp);
                const int rs = r0 + st;  // row that output 0 of this wave meets with tap 0 of the stage
                const float* up = us + rs * kChan + lane;
                const float* hp = ts + lane;
                int j = 0;
                auto tap_block = [&](auto nb_c, auto whole_c) {  // the next nb taps of the stage
                    constexpr int NB = decltype(nb_c)::value;
                    float uw[kR + NB - 1], hw[NB];
#pragma unroll
                    for (int i = 0; i < NB; ++i) hw[i] = hp[i * kTapStride];
#pragma unroll
                    for (int i = 0; i < kR + NB - 1; ++i) uw[i] = up[i * kChan];
                    if constexpr (decltype(whole_c)::value) {
#pragma unroll
                        for (int i = 0; i < NB; ++i)
#pragma unroll
                            for (int r = 0; r < kR; ++r) acc[r] = __builtin_fmaf(hw[i], uw[r + i], acc[r]);
                    } else {  // rows outside [vlo, vhi) have no term
                        const int lo = vlo - rs - j, hi = vhi - rs - j;
#pragma unroll
                        for (int x = 0; x < kR + NB - 1; ++x) {
                            const bool has = x >= lo && x < hi;
#pragma unroll
                            for (int i = 0; i < NB; ++i)
                                if (x - i >= 0 && x - i < kR) {
                                    const float y = __builtin_fmaf(hw[i], uw[x], acc[x - i]);
                                    acc[x - i] = has ? y : acc[x - i];
                                }
                        }
                    }
                    j += NB;
                    hp += NB * kTapStride;
                    up += NB * kChan;
                };
                using Blk = std::integral_constant<int, kBlk>;
                using One = std::integral_constant<int, 1>;
                while (j + kBlk <= n && rs + j + kR + kBlk - 2 < vlo) {  // no row of the block holds data
                    j += kBlk;
                    hp += kBlk * kTapStride;
                    up += kBlk * kChan;
                }
                while (j + kBlk <= n && rs + j < vlo) tap_block(Blk{}, std::false_type{});
                while (j + kBlk <= n && rs + j + kR + kBlk - 2 < vhi) tap_block(Blk{}, std::true_type{});
                while (j + kBlk <= n && rs + j < vhi) tap_block(Blk{}, std::false_type{});
                while (j < n && rs + j < vhi) tap_block(One{}, std::false_type{});
                if (more) {
                    __syncthreads();
                    write_taps(tp);
                    __syncthreads();
                }
            }
        }

        put(t0 + r0, acc, pr.gate, pr.out);
        if (pr.out2) put(t0 + r0, acc, pr.gate2, pr.out2);
    }
}

template <typename T, int VEC, int kR>
hy_status launch_r(FirArgs& a, int nprob, int64_t B, hipStream_t st) {
    constexpr int TR = kWaves * kR;
    const int64_t tiles = (a.L + TR - 1) / TR;
    // two workgroups per compute unit where there are tiles enough: each then walks its share of a sequence, loading the
    // next tile's rows while it computes
    int64_t walks = 512 / (B * a.ncb * nprob);
    if (walks < 1) walks = 1;
    if (walks > tiles) walks = tiles;
    const int64_t steps = (tiles + walks - 1) / walks;
    walks = (tiles + steps - 1) / steps;
    if (steps > 0x7fffffffLL || B > 0x7fffffffLL || B * walks > 0x7fffffffLL / a.ncb) return HY_ERR_UNSUPPORTED;
    a.steps = (int32_t)steps;
    a.walks_per_seq = (int32_t)walks;
    return launch_kernel((fir_kernel<T, VEC, kR>), dim3((uint32_t)(B * walks * a.ncb), (uint32_t)nprob), dim3(kThreads), st, a);
}

template <typename T, int VEC>
hy_status launch_vec(FirArgs& a, int nprob, int64_t B, hipStream_t st) {
    // 128-row tiles amortise the 127 halo rows of a 128-tap filter; a problem that leaves compute units without a
    // workgroup that way is cut into 32-row tiles instead
    const int64_t wg = B * ((a.L + 127) / 128) * a.ncb * nprob;
    return wg >= 256 ? launch_r<T, VEC, 32>(a, nprob, B, st) : launch_r<T, VEC, 8>(a, nprob, B, st);
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
    a.lh = lh;
    a.group = group;
    const int64_t ncb = (D + kChan - 1) / kChan;
    if (ncb > 0x7fffffffLL) return HY_ERR_UNSUPPORTED;
    a.ncb = (int32_t)ncb;
    return dtype == HY_BF16 ? launch_t<BF16>(a, nprob, B, st) : launch_t<F32>(a, nprob, B, st);
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
    return launch_fir(f, nprob, s.B, s.L, s.D, s.lh, s.group, s.dtype, st);
}

}  // namespace hy
