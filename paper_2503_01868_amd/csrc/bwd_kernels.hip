// Backward of the gated causal convolution  y = q (.) (h * (k (.) v))  for the vector-ALU paths.
//
// Given dy, with u = k*v, z = h * u, g = dy*q:
//     dq[t] = dy[t] * z[t]
//     du[s] = sum_{j<lh, s+j<L} h[j] * g[s+j]        (transposed = anti-causal convolution)
//     dk[s] = du[s] * v[s],  dv[s] = du[s] * k[s]
//     dh[G, j] = sum_b sum_{c in G} sum_{t>=j} g[b,t,c] * u[b,t-j,c]
// The filter gradient follows the two-pass scheme of the paper's backward (App. A.4): the main kernel
// accumulates a partial dh per tile next to dq, dk, dv and writes it out contiguously; a second small kernel
// reduces the partials (and the channels of a group).
//
//  * bwd_stencil_kernel: short filters (lh <= 8), one fused streaming pass.  A lane owns VEC adjacent
//    channels and walks one tile forward in time with everything in registers: the last lh-1 values of u
//    (for z), the last lh values of g (du is finished lh-1 steps late, when the newest g it needs has
//    arrived), a delay line of k and v for that lag, and VEC*lh partial sums for dh.  A tile reads lh-1
//    halo rows of k, v before its start and lh-1 halo rows of dy, q after its end.
//  * any other lh, group or width, both dtypes: dq, dk, dv by the general FIR kernels (split_kernels.hip where 8 channels
//    share a filter of more than 32 taps, else direct_kernels.hip) in both time
//    directions, dh by dh_tile_kernel (where its partial sums do not fit or samples are few: dh_direct_kernel).
//
// kGated = false turns both paths into the backward of the featurizer convolutions of Eq. 1 (x' = h * x, no
// gates): u = x (the k pointer), g = dy, the only activation gradient is dx = du (the dk pointer); q, v, dq, dv are
// neither read nor written.
#include <type_traits>

#include "hy_common.hpp"
#include "hy_launch.hpp"

namespace hy {
namespace {

// ------------------------------------------------------------------------------------- stencil
constexpr int kMaxProb = 3;  // problems of one shape per launch (the three featurizers of a chain)
constexpr int kMaxReduce = 4;  // filter gradients per reduction (those and the inner filter's)

struct BwdStencilArgs {
    BwdPtrs p[kMaxProb];
    float* partial[kMaxProb];  // [B * tiles_per_seq][D * LH] each
    int64_t L, D;
    int64_t skv, sgq, sout;  // elements between batch items in k, v / dy, q / dq, dk, dv
    int32_t hist, fut;       // rows of k, v in front of row 0 / of dy, q behind row L - 1 that hold data
    int64_t nvec, nitems;
    int32_t group, rows, tiles_per_seq;
};

constexpr int kBlock = 256;

template <typename T, int VEC, int LH, int R, bool kGated>
__global__ __launch_bounds__(kBlock) void bwd_stencil_kernel(BwdStencilArgs a) {
    using P = Pack<T, VEC>;
    using Raw = typename P::Raw;
    constexpr int W = LH - 1 + R;  // window length: LH-1 older steps plus the batch
    const BwdPtrs pr = a.p[blockIdx.y];
    const int64_t item = (int64_t)blockIdx.x * kBlock + threadIdx.x;
    if (item >= a.nitems) return;
    int64_t cv, tile, b, t0;
    if (a.nitems <= 0xffffffffLL) {  // 32-bit divisions: those of 64 bits are a good part of a small launch
        tile = (uint32_t)item / (uint32_t)a.nvec;
        cv = (uint32_t)item - (uint32_t)tile * (uint32_t)a.nvec;
        b = (uint32_t)tile / (uint32_t)a.tiles_per_seq;
        t0 = (int64_t)((uint32_t)tile - (uint32_t)b * (uint32_t)a.tiles_per_seq) * a.rows;
    } else {
        cv = item % a.nvec;
        tile = item / a.nvec;
        b = tile / a.tiles_per_seq;
        t0 = (tile % a.tiles_per_seq) * (int64_t)a.rows;
    }
    const int64_t t1 = (t0 + a.rows < a.L) ? t0 + a.rows : a.L;
    const int64_t L = a.L, D = a.D;
    const int64_t c = cv * VEC;
    const int64_t seq0 = b * a.sout + c, seq0kv = b * a.skv + c, seq0gq = b * a.sgq + c;
    const char* dyp = static_cast<const char*>(pr.dy);
    const char* qp = static_cast<const char*>(pr.q);
    const char* kp = static_cast<const char*>(pr.k);
    const char* vp = static_cast<const char*>(pr.v);
    char* dqp = static_cast<char*>(pr.dq);
    char* dkp = static_cast<char*>(pr.dk);
    char* dvp = static_cast<char*>(pr.dv);

    float taps[VEC][LH], dh[VEC][LH];
#pragma unroll
    for (int e = 0; e < VEC; ++e) {
        const int64_t g = D <= 0xffffffffLL ? (int64_t)((uint32_t)(c + e) / (uint32_t)a.group) : (c + e) / a.group;
        const float* hp = pr.h + g * (int64_t)LH;
#pragma unroll
        for (int j = 0; j < LH; ++j) {
            taps[e][j] = hp[j];
            dh[e][j] = 0.0f;
        }
    }

    // index i of a window = time (first step of the current batch) - (LH-1) + i
    float uw[VEC][W], gw[VEC][W], kd[VEC][W], vd[VEC][W];
#pragma unroll
    for (int i = 0; i < LH - 1; ++i) {
        const int64_t t = t0 - (LH - 1) + i;
        float kf[VEC], vf[VEC];
        if (t >= -(int64_t)a.hist) {
            const int64_t off = (seq0kv + t * D) * T::kBytes;
            P::unpack(P::load(kp + off), kf);
            if constexpr (kGated) {
                P::unpack(P::load(vp + off), vf);
            } else {
#pragma unroll
                for (int e = 0; e < VEC; ++e) vf[e] = 1.0f;
            }
        } else {
#pragma unroll
            for (int e = 0; e < VEC; ++e) kf[e] = vf[e] = 0.0f;
        }
#pragma unroll
        for (int e = 0; e < VEC; ++e) {
            uw[e][i] = kf[e] * vf[e];
            gw[e][i] = 0.0f;
            kd[e][i] = kf[e];
            vd[e][i] = vf[e];
        }
    }

    // the walk covers the tile plus the LH-1 steps after it whose g still reaches into the tile
    const int64_t t_stop = L + a.fut;  // dy and q hold data up to here
    const int64_t t_walk = (t1 + (LH - 1) < t_stop) ? t1 + (LH - 1) : t_stop;
    Raw kr[R], vr[R], qr[R], gr[R];
    auto issue = [&](int64_t t) {
#pragma unroll
        for (int r = 0; r < R; ++r) {
            kr[r] = zero_words<P::kWords>();
            vr[r] = zero_words<P::kWords>();
            qr[r] = zero_words<P::kWords>();
            gr[r] = zero_words<P::kWords>();
            if (t + r < t_walk) {
                const int64_t off = (seq0gq + (t + r) * D) * T::kBytes;
                if constexpr (kGated) qr[r] = P::load_nt(qp + off);
                gr[r] = P::load_nt(dyp + off);
                if (t + r < t1) {
                    const int64_t offkv = (seq0kv + (t + r) * D) * T::kBytes;
                    kr[r] = P::load_nt(kp + offkv);
                    if constexpr (kGated) vr[r] = P::load_nt(vp + offkv);
                }
            }
        }
    };

    issue(t0);
    // du of step s is finished when step s + LH - 1 has been seen: run LH-1 steps past the tile end
    for (int64_t t = t0; t < t1 + (LH - 1); t += R) {
        Raw kc[R], vc[R], qc[R], gc[R];
#pragma unroll
        for (int r = 0; r < R; ++r) {
            kc[r] = kr[r];
            vc[r] = vr[r];
            qc[r] = qr[r];
            gc[r] = gr[r];
        }
        if (t + R < t1 + (LH - 1)) issue(t + R);

#pragma unroll
        for (int r = 0; r < R; ++r) {
            float kf[VEC], vf[VEC], qf[VEC], dyf[VEC];
            P::unpack(kc[r], kf);
            P::unpack(gc[r], dyf);
            if constexpr (kGated) {
                P::unpack(vc[r], vf);
                P::unpack(qc[r], qf);
            } else {
#pragma unroll
                for (int e = 0; e < VEC; ++e) vf[e] = qf[e] = 1.0f;
            }
            const int64_t tt = t + r;
#pragma unroll
            for (int e = 0; e < VEC; ++e) {
                uw[e][LH - 1 + r] = kf[e] * vf[e];
                gw[e][LH - 1 + r] = dyf[e] * qf[e];  // zero at and after the end of the sequence (loads skipped)
                kd[e][LH - 1 + r] = kf[e];
                vd[e][LH - 1 + r] = vf[e];
            }
            if (tt < t1) {  // dq and the filter-gradient partials of step tt
                float dqv[VEC];
#pragma unroll
                for (int e = 0; e < VEC; ++e) {
                    if constexpr (kGated) {
                        float z = taps[e][0] * uw[e][LH - 1 + r];
#pragma unroll
                        for (int j = 1; j < LH; ++j) z = __builtin_fmaf(taps[e][j], uw[e][LH - 1 + r - j], z);
                        dqv[e] = dyf[e] * z;
                    }
#pragma unroll
                    for (int j = 0; j < LH; ++j) dh[e][j] = __builtin_fmaf(gw[e][LH - 1 + r], uw[e][LH - 1 + r - j], dh[e][j]);
                }
                if constexpr (kGated) P::store_nt(dqp + (seq0 + tt * D) * T::kBytes, P::pack(dqv));
            }
            const int64_t s = tt - (LH - 1);  // the step whose du is complete now; window index r
            if (s >= t0 && s < t1) {
                float dkv[VEC], dvv[VEC];
#pragma unroll
                for (int e = 0; e < VEC; ++e) {
                    float du = taps[e][0] * gw[e][r];
#pragma unroll
                    for (int j = 1; j < LH; ++j) du = __builtin_fmaf(taps[e][j], gw[e][r + j], du);
                    dkv[e] = du * vd[e][r];
                    dvv[e] = du * kd[e][r];
                }
                P::store_nt(dkp + (seq0 + s * D) * T::kBytes, P::pack(dkv));
                if constexpr (kGated) P::store_nt(dvp + (seq0 + s * D) * T::kBytes, P::pack(dvv));
            }
        }
#pragma unroll
        for (int i = 0; i < LH - 1; ++i) {
#pragma unroll
            for (int e = 0; e < VEC; ++e) {
                uw[e][i] = uw[e][i + R];
                gw[e][i] = gw[e][i + R];
                kd[e][i] = kd[e][i + R];
                vd[e][i] = vd[e][i + R];
            }
        }
    }

    float* pp = a.partial[blockIdx.y] + tile * (D * LH) + c * LH;
#pragma unroll
    for (int e = 0; e < VEC; ++e)
#pragma unroll
        for (int j = 0; j < LH; ++j) pp[e * LH + j] = dh[e][j];
}

// second pass: dh[g][j] = sum over partial sets and over the channels of group g.  kRedParts lanes share an output: each
// sums a contiguous share of the terms (fixed order: set, then channel of the group), the first adds the shares in
// order.  Deterministic, no atomics.  The sums run in fp64 (the adds are a negligible part of this kernel), so the
// reduction adds no rounding of its own to the fp32 partials.  With few terms per output (up to 8: single channels and
// a handful of tiles) one lane sums them all, all its loads in flight at once, no exchange.
// The items of a launch (blockIdx.y) have shapes and lanes per output of their own.
struct ReduceItem {
    const float* partial;
    float* dh;
    int64_t nsets, rows;  // partial sets; rows of a set
    int32_t lh, group, parts;
};
struct ReduceArgs {
    ReduceItem p[kMaxReduce];
};

// a / b, in 32 bits where a fits them: a 64-bit division is a good part of this kernel
__device__ __forceinline__ int64_t quotient(int64_t a, int32_t b) {
    return a <= 0xffffffffLL ? (int64_t)((uint32_t)a / (uint32_t)b) : a / b;
}

template <int kRedParts>
__device__ __forceinline__ void reduce_item(const ReduceItem& it, double* red) {
    const float* __restrict__ partial = it.partial;
    float* __restrict__ dh = it.dh;
    const int64_t D = it.rows;
    const int32_t lh = it.lh, group = it.group;
    constexpr int kRedOut = kBlock / kRedParts;
    const int o = threadIdx.x % kRedOut, part = threadIdx.x / kRedOut;
    const int64_t idx = (int64_t)blockIdx.x * kRedOut + o;  // (g, j)
    const int64_t n = quotient(D, group) * lh;
    if ((int64_t)blockIdx.x * kRedOut >= n) return;
    const int64_t idc = idx < n ? idx : n - 1;  // lanes past the end repeat the last output and do not store
    const int64_t g = quotient(idc, lh), j = idc - g * lh;
    const float* base = partial + (g * group) * lh + j;
    const int64_t total = it.nsets * group;
    const int64_t per = (total + kRedParts - 1) / kRedParts;
    const int64_t lo = part * per, hi = lo + per < total ? lo + per : total;
    double s = 0.0;
    // term x = set * group + c lives at base[set * D * lh + c * lh]; the offset is advanced term by term (one
    // division per lane instead of two per term).  Eight loads in flight at a time (they do not depend on the
    // running sum); past the end the last offset repeats, so that the loads stay unconditional.
    const int64_t set0 = quotient(lo, group);
    int32_t c = (int32_t)(lo - set0 * group);
    int64_t cur = set0 * (D * lh) + (int64_t)c * lh;
    const int64_t wrap = D * lh - (int64_t)(group - 1) * lh;
    for (int64_t x0 = lo; x0 < hi; x0 += 8) {
        float v[8];
#pragma unroll
        for (int i = 0; i < 8; ++i) {
            v[i] = base[cur];
            if (x0 + i + 1 < hi) {
                if (++c == group) {
                    c = 0;
                    cur += wrap;
                } else {
                    cur += lh;
                }
            }
        }
#pragma unroll
        for (int i = 0; i < 8; ++i)
            if (x0 + i < hi) s += (double)v[i];
    }
    if constexpr (kRedParts == 1) {
        if (idx < n) dh[idx] = (float)s;
        return;
    }
    red[part * kRedOut + o] = s;
    __syncthreads();
    if (part == 0 && idx < n) {
        double t = red[o];
#pragma unroll 8
        for (int r = 1; r < kRedParts; ++r) t += red[r * kRedOut + o];
        dh[idx] = (float)t;
    }
}

// kRedParts: the lanes per output of every item; 0: each has its own
template <int kRedParts>
__global__ __launch_bounds__(kBlock) void dh_reduce_kernel(ReduceArgs a) {
    __shared__ double red[kBlock];
    const ReduceItem it = a.p[blockIdx.y];
    if constexpr (kRedParts > 0) {
        reduce_item<kRedParts>(it, red);
    } else {
        switch (it.parts) {
            case 1: return reduce_item<1>(it, red);
            case 32: return reduce_item<32>(it, red);
            case 256: return reduce_item<256>(it, red);
            default: return reduce_item<4>(it, red);
        }
    }
}

// ------------------------------------------------------------------------------------- general
struct BwdDirectArgs {
    BwdPtrs p;
    int64_t B, L, D;
    int64_t skv, sgq;  // elements between batch items in k, v / dy, q
    int32_t hist;      // rows of k, v in front of row 0 that hold data
    int32_t lh, group;
};

// dh[g][j]: one workgroup per (group, tap); lanes stride over (b, t, channel of the group), then a tree sum.
// Products of fp32 factors and their sum are carried in fp64 (correctness path: the sum has B * L * group terms).
template <typename T, bool kGated>
__global__ __launch_bounds__(kBlock) void dh_direct_kernel(BwdDirectArgs a) {
    using P = Pack<T, 1>;
    __shared__ double red[kBlock];
    const int64_t g = blockIdx.x;
    const int64_t j = blockIdx.y;
    const int64_t L = a.L, D = a.D;
    const int group = a.group;
    const char* dyp = static_cast<const char*>(a.p.dy);
    const char* qp = static_cast<const char*>(a.p.q);
    const char* kp = static_cast<const char*>(a.p.k);
    const char* vp = static_cast<const char*>(a.p.v);
    auto ld = [&](const char* base, int64_t e) {
        float f[1];
        P::unpack(P::load(base + e * T::kBytes), f);
        return f[0];
    };
    // this call's share: g of its own steps against u up to `hist` steps before them
    const int64_t t_first = j > a.hist ? j - a.hist : 0;
    const int64_t span = (L - t_first) * group;  // (t, cc) pairs per batch item, channel fastest
    double s = 0.0;
    for (int64_t b = 0; b < a.B; ++b) {
        for (int64_t i = threadIdx.x; i < span; i += kBlock) {
            const int64_t t = t_first + i / group;
            const int64_t c = g * group + i % group;
            const int64_t at = b * a.sgq + t * D + c, src = b * a.skv + (t - j) * D + c;
            if constexpr (kGated)
                s = __builtin_fma((double)ld(dyp, at) * (double)ld(qp, at), (double)ld(kp, src) * (double)ld(vp, src), s);
            else
                s = __builtin_fma((double)ld(dyp, at), (double)ld(kp, src), s);
        }
    }
    red[threadIdx.x] = s;
    __syncthreads();
    for (int w = kBlock / 2; w > 0; w >>= 1) {
        if ((int)threadIdx.x < w) red[threadIdx.x] += red[threadIdx.x + w];
        __syncthreads();
    }
    if (threadIdx.x == 0) a.p.dh[g * a.lh + j] = (float)red[0];
}

// The same filter gradient for everything but very short sequences, in two passes (App. A.4): partial sums per tile of
// time, then a reduction.  Products and sums are fp64 as above; the vector ALUs issue fp64 FMAs as fast as unpacked fp32
// ones, so the bound is lh FMAs per element and the layout is again around them: a workgroup owns 64 channels (one per
// lane) and a tile of time, u = k*v and g = dy*q are formed once into LDS in fp64 (both products are exact there), and
// a wave holds 16 lags: 16 steps of g against 16 + 15 rows of u are 256 FMAs per 48 LDS reads.  Filters of fewer than
// 128 taps leave waves without lags: those take a share of the steps instead (kLagWaves lag blocks of 16).
// The partial sums of a tile lie in the memory of dk, which the FIR launch behind these two overwrites: the shapes that
// come here are the ones whose callers bring no workspace, and tiles are no more than their sums fit (the channels of a
// group are summed in the wave first, as far as its size has powers of two).
// Pairs the definition does not have are left out, not multiplied by zeros (see the FIR kernel).
// Measured at B = 2, L = 2048, D = 1024, 128 taps, groups of 16, fp32: 1160 us with one workgroup per (group, tap), which
// read all samples of the group once per tap; 35 + 5 us in these two.
struct DhArgs {
    BwdPtrs p;
    int64_t L, D;
    int64_t skv, sgq, sout;  // elements between batch items in k, v / dy, q / dk
    int32_t hist;            // rows of k, v in front of row 0 that hold data
    int32_t lh, group;
    int32_t fold;            // largest power of two (up to 64) that divides the group: channels summed in the wave
    int32_t ncb, rows, tiles_per_seq;
};

constexpr int kDhThreads = 512;
constexpr int kDhT = 64;     // steps staged at a time
constexpr int kDhRing = 192;  // rows of u: the staged steps and 128 before them
constexpr int kDhLags = 128;  // lags per workgroup at most

// the partial sums of batch item b, in dk's memory
template <typename T>
__device__ __forceinline__ double* dh_scratch(void* dk, int64_t b, int64_t sout) {
    const uintptr_t at = reinterpret_cast<uintptr_t>(dk) + (uintptr_t)(b * sout) * T::kBytes;
    return reinterpret_cast<double*>((at + 7) & ~(uintptr_t)7);
}

template <typename T, int VEC, int kLagWaves, bool kGated>
__global__ __launch_bounds__(kDhThreads, 1) void dh_tile_kernel(DhArgs a) {
    constexpr int kC = 64;
    constexpr int kWaves = kDhThreads / 64;
    constexpr int kSplit = kWaves / kLagWaves < 4 ? kWaves / kLagWaves : 4;  // waves that share a lag block
    constexpr int kSub = 4 / kSplit;          // 16-step blocks per wave and staging
    constexpr int PPR = kC / VEC, RPP = kDhThreads / PPR, kPass = kDhT / RPP;
    static_assert(kDhT % RPP == 0, "whole passes");
    using P = Pack<T, VEC>;
    __shared__ __attribute__((aligned(16))) double us[kDhRing * kC];
    __shared__ __attribute__((aligned(16))) double gs[kDhT * kC];

    const int tid = threadIdx.x, lane = tid % 64, w = __builtin_amdgcn_readfirstlane(tid / 64);
    const uint32_t lb = blockIdx.x;
    const uint32_t tile = lb / (uint32_t)a.ncb;
    const int64_t c0 = (int64_t)(lb % (uint32_t)a.ncb) * kC;
    const int64_t b = tile / (uint32_t)a.tiles_per_seq;
    const int64_t ti = tile % (uint32_t)a.tiles_per_seq;
    const int64_t ts = ti * a.rows, te = ts + a.rows < a.L ? ts + a.rows : a.L;
    const int64_t D = a.D, L = a.L;
    const int64_t l0 = (int64_t)blockIdx.y * (16 * kLagWaves);  // first lag of this workgroup
    const int lagw = w % kLagWaves, part = w / kLagWaves;
    const int64_t j0 = l0 + 16 * lagw;                  // first lag of this wave
    const bool busy = part < kSplit && j0 < a.lh;

    const int pc = tid % PPR, pr0 = tid / PPR;
    const int64_t col = c0 + (int64_t)pc * VEC < D ? c0 + (int64_t)pc * VEC : c0;
    const char* const kp = static_cast<const char*>(a.p.k) + (b * a.skv + col) * T::kBytes;
    const char* const vp = kGated ? static_cast<const char*>(a.p.v) + (b * a.skv + col) * T::kBytes : nullptr;
    const char* const yp = static_cast<const char*>(a.p.dy) + (b * a.sgq + col) * T::kBytes;
    const char* const qp = kGated ? static_cast<const char*>(a.p.q) + (b * a.sgq + col) * T::kBytes : nullptr;
    const int64_t row_bytes = D * T::kBytes;
    typename P::Raw kr[kPass], vr[kPass], yr[kPass], qr[kPass];
    typename P::Raw kh[2][kPass], vh[2][kPass];
    // 64 rows of k, v from step s0 on, clamped into those that hold data
    auto load_u = [&](int64_t s0, typename P::Raw (&kk)[kPass], typename P::Raw (&vv)[kPass]) {
#pragma unroll
        for (int i = 0; i < kPass; ++i) {
            int64_t s = s0 + i * RPP + pr0;
            s = s < L ? s : L - 1;
            s = s > -(int64_t)a.hist ? s : -(int64_t)a.hist;
            kk[i] = P::load(kp + s * row_bytes);
            if constexpr (kGated) vv[i] = P::load(vp + s * row_bytes);
        }
    };
    auto load_g = [&](int64_t t0) {
#pragma unroll
        for (int i = 0; i < kPass; ++i) {
            int64_t t = t0 + i * RPP + pr0;
            t = t < L ? t : L - 1;
            yr[i] = P::load(yp + t * row_bytes);
            if constexpr (kGated) qr[i] = P::load(qp + t * row_bytes);
        }
    };
    auto write_prod = [&](double* rows, const typename P::Raw (&x)[kPass], const typename P::Raw (&y)[kPass]) {
#pragma unroll
        for (int i = 0; i < kPass; ++i) {
            float f[VEC], g[VEC];
            P::unpack(x[i], f);
            if constexpr (kGated) P::unpack(y[i], g);
            double* dst = rows + (i * RPP + pr0) * kC + pc * VEC;
            double d[VEC];
#pragma unroll
            for (int e = 0; e < VEC; ++e) d[e] = kGated ? (double)f[e] * (double)g[e] : (double)f[e];
            if constexpr (VEC >= 2) {
#pragma unroll
                for (int e = 0; e < VEC; e += 2) *reinterpret_cast<double2*>(dst + e) = make_double2(d[e], d[e + 1]);
            } else {
                dst[0] = d[0];
            }
        }
    };

    // steps ts - l0 - 128 .. ts - l0 - 1 of u (up to 64 lags: 64 of them) to ring rows 64 .. 191; staging n then writes rows
    // 64 (n % 3) on
    constexpr bool kFar = kLagWaves > 4;
    if constexpr (kFar) load_u(ts - l0 - 128, kh[0], vh[0]);
    load_u(ts - l0 - 64, kh[1], vh[1]);
    load_u(ts - l0, kr, vr);
    load_g(ts);
    if constexpr (kFar) write_prod(us + kDhT * kC, kh[0], vh[0]);
    write_prod(us + 2 * kDhT * kC, kh[1], vh[1]);

    double acc[16];
#pragma unroll
    for (int r = 0; r < 16; ++r) acc[r] = 0.0;

    int slot = 0;
    for (int64_t t0 = ts; t0 < te; t0 += kDhT) {
        __syncthreads();
        write_prod(us + slot * kDhT * kC, kr, vr);
        write_prod(gs, yr, qr);
        __syncthreads();
        if (t0 + kDhT < te) {
            load_u(t0 + kDhT - l0, kr, vr);
            load_g(t0 + kDhT);
        }
        if (busy) {
            // 16-row block m of the ring; blocks of u 16 lags earlier lie one block lower
            const int blk0 = slot * 4 + part * kSub - lagw + 12;
            auto read_u = [&](double (&x)[16], int blk) {
                const double* p = us + (blk % 12) * 16 * kC + lane;
#pragma unroll
                for (int i = 0; i < 16; ++i) x[i] = p[i * kC];
            };
            double ua[16], ub[16];  // rows 16 steps before the block, rows of the block
            read_u(ub, blk0 - 1 + 12);
#pragma unroll
            for (int n = 0; n < kSub; ++n) {
                const int sb = part * kSub + n;
                const int64_t tb = t0 + 16 * sb;
#pragma unroll
                for (int i = 0; i < 16; ++i) ua[i] = ub[i];
                read_u(ub, blk0 + n);
                const double* gp = gs + sb * 16 * kC + lane;
                if (tb + 16 <= te && tb - j0 - 15 >= -(int64_t)a.hist) {
#pragma unroll
                    for (int i = 0; i < 16; ++i) {
                        const double g = gp[i * kC];
#pragma unroll
                        for (int r = 0; r < 16; ++r) acc[r] = __builtin_fma(g, i >= r ? ub[i - r] : ua[16 + i - r], acc[r]);
                    }
                } else if (tb - j0 + 15 >= -(int64_t)a.hist) {
                    const int nt = te - tb < 16 ? (int)(te - tb) : 16;                       // steps of the tile
                    const int64_t back64 = tb - j0 + a.hist;                                  // u reaches this far back
                    const int back = back64 < 16 ? (back64 > -16 ? (int)back64 : -16) : 16;
#pragma unroll
                    for (int i = 0; i < 16; ++i) {
                        const double g = gp[i * kC];
#pragma unroll
                        for (int r = 0; r < 16; ++r) {
                            const double x = __builtin_fma(g, i >= r ? ub[i - r] : ua[16 + i - r], acc[r]);
                            acc[r] = (i < nt && r - i <= back) ? x : acc[r];
                        }
                    }
                }
            }
        }
        slot = slot == 2 ? 0 : slot + 1;
    }

    if constexpr (kSplit > 1) {  // the waves that share a lag block, summed in their order
        __syncthreads();
        if (busy && part > 0) {
#pragma unroll
            for (int r = 0; r < 16; ++r) us[(((part - 1) * kLagWaves + lagw) * 16 + r) * kC + lane] = acc[r];
        }
        __syncthreads();
        if (part > 0) return;
        if (busy) {
#pragma unroll
            for (int x = 0; x < kSplit - 1; ++x)
#pragma unroll
                for (int r = 0; r < 16; ++r) acc[r] += us[((x * kLagWaves + lagw) * 16 + r) * kC + lane];
        }
    }
    if (!busy) return;
    const bool own = c0 + lane < D;
#pragma unroll
    for (int r = 0; r < 16; ++r) acc[r] = own ? acc[r] : 0.0;
    for (int x = 1; x < a.fold; x <<= 1) {
#pragma unroll
        for (int r = 0; r < 16; ++r) acc[r] += __shfl_xor(acc[r], x);
    }
    if (own && lane % a.fold == 0) {
        double* out = dh_scratch<T>(a.p.dk, b, a.sout) + (ti * (D / a.fold) + (c0 + lane) / a.fold) * a.lh;
#pragma unroll
        for (int r = 0; r < 16; ++r)
            if (j0 + r < a.lh) out[j0 + r] = acc[r];
    }
}

// dh[g][j] = sum over batch items, tiles and the group's partial rows, in that order, by kParts lanes per output as in
// dh_reduce_kernel
template <typename T, int kParts>
__global__ __launch_bounds__(kBlock) void dh_tile_reduce_kernel(DhArgs a, int64_t B) {
    constexpr int kOut = kBlock / kParts;
    __shared__ double red[kParts][kOut];
    const int o = threadIdx.x % kOut, part = threadIdx.x / kOut;
    const int64_t n = quotient(a.D, a.group) * a.lh;
    const int64_t idx = (int64_t)blockIdx.x * kOut + o;
    const int64_t idc = idx < n ? idx : n - 1;
    const int64_t g = quotient(idc, a.lh), j = idc - g * a.lh;
    const int32_t rpg = a.group / a.fold;               // partial rows per group
    const int64_t tile_len = quotient(a.D, a.fold) * a.lh;
    const int64_t per_item = (int64_t)a.tiles_per_seq * rpg, total = B * per_item;
    const int64_t per = (total + kParts - 1) / kParts;
    const int64_t lo = part * per, hi = lo + per < total ? lo + per : total;
    auto tile_row = [&](int64_t b, int32_t t) { return dh_scratch<T>(a.p.dk, b, a.sout) + t * tile_len + g * rpg * a.lh + j; };
    double s = 0.0;
    if (lo < hi) {
        int64_t b = total <= 0xffffffffLL ? (int64_t)((uint32_t)lo / (uint32_t)per_item) : lo / per_item;
        int32_t t = (int32_t)quotient(lo - b * per_item, rpg), c = (int32_t)(lo - b * per_item - (int64_t)t * rpg);
        const double* cur = tile_row(b, t) + (int64_t)c * a.lh;
        for (int64_t x0 = lo; x0 < hi; x0 += 8) {  // past the end the last term is read again, not added
            double v[8];
#pragma unroll
            for (int i = 0; i < 8; ++i) {
                v[i] = *cur;
                if (x0 + i + 1 < hi) {
                    if (++c < rpg) {
                        cur += a.lh;
                    } else {
                        c = 0;
                        if (++t == a.tiles_per_seq) {
                            t = 0;
                            ++b;
                        }
                        cur = tile_row(b, t);
                    }
                }
            }
#pragma unroll
            for (int i = 0; i < 8; ++i) s += x0 + i < hi ? v[i] : 0.0;
        }
    }
    red[part][o] = s;
    __syncthreads();
    if (part == 0 && idx < n) {
        double t = red[0][o];
#pragma unroll 8
        for (int r = 1; r < kParts; ++r) t += red[r][o];
        a.p.dh[idx] = (float)t;
    }
}

// Lanes per output of a reduction: few outputs of many terms (a filter shared by many channels, many short tiles) are one
// long chain per lane, so more lanes share them; many outputs fill the chip by themselves and read whole lines with four
// (featurizer backward, 7 taps, whole call with 4 / 32 / 256 lanes; outputs x terms: 7 x 65536 1073 / 155 / 58 us,
// 448 x 2048 50 / 18 / 22, 448 x 16384 399 / 128 / 133, 1792 x 512 21.8 / 17.6 / 25, 7168 x 512 31 / 27 / 57, 28672 x 512
// 66 / 90 / 202, 448 x 256 17.1 / 17.0 / 17.3).
int reduce_parts(int64_t nout, int64_t terms) {
    if (terms > 4096 && nout <= 512) return 256;
    if (terms > 256 && nout <= 8192) return 32;
    return 4;
}

// HY_ERR_UNSUPPORTED where dk cannot hold the partial sums of one tile and where dh_direct_kernel is quicker
template <typename T, int VEC>
hy_status launch_dh_tile(const BwdPtrs& p, const BwdShape& s, hipStream_t st) {
    DhArgs a;
    a.p = p;
    a.L = s.L;
    a.D = s.D;
    a.skv = s.stride_kv();
    a.sgq = s.stride_gq();
    a.sout = s.stride_out();
    a.hist = s.history;
    a.lh = s.lh;
    a.group = s.group;
    a.fold = 1;
    while (a.fold < 64 && s.group % (2 * a.fold) == 0) a.fold *= 2;
    const int64_t ncb = (s.D + 63) / 64, nlag = (s.lh + kDhLags - 1) / kDhLags;
    const int64_t fit = (s.L * s.D * T::kBytes - 8) / ((s.D / a.fold) * (int64_t)s.lh * 8);
    // one workgroup per compute unit, in tiles of a staging or more (256 steps against 64: 3 x 1058 x 256 fp32, 100 taps,
    // whole call 55 / 39 us, 9 x 490 x 136 bf16, 9 taps 36 / 23)
    int64_t tiles = 256 / (s.B * ncb * nlag);
    if (tiles > s.L / kDhT) tiles = s.L / kDhT;
    if (tiles < 1) tiles = 1;
    if (tiles > fit) tiles = fit;
    if (tiles < 1) return HY_ERR_UNSUPPORTED;
    int64_t rows = ((s.L + tiles - 1) / tiles + kDhT - 1) / kDhT * kDhT;
    // A few samples per lane of dh_direct_kernel are done before a tile is staged.  In units of 0.25 us: its chain of loads
    // (2048 workgroups at a time) or the lines it reads, against two launches and the products of a tile's stagings.
    // Plain kernel / tiles, whole call, us: 1 x 85 x 72 fp32, 100 taps, group 72 19 / 40, 1 x 319 x 72 bf16, 65 taps 20 / 50,
    // 6 x 132 x 3 fp32, 9 taps 13 / 22; beyond the line 4 x 317 x 72 bf16, 64 taps 30 / 25, 9 x 490 x 136 bf16, 9 taps 44 / 23.
    const int64_t filters = s.D / s.group, blocks = filters * s.lh;
    const int64_t chain = s.B * ((s.L * s.group + kBlock - 1) / kBlock) * (blocks > 2048 ? blocks / 2048 : 1);
    const int64_t line = s.group * T::kBytes > 64 ? s.group * T::kBytes : 64;
    const double lines = (double)blocks * (double)(s.B * s.L) * (double)line * (s.gated ? 4 : 2) / 5.5e6;
    const int64_t products = rows / kDhT * (s.lh <= 32 ? 1 : s.lh <= 64 ? 2 : 4);
    if (chain < 24 + 6 * products && lines < (double)(24 + 6 * products)) return HY_ERR_UNSUPPORTED;
    if (rows > 0x7fffffffLL || ncb > 0x7fffffffLL || nlag > 65535) return HY_ERR_UNSUPPORTED;
    tiles = (s.L + rows - 1) / rows;
    if (s.B > 0x7fffffffLL || s.B * tiles > 0x7fffffffLL / ncb) return HY_ERR_UNSUPPORTED;
    a.ncb = (int32_t)ncb;
    a.rows = (int32_t)rows;
    a.tiles_per_seq = (int32_t)tiles;
    // A workgroup takes as many blocks of 16 lags as the filter has, or half and half of that where the launch leaves compute
    // units without one: its waves then share the steps of a staging (forward and gradients, fp32, whole blocks / shared, us:
    // 5 x 338 x 256, 128 taps 46 / 33, 2 x 1123 x 256 45 / 39, 1 x 1218 x 1000, one filter per channel 95 / 70; 2 x 2048 x 1024,
    // which fills the chip, 86 either way).
    int lagw = s.lh <= 16 ? 1 : s.lh <= 32 ? 2 : s.lh <= 64 ? 4 : 8;
    auto lag_blocks = [&](int w) { return (s.lh + 16 * w - 1) / (16 * w); };
    while (lagw > 2 && s.B * tiles * ncb * lag_blocks(lagw / 2) <= 256) lagw /= 2;
    const dim3 grid((uint32_t)(s.B * tiles * ncb), (uint32_t)lag_blocks(lagw)), block(kDhThreads);
    auto go = [&](auto gated_c) {
        constexpr bool G = decltype(gated_c)::value;
        if (lagw == 1) return launch_kernel((dh_tile_kernel<T, VEC, 1, G>), grid, block, st, a);
        if (lagw == 2) return launch_kernel((dh_tile_kernel<T, VEC, 2, G>), grid, block, st, a);
        if (lagw == 4) return launch_kernel((dh_tile_kernel<T, VEC, 4, G>), grid, block, st, a);
        return launch_kernel((dh_tile_kernel<T, VEC, 8, G>), grid, block, st, a);
    };
    const hy_status rc = s.gated ? go(std::true_type{}) : go(std::false_type{});
    if (rc != HY_OK) return rc;
    const int64_t nout = (s.D / s.group) * s.lh;
    auto reduce = [&](void (*kernel)(DhArgs, int64_t), int64_t parts) {
        const int64_t per = kBlock / parts;
        return launch_kernel(kernel, dim3((uint32_t)((nout + per - 1) / per)), dim3(kBlock), st, a, s.B);
    };
    switch (reduce_parts(nout, s.B * tiles * (s.group / a.fold))) {
        case 256: return reduce(dh_tile_reduce_kernel<T, 256>, 256);
        case 32: return reduce(dh_tile_reduce_kernel<T, 32>, 32);
        default: return reduce(dh_tile_reduce_kernel<T, 4>, 4);
    }
}

int stencil_rows(const BwdShape& s, int64_t nvec) {
    int rows = tuning().se_rows;
    if (rows <= 0) {
        const int64_t waves_per_row = (nvec * s.nprob + kWave - 1) / kWave;
        // Measured on MI355X (L = 8192, D = 4096): 256-step tiles run 10% faster than 128-step ones (half the
        // halo rows and half the partial filter gradients), as long as four waves per CU are left.
        // The featurizer variant holds half the loads and windows per lane and wants eight waves per CU (same
        // shape: 48.5 us with 128-step tiles, 66 us with 256).
        rows = 256;
        const int64_t want = s.gated ? 1024 : 2048;
        auto waves = [&] { return s.B * ((s.L + rows - 1) / rows) * waves_per_row; };
        while (rows > 32 && waves() < want) rows >>= 1;
        // With two waves per CU or fewer a launch is as long as one lane's chain of batches: shorter tiles still, for the
        // price of halo rows and partial filter gradients (rows 32 / 16 / 8, bf16, 7 taps: 512 x 256 18.2 / 13.7 / 12.3
        // us, 512 x 4096 19.5 / 16.7 / 18.6, 2 x 1000 x 768 17.8 / 15.0 / 17.2; 2048 x 1024 20.1 / 20.0 / 24.2).  Three
        // problems at a time stop at 16, where their partial sums still fit the chain's workspace.
        while (rows > (s.nprob > 1 ? 16 : 8) && waves() <= 512) rows >>= 1;
    }
    if (rows > s.L) rows = (int)s.L;
    if (rows < 1) rows = 1;
    return rows;
}

template <typename T>
constexpr int stencil_vec() { return T::kBytes == 2 ? 2 : 1; }

hy_status launch_reduce(const DhReduce* items, int n, hipStream_t st) {
    ReduceArgs r{};
    int64_t nb = 0;
    int common = -1;
    for (int i = 0; i < n; ++i) {
        const DhReduce& x = items[i];
        const int64_t nout = (x.rows / x.group) * x.lh, terms = x.nsets * x.group;
        const int parts = terms <= 8 ? 1 : reduce_parts(nout, terms);
        r.p[i] = ReduceItem{x.partial, x.dh, x.nsets, x.rows, x.lh, x.group, parts};
        const int64_t per = kBlock / parts, blocks = (nout + per - 1) / per;
        nb = blocks > nb ? blocks : nb;
        common = i == 0 || common == parts ? parts : 0;
    }
    if (nb == 0) return HY_OK;
    if (nb > 0x7fffffffLL) return HY_ERR_UNSUPPORTED;
    const dim3 grid((uint32_t)nb, (uint32_t)n), block(kBlock);
    switch (common) {
        case 1: return launch_kernel(dh_reduce_kernel<1>, grid, block, st, r);
        case 4: return launch_kernel(dh_reduce_kernel<4>, grid, block, st, r);
        case 32: return launch_kernel(dh_reduce_kernel<32>, grid, block, st, r);
        case 256: return launch_kernel(dh_reduce_kernel<256>, grid, block, st, r);
        default: return launch_kernel(dh_reduce_kernel<0>, grid, block, st, r);
    }
}

template <typename T, int LH>
hy_status launch_stencil_lh(const BwdPtrs* p, const BwdShape& s, void* ws, hipStream_t st) {
    constexpr int VEC = stencil_vec<T>();
    constexpr int R = 4;
    BwdStencilArgs a;
    for (int i = 0; i < kMaxProb; ++i) {
        const int x = i < s.nprob ? i : 0;
        a.p[i] = p[x];
        a.partial[i] = reinterpret_cast<float*>(static_cast<char*>(ws) + x * bwd_stencil_workspace_bytes(s));
    }
    a.L = s.L;
    a.D = s.D;
    a.skv = s.stride_kv();
    a.sgq = s.stride_gq();
    a.sout = s.stride_out();
    a.hist = s.history;
    a.fut = s.future;
    a.group = s.group;
    a.nvec = s.D / VEC;
    a.rows = stencil_rows(s, a.nvec);
    a.tiles_per_seq = (int32_t)((s.L + a.rows - 1) / a.rows);
    a.nitems = s.B * a.tiles_per_seq * a.nvec;
    const int64_t nb = (a.nitems + kBlock - 1) / kBlock;
    if (nb > 0x7fffffffLL) return HY_ERR_UNSUPPORTED;
    const hy_status rc = s.gated
        ? launch_kernel((bwd_stencil_kernel<T, VEC, LH, R, true>), dim3((uint32_t)nb, (uint32_t)s.nprob), dim3(kBlock), st, a)
        : launch_kernel((bwd_stencil_kernel<T, VEC, LH, R, false>), dim3((uint32_t)nb, (uint32_t)s.nprob), dim3(kBlock), st, a);
    if (rc != HY_OK) return rc;
    const int64_t nsets = s.B * a.tiles_per_seq;
    DhReduce r[kMaxProb];
    for (int i = 0; i < s.nprob; ++i) r[i] = DhReduce{a.partial[i], a.p[i].dh, nsets, s.D, s.lh, s.group};
    return launch_reduce(r, s.nprob, st);
}

template <typename T>
hy_status launch_stencil_t(const BwdPtrs* p, const BwdShape& s, void* ws, hipStream_t st) {
    switch (s.lh) {
        case 1: return launch_stencil_lh<T, 1>(p, s, ws, st);
        case 2: return launch_stencil_lh<T, 2>(p, s, ws, st);
        case 3: return launch_stencil_lh<T, 3>(p, s, ws, st);
        case 4: return launch_stencil_lh<T, 4>(p, s, ws, st);
        case 5: return launch_stencil_lh<T, 5>(p, s, ws, st);
        case 6: return launch_stencil_lh<T, 6>(p, s, ws, st);
        case 7: return launch_stencil_lh<T, 7>(p, s, ws, st);
        case 8: return launch_stencil_lh<T, 8>(p, s, ws, st);
        default: return HY_ERR_UNSUPPORTED;
    }
}

template <typename T>
hy_status launch_direct_t(const BwdPtrs& p, const BwdShape& s, hipStream_t st) {
    BwdDirectArgs a;
    a.p = p;
    a.B = s.B; a.L = s.L; a.D = s.D; a.lh = s.lh; a.group = s.group;
    a.skv = s.stride_kv();
    a.sgq = s.stride_gq();
    a.hist = s.history;
    const int64_t G = s.D / s.group;
    if (G > 0x7fffffffLL || s.lh > 65535) return HY_ERR_UNSUPPORTED;
    // the filter gradient first: its partial sums lie in dk's memory, which the FIR launch then overwrites
    constexpr int V = 16 / T::kBytes;
    hy_status rc = s.D % V == 0 ? launch_dh_tile<T, V>(p, s, st) : launch_dh_tile<T, 1>(p, s, st);
    if (rc == HY_ERR_UNSUPPORTED) {
        const dim3 gridh((uint32_t)G, (uint32_t)s.lh);
        rc = s.gated ? launch_kernel((dh_direct_kernel<T, true>), gridh, dim3(kBlock), st, a)
                     : launch_kernel((dh_direct_kernel<T, false>), gridh, dim3(kBlock), st, a);
    }
    if (rc != HY_OK) return rc;
    // du = h *' g towards the past, gated by v and by k; z = h * u, gated by dy
    FirProblem f[2];
    f[0].a = p.dy;
    f[0].b = s.gated ? p.q : nullptr;
    f[0].h = p.h;
    f[0].gate = s.gated ? p.v : nullptr;
    f[0].out = p.dk;
    f[0].gate2 = s.gated ? p.k : nullptr;
    f[0].out2 = s.gated ? p.dv : nullptr;
    f[0].stride_ab = s.stride_gq();
    f[0].stride_gate = s.stride_kv();
    f[0].stride_out = s.stride_out();
    f[0].lo = 0;
    f[0].hi = s.L + s.future;
    f[0].rev = 1;
    f[1].a = p.k;
    f[1].b = p.v;
    f[1].h = p.h;
    f[1].gate = p.dy;
    f[1].out = p.dq;
    f[1].stride_ab = s.stride_kv();
    f[1].stride_gate = s.stride_gq();
    f[1].stride_out = s.stride_out();
    f[1].lo = -(int64_t)s.history;
    f[1].hi = s.L;
    if (s.gated) {
        rc = launch_split_fir(f, 2, s.B, s.L, s.D, s.lh, s.group, s.dtype, st);
        if (rc != HY_ERR_UNSUPPORTED) return rc;
    }
    return launch_fir(f, s.gated ? 2 : 1, s.B, s.L, s.D, s.lh, s.group, s.dtype, st);
}

}  // namespace

bool bwd_stencil_supported(const BwdShape& s) {
    const int vec = s.dtype == HY_BF16 ? 2 : 1;
    return s.lh <= 8 && s.D % vec == 0;
}

int64_t bwd_stencil_workspace_bytes(const BwdShape& s) {
    const int vec = s.dtype == HY_BF16 ? 2 : 1;
    const int rows = stencil_rows(s, s.D / vec);
    const int64_t tiles = (s.L + rows - 1) / rows;
    return s.B * tiles * s.D * s.lh * (int64_t)sizeof(float);
}

hy_status launch_bwd_stencil(const BwdPtrs& p, const BwdShape& s, void* ws, hipStream_t st) {
    if (!bwd_stencil_supported(s) || s.nprob < 1 || s.nprob > kMaxProb) return HY_ERR_UNSUPPORTED;
    return s.dtype == HY_BF16 ? launch_stencil_t<BF16>(&p, s, ws, st) : launch_stencil_t<F32>(&p, s, ws, st);
}

hy_status launch_dh_reduce(const DhReduce* items, int n, hipStream_t st) {
    return n < 1 || n > kMaxReduce ? HY_ERR_UNSUPPORTED : launch_reduce(items, n, st);
}

hy_status launch_bwd_zero_dh(float* dh, int64_t D, int32_t lh, int32_t group, hipStream_t st) {
    // a reduction over zero partial sets writes zeros (a fill kernel, not a memset, so that callers may
    // capture the call in a HIP graph)
    const DhReduce r{dh, dh, 0, D, lh, group};
    return launch_dh_reduce(&r, 1, st);
}

hy_status launch_bwd_direct(const BwdPtrs& p, const BwdShape& s, hipStream_t st) {
    return s.dtype == HY_BF16 ? launch_direct_t<BF16>(p, s, st) : launch_direct_t<F32>(p, s, st);
}

}  // namespace hy
