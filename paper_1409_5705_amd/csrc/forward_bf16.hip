// Logits of the bf16 multiclass-logistic path where the 256 x 256 tiles of
// sf_gemm_kernel (gemm_bf16.hip) would leave most of the chip idle:
//
//   Z[b][j] = sum_d X[b][d] * bf16(W[j][d]),   fp32 accumulate.
//
// A workgroup takes 64 or 128 classes and up to 256 samples, over the whole of d or,
// where that leaves CUs idle, over a part of it (the partial sums go to planes of
// their own, which the softmax adds up).  The rows of W are the long stream (every
// one is read once per 256 samples): four of the eight wavefronts carry them through
// registers, several k-slices ahead, into LDS; where W has no bf16 copy they are read
// as fp32 and rounded on the way, which saves the pass that makes the copy.  The
// samples are small and come from the L2: the other four wavefronts bring them
// straight into three LDS stages.  All eight multiply what LDS holds.
#include "device.h"
#include "forward_index.h"
#include "kernels.h"

#include <cmath>

namespace sfb {
namespace {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float floatx4 __attribute__((ext_vector_type(4)));
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));

constexpr int NT = 512;
constexpr int KS = 64;       // k-slice
constexpr int NX = 3;        // LDS stages of the samples

struct FwdParams {
    const uint16_t* X;       // samples in the operand layout (blocks of 256 x 64, pitch P)
    int64_t x_pitch;         // or, where this is not 0, as rows of x_pitch elements, a multiple of 64
    const void* W;           // fp32 [J][D], or bf16 in the operand layout
    float* Z;                // per k-split: 256 x 256 tiles, tile (b / 256, j / 256) at index (j / 256) * tiles_b + b / 256
    int64_t plane;           // floats from one split's logits to the next
    int64_t B, J, D, P;
    int tiles_b;             // of 256
    int tiles_m;             // of this kernel
    int per_split;           // k-slices per split
    int num_xcd;
};

// 4 x 2 wavefronts, each MT x NTL MFMA tiles of 16 x 16 (samples x classes).  Wavefronts 0-3 bring the samples
// (direct-to-LDS loads, NX stages), wavefronts 4-7 the rows of W (DW slices in registers, two stages): each kind waits
// for its own loads only, so the long latency of W does not hold up the samples.
template <int MT, int NTL, int DW, bool FP32>
__global__ __launch_bounds__(NT, 2) void fwd_stream_kernel(FwdParams p)
{
    constexpr int BM = 64 * MT, BN = 32 * NTL;
    constexpr int XS = BM * 128, WS = BN * 128;           // bytes of a slice in LDS: rows of 64 bf16, chunks swizzled
    constexpr int LX = BM / 8 / 4;                        // 1 KB loads of the samples per wavefront and slice
    constexpr int PER = FP32 ? 16 : 8, RSTEP = 256 / PER, PIECES = BN / RSTEP;   // 16-byte pieces of a row of W; rows per step; pieces a thread
    extern __shared__ u32x4 fwd_smem[];
    char* const lds = reinterpret_cast<char*>(fwd_smem);
    const uint32_t lds_base = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) char*)fwd_smem;

    const int tid = threadIdx.x, lane = tid & 63, l16 = lane & 15, quad = lane >> 4;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int wm0 = (wave >> 1) * (16 * MT), wn0 = (wave & 1) * (16 * NTL);

    // tiles of one class range are neighbours under one L2
    int64_t m0, n0;
    {
        const uint32_t tiles = gridDim.x, xcds = (uint32_t)p.num_xcd, tm = (uint32_t)p.tiles_m;
        const uint32_t x = blockIdx.x % xcds, wi = blockIdx.x / xcds, q = tiles / xcds, r = tiles % xcds;
        const uint32_t t = x * q + (x < r ? x : r) + wi;
        m0 = (int64_t)(t % tm) * BM;
        n0 = (int64_t)(t / tm) * BN;
    }
    const int nk_all = (int)((p.D + KS - 1) / KS), first = (int)blockIdx.y * p.per_split;
    const int nk = nk_all - first < p.per_split ? nk_all - first : p.per_split;       // (>= 1: no empty split)
    // the workgroups start at different k: all at the same one would ask the same memory channels for it (rows of W are
    // often a multiple of 4 KB apart).  The order in which a logit is summed so depends on its tile.
    const int turn = (int)((blockIdx.x * 5u) % (uint32_t)nk);
    auto at = [&](int s) {
        s = s < nk ? s : nk - 1;
        return first + (s + turn < nk ? s + turn : s + turn - nk);
    };

    floatx4 acc[MT][NTL];
#pragma unroll
    for (int i = 0; i < MT; ++i)
#pragma unroll
        for (int n = 0; n < NTL; ++n) acc[i][n] = floatx4{0.f, 0.f, 0.f, 0.f};
    uint32_t xoff[MT], roff[NTL];
#pragma unroll
    for (int i = 0; i < MT; ++i) {
        const int r = wm0 + 16 * i + l16;
        xoff[i] = (uint32_t)(r * 128 + ((quad ^ swz(r)) << 4));
    }
#pragma unroll
    for (int n = 0; n < NTL; ++n) {
        const int r = wn0 + 16 * n + l16;
        roff[n] = (uint32_t)(NX * XS + r * 128 + ((quad ^ swz(r)) << 4));
    }
    // A slice is two k-steps of 32.  The fragments of a step are read under the MFMAs of the step before it, across the
    // barrier in the middle of a slice: in front of it a wavefront has read all of slice s and waited for its own part
    // of slice s + 1; behind it the stage of slice s is free and slice s + 1 can be read.
    struct Frags {
        bf16x8 x[MT], w[NTL];
    };
    Frags f0, f1;
    auto read_one = [&](Frags& f, int xstage, int wstage, int ks, int i) {
        if (i < NTL)
            f.w[i] = *reinterpret_cast<const bf16x8*>(lds + wstage * WS + (roff[i] ^ (64u * ks)));
        else
            f.x[i - NTL] = *reinterpret_cast<const bf16x8*>(lds + xstage * XS + (xoff[i - NTL] ^ (64u * ks)));
    };
    auto step = [&](const Frags& f, Frags& next, int xstage, int wstage, int ks, auto&& beside) {
        __builtin_amdgcn_sched_barrier(0);
        static_for<0, MT * NTL>([&](auto J) {
            constexpr int j = decltype(J)::value, i = j / NTL, n = j % NTL, NR = MT + NTL, M = MT * NTL;
            acc[i][n] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(f.x[i], f.w[n], acc[i][n], 0, 0, 0);
            static_for<j * NR / M, (j + 1) * NR / M>([&](auto Q) { read_one(next, xstage, wstage, ks, decltype(Q)::value); });
            beside(J);
            __builtin_amdgcn_sched_barrier(0);
        });
    };

    const int rounds = (nk + DW - 1) / DW;      // both kinds of wavefronts run rounds of DW slices: the same barriers
    if (wave < 4) {
        // unit u of a slice is rows 8 u .. + 7 of the tile; lane l fetches chunk (l & 7) ^ swz of row + l / 8.  Rows past
        // the last sample are clamped.
        uint32_t voff[LX];
#pragma unroll
        for (int i = 0; i < LX; ++i) {
            const int r = 8 * (LX * wave + i) + (lane >> 3);
            int64_t b = m0 + r;
            if (b >= p.B) b = p.B - 1;
            const int64_t row = p.x_pitch ? (b - m0) * p.x_pitch : (b / 256 - m0 / 256) * (p.P / 64) * 16384 + (b % 256) * 64;
            voff[i] = (uint32_t)(row * 2) + (uint32_t)(((lane & 7) ^ swz(r)) << 4);
        }
        const uint64_t base = uniform64(reinterpret_cast<uint64_t>(p.X) +
                                        (p.x_pitch ? (uint64_t)(m0 * p.x_pitch) * 2 : (uint64_t)(m0 / 256) * (uint64_t)(p.P / 64) * 32768));
        const uint64_t x_slice = p.x_pitch ? 128 : 32768;
        auto issue_one = [&](int i, int stage, uint64_t from) {
            load_to_lds_16(lds_base + (uint32_t)(stage * XS + (LX * wave + i) * 1024), from, voff[i]);
        };
        auto issue = [&](int s, int stage) {
#pragma unroll
            for (int i = 0; i < LX; ++i) issue_one(i, stage, base + (uint64_t)at(s) * x_slice);
        };
        static_for<0, NX>([&](auto S) { issue(decltype(S)::value, decltype(S)::value); });
        asm volatile("s_waitcnt vmcnt(%0)" ::"n"((NX - 1) * LX) : "memory");
        __syncthreads();
        static_for<0, MT + NTL>([&](auto Q) { read_one(f0, 0, 0, 0, decltype(Q)::value); });
        int xs = 0;
        for (int s0 = 0; s0 < rounds * DW; s0 += DW) {
            static_for<0, DW>([&](auto U) {
                constexpr int u = decltype(U)::value;
                const int xn = xs + 1 == NX ? 0 : xs + 1;
                step(f0, f1, xs, u & 1, 1, [](auto) {});
                asm volatile("s_waitcnt vmcnt(%0)" ::"n"((NX - 2) * LX) : "memory");
                __syncthreads();
                const uint64_t from = base + (uint64_t)at(s0 + u + NX) * x_slice;
                step(f1, f0, xn, (u + 1) & 1, 0, [&](auto J) {
                    constexpr int j = decltype(J)::value, M = MT * NTL;
                    static_for<j * LX / M, (j + 1) * LX / M>([&](auto Q) { issue_one(decltype(Q)::value, xs, from); });
                });
                xs = xn;
            });
        }
        asm volatile("s_waitcnt vmcnt(0)" ::: "memory");      // no direct load may be in flight when the LDS is released
    } else {
        const int wt = tid - 256, part = wt % PER;
        uint64_t wsrc[PIECES];
        uint32_t wdst[PIECES];
#pragma unroll
        for (int i = 0; i < PIECES; ++i) {
            const int row = wt / PER + i * RSTEP;             // class of the tile
            int64_t j = n0 + row;
            if (j >= p.J) j = p.J - 1;
            if (FP32)
                wsrc[i] = reinterpret_cast<uint64_t>(p.W) + (uint64_t)(j * p.D) * 4;
            else
                wsrc[i] = reinterpret_cast<uint64_t>(p.W) + (uint64_t)((j / 256) * (p.P / 64) * 16384 + (j % 256) * 64 + part * 8) * 2;
            // class c of a wavefront's block sits in LDS row 16 (c % NTL) + c / NTL: a lane's NTL columns are neighbours
            const int blk = row / (16 * NTL), c = row % (16 * NTL), r = blk * 16 * NTL + 16 * (c % NTL) + c / NTL;
            const int chunk = FP32 ? part / 2 : part;
            wdst[i] = (uint32_t)(NX * XS + r * 128 + ((chunk ^ swz(r)) << 4) + (FP32 ? (part & 1) * 8 : 0));
        }
        u32x4 wreg[DW][PIECES];
        // (No branch around a load: where paths with and without it meet, the compiler can only wait for everything.
        // Past the last slice the loads repeat it and W counts as zero, as do fp32 columns past D.)
        auto live = [&](int s) { return s < nk && (!FP32 || (int64_t)at(s) * KS + 4 * part < p.D); };
        auto fetch = [&](int s, u32x4 (&dst)[PIECES]) {
            const uint64_t off = FP32 ? (uint64_t)fwd_w_column((int64_t)at(s) * KS, part, p.D) * 4 : (uint64_t)at(s) * 32768;
#pragma unroll
            for (int i = 0; i < PIECES; ++i) dst[i] = *reinterpret_cast<const __attribute__((address_space(1))) u32x4*>(wsrc[i] + off);
        };
        auto store = [&](int s, int stage, const u32x4 (&src)[PIECES]) {
            const bool on = live(s);
#pragma unroll
            for (int i = 0; i < PIECES; ++i) {
                char* const to = lds + stage * WS + wdst[i];
                uint32_t a = src[i][0], b = src[i][1], c = src[i][2], d = src[i][3];
                if (FP32) {
                    a = pack_bf16(__uint_as_float(a), __uint_as_float(b));
                    b = pack_bf16(__uint_as_float(c), __uint_as_float(d));
                    *reinterpret_cast<u32x2*>(to) = u32x2{on ? a : 0u, on ? b : 0u};
                } else {
                    *reinterpret_cast<u32x4*>(to) = u32x4{on ? a : 0u, on ? b : 0u, on ? c : 0u, on ? d : 0u};
                }
            }
        };
        static_for<0, DW>([&](auto S) {
            fetch(decltype(S)::value, wreg[decltype(S)::value]);
            __builtin_amdgcn_sched_barrier(0);      // (left alone the compiler gathers loads and sinks them to their use)
        });
        store(0, 0, wreg[0]);
        fetch(DW, wreg[0]);
        __syncthreads();
        static_for<0, MT + NTL>([&](auto Q) { read_one(f0, 0, 0, 0, decltype(Q)::value); });
        int xs = 0;
        for (int s0 = 0; s0 < rounds * DW; s0 += DW) {
            static_for<0, DW>([&](auto U) {
                constexpr int u = decltype(U)::value, v = (u + 1) % DW;
                const int xn = xs + 1 == NX ? 0 : xs + 1;
                store(s0 + u + 1, (u + 1) & 1, wreg[v]);
                fetch(s0 + u + 1 + DW, wreg[v]);
                step(f0, f1, xs, u & 1, 1, [](auto) {});
                __syncthreads();
                step(f1, f0, xn, (u + 1) & 1, 0, [](auto) {});
                xs = xn;
            });
        }
    }

    // register e of lane (quad, l16) of tile (i, n): sample 16 i + 4 quad + e, class NTL l16 + n of the wavefront's block
    float* const Z = p.Z + (int64_t)blockIdx.y * p.plane;
    const int64_t j = n0 + wn0 + NTL * l16;
    typedef float VecN __attribute__((ext_vector_type(NTL)));
#pragma unroll
    for (int i = 0; i < MT; ++i)
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            const int64_t b = m0 + wm0 + 16 * i + 4 * quad + e;
            if (b >= p.B || j >= p.J) continue;            // (whole tiles are allocated: a group across J is in bounds)
            VecN v;
#pragma unroll
            for (int n = 0; n < NTL; ++n) v[n] = acc[i][n][e];
            *reinterpret_cast<VecN*>(Z + ((j / 256) * p.tiles_b + b / 256) * 65536 + (b % 256) * 256 + j % 256) = v;
        }
}

template <int MT, int NTL, int DW, bool FP32>
hipError_t launch_fwd(FwdParams p, int split, DeviceInfo& dev, int slot, hipStream_t stream)
{
    constexpr int BM = 64 * MT, BN = 32 * NTL, LDS = NX * BM * 128 + 2 * BN * 128;
    const int64_t tm = (p.B + BM - 1) / BM, tn = (p.J + BN - 1) / BN, nk = (p.D + KS - 1) / KS;
    if (tm * tn > 0x7fffffffLL || nk > 0x3fffffffLL) return hipErrorInvalidValue;
    p.tiles_m = (int)tm;
    p.per_split = (int)((nk + split - 1) / split);
    if ((nk + p.per_split - 1) / p.per_split != split) return hipErrorInvalidValue;      // (every plane is written)
    if (!dev.fwd_stream_lds_set[slot]) {
        hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(&fwd_stream_kernel<MT, NTL, DW, FP32>),
                                           hipFuncAttributeMaxDynamicSharedMemorySize, LDS);
        if (e != hipSuccess) return e;
        dev.fwd_stream_lds_set[slot] = true;
    }
    hipLaunchKernelGGL((fwd_stream_kernel<MT, NTL, DW, FP32>), dim3((unsigned)(tm * tn), (unsigned)split), dim3(NT), LDS, stream, p);
    return hipGetLastError();
}

}  // namespace

// Measured (us; f: W as fp32, h: from its bf16 copy; the conversion that f saves and the 256 x 256 kernel in
// brackets): 256 samples, 8192 x 4096: f 36 [33 + 75], h 28 [75]; 200, 1504 x 9000: f 22, h 18 [160]; 100, 20000 x
// 3000: f 57 [72 + 55], h 31 [55]; 1000, 4000 x 2000: f 34, h 27 [10 + 43]; 256, 40000 x 2048: f 114 [98 + 42],
// h 74 [42].  Per tile and slice the kernel takes 0.5 to 0.9 us, bound by what a CU pulls from the L2 (48 KB in f)
// and by its LDS; W as fp32 arrives at 4.6 TB/s.
MlrForwardPlan mlr_forward_plan(int64_t B, int64_t J, int64_t D, bool have_copy, bool may_split)
{
    const int64_t nk = (D + KS - 1) / KS;
    // The CU count of an MI355X, not the context's: the workspace is sized from the plan, and that query has no device.
    const double cus = 256.0, w = (double)J * (double)D;
    MlrForwardPlan best = {};
    best.split = 1;
    const int64_t tiles = ((B + 255) / 256) * ((J + 255) / 256);
    double best_t = 3.0 + std::ceil((double)tiles / cus) * ((double)nk * 1.12 + 6.0);
    if (!have_copy) best_t += 3.0 + w * 6.0 / 5e6;
    // shape: MT, NTL; us per slice with the chip full
    struct Shape {
        int mt, ntl;
        double us;
    };
    static const Shape copy_shapes[3] = {{4, 2, 0.64}, {2, 4, 0.60}, {1, 2, 0.30}}, fp32_shapes[3] = {{4, 2, 0.86}, {2, 2, 0.62}, {1, 2, 0.52}};
    for (int i = 0; i < 3; ++i) {
        const Shape& sh = have_copy ? copy_shapes[i] : fp32_shapes[i];
        const int64_t tm = (B + 64 * sh.mt - 1) / (64 * sh.mt), tn = (J + 32 * sh.ntl - 1) / (32 * sh.ntl);
        for (int s = 1; s <= (may_split ? 16 : 1); ++s) {
            const int64_t per = (nk + s - 1) / s;
            if (s > 1 && (J > MLR_SOFTMAX_ROW_MAX || per < 4)) break;      // (so for every larger s)
            if (s > 1 && (nk + per - 1) / per != s) continue;
            const double rounds = std::ceil((double)(tm * tn * s) / cus);
            double t = 3.0 + rounds * ((double)per * sh.us + 4.5) + (s > 1 ? (double)s * (double)B * (double)J * 8.0 / 4e6 : 0.0);
            const double stream_us = w * (have_copy ? 2.0 : 4.0) * (double)tm / 4.6e6 + 5.0;
            if (t < stream_us) t = stream_us;
            if (t < best_t) {
                best_t = t;
                best = MlrForwardPlan{sh.mt, sh.ntl, s};
            }
        }
    }
    return best;
}

// Whole k-slices need no padding with zeros, and a piece of a sample in one is a line of 128 bytes in either layout: the
// samples are then read as they come (32-bit offsets inside a tile of 256).  Rows that end inside a slice would bring the
// next sample's features, which zeros of W do not cancel where they are infinite.  Copy in front / none (us of the whole
// factor computation, samples x classes x features, W as fp32; from its copy): 16 x 1000 x 1024 15.0 / 9.7; 15.0 / 10.2,
// 256 x 1504 x 8960 38.8 / 32.8; 33.5 / 27.5, 256 x 8192 x 4096 48.6 / 46.1; 41.0 / 37.7, 1000 x 4000 x 2048 46.2 / 42.4;
// 39.9 / 35.7, 256 x 40000 x 2048 130.7 / 127.5; 78.0 / 76.8, 64 x 325000 x 10048 2548 / 2556 (fp32).
bool fwd_stream_takes_rows(const MlrForwardPlan& plan, int64_t D) { return plan.mt > 0 && D % KS == 0 && D < (1LL << 22); }

hipError_t launch_fwd_stream(const MlrForwardPlan& plan, const uint16_t* X, bool rows, const float* W, const uint16_t* W_shadow, float* Z, int64_t B,
                             int64_t J, int64_t D, DeviceInfo& dev, hipStream_t stream)
{
    FwdParams p = {};
    p.X = X;
    p.x_pitch = rows ? D : 0;
    p.W = W_shadow ? static_cast<const void*>(W_shadow) : static_cast<const void*>(W);
    p.Z = Z;
    p.plane = mlr_logits_floats(B, J);
    p.B = B; p.J = J; p.D = D; p.P = bf16_pitch(D);
    p.tiles_b = (int)((B + 255) / 256);
    p.num_xcd = dev.xcds > 0 ? dev.xcds : 1;
    if (W_shadow) {
        if (plan.mt == 4) return launch_fwd<4, 2, 8, false>(p, plan.split, dev, 0, stream);
        if (plan.mt == 2) return launch_fwd<2, 4, 4, false>(p, plan.split, dev, 1, stream);
        return launch_fwd<1, 2, 8, false>(p, plan.split, dev, 2, stream);
    }
    if (plan.mt == 4) return launch_fwd<4, 2, 6, true>(p, plan.split, dev, 3, stream);
    if (plan.mt == 2) return launch_fwd<2, 2, 8, true>(p, plan.split, dev, 4, stream);
    return launch_fwd<1, 2, 8, true>(p, plan.split, dev, 5, stream);
}

}  // namespace sfb
