// The fp32 contractions of gemm_f32.hip where they are large, on the bf16 matrix pipes.
//
// A value of 24 bits is the sum of three bf16 values of 8 bits each, x = h + m + l (h cut off, m rounded, l what is left:
// exact for |x| >= 2^-110, below that to 2^-134).  A product of two values is taken as the six products
//   h h' + (h m' + m h') + (h l' + m m' + l h')
// which leave out less than 2^-24 of it; every one of them is exact in fp32, and v_mfma_f32_32x32x16_bf16 adds sixteen of
// them with two roundings.  The leading products have accumulators of their own, so that the running sum is rounded as
// rarely as possible: the 2-norm of the error of a product of 1000 x 2048 over 2048 pairs, N(0,1), is 1.5e-7 (5.7e-7 with
// fp32 MFMAs), of 512 x 4096 over 1024 0.9e-7, over 64 0.5e-7 (1.4e-7).  Infinities and NaN: where the sum of the leading
// products is not finite it is the result (the others then hold Inf - Inf).
//
// One workgroup of four wavefronts, one per SIMD, owns an output tile; each wavefront multiplies 128 x 64 of it over its
// own blocks of 32 of k (KW wavefronts take turns), and the partial sums meet in LDS at the end.  No wavefront shares
// operand data with another, so the loop has no LDS and no barrier: a lane loads what it multiplies (16 bytes a lane
// along the rows of a k-strided operand, 512 contiguous bytes per 32 lanes), two steps of 16 ahead, cuts it into its terms between the
// MFMAs (11 instructions per pair; 5.5 of them per MFMA of 32 cycles, which hides that many) and multiplies.
//
// 32x32x16 rather than 16x16x32 MFMAs: the latter hide two vector instructions each, and the loop has three times as many.
//
// What bounds it: power.  The launch of 1000 x 2048 over 2048 takes 79000 cycles of which the matrix pipes are busy for
// 49000; on zeros the clock is 2.37 GHz and the launch takes 36 us, on N(0,1) values 1.65 to 1.8 GHz and 46 to 49.
#include "gemm_f32.h"

#include <type_traits>

namespace sfb {
namespace {

typedef float floatx4 __attribute__((ext_vector_type(4)));
typedef float floatx2 __attribute__((ext_vector_type(2)));
typedef float floatx16 __attribute__((ext_vector_type(16)));
typedef float floatx4u __attribute__((ext_vector_type(4), aligned(4)));
typedef uint32_t uintx2 __attribute__((ext_vector_type(2)));
typedef uint32_t uintx4 __attribute__((ext_vector_type(4)));
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef __amdgpu_buffer_rsrc_t Rsrc;

constexpr int TA = 4, TB = 2;      // a wavefront's 32 x 32 MFMA tiles along the rows and columns of C
constexpr int NT = 256;

// WN wavefronts side by side along n, KW over k.
template <int WN_, int KW_>
struct Tile {
    static constexpr int WN = WN_, KW = KW_, BM = 32 * TA, BN = 32 * TB * WN;
    static constexpr int LDS = KW * BM * BN * 4;      // the partial sums
    static_assert(WN * KW * 64 == NT, "four wavefronts");
};

// The three terms of eight values of k of a row, packed as MFMA operands.
struct Terms {
    uint32_t t[3][4];
};
__device__ __forceinline__ bf16x8 fragment(const uint32_t* t)
{
    const uintx4 v = {t[0], t[1], t[2], t[3]};
    return __builtin_bit_cast(bf16x8, v);
}
// (h is cut off rather than rounded: rounded, the largest fp32 values would become infinite)
__device__ __forceinline__ void cut_pair(float x0, float x1, Terms& s, int i)
{
    const uint32_t h = __builtin_amdgcn_perm(__float_as_uint(x1), __float_as_uint(x0), 0x07060302u);
    const float r0 = x0 - __uint_as_float(__float_as_uint(x0) & 0xffff0000u), r1 = x1 - __uint_as_float(__float_as_uint(x1) & 0xffff0000u);
    const uint32_t m = pack_bf16(r0, r1);
    const float s0 = r0 - __uint_as_float(m << 16), s1 = r1 - __uint_as_float(m & 0xffff0000u);
    s.t[0][i] = h;
    s.t[1][i] = m;
    s.t[2][i] = pack_bf16(s0, s1);
}

// One operand of a wavefront ([k][rows]): 32 T rows.  Lane (l32, half) holds of MFMA tile x the row T l32 + x and the k
// 8 half .. + 7 of a step of 16; a block is two steps.  Loads go through a buffer descriptor that ends with the matrix:
// what lies behind its end reads as zero, and rows past the last one reach only elements of C that are not stored.
template <int T>
struct Operand {
    float raw[2][T][8];      // two steps
    uint32_t voff, ld4;
    uint64_t base, end;      // uniform

    __device__ __forceinline__ void init(const float* P, int64_t ld, int64_t row0, int64_t rows, int64_t K, int l32, int half)
    {
        ld4 = (uint32_t)ld * 4u;
        base = uniform64(reinterpret_cast<uint64_t>(P) + (uint64_t)row0 * 4);
        end = uniform64(reinterpret_cast<uint64_t>(P) + (uint64_t)((K - 1) * ld + rows) * 4);
        voff = 8u * half * ld4 + 4u * T * l32;
    }
    __device__ __forceinline__ Rsrc at(int block) const
    {
        const uint64_t b = uniform64(base + (uint64_t)block * 32 * ld4);
        const uint64_t left = b < end ? end - b : 0;
        return __builtin_amdgcn_make_buffer_rsrc(reinterpret_cast<void*>(b), 0, left > 0xffffffffu ? 0xffffffffu : (uint32_t)left, 0x00020000);
    }
    // step j of the block at r
    __device__ __forceinline__ void load(Rsrc r, int j, int slot)
    {
#pragma unroll
        for (int i = 0; i < 8; ++i) {
            if (T == 4) {
                const uintx4 v = __builtin_amdgcn_raw_buffer_load_b128(r, voff, (16u * j + i) * ld4, 0);
#pragma unroll
                for (int x = 0; x < T; ++x) raw[slot][x][i] = __uint_as_float(v[x & 3]);
            } else {
                const uintx2 v = __builtin_amdgcn_raw_buffer_load_b64(r, voff, (16u * j + i) * ld4, 0);
#pragma unroll
                for (int x = 0; x < T; ++x) raw[slot][x][i] = __uint_as_float(v[x & 1]);
            }
        }
    }
    // pair i (values 2 i, 2 i + 1) of the terms of tile x; MASKED: zeros from value `left` of the step on
    template <bool MASKED>
    __device__ __forceinline__ void cut(Terms& s, int x, int slot, int i, int left, int half) const
    {
        const float x0 = raw[slot][x][2 * i], x1 = raw[slot][x][2 * i + 1];
        if (MASKED)
            cut_pair(8 * half + 2 * i < left ? x0 : 0.f, 8 * half + 2 * i + 1 < left ? x1 : 0.f, s, i);
        else
            cut_pair(x0, x1, s, i);
    }
};

template <class TL, int EPI>
__global__ __launch_bounds__(NT) __attribute__((amdgpu_waves_per_eu(1, 1))) void gemm_f32x3_kernel(GemmF32Params p)
{
    constexpr int WN = TL::WN, KW = TL::KW, BM = TL::BM, BN = TL::BN;
    extern __shared__ floatx4 x3_smem[];
    const int tid = threadIdx.x, lane = tid & 63, l32 = lane & 31, half = lane >> 5;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int kw = wave / WN, wn0 = (wave % WN) * (32 * TB);
    uint32_t tile_m, tile_n;
    gemm_tile_of(p, tile_m, tile_n);
    const int64_t m0 = (int64_t)tile_m * BM, n0 = (int64_t)tile_n * BN;
    // blocks of 32 of k of this workgroup, and how many of them are this wavefront's (its first and every KW-th from there).
    // The partial block at the end of K, if it has that one, is taken first: the only one with masks.
    const int z = blockIdx.y, all = (int)((p.K + 31) / 32), left = (int)(p.K % 32);
    const int b0 = p.split_k > 1 ? z * (int)p.per_split : 0, per = p.split_k > 1 ? (int)p.per_split : all;
    const int blocks = (b0 + per < all ? b0 + per : all) - b0;
    const int n = blocks > kw ? (blocks - kw + KW - 1) / KW : 0;
    const bool tail = left && b0 + blocks == all && n > 0 && (blocks - 1) % KW == kw;

    floatx16 acc[TA][TB], cor[TA][TB];      // sums of h h'; of the rest
#pragma unroll
    for (int a = 0; a < TA; ++a)
#pragma unroll
        for (int b = 0; b < TB; ++b)
#pragma unroll
            for (int e = 0; e < 16; ++e) acc[a][b][e] = cor[a][b][e] = 0.f;

    if (n > 0) {
        Operand<TA> A;
        Operand<TB> B;
        A.init(p.A, p.lda, m0, p.M, p.K, l32, half);
        B.init(p.B, p.ldb, n0 + wn0, p.N, p.K, l32, half);
        const int first = tail ? all - 1 : b0 + kw, lim = tail ? left : 32;
        const int second = n < 2 ? first : (tail ? b0 + kw : b0 + kw + KW);      // (no further block: the last one again)
        {
            const Rsrc ra = A.at(first), rb = B.at(first);
            B.load(rb, 0, 0);
            A.load(ra, 0, 0);
            B.load(rb, 1, 1);
            A.load(ra, 1, 1);
        }
        // A tile a of step j has its terms in at[(j + a) % 3], B tile b in bt[j][b]
        Terms at[3], bt[2][TB];
#pragma unroll
        for (int i = 0; i < 4; ++i) {
#pragma unroll
            for (int b = 0; b < TB; ++b) B.template cut<true>(bt[0][b], b, 0, i, lim, half);
            A.template cut<true>(at[0], 0, 0, i, lim, half);
        }
        B.load(B.at(second), 0, 0);
        auto products = [&](const Terms& ta, const Terms& tb, floatx16& ac, floatx16& co) {
            constexpr int PA[6] = {2, 0, 0, 1, 1, 0}, PB[6] = {0, 2, 0, 1, 0, 1};
#pragma unroll
            for (int q = 0; q < 6; ++q) {
                floatx16& c = q == 2 ? ac : co;
                c = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fragment(ta.t[PA[q]]), fragment(tb.t[PB[q]]), c, 0, 0, 0);
            }
            static_for<0, 6>([&](auto) {
                __builtin_amdgcn_sched_group_barrier(0x8, 1, 0);      // an MFMA,
                __builtin_amdgcn_sched_group_barrier(0x2, 6, 0);      // six vector instructions
            });
            __builtin_amdgcn_sched_barrier(0);
        };
        // One block: eight phases a step, the six products of one MFMA tile each.  Beside them 24 pairs are cut, three a
        // phase: of A tiles 1, 2, 3 and, for the next step, of B tiles 0, 1 and A tile 0.  A step's raw values are
        // requested again (for the step behind the next; B for the one behind that) as soon as all of them are cut.
        auto block = [&](auto first_tag, Rsrc a_next, Rsrc b_next, Rsrc b_after) {
            constexpr bool FIRST = decltype(first_tag)::value;
            static_for<0, 2>([&](auto j_) {
                constexpr int j = decltype(j_)::value;
                __builtin_amdgcn_sched_barrier(0);
                auto cut = [&](auto c_) {
                    constexpr int c = decltype(c_)::value, set = c / 4, i = c % 4;
                    constexpr bool MASKED = FIRST && (set < 3 || j == 0);
                    if constexpr (set < 3)
                        A.template cut<MASKED>(at[(j + set + 1) % 3], set + 1, j, i, lim - 16 * j, half);
                    else if constexpr (set < 5)
                        B.template cut<MASKED>(bt[j ^ 1][set - 3], set - 3, j ^ 1, i, lim - 16, half);
                    else
                        A.template cut<MASKED>(at[(j + 4) % 3], 0, j ^ 1, i, lim - 16, half);
                };
                static_for<0, 8>([&](auto ph_) {
                    constexpr int ph = decltype(ph_)::value, a = ph / 2, b = (a & 1) ? 1 - ph % 2 : ph % 2;
                    static_for<3 * ph, 3 * ph + 3>(cut);
                    if constexpr (ph == 4) A.load(a_next, j, j);
                    if constexpr (ph == 7) B.load(j ? b_after : b_next, j ^ 1, j ^ 1);
                    products(at[(j + a) % 3], bt[j][b], acc[a][b], cor[a][b]);
                });
            });
            at[0] = at[2];
        };
        int next = n < 3 ? second : second + KW;
        block(std::true_type{}, A.at(second), B.at(second), B.at(next));
        for (int i = 1; i < n; ++i) {
            const int after = i + 2 < n ? next + KW : next;
            block(std::false_type{}, A.at(next), B.at(next), B.at(after));
            next = after;
        }
    }

    // ---- the partial sums meet in LDS as [kw][row][column]; a thread takes four neighbouring columns of a row
    float* const meet = reinterpret_cast<float*>(x3_smem);
    const bool direct = EPI == EPI_STORE || p.split_k > 1;
    float* const out = p.split_k > 1 ? p.partial + (int64_t)z * p.M * p.N : p.C;
    const int64_t ldo = p.split_k > 1 ? p.N : p.ldc;
    constexpr int PER = BM * BN / 4 / NT, PO = EPI == EPI_STORE ? 1 : PER;
    floatx4 old[PO];
    float invL = 0.f, th = 0.f;
    if (EPI != EPI_STORE && !direct) {      // (on their way while the sums meet)
        if (EPI == EPI_SHRINK) {
            invL = 1.0f / p.L_ptr[0];
            th = p.lambda * invL;
        }
        const float* src = EPI == EPI_RMW ? p.C : p.aux;      // (EPI_SHRINK, null: zeros)
#pragma unroll
        for (int i = 0; i < PO; ++i) {
            const int u = tid + NT * i;
            const int64_t row = m0 + u / (BN / 4), col = n0 + 4 * (u % (BN / 4));
            old[i] = floatx4{0.f, 0.f, 0.f, 0.f};
            if (row < p.M && (EPI != EPI_SHRINK || src)) {
                const float* s = src + row * p.ldc + col;
                if (col + 4 <= p.N) {
                    const floatx4u v = *reinterpret_cast<const floatx4u*>(s);
                    old[i] = floatx4{v[0], v[1], v[2], v[3]};
                } else {
#pragma unroll
                    for (int c = 0; c < 4; ++c)
                        if (col + c < p.N) old[i][c] = s[c];
                }
            }
        }
    }
#pragma unroll
    for (int a = 0; a < TA; ++a)
#pragma unroll
        for (int e = 0; e < 16; ++e) {
            floatx2 v;
#pragma unroll
            for (int b = 0; b < TB; ++b) {      // (a sum of leading products that is not finite is the result)
                const float x = acc[a][b][e], y = x + cor[a][b][e];
                v[b] = __builtin_fabsf(x) < __builtin_inff() ? y : x;
            }
            *reinterpret_cast<floatx2*>(meet + (kw * BM + TA * (8 * (e / 4) + 4 * half + e % 4) + a) * BN + wn0 + TB * l32) = v;
        }
    __syncthreads();
#pragma unroll
    for (int i = 0; i < PER; ++i) {
        const int u = tid + NT * i;
        const int64_t row = m0 + u / (BN / 4), col = n0 + 4 * (u % (BN / 4));
        floatx4 sum = *reinterpret_cast<const floatx4*>(meet + 4 * u);
#pragma unroll
        for (int k = 1; k < KW; ++k) sum += *reinterpret_cast<const floatx4*>(meet + k * BM * BN + 4 * u);
        if (row >= p.M) continue;
        if (!direct) {
#pragma unroll
            for (int c = 0; c < 4; ++c) sum[c] = gemm_combine<EPI>(old[EPI == EPI_STORE ? 0 : i][c], sum[c], p.eta, invL, th);
        }
        float* dst = out + row * ldo + col;
        if (col + 4 <= p.N) {
            *reinterpret_cast<floatx4u*>(dst) = floatx4u{sum[0], sum[1], sum[2], sum[3]};
        } else {
#pragma unroll
            for (int c = 0; c < 4; ++c)
                if (col + c < p.N) dst[c] = sum[c];
        }
    }
}

typedef Tile<1, 4> X0;      // 128 x 64
typedef Tile<2, 2> X1;      // 128 x 128
constexpr int NTILES = 2;

template <class TL, int EPI>
hipError_t launch_tile(GemmF32Params& p, DeviceInfo& dev, int slot, int split, hipStream_t stream)
{
    const int64_t tm = (p.M + TL::BM - 1) / TL::BM, tn = (p.N + TL::BN - 1) / TL::BN;
    if (!dev.gemm_f32x3_lds_set[slot]) {
        hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(&gemm_f32x3_kernel<TL, EPI>),
                                           hipFuncAttributeMaxDynamicSharedMemorySize, TL::LDS);
        if (e != hipSuccess) return e;
        dev.gemm_f32x3_lds_set[slot] = true;
    }
    const int64_t blocks = (p.K + 31) / 32;
    p.per_split = split > 1 ? (blocks + split - 1) / split : blocks;
    p.split_k = split > 1 ? (int)((blocks + p.per_split - 1) / p.per_split) : 1;      // (no empty split)
    gemm_f32_raster(p, tm, tn, TL::BM, TL::BN, dev);
    hipLaunchKernelGGL((gemm_f32x3_kernel<TL, EPI>), dim3((unsigned)(tm * tn), (unsigned)p.split_k), dim3(NT), TL::LDS, stream, p);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess || p.split_k <= 1) return e;
    return launch_splitk_reduce(p, EPI, stream);
}

}  // namespace

// Estimated duration (us): the launch (more with the chip full), and rounds of one workgroup per CU, each `own` for its
// first loads, meeting and epilogue and `step` for every block of 32 of k of a wavefront (less where CUs are idle); a
// k-split pays a second launch and the traffic of the partial sums.  Fitted to 60 shapes of sfb_apply, 100 x 100 with 32
// pairs to 4100 x 8200 with 4000 (rms of the logarithm 8 %); with the estimates of the fp32 kernel the choice between the
// two was 13.1 % faster in the mean than that kernel alone, the better one each time 13.2 %.  fp32 kernel / this one (us):
//   1000 x 2048, 2048 pairs 77 / 50    4096 x 4096, 2048 483 / 339    1003 x 2047, 800 43 / 29    1024 x 4096, 512 41 / 30
//   616 x 2488, 327 19 / 17            1720 x 208, 1531 19.2 / 19.0   284 x 850, 1340 14.8 / 16.3  1561 x 5818, 37 34 / 39
// What is within 3 % stays with the fp32 kernel.
GemmF32x3Plan gemm_f32x3_plan(const GemmF32Args& a, int max_split)
{
    GemmF32x3Plan best = {-1, 1, 1e30};
    if (!a.a_kstrided || !a.b_kstrided || a.epilogue != EPI_RMW) return best;
    // a handful of blocks of k for a wavefront (with 128 pairs it was never faster); 32-bit offsets inside a block
    if (a.K < 160 || a.K > (1LL << 30) || a.lda >= (1LL << 24) || a.ldb >= (1LL << 24)) return best;
    static const double own[NTILES] = {5.1, 10.1}, step[NTILES] = {2.07, 2.02};
    const int cus = a.dev->cus > 0 ? a.dev->cus : 256;
    const int64_t blocks = (a.K + 31) / 32;
    for (int t = 0; t < NTILES; ++t) {
        const int64_t bn = t ? X1::BN : X0::BN, kw = t ? X1::KW : X0::KW, tiles = ((a.M + 127) / 128) * ((a.N + bn - 1) / bn);
        if (tiles > 0x7fffffffLL) continue;
        for (int s = 1; s <= max_split; ++s) {
            const int64_t steps = ((blocks + s - 1) / s + kw - 1) / kw, wgs = tiles * s;
            const double idle = wgs < cus ? 1.0 - (double)wgs / cus : 0.0;
            double us = 4.5 + 1.8 * (1.0 - idle) + (double)((wgs + cus - 1) / cus) * (own[t] + (double)steps * step[t] * (1.0 - 0.18 * idle));
            if (s > 1) us += 4.0 + (double)(s + 1) * (double)a.M * (double)a.N * 4.0 / 6e6;
            if (us < best.us) best = GemmF32x3Plan{t, s, us};
        }
    }
    best.us /= 0.97;
    return best;
}

hipError_t launch_gemm_f32x3(const GemmF32Args& a, GemmF32Params p, const GemmF32x3Plan& plan, hipStream_t stream)
{
    if (plan.tile == 0) return launch_tile<X0, EPI_RMW>(p, *a.dev, 0, plan.split, stream);
    return launch_tile<X1, EPI_RMW>(p, *a.dev, 1, plan.split, stream);
}

}  // namespace sfb
