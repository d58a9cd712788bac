// The fp32 contractions of gemm_f32.hip where they are large, on the bf16 matrix pipes.
//
// A value of 24 bits is the sum of three bf16 values of 8 bits each, x = h + m + l (h and m rounded to nearest, l what is
// left).  bf16 ends at 2^-133, so the values are multiplied by 2^16 first and the sums by 2^-32 at the end: exact down to the
// smallest denormal (without that only from 2^-110 on, and values below 2^-134 were lost).  A product is taken as the six
//   h h' + (h m' + m h') + (h l' + m m' + l h')
// Every one of them is exact in fp32, and v_mfma_f32_32x32x16_bf16 adds sixteen of them with two roundings.  The rest,
// m l' + l m' + l l', is at most 2 * 2^-8 * 2^-17 of the product and a little: (1 + 2^-9) 2^-24, typically 2^-26 (h cut off
// instead of rounded it is up to 2^-22).  The leading products have accumulators of their own, so that the running sum is
// rounded as rarely as possible.  rms error over the sum of the products' sizes in units of 2^-24, here / with fp32 MFMAs,
// by the number of products that are not zero: one 0.44 / 0.42, two 0.48 / 0.47, three 0.49 / 0.48, five 0.44 / 0.46, twelve
// 0.33 / 0.40, fifty 0.19 / 0.35.  2-norm of the error of a product of 1003 x 2047 over 300 pairs, N(0,1): 0.7e-7 (2.2e-7).
// Infinities and NaN: the terms do not hold them apart (Inf - Inf), and values from 2^112 and sums from 2^96 on become infinite
// here, so a workgroup with a sum that is not finite multiplies its part again with fp32 MFMAs and takes those results.
//
// One workgroup of four wavefronts, one per SIMD, owns an output tile; each wavefront multiplies 128 x 64 of it over its
// own blocks of 32 of k (KW wavefronts take turns), and the partial sums meet in LDS at the end.  No wavefront shares
// operand data with another, so the loop has no barrier.  Two k-strided operands: a lane loads what it multiplies (16
// bytes a lane along the rows, 512 contiguous bytes per 32 lanes), two steps of 16 ahead.  Otherwise a wavefront brings a
// block of its operands into LDS of its own while it multiplies the one before.  It cuts the values into their terms
// between the MFMAs (13 instructions per pair, 6.5 of them per MFMA of 32 cycles; without the multiplications by 2^16 five and
// a half, and 1000 x 2048 over 2048 takes 47.5 instead of 48.9 us, 4096 x 4096 over 2048 335 instead of 347).
//
// 32x32x16 rather than 16x16x32 MFMAs: the latter hide two vector instructions each, and the loop has three times as many.
//
// What bounds it: power and instruction issue.  The launch of 1000 x 2048 over 2048 takes 84600 cycles of which the matrix
// pipes are busy for 49000; on zeros the clock is 2.35 GHz and the launch takes 36 us, on N(0,1) values 1.75 GHz and 47 to 49.
// Where k is short the launch, first loads and epilogue (8 us in all) count as much.  The epilogue goes through buffer
// descriptors because the branches of a bounds check per access made it wait for each old value in turn (24 instead of 29 us
// at 1003 x 2047 over 800).  The launch takes 190 us where every sum is multiplied again (factors of nothing but NaN; the fp32
// kernel 65).  Factors that rotate through 320 MB instead of coming from the caches: 48.2 / 49.0 us, 1003 x 2047 over 800
// 24.9 / 26.1.
#include "gemm_f32.h"

#include <type_traits>

namespace sfb {
namespace {

typedef float floatx4 __attribute__((ext_vector_type(4)));
typedef float floatx2 __attribute__((ext_vector_type(2)));
typedef float floatx16 __attribute__((ext_vector_type(16)));
typedef uint32_t uintx2 __attribute__((ext_vector_type(2)));
typedef uint32_t uintx4 __attribute__((ext_vector_type(4)));
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef __amdgpu_buffer_rsrc_t Rsrc;

constexpr int TA = 4, TB = 2;      // a wavefront's 32 x 32 MFMA tiles along the rows and columns of C
constexpr int NT = 256;
constexpr float SCALE = 0x1p16f, UNSCALE = 0x1p-32f;      // of the values before they are cut; of a sum

// WN wavefronts side by side along n, KW over k.
template <int WN_, int KW_>
struct Tile {
    static constexpr int WN = WN_, KW = KW_, BM = 32 * TA, BN = 32 * TB * WN;
    static constexpr int SUMS = KW * BM * BN * 4, LDS = SUMS + 16;      // the partial sums (before: 24 KB a wavefront); a flag
    static_assert(WN * KW * 64 == NT && SUMS >= 4 * 4096 * (TA + TB), "four wavefronts");
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
// (the largest values become infinite: their sums are then not finite and multiplied again)
__device__ __forceinline__ void cut_pair(float x0, float x1, Terms& s, int i)
{
    x0 *= SCALE;
    x1 *= SCALE;
    const uint32_t h = pack_bf16(x0, x1);
    const float r0 = x0 - __uint_as_float(h << 16), r1 = x1 - __uint_as_float(h & 0xffff0000u);
    const uint32_t m = pack_bf16(r0, r1);
    const float s0 = r0 - __uint_as_float(m << 16), s1 = r1 - __uint_as_float(m & 0xffff0000u);
    s.t[0][i] = h;
    s.t[1][i] = m;
    s.t[2][i] = pack_bf16(s0, s1);
}

// What both kinds of operands have of a wavefront's 32 T rows: lane (l32, half) holds of MFMA tile x the row T l32 + x and
// the k 8 half .. + 7 of a step of 16; a block is two steps.
template <int T>
struct Raw {
    float raw[2][T][8];      // two steps

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

// Loads go through a buffer descriptor that ends with the matrix: what lies behind its end is not read (and masked), and
// rows past the last one reach only elements of C that are not stored.
template <bool KS>
struct Extent {
    uint64_t base, end;      // uniform
    uint32_t ld4;
    __device__ __forceinline__ void init(const float* P, int64_t ld, int64_t row0, int64_t rows, int64_t K)
    {
        ld4 = (uint32_t)ld * 4u;
        base = uniform64(reinterpret_cast<uint64_t>(P) + (uint64_t)(KS ? row0 : row0 * ld) * 4);
        end = uniform64(reinterpret_cast<uint64_t>(P) + (uint64_t)(KS ? (K - 1) * ld + rows : (rows - 1) * ld + K) * 4);
    }
    __device__ __forceinline__ uint64_t start(int block) const { return uniform64(base + (uint64_t)block * (KS ? 32 * (uint64_t)ld4 : 128)); }
    __device__ __forceinline__ uint32_t bytes(uint64_t b) const
    {
        const uint64_t left = b < end ? end - b : 0;
        return left > 0xffffffffu ? 0xffffffffu : (uint32_t)left;
    }
};

// An operand that is strided along k ([k][rows]): a lane loads what it multiplies, at any alignment.
template <int T>
struct StridedOperand : Raw<T> {
    Extent<true> ext;
    uint32_t voff;

    __device__ __forceinline__ void init(const float* P, int64_t ld, int64_t row0, int64_t rows, int64_t K, int lane)
    {
        ext.init(P, ld, row0, rows, K);
        voff = 8u * (lane >> 5) * ext.ld4 + 4u * T * (lane & 31);
    }
    __device__ __forceinline__ Rsrc at(int block) const
    {
        const uint64_t b = ext.start(block);
        return __builtin_amdgcn_make_buffer_rsrc(reinterpret_cast<void*>(b), 0, ext.bytes(b), 0x00020000);
    }
    // step j of the block at r
    __device__ __forceinline__ void load(Rsrc r, int j, int slot)
    {
#pragma unroll
        for (int i = 0; i < 8; ++i) {
            if (T == 4) {
                const uintx4 v = __builtin_amdgcn_raw_buffer_load_b128(r, voff, (16u * j + i) * ext.ld4, 0);
#pragma unroll
                for (int x = 0; x < T; ++x) this->raw[slot][x][i] = __uint_as_float(v[x & 3]);
            } else {
                const uintx2 v = __builtin_amdgcn_raw_buffer_load_b64(r, voff, (16u * j + i) * ext.ld4, 0);
#pragma unroll
                for (int x = 0; x < T; ++x) this->raw[slot][x][i] = __uint_as_float(v[x & 1]);
            }
        }
    }
};

// An operand whose rows are 16-byte aligned, by way of the wavefront's own LDS (4 KB for 32 rows and a block, no other
// wavefront reads it).  Loading k-contiguous rows lane by lane as they are multiplied costs the address unit 72 cycles
// per kilobyte (32 rows at the same offset), direct loads of eight lanes a row 16.
//   k-contiguous: a unit is a tile, 32 rows of 128 bytes, the 16-byte chunks of row r swizzled by swz(r);
//   k-strided (T = 2): a unit is a step, 16 rows of 64 columns as in memory.
template <int T, bool KS>
struct LdsOperand : Raw<T> {
    Extent<KS> ext;
    uint32_t voff[KS ? 1 : 4];       // of the direct loads
    uint32_t from[KS ? 1 : 4];       // of the LDS reads
    uint32_t lds;                    // of the first unit (uniform)

    __device__ __forceinline__ void init(const float* P, int64_t ld, int64_t row0, int64_t rows, int64_t K, int lane, uint32_t lds_at)
    {
        ext.init(P, ld, row0, rows, K);
        lds = lds_at;
        const int l32 = lane & 31, half = lane >> 5;
        if (KS) {
            voff[0] = (lane >> 4) * ext.ld4 + 16u * (lane & 15);
            from[0] = 8u * half * 256 + 8u * l32;
        } else {
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                voff[KS ? 0 : i] = T * (lane >> 3) * ext.ld4 + 16u * ((lane & 7) ^ swz(8 * i + (lane >> 3)));
                from[KS ? 0 : i] = l32 * 128u + (((4 * (i >> 1) + 2 * half + (i & 1)) ^ swz(l32)) << 4);
            }
        }
    }
    __device__ __forceinline__ uintx4 at(int block) const
    {
        const uint64_t b = ext.start(block);
        return uintx4{(uint32_t)b, (uint32_t)(b >> 32) & 0xffffu, (uint32_t)__builtin_amdgcn_readfirstlane((int)ext.bytes(b)), 0x00020000u};
    }
    // request q of the 4 T of a block
    __device__ __forceinline__ void request(uintx4 r, int q)
    {
        const uint32_t dst = lds + 1024u * q, v = voff[KS ? 0 : q % 4];
        const uint32_t soff = KS ? 4u * q * ext.ld4 : (T * 8u * (q % 4) + q / 4) * ext.ld4;
        asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tbuffer_load_dwordx4 %1, %2, %3 offen lds" ::"s"(dst), "v"(v), "s"(r), "s"(soff) : "memory");
    }
    // both steps of tiles x0 .. x1 - 1 (k-strided: of both tiles)
    __device__ __forceinline__ void read(int x0, int x1)
    {
        typedef __attribute__((address_space(3))) const char* LdsPtr;
        if (KS) {
#pragma unroll
            for (int j = 0; j < 2; ++j)
#pragma unroll
                for (int i = 0; i < 8; ++i) {
                    const floatx2 v = *reinterpret_cast<__attribute__((address_space(3))) const floatx2*>((LdsPtr)(uintptr_t)(lds + from[0] + 4096u * j + 256u * i));
#pragma unroll
                    for (int x = 0; x < T; ++x) this->raw[j][x][i] = v[x & 1];
                }
        } else {
#pragma unroll
            for (int x = x0; x < x1; ++x)
#pragma unroll
                for (int q = 0; q < 4; ++q) {
                    const floatx4 v = *reinterpret_cast<__attribute__((address_space(3))) const floatx4*>((LdsPtr)(uintptr_t)(lds + from[KS ? 0 : q] + 4096u * x));
#pragma unroll
                    for (int e = 0; e < 4; ++e) this->raw[q >> 1][x][4 * (q & 1) + e] = v[e];
                }
        }
    }
};

template <class TL, bool A_KS, bool B_KS, int EPI>
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
        constexpr bool LDS = !A_KS;      // (rows are 16-byte aligned then)
        typename std::conditional<LDS, LdsOperand<TA, A_KS>, StridedOperand<TA>>::type A;
        typename std::conditional<LDS, LdsOperand<TB, B_KS>, StridedOperand<TB>>::type B;
        const int first = tail ? all - 1 : b0 + kw, lim = tail ? left : 32;
        const int second = n < 2 ? first : (tail ? b0 + kw : b0 + kw + KW);      // (no further block: the last one again)
        // (LDS) the 24 requests of a block, B and A tile 0 first, in four parts
        [[maybe_unused]] auto request = [&](auto ra, auto rb, auto part_) {
            if constexpr (LDS) {
                constexpr int part = decltype(part_)::value;
#pragma unroll
                for (int q = 6 * part; q < 6 * part + 6; ++q) {
                    if (q < 4 * TB)
                        B.request(rb, q);
                    else
                        A.request(ra, q - 4 * TB);
                }
            }
        };
        if constexpr (LDS) {
            const uint32_t at0 = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) char*)x3_smem + (uint32_t)wave * (4096u * (TA + TB));
            A.init(p.A, p.lda, m0, p.M, p.K, lane, at0 + 4096u * TB);
            B.init(p.B, p.ldb, n0 + wn0, p.N, p.K, lane, at0);
            const uintx4 ra = A.at(first), rb = B.at(first);
            static_for<0, 4>([&](auto part) { request(ra, rb, part); });
            asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
            B.read(0, TB);
            A.read(0, TA);
            asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
            request(A.at(second), B.at(second), std::integral_constant<int, 0>{});
        } else {
            A.init(p.A, p.lda, m0, p.M, p.K, lane);
            B.init(p.B, p.ldb, n0 + wn0, p.N, p.K, lane);
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
        if constexpr (!LDS) B.load(B.at(second), 0, 0);
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
        // phase: of A tiles 1, 2, 3 and, for the next step, of B tiles 0, 1 and A tile 0.  Raw values follow as soon as
        // those of both steps (by way of LDS) or of a step are cut: the block behind this one is read from LDS, where it
        // has been on its way for a step, and the one behind that requested; or a step's values are loaded for the step
        // behind the next (B: for the one behind that).
        auto block = [&](auto first_tag, auto a_next, auto b_next, auto a_after, auto b_after) {
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
                    if constexpr (!LDS) {
                        if constexpr (ph == 4) A.load(a_next, j, j);
                        if constexpr (ph == 7) B.load(j ? b_after : b_next, j ^ 1, j ^ 1);
                    } else if constexpr (j == 0) {
                        if constexpr (ph < 3) request(a_next, b_next, std::integral_constant<int, ph + 1>{});
                    } else if constexpr (ph == 0) {
                        asm volatile("s_waitcnt vmcnt(12)" ::: "memory");      // (all but A tiles 1 to 3)
                        B.read(0, TB);
                        A.read(0, 1);
                    } else if constexpr (ph == 4) {
                        asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
                        A.read(1, TA);
                    } else if constexpr (ph == 7) {
                        asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");     // (read out: the LDS is free again)
                        request(a_after, b_after, std::integral_constant<int, 0>{});
                    }
                    products(at[(j + a) % 3], bt[j][b], acc[a][b], cor[a][b]);
                });
            });
            at[0] = at[2];
        };
        int next = n < 3 ? second : second + KW;
        block(std::true_type{}, A.at(second), B.at(second), A.at(next), B.at(next));
        for (int i = 1; i < n; ++i) {
            const int after = i + 2 < n ? next + KW : next;
            block(std::false_type{}, A.at(next), B.at(next), A.at(after), B.at(after));
            next = after;
        }
        if (LDS) asm volatile("s_waitcnt vmcnt(0)" ::: "memory");      // (requested once too often: the sums go there)
    }
    if (!A_KS) __syncthreads();

    // ---- the partial sums meet in LDS, four accumulators of a lane as one word; of the KW wavefronts with the same part of
    // C each finishes TA / KW row tiles: rows TA (8 (e / 4) + 4 half + e % 4) + a, columns 2 l32 and 2 l32 + 1
    floatx4* const meet = x3_smem;
    const bool direct = EPI == EPI_STORE || p.split_k > 1;
    float* const out = p.split_k > 1 ? p.partial + (int64_t)z * p.M * p.N : p.C;
    const int64_t ldo = p.split_k > 1 ? p.N : p.ldc;
    constexpr int AT = TA / KW;
    // C, aux and the partial sums through buffer descriptors that end with the matrix: rows past the last one are not
    // accessed; a column past the last one is read from the next row and not stored
    auto tile_rsrc = [&](const float* P, int64_t ld) {
        const uint64_t at = uniform64(reinterpret_cast<uint64_t>(P) + (uint64_t)(m0 * ld + n0 + wn0) * 4);
        const uint64_t end = uniform64(reinterpret_cast<uint64_t>(P) + (uint64_t)((p.M - 1) * ld + p.N) * 4), left = at < end ? end - at : 0;
        return __builtin_amdgcn_make_buffer_rsrc(reinterpret_cast<void*>(at), 0, left > 0xffffffffu ? 0xffffffffu : (uint32_t)left, 0x00020000);
    };
    auto row_of = [&](int t, int e) { return (uint32_t)(TA * (8 * (e / 4) + 4 * half + e % 4) + AT * kw + t); };
    floatx2 old[EPI == EPI_STORE ? 1 : AT][16];
    float invL = 0.f, th = 0.f;
    if (EPI != EPI_STORE && !direct) {      // (on their way while the sums meet)
        if (EPI == EPI_SHRINK) {
            invL = 1.0f / p.L_ptr[0];
            th = p.lambda * invL;
        }
        const float* src = EPI == EPI_RMW ? p.C : p.aux;
        const Rsrc rs = EPI != EPI_SHRINK || src ? tile_rsrc(src, p.ldc) : __builtin_amdgcn_make_buffer_rsrc(p.C, 0, 0, 0x00020000);   // (null: zeros)
#pragma unroll
        for (int t = 0; t < AT; ++t)
#pragma unroll
            for (int e = 0; e < 16; ++e) {
                const uintx2 v = __builtin_amdgcn_raw_buffer_load_b64(rs, row_of(t, e) * ((uint32_t)p.ldc * 4u) + 4u * TB * l32, 0, 0);
                old[EPI == EPI_STORE ? 0 : t][e] = floatx2{__uint_as_float(v[0]), __uint_as_float(v[1])};
            }
    }
    auto put = [&](auto single_tag) {
#pragma unroll
        for (int a = 0; a < TA; ++a)
#pragma unroll
            for (int b = 0; b < TB; ++b)
#pragma unroll
                for (int q = 0; q < 4; ++q) {
                    floatx4 v;
#pragma unroll
                    for (int e = 0; e < 4; ++e) v[e] = acc[a][b][4 * q + e] + (decltype(single_tag)::value ? 0.f : cor[a][b][4 * q + e]);
                    meet[(((kw * WN + wave % WN) * TA + a) * TB + b) * 256 + q * 64 + lane] = v;
                }
    };
    float sum[AT][16][TB];
    auto get = [&](auto&& take) {
#pragma unroll
        for (int t = 0; t < AT; ++t)
#pragma unroll
            for (int b = 0; b < TB; ++b)
#pragma unroll
                for (int q = 0; q < 4; ++q) {
                    floatx4 v = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
                    for (int k = 0; k < KW; ++k) {
                        const floatx4 w = meet[(((k * WN + wave % WN) * TA + AT * kw + t) * TB + b) * 256 + q * 64 + lane];
                        v = k ? v + w : w;
                    }
#pragma unroll
                    for (int e = 0; e < 4; ++e) take(sum[t][4 * q + e][b], v[e]);
                }
    };
    int* const flag = reinterpret_cast<int*>(x3_smem) + TL::SUMS / 4;
    if (tid == 0) *flag = 0;
    put(std::false_type{});
    __syncthreads();
    bool finite = true;
    get([&](float& s, float v) {
        s = v * UNSCALE;
        finite &= __builtin_fabsf(v) < __builtin_inff();
    });
    if (!finite) *flag = 1;
    __syncthreads();
    if (*flag) {      // such sums are those of fp32 products
        static_for<0, TA>([&](auto a) { static_for<0, TB>([&](auto b) { acc[a][b] = floatx16{}; }); });
        // (the arguments and the lane read again: kept since the start they would take registers from the loop)
        uint64_t args = (uint64_t)__builtin_amdgcn_kernarg_segment_ptr();
        int l = threadIdx.x & 63;
        asm volatile("" : "+s"(args), "+v"(l));
        const auto* q = (const __attribute__((address_space(4))) GemmF32Params*)args;
        const int64_t M = q->M, N = q->N, K = q->K, ka = A_KS ? q->lda : 1, kb = B_KS ? q->ldb : 1;
        const float *pa[TA], *pb[TB];
#pragma unroll
        for (int a = 0; a < TA; ++a) {
            const int64_t r = m0 + TA * (l & 31) + a, row = r < M ? r : M - 1;
            pa[a] = q->A + (A_KS ? row : row * q->lda);
        }
#pragma unroll
        for (int b = 0; b < TB; ++b) {
            const int64_t c = n0 + wn0 + TB * (l & 31) + b, col = c < N ? c : N - 1;
            pb[b] = q->B + (B_KS ? col : col * q->ldb);
        }
        for (int i = 0; i < n; ++i) {
            const int64_t k0 = 32 * (int64_t)(b0 + kw + KW * i);
#pragma unroll 4
            for (int j = 0; j < 32; j += 2) {
                const bool in = k0 + j + (l >> 5) < K;
                const int64_t k = in ? k0 + j + (l >> 5) : K - 1;
                float av[TA], bv[TB];
#pragma unroll
                for (int a = 0; a < TA; ++a) av[a] = pa[a][k * ka];
#pragma unroll
                for (int b = 0; b < TB; ++b) bv[b] = pb[b][k * kb];
#pragma unroll
                for (int a = 0; a < TA; ++a)
#pragma unroll
                    for (int b = 0; b < TB; ++b)
                        acc[a][b] = __builtin_amdgcn_mfma_f32_32x32x2f32(in ? av[a] : 0.f, in ? bv[b] : 0.f, acc[a][b], 0, 0, 0);
            }
        }
        put(std::true_type{});
        __syncthreads();
        get([&](float& s, float v) { s = __builtin_fabsf(s) < __builtin_inff() ? s : v; });
    }
    const Rsrc ro = tile_rsrc(out, ldo);
    const int64_t cols = p.N - (n0 + wn0) - TB * l32;      // (left in the row from this lane's first one)
#pragma unroll
    for (int t = 0; t < AT; ++t)
#pragma unroll
        for (int e = 0; e < 16; ++e) {
            uint32_t r[TB];
#pragma unroll
            for (int b = 0; b < TB; ++b)
                r[b] = __float_as_uint(direct ? sum[t][e][b]
                                              : gemm_combine<EPI>(old[EPI == EPI_STORE ? 0 : t][e][b], sum[t][e][b], p.eta, invL, th));
            const uint32_t at = row_of(t, e) * ((uint32_t)ldo * 4u) + 4u * TB * l32;
            if (cols >= TB)
                __builtin_amdgcn_raw_buffer_store_b64(uintx2{r[0], r[1]}, ro, at, 0, 0);
            else if (cols > 0)
                __builtin_amdgcn_raw_buffer_store_b32(r[0], ro, at, 0, 0);
        }
}

typedef Tile<1, 4> X0;      // 128 x 64
typedef Tile<2, 2> X1;      // 128 x 128
constexpr int NTILES = 2;

template <class TL, bool A_KS, bool B_KS, int EPI>
hipError_t launch_tile(GemmF32Params p, DeviceInfo& dev, int slot, int split, hipStream_t stream)
{
    const int64_t tm = (p.M + TL::BM - 1) / TL::BM, tn = (p.N + TL::BN - 1) / TL::BN;
    if (!dev.gemm_f32x3_lds_set[slot]) {
        hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(&gemm_f32x3_kernel<TL, A_KS, B_KS, EPI>),
                                           hipFuncAttributeMaxDynamicSharedMemorySize, TL::LDS);
        if (e != hipSuccess) return e;
        dev.gemm_f32x3_lds_set[slot] = true;
    }
    const int64_t blocks = (p.K + 31) / 32;
    p.per_split = split > 1 ? (blocks + split - 1) / split : blocks;
    p.split_k = split > 1 ? (int)((blocks + p.per_split - 1) / p.per_split) : 1;      // (no empty split)
    gemm_f32_raster(p, tm, tn, TL::BM, TL::BN, dev);
    hipLaunchKernelGGL((gemm_f32x3_kernel<TL, A_KS, B_KS, EPI>), dim3((unsigned)(tm * tn), (unsigned)p.split_k), dim3(NT), TL::LDS, stream, p);
    hipError_t e = hipGetLastError();
    if (p.parts) *p.parts = p.split_k;
    if (e != hipSuccess || p.split_k <= 1 || p.parts) return e;
    return launch_splitk_reduce(p, EPI, stream);
}

template <bool A_KS, bool B_KS, int EPI>
hipError_t launch_any(const GemmF32Params& p, DeviceInfo& dev, int combo, const GemmF32Plan& plan, hipStream_t stream)
{
    if (plan.tile == 0) return launch_tile<X0, A_KS, B_KS, EPI>(p, dev, combo * NTILES, plan.split, stream);
    return launch_tile<X1, A_KS, B_KS, EPI>(p, dev, combo * NTILES + 1, plan.split, stream);
}

}  // namespace

// Estimated duration (us): the launch (more with the chip full), and rounds of one workgroup per CU, each OWN_US for its
// first loads, meeting and epilogue and STEP_US for every block of 32 of k of a wavefront (less where CUs are idle); a
// k-split pays the traffic of the partial sums and, unless the caller's row kernel adds them up, a second launch.  Fitted to
// 69 shapes of sfb_apply (100 x 100 with 16 pairs to 4096 x 8192 with 3000; rms of the logarithm 4 %); with the estimates of
// the fp32 kernel the plan is within 1.2 % of the best one of all tiles, splits and both kernels in the mean, on 147 others
// within 3 %.  fp32 kernel / this one (us):
//   1000 x 2048, 2048 pairs 77 / 49    4096 x 4096, 2048 483 / 347    1003 x 2047, 800 43 / 25    1024 x 4096, 512 41 / 29.5
//   616 x 2488, 327 19 / 13.8          2090 x 831, 148 15.9 / 11.3    1561 x 5818, 37 34 / 30     284 x 850, 1340 14.8 / 16
//   by way of LDS: 512 x 4096 over 1024 41 / 27.5, 512 x 1024 over 4096 41 / 34 and (k-strided B) 43 / 35 with a k-split of
//   four, 454 x 2559 over 476 21 / 16, 678 x 1365 over 712 17.9 / 18.1, 256 x 1000 over 2048 13.0 / 18.2
//   (loading those lane by lane: 33, 39 and 36 of the first three).
// What is within 5 % stays with the fp32 kernel.
namespace {
constexpr double LAUNCH_US = 1.5, OWN_US[NTILES] = {5.2, 6.8}, STEP_US[NTILES] = {2.3, 2.12}, IDLE_GAIN = 0.2, MARGIN = 0.95;
}  // namespace

// One workgroup on an idle chip, one block of k (8.99 us).
double gemm_f32x3_least_us() { return (LAUNCH_US + OWN_US[0] + STEP_US[0] * (1.0 - IDLE_GAIN)) / MARGIN; }

GemmF32Plan gemm_f32x3_plan(const GemmF32Args& a, int max_split)
{
    GemmF32Plan best = {true, -1, 1, false, 1e30};
    // a whole block of k; 32-bit offsets inside a block and tile
    if (a.K < 32 || a.K > (1LL << 30) || a.lda >= (1LL << 22) || a.ldb >= (1LL << 22) || a.ldc >= (1LL << 22) || a.N >= (1LL << 22)) return best;
    auto aligned = [](const float* P, int64_t ld) { return ld % 4 == 0 && reinterpret_cast<uintptr_t>(P) % 16 == 0; };
    if (!a.a_kstrided && !(aligned(a.A, a.lda) && aligned(a.B, a.ldb))) return best;      // (direct loads)
    const int cus = a.dev->cus > 0 ? a.dev->cus : 256;
    const int64_t blocks = (a.K + 31) / 32;
    for (int t = 0; t < NTILES; ++t) {
        const int64_t bn = t ? X1::BN : X0::BN, kw = t ? X1::KW : X0::KW, tiles = ((a.M + 127) / 128) * ((a.N + bn - 1) / bn);
        if (tiles > 0x7fffffffLL) continue;
        for (int s = 1; s <= max_split; ++s) {
            const int64_t steps = ((blocks + s - 1) / s + kw - 1) / kw, wgs = tiles * s;
            const double idle = wgs < cus ? 1.0 - (double)wgs / cus : 0.0;
            double us = LAUNCH_US + 0.8 * (1.0 - idle) + (double)((wgs + cus - 1) / cus) * (OWN_US[t] + (double)steps * STEP_US[t] * (1.0 - IDLE_GAIN * idle));
            if (s > 1) us += (a.parts ? 0.0 : 3.0) + (double)(s + 1) * (double)a.M * (double)a.N * 4.0 / 6e6;
            if (us < best.us) best = GemmF32Plan{true, t, s, false, us};
        }
    }
    best.us /= MARGIN;
    return best;
}

hipError_t launch_gemm_f32x3(const GemmF32Args& a, GemmF32Params p, const GemmF32Plan& plan, hipStream_t stream)
{
    const bool aks = a.a_kstrided, bks = a.b_kstrided;
    if (!aks && !bks && a.epilogue == EPI_STORE) return launch_any<false, false, EPI_STORE>(p, *a.dev, 0, plan, stream);
    if (!aks && !bks && a.epilogue == EPI_SHRINK) return launch_any<false, false, EPI_SHRINK>(p, *a.dev, 1, plan, stream);
    if (!aks && bks && a.epilogue == EPI_RESID) return launch_any<false, true, EPI_RESID>(p, *a.dev, 2, plan, stream);
    if (aks && bks && a.epilogue == EPI_RMW) return launch_any<true, true, EPI_RMW>(p, *a.dev, 3, plan, stream);
    return hipErrorInvalidValue;
}

}  // namespace sfb
