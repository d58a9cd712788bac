// fp32 MFMA GEMM family for gfx950 (v_mfma_f32_16x16x4_f32), used by every
// fp32 workload: MLR logits, DML projections, the two ISTA contractions of
// sparse coding, and the reconstruction + application of the SF sum.  It keeps the
// contractions of less than some 10 us, the ones with a k below 32 and the k-contiguous
// ones off 16-byte alignment; the larger ones go to the bf16 matrix instructions on three
// terms per value (gemm_f32x3.hip) wherever the two cost models find that faster.
//
//   acc[m][n] = sum_k A(m,k) * B(n,k)
//
// Either operand may be k-contiguous ([rows][k], e.g. W[J][D] against the
// feature index) or k-strided ([k][rows], e.g. the SF matrices U[N][J], V[N][D]
// against the SF index), so "U^T V" needs no transposed copy: a k-strided tile
// is kept in LDS as it sits in memory.
//
// One workgroup of eight wavefronts (two per SIMD) owns one output tile; where its
// walk over k is short, several workgroups share a CU.  Operands go from global memory
// straight into LDS, several k-slices ahead; the wavefronts divide the tile between
// them, and the k of every slice two, four or eight ways (their partial sums meet in
// LDS at the end), so that a contraction with few outputs and a long k fills the chip
// in one launch.
//
// What bounds it (MI355X, us of one launch in a row of dependent ones; in front of the
// arrow the kernel this one replaced: four wavefronts of 32x32x2 MFMAs, a k-split over
// workgroups with a second launch, rows off 16-byte alignment through a scalar path):
//   256 x 1000 x 2048                        21 -> 12
//   100 x 1000 x 300                         14 -> 4.9  launch, first loads, epilogue; two workgroups share a CU
//   100 x 300 x 1000                         14 -> 5.7
//   100 x 1003 x 2047 (nothing aligned)      20 -> 14
// and, where it ran before gemm_f32x3.hip took them (now 48, 29, 34 and 25 us),
//   1000 x 2048 x 2048 (both k-strided)      92 -> 74   64.7 us in the k-loop (54.5 at 2.4 GHz; the clock is 2.2
//                                                       in kernels this short), 2.3 first loads, 2.5 epilogue
//   512 x 4096 x 1024  (both k-contiguous)   45 -> 40   32 in the loop, 27.9 at 2.4 GHz
//   512 x 1024 x 4096  (k-contiguous x strided) 47 -> 43   k divided inside the workgroup, no second launch
//   1003 x 2047 x 800 (nothing aligned)      60 -> 41
// 16x16x4 MFMAs rather than 32x32x2: in a kernel of 60 us a loop of nothing but MFMAs on
// random operands runs at 2.40 GHz with the former and 2.23 with the latter.  Two
// wavefronts per SIMD hide each other's LDS latency, barriers and load issue: a launch of
// 1000 x 2048 x 2048 without any loads or reads in its loop takes 68 instead of 74 us.
#include "gemm_f32.h"

#include <cmath>
#include <type_traits>

namespace sfb {
namespace {

typedef float floatx4 __attribute__((ext_vector_type(4)));

constexpr int NWAVES = 8, NT = 64 * NWAVES;
constexpr int LDS_CU = 160 * 1024, LDS_MAX = 152 * 1024;      // of a CU; of one workgroup

typedef GemmF32Params Params;

// A workgroup tile of BM x BN, WM x WN wavefronts over it and KW (at least two) over k: each wavefront multiplies a block
// of 16 TA x 16 TB over its 16 of the KB = 16 KW values of k of a slice.
template <int BM_, int BN_, int WM_, int WN_, int KW_, int MAX_NS = 5>
struct Tile {
    static constexpr int BM = BM_, BN = BN_, WM = WM_, WN = WN_, KW = KW_, KB = 16 * KW;
    static constexpr int TA = BM / WM / 16, TB = BN / WN / 16;  // 16 x 16 MFMA tiles of a wavefront
    static constexpr int A_BYTES = BM * KB * 4, B_BYTES = BN * KB * 4, STAGE = A_BYTES + B_BYTES;
    static constexpr int MEET = NWAVES * TA * TB * 1024;                   // LDS of the partial sums
    static constexpr int NS = LDS_MAX / STAGE < MAX_NS ? LDS_MAX / STAGE : MAX_NS;   // LDS stages
    static constexpr int NSR = NS > 5 ? NS : 3;                            // the same where slices wait in registers first
    // LDS of a workgroup that walks n slices: a short walk does not use all stages
    static constexpr int stages(bool direct) { return direct ? NS : NSR; }
    static constexpr int lds(bool direct, int64_t n)
    {
        const int used = (n < stages(direct) ? (int)n : stages(direct)) * STAGE;
        return used > MEET ? used : MEET;
    }
    static_assert(WM * WN * KW == NWAVES && KW % 2 == 0 && NS >= 3 && MEET <= LDS_MAX, "tile");
};

// LDS image of one operand's slice (ROWS x KB floats):
//   k-contiguous: per 32 of k, ROWS rows of 32 floats (128 bytes), the eight 16-byte chunks of row r XOR-swizzled by
//     (r ^ r / 8) & 7, so that the 16-byte fragment reads of 16 consecutive rows meet every bank once;
//   k-strided: [k][rows] as in memory; a fragment is four reads of T consecutive floats.
// MFMA tile x, lane l of a wavefront's block of 16 T rows is row T l + x of the block in both images (LDS row 16 x + l
// of a k-contiguous block holds it): a lane's T columns of C are neighbours and its fragments of a k-strided operand
// one read.  Rows past the end of the matrix are clamped (they feed accumulators that are not stored).
template <int T>
__device__ __forceinline__ int tile_row(int r) { return (r / (16 * T)) * (16 * T) + T * (r % 16) + (r % (16 * T)) / 16; }

// T consecutive floats, at any float of global memory.
template <int T> struct Vec;
template <> struct Vec<1> { typedef float type __attribute__((ext_vector_type(1), aligned(4))); };
template <> struct Vec<2> { typedef float type __attribute__((ext_vector_type(2), aligned(4))); };
template <> struct Vec<4> { typedef float type __attribute__((ext_vector_type(4), aligned(4))); };

// Which 16 bytes of the operand lane `lane` of 1 KB unit u of a slice takes: row (k-contiguous) or k (k-strided) and the
// first of four floats along the other index, relative to the tile and the slice.
template <int ROWS, bool KS, int T>
__device__ __forceinline__ void unit_place(int u, int lane, int& row, int& k)
{
    if (KS) {
        const int f = 256 * u + 4 * lane;
        k = f / ROWS;
        row = f % ROWS;
    } else {
        const int r = 8 * (u % (ROWS / 8)) + (lane >> 3);
        row = tile_row<T>(r);
        k = 32 * (u / (ROWS / 8)) + 4 * ((lane & 7) ^ swz(r));
    }
}

// Direct loads of one operand whose rows are 16-byte aligned.
template <int ROWS, int KB, bool KS, int T>
struct DirectLoader {
    static constexpr int L = ROWS * KB * 4 / 1024 / NWAVES;
    static_assert(L * 1024 * NWAVES == ROWS * KB * 4, "loads per wavefront");
    uint64_t base[L];      // uniform: the address of the unit's first row and k
    uint32_t voff[L];
    uint64_t step;

    __device__ __forceinline__ void init(const float* P, int64_t ld, int64_t row0, int64_t rows, int64_t k0, int wave, int lane)
    {
        step = (uint64_t)(KS ? KB * ld : KB) * 4;
#pragma unroll
        for (int i = 0; i < L; ++i) {
            int r, k, r_first, k_first;
            unit_place<ROWS, KS, T>(L * wave + i, lane, r, k);
            if (KS) {
                k_first = 256 * (L * wave + i) / ROWS;
                int64_t m = row0 + r;
                if (m + 4 > rows) m = rows - 4;               // (rows % 4 == 0 and rows >= 4 here)
                base[i] = uniform64(reinterpret_cast<uint64_t>(P) + (uint64_t)((k0 + k_first) * ld + row0) * 4);
                voff[i] = (uint32_t)((k - k_first) * ld * 4) + (uint32_t)((m - row0) * 4);
            } else {
                r_first = tile_row<T>(8 * ((L * wave + i) % (ROWS / 8)));
                k_first = 32 * ((L * wave + i) / (ROWS / 8));
                int64_t br = row0 + r_first, gr = row0 + r;
                if (br >= rows) br = rows - 1;
                if (gr >= rows) gr = rows - 1;
                base[i] = uniform64(reinterpret_cast<uint64_t>(P) + (uint64_t)(br * ld + k0 + k_first) * 4);
                voff[i] = (uint32_t)((gr - br) * ld * 4) + (uint32_t)((k - k_first) * 4);
            }
        }
    }
    __device__ __forceinline__ void issue(int i, uint32_t dst, int wave)
    {
        load_to_lds_16(dst + (uint32_t)(L * wave + i) * 1024u, base[i], voff[i]);
        base[i] += step;
    }
};

// The same for rows at any alignment: 16-byte loads at 4-byte alignment into registers, then to LDS.  (Direct loads of
// 4 bytes a lane, the alternative, keep the address unit busy four times as long per byte.)
template <int ROWS, int KB, bool KS, int T>
struct RegLoader {
    static constexpr int L = ROWS * KB * 4 / 1024 / NWAVES;
    uint64_t at[L];        // the lane's own address
    int shift[L];          // k-strided, last rows: the four floats are loaded `shift` floats early (they end with the row)
    uint64_t step;
    int last;              // k-strided with fewer than four rows in all: the last row (float by float); otherwise -1

    __device__ __forceinline__ void init(const float* P, int64_t ld, int64_t row0, int64_t rows, int64_t k0, int wave, int lane)
    {
        step = (uint64_t)(KS ? KB * ld : KB) * 4;
        last = KS && rows < 4 ? (int)rows - 1 : -1;
#pragma unroll
        for (int i = 0; i < L; ++i) {
            int r, k;
            unit_place<ROWS, KS, T>(L * wave + i, lane, r, k);
            int64_t m = row0 + r;
            shift[i] = 0;
            if (KS && last < 0) {
                if (m >= rows) m = rows - 1;
                if (m + 4 > rows) {
                    shift[i] = (int)(m + 4 - rows);
                    m = rows - 4;
                }
            } else if (m >= rows) {
                m = KS ? 0 : rows - 1;
            }
            at[i] = reinterpret_cast<uint64_t>(P) + (uint64_t)(KS ? (k0 + k) * ld + m : m * ld + k0 + k) * 4;
        }
    }
    __device__ __forceinline__ floatx4 fetch(int i)
    {
        const float* src = reinterpret_cast<const float*>(at[i]);
        at[i] += step;
        if (KS && last >= 0) return floatx4{src[0], src[last < 1 ? last : 1], src[last < 2 ? last : 2], src[last]};
        const typename Vec<4>::type v = *reinterpret_cast<const typename Vec<4>::type*>(src);
        return floatx4{v[0], v[1], v[2], v[3]};
    }
    __device__ __forceinline__ void store(int i, char* dst, int wave, int lane, floatx4 v) const
    {
        if (KS) {
            const bool one = shift[i] & 1, two = shift[i] & 2;
            const float a0 = one ? v[1] : v[0], a1 = one ? v[2] : v[1], a2 = one ? v[3] : v[2], a3 = v[3];
            v = floatx4{two ? a2 : a0, two ? a3 : a1, a2, a3};
        }
        *reinterpret_cast<floatx4*>(dst + (L * wave + i) * 1024 + lane * 16) = v;
    }
};

// The values of a partial slice (k0 .. K) that this thread puts into LDS itself, zero past K.
template <int ROWS, int KB, bool KS, int T>
struct TailPart {
    static_assert(ROWS * KB % NT == 0, "whole parts");
    static constexpr int PER = ROWS * KB / NT;
    float v[PER];
    __device__ __forceinline__ void fetch(const float* P, int64_t ld, int64_t row0, int64_t rows, int64_t k0, int64_t K, int tid)
    {
#pragma unroll
        for (int i = 0; i < PER; ++i) {
            const int f = tid + NT * i;
            const int kk = KS ? f / ROWS : (f / (ROWS * 32)) * 32 + f % 32;
            int64_t row = row0 + (KS ? f % ROWS : tile_row<T>((f / 32) % ROWS));
            if (row >= rows) row = rows - 1;
            v[i] = k0 + kk < K ? P[KS ? (k0 + kk) * ld + row : row * ld + k0 + kk] : 0.f;
        }
    }
    __device__ __forceinline__ void store(char* dst, int tid) const
    {
#pragma unroll
        for (int i = 0; i < PER; ++i) {
            const int f = tid + NT * i, r = (f / 32) % ROWS, pos = f % 32;
            const int at = KS ? f : (f / 32) * 32 + (((pos >> 2) ^ swz(r)) << 2) + (pos & 3);
            *reinterpret_cast<float*>(dst + at * 4) = v[i];
        }
    }
};

template <class TL, bool A_KS, bool B_KS, int EPI, bool DIRECT>
__global__ __launch_bounds__(NT, 2) void gemm_f32_kernel(Params p)
{
    constexpr int BM = TL::BM, BN = TL::BN, WM = TL::WM, WN = TL::WN, KW = TL::KW, KB = TL::KB;
    constexpr int TA = TL::TA, TB = TL::TB, STAGE = TL::STAGE, A_BYTES = TL::A_BYTES, NS = DIRECT ? TL::NS : TL::NSR;
    extern __shared__ floatx4 gemm_smem[];
    char* const lds = reinterpret_cast<char*>(gemm_smem);
    const uint32_t lds_base = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) char*)gemm_smem;

    const int tid = threadIdx.x, lane = tid & 63, l16 = lane & 15, quad = lane >> 4;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int kw = wave / (WM * WN), wm0 = ((wave / WN) % WM) * (16 * TA), wn0 = (wave % WN) * (16 * TB);

    uint32_t tile_m, tile_n;
    gemm_tile_of(p, tile_m, tile_n);
    const int64_t m0 = (int64_t)tile_m * BM, n0 = (int64_t)tile_n * BN;
    const int64_t z = blockIdx.y;
    // slices of this workgroup: the whole ones [k_first, k_end) and, for the last split, the partial one, which comes
    // first (stage 0, through registers, under the latency of the direct loads of the others)
    const int64_t whole = p.K / KB, all = (p.K + KB - 1) / KB;
    const int64_t k_first = p.split_k > 1 ? z * p.per_split : 0;
    int64_t k_end = p.split_k > 1 ? k_first + p.per_split : all;
    const bool tail = k_end >= all && all > whole;
    if (k_end > whole) k_end = whole;
    const int64_t n = (k_end > k_first ? k_end - k_first : 0) + (tail ? 1 : 0);

    floatx4 acc[TA][TB];
#pragma unroll
    for (int a = 0; a < TA; ++a)
#pragma unroll
        for (int b = 0; b < TB; ++b) acc[a][b] = floatx4{0.f, 0.f, 0.f, 0.f};

    // ---- fragments of a slice: this wavefront's 16 k are 16 kw .. + 15; lane quad q owns k = 4 q + e, the e-th MFMA
    // takes element e of all four
    struct Frag {
        float a[TA][4], b[TB][4];
    };
    uint32_t ra[A_KS ? 1 : TA], rb[B_KS ? 1 : TB];
    if (A_KS) {
        ra[0] = (uint32_t)((16 * kw + 4 * quad) * BM + wm0 + TA * l16) * 4u;
    } else {
#pragma unroll
        for (int x = 0; x < TA; ++x) {
            const int r = wm0 + 16 * x + l16;
            ra[A_KS ? 0 : x] = (uint32_t)((kw / 2) * (BM * 128) + r * 128 + (((4 * (kw & 1) + quad) ^ swz(r)) << 4));
        }
    }
    if (B_KS) {
        rb[0] = (uint32_t)(A_BYTES + ((16 * kw + 4 * quad) * BN + wn0 + TB * l16) * 4);
    } else {
#pragma unroll
        for (int x = 0; x < TB; ++x) {
            const int r = wn0 + 16 * x + l16;
            rb[B_KS ? 0 : x] = (uint32_t)(A_BYTES + (kw / 2) * (BN * 128) + r * 128 + (((4 * (kw & 1) + quad) ^ swz(r)) << 4));
        }
    }
    constexpr int NRA = A_KS ? 4 : TA, NRB = B_KS ? 4 : TB, NR = NRA + NRB;   // LDS reads per slice
    auto read_op = [&](const char* stage, int q, Frag& f) {    // q: a constant after unrolling
        if (q < NRA) {
            if (A_KS) {
                typedef float V __attribute__((ext_vector_type(TA)));
                const V v = *reinterpret_cast<const V*>(stage + ra[0] + q * (BM * 4));
#pragma unroll
                for (int x = 0; x < TA; ++x) f.a[x][A_KS ? q : 0] = v[x];
            } else {
                const floatx4 v = *reinterpret_cast<const floatx4*>(stage + ra[A_KS ? 0 : q]);
#pragma unroll
                for (int e = 0; e < 4; ++e) f.a[A_KS ? 0 : q][e] = v[e];
            }
        } else {
            const int qq = q - NRA;
            if (B_KS) {
                typedef float V __attribute__((ext_vector_type(TB)));
                const V v = *reinterpret_cast<const V*>(stage + rb[0] + qq * (BN * 4));
#pragma unroll
                for (int x = 0; x < TB; ++x) f.b[x][B_KS ? qq : 0] = v[x];
            } else {
                const floatx4 v = *reinterpret_cast<const floatx4*>(stage + rb[B_KS ? 0 : qq]);
#pragma unroll
                for (int e = 0; e < 4; ++e) f.b[B_KS ? 0 : qq][e] = v[e];
            }
        }
    };

    typename std::conditional<DIRECT, DirectLoader<BM, KB, A_KS, TA>, RegLoader<BM, KB, A_KS, TA>>::type la;
    typename std::conditional<DIRECT, DirectLoader<BN, KB, B_KS, TB>, RegLoader<BN, KB, B_KS, TB>>::type lb;
    constexpr int LA = decltype(la)::L, LB = decltype(lb)::L, LL = LA + LB;
    [[maybe_unused]] auto issue_one = [&](int i, int stage) {
        if constexpr (DIRECT) {
            const uint32_t dst = lds_base + (uint32_t)stage * STAGE;
            if (i < LA)
                la.issue(i, dst, wave);
            else
                lb.issue(i - LA, dst + A_BYTES, wave);
        }
    };
    [[maybe_unused]] floatx4 held[2][DIRECT ? 1 : LL];       // (not DIRECT) the next two slices to go to LDS, on their way
    [[maybe_unused]] auto fetch_one = [&](int i) -> floatx4 {
        if constexpr (DIRECT)
            return floatx4{};
        else
            return i < LA ? la.fetch(i < LA ? i : 0) : lb.fetch(i < LA ? 0 : i - LA);
    };
    [[maybe_unused]] auto store_one = [&](int i, int stage, floatx4 v) {
        if constexpr (!DIRECT) {
            if (i < LA)
                la.store(i < LA ? i : 0, lds + stage * STAGE, wave, lane, v);
            else
                lb.store(i < LA ? 0 : i - LA, lds + stage * STAGE + A_BYTES, wave, lane, v);
        }
    };

    // Slice s lives in stage s % NS and is multiplied in two halves (elements 0, 1 and 2, 3 of the fragments).
    // Between them every wavefront waits until slice s + 1 has landed and meets the others: after that barrier the
    // stage of slice s - 1 is free (the loads of slice s + NS - 1 go there) and the fragments of slice s + 1 can be
    // read, so that the MFMA pipe does not drain at a slice boundary.  Direct loads complete in order: "slice s + 1
    // has landed" = at most the loads of the NS - 3 slices after it are outstanding.  (Through registers: slice
    // s + NS - 1, requested two slices earlier, is written to that stage, and slice s + NS + 1 requested.)  Reads and loads
    // follow the MFMAs one at a time (a burst of loads blocks the wavefront in the memory-issue stage); the order is
    // pinned.
    constexpr int HM = 2 * TA * TB;
    auto mfma = [&](const Frag& f, int j) {
        const int e = j / (TA * TB), a = (j / TB) % TA, b = j % TB;
        acc[a][b] = __builtin_amdgcn_mfma_f32_16x16x4f32(f.a[a][e], f.b[b][e], acc[a][b], 0, 0, 0);
    };
    // FEED 2: everything above; 1: write the held slice, request none; 0: no slice left to bring
    auto slice = [&](const Frag& cur, Frag& next, floatx4* hold, int st, int st_next, auto feed_tag) {
        constexpr int FEED = decltype(feed_tag)::value, OVER = DIRECT ? HM : HM / 2;
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int j = 0; j < HM; ++j) mfma(cur, j);
        __builtin_amdgcn_sched_barrier(0);
        if (DIRECT && FEED)
            asm volatile("s_waitcnt vmcnt(%0)" ::"n"((NS - 3) * LL) : "memory");
        else if (DIRECT)
            asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
        __syncthreads();
        const char* nxt = lds + st_next * STAGE;
        const int st_load = st >= 1 ? st - 1 : NS - 1;
#pragma unroll
        for (int j = 0; j < HM; ++j) {
            mfma(cur, HM + j);
#pragma unroll
            for (int q = j * NR / (HM / 2); q < (j + 1) * NR / (HM / 2) && q < NR; ++q) read_op(nxt, q, next);
            if (FEED) {
#pragma unroll
                for (int q = j * LL / OVER; q < (j + 1) * LL / OVER && q < LL; ++q) {
                    if (DIRECT) {
                        issue_one(q, st_load);
                    } else {
                        store_one(q, st_load, hold[DIRECT ? 0 : q]);
                        if (FEED == 2) hold[DIRECT ? 0 : q] = fetch_one(q);
                    }
                }
            }
            __builtin_amdgcn_sched_barrier(0);
        }
    };

    // ---- epilogue units: EU accumulator registers e of one a (rows TA (4 quad + e) + a of the wavefront's block) and
    // all TB tiles along n (columns TB l16 .. + TB - 1); the KW wavefronts of a block share its units
    constexpr int EU = TA >= KW ? 4 : (2 * TA >= KW ? 2 : 1), UNITS = TA * 4 / EU, PER = (UNITS + KW - 1) / KW;
    typedef typename Vec<TB>::type VecC;
    float* const out = p.split_k > 1 ? p.partial + z * p.M * p.N : p.C;
    const int64_t ldo = p.split_k > 1 ? p.N : p.ldc;
    const int64_t col = n0 + wn0 + TB * l16;
    const bool direct = EPI == EPI_STORE || p.split_k > 1;
    constexpr int PO = EPI == EPI_STORE ? 1 : PER;
    float old[PO][EU][TB];
    auto unit_row = [&](int unit, int e) { return m0 + wm0 + TA * (4 * quad + (unit % (4 / EU)) * EU + e) + unit / (4 / EU); };
    auto load_old = [&]() {
        if (direct) return;
        const float* src = EPI == EPI_RMW ? p.C : p.aux;      // (EPI_SHRINK, null: zeros)
#pragma unroll
        for (int i = 0; i < PO; ++i) {
            const int unit = kw * PER + i;
#pragma unroll
            for (int e = 0; e < EU; ++e) {
                const int64_t row = unit_row(unit, e);
#pragma unroll
                for (int b = 0; b < TB; ++b) old[i][e][b] = 0.f;
                if (unit < UNITS && row < p.M && (EPI != EPI_SHRINK || src)) {
                    const float* s = src + row * p.ldc + col;
                    if (col + TB <= p.N) {
                        const VecC v = *reinterpret_cast<const VecC*>(s);
#pragma unroll
                        for (int b = 0; b < TB; ++b) old[i][e][b] = v[b];
                    } else {
#pragma unroll
                        for (int b = 0; b < TB; ++b)
                            if (col + b < p.N) old[i][e][b] = s[b];
                    }
                }
            }
        }
    };

    if (n > 0) {
        const int64_t k0 = k_first * KB;
        la.init(p.A, p.lda, m0, p.M, k0, wave, lane);
        lb.init(p.B, p.ldb, n0, p.N, k0, wave, lane);
        auto bring = [&](int first) {      // slices first .. NS - 2 on their way, and (through registers) NS - 1 and NS held
            if constexpr (DIRECT) {
#pragma unroll
                for (int s = 0; s < NS - 1; ++s)
                    if (s >= first && s < n) {
#pragma unroll
                        for (int i = 0; i < LL; ++i) issue_one(i, s);
                    }
            } else {
                floatx4 early[NS - 1][LL];
#pragma unroll
                for (int s = 0; s < NS + 1; ++s)
                    if (s >= first && s < n) {
#pragma unroll
                        for (int i = 0; i < LL; ++i) {
                            if (s < NS - 1)
                                early[s < NS - 1 ? s : 0][i] = fetch_one(i);
                            else
                                held[(s - NS + 1) & 1][i] = fetch_one(i);
                        }
                    }
#pragma unroll
                for (int s = 0; s < NS - 1; ++s)
                    if (s >= first && s < n) {
#pragma unroll
                        for (int i = 0; i < LL; ++i) store_one(i, s, early[s][i]);
                    }
            }
        };
        if (tail) {
            TailPart<BM, KB, A_KS, TA> ta;
            TailPart<BN, KB, B_KS, TB> tb;
            ta.fetch(p.A, p.lda, m0, p.M, whole * KB, p.K, tid);
            tb.fetch(p.B, p.ldb, n0, p.N, whole * KB, p.K, tid);
            bring(1);
            ta.store(lds, tid);
            tb.store(lds + A_BYTES, tid);
        } else {
            bring(0);
            if (DIRECT && n >= NS - 1)
                asm volatile("s_waitcnt vmcnt(%0)" ::"n"((NS - 2) * LL) : "memory");
            else if (DIRECT)
                asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
        }
        __syncthreads();
        Frag f0, f1;
#pragma unroll
        for (int q = 0; q < NR; ++q) read_op(lds, q, f0);
        int st = 0;
        auto next_of = [](int x) { return x + 1 == NS ? 0 : x + 1; };
        typedef std::integral_constant<int, 2> Feed;
        int64_t s = 0;
        const int64_t feeds = n - NS - (DIRECT ? 0 : 2);       // slices 0 .. feeds bring another one
        for (; s < feeds; s += 2) {
            const int s1 = next_of(st), s2 = next_of(s1);
            slice(f0, f1, held[0], st, s1, Feed{});
            slice(f1, f0, held[1], s1, s2, Feed{});
            st = s2;
        }
        auto single = [&](auto feed_tag) {
            slice(f0, f1, held[0], st, next_of(st), feed_tag);
            f0 = f1;
            if (!DIRECT) {
#pragma unroll
                for (int i = 0; i < LL; ++i) {
                    const floatx4 t = held[0][DIRECT ? 0 : i];
                    held[0][DIRECT ? 0 : i] = held[1][DIRECT ? 0 : i];
                    held[1][DIRECT ? 0 : i] = t;
                }
            }
            st = next_of(st);
            ++s;
        };
        if (s <= feeds) single(Feed{});
        if (!DIRECT)
            while (s + NS - 1 < n) single(std::integral_constant<int, 1>{});
        while (s + 1 < n) single(std::integral_constant<int, 0>{});
        load_old();      // (their latency runs under the last slice)
#pragma unroll
        for (int j = 0; j < 2 * HM; ++j) mfma(f0, j);
    } else {
        load_old();
    }

    float invL = 0.f, th = 0.f;
    if (EPI == EPI_SHRINK) {
        invL = 1.0f / p.L_ptr[0];
        th = p.lambda * invL;
    }
    // partial sums: EU floats a lane per (tile, unit of it), added in the order of kw
    typedef float VecE __attribute__((ext_vector_type(EU)));
    VecE* const meet = reinterpret_cast<VecE*>(gemm_smem);
    __syncthreads();
#pragma unroll
    for (int t = 0; t < TA * TB; ++t)
#pragma unroll
        for (int q = 0; q < 4 / EU; ++q) {
            VecE v;
#pragma unroll
            for (int e = 0; e < EU; ++e) v[e] = acc[t / TB][t % TB][q * EU + e];
            meet[((wave * TA * TB + t) * (4 / EU) + q) * 64 + lane] = v;
        }
    __syncthreads();
#pragma unroll
    for (int i = 0; i < PER; ++i) {
        const int unit = kw * PER + i;
        if (unit >= UNITS) break;
        float v[TB][EU];
#pragma unroll
        for (int b = 0; b < TB; ++b) {
            const int w0 = wave % (WM * WN), t = unit / (4 / EU) * TB + b, q = unit % (4 / EU);
            VecE sum = meet[((w0 * TA * TB + t) * (4 / EU) + q) * 64 + lane];
#pragma unroll
            for (int k = 1; k < KW; ++k) sum += meet[(((w0 + k * WM * WN) * TA * TB + t) * (4 / EU) + q) * 64 + lane];
#pragma unroll
            for (int e = 0; e < EU; ++e) v[b][e] = sum[e];
        }
#pragma unroll
        for (int e = 0; e < EU; ++e) {
            const int64_t row = unit_row(unit, e);
            if (row >= p.M) continue;
            float r[TB];
#pragma unroll
            for (int b = 0; b < TB; ++b)
                r[b] = direct ? v[b][e] : gemm_combine<EPI>(old[EPI == EPI_STORE ? 0 : i][e][b], v[b][e], p.eta, invL, th);
            float* dst = out + row * ldo + col;
            if (col + TB <= p.N) {
                VecC w;
#pragma unroll
                for (int b = 0; b < TB; ++b) w[b] = r[b];
                *reinterpret_cast<VecC*>(dst) = w;
            } else {
#pragma unroll
                for (int b = 0; b < TB; ++b)
                    if (col + b < p.N) dst[b] = r[b];
            }
        }
    }
}

// Sum of the k-splits in index order, then the epilogue; four columns of a row a thread.
template <int EPI>
__global__ __launch_bounds__(256) void splitk_reduce_kernel(Params p)
{
    typedef typename Vec<4>::type V;
    float invL = 0.f, th = 0.f;
    if (EPI == EPI_SHRINK) {
        invL = 1.0f / p.L_ptr[0];
        th = p.lambda * invL;
    }
    const int64_t groups = (p.N + 3) / 4, total = p.M * groups, plane = p.M * p.N, stride = (int64_t)gridDim.x * 256;
    const float* aux = EPI == EPI_RMW ? p.C : p.aux;      // (EPI_SHRINK, null: zeros)
    for (int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x; i < total; i += stride) {
        // (a 32-bit division where that is enough)
        const int64_t row = total <= 0xffffffffLL ? (int64_t)((uint32_t)i / (uint32_t)groups) : i / groups, col = 4 * (i - row * groups);
        const float* src = p.partial + row * p.N + col;
        float* dst = p.C + row * p.ldc + col;
        if (col + 4 <= p.N) {
            V old = {0.f, 0.f, 0.f, 0.f};
            if (EPI != EPI_STORE && (EPI != EPI_SHRINK || aux)) old = *reinterpret_cast<const V*>(aux + row * p.ldc + col);
            V sum = *reinterpret_cast<const V*>(src);
#pragma unroll 4
            for (int z = 1; z < p.split_k; ++z) sum += *reinterpret_cast<const V*>(src + z * plane);
#pragma unroll
            for (int c = 0; c < 4; ++c) sum[c] = gemm_combine<EPI>(old[c], sum[c], p.eta, invL, th);
            *reinterpret_cast<V*>(dst) = sum;
        } else {
            for (int c = 0; col + c < p.N; ++c) {
                float sum = src[c];
                for (int z = 1; z < p.split_k; ++z) sum += src[z * plane + c];
                const float old = EPI == EPI_STORE || (EPI == EPI_SHRINK && !aux) ? 0.f : aux[row * p.ldc + col + c];
                dst[c] = gemm_combine<EPI>(old, sum, p.eta, invL, th);
            }
        }
    }
}

// ---- tile shape and k-split by a small cost model ----
typedef Tile<128, 128, 2, 2, 2> T0;
typedef Tile<128, 64, 2, 2, 2> T1;
typedef Tile<64, 64, 2, 1, 4> T2;
typedef Tile<64, 32, 2, 1, 4> T3;
typedef Tile<32, 32, 1, 1, 8> T4;
typedef Tile<16, 16, 1, 1, 8, 9> T5;
constexpr int NTILES = 6;

// Estimated duration (us) of a contraction as `rounds` of one workgroup per CU, each walking its k-slices.  Per tile
// shape: us per slice with every CU busy, and us per tile beside the slices (first loads, partial sums, epilogue).
// Measured (direct, us of one launch, 2.5 of them between dependent launches): 1000 x 2048 x 2048 73 with T1, 78 T2,
// 89 T3, 100 T4; 256 x 1000 x 2048 12.0 T4, 20.5 T3, 20.7 T5, 16 T3 split in two; 100 x 300 x 1000 5.7 T5, 9.4 T4,
// 13 T3; 4096 x 4096 x 1024 260 T0, 283 T1.  The smallest tile waits for memory rather than for the matrix pipes, and
// waits less where it leaves CUs idle.
// A contraction of few slices needs less LDS, and several workgroups share a CU where registers allow it: each takes
// longer (`share` of its time per neighbour), the round of all of them less.  Measured (us of sfb_apply, one workgroup
// per CU / several, with the same tile): 16 x 100000 with 100 pairs 55 / 22 T5, 32 x 200000 with 256 103 / 66 T4,
// 100000 x 16 with 100 34 / 20 T3, 5000 x 3000 with 10 49 / 35 T1.
// The sum of a k-split is a launch of its own or, where the caller's row kernel adds the parts up (GemmF32Args::parts), the
// traffic and a microsecond: 209 shapes of logits and 169 of projections (16 to 700 samples) are 1.4 and 1.2 % faster in the mean
// than with the cost of the launch (22 x 20 over 6615 20.7 / 13.5, 64 x 624 over 5496 18.2 / 15.2; 104 x 520 over 4200
// 13.5 / 14.9), those that the kernel on three bf16 terms takes among them.
struct TileCost {
    double slice_us, tile_us, idle_gain, share;
    int wgs;       // workgroups a CU has registers for
};
template <class TL>
double plan_time(int64_t M, int64_t N, int64_t K, int cus, int s, bool direct, bool parts, const TileCost& c)
{
    const int64_t tiles = ((M + TL::BM - 1) / TL::BM) * ((N + TL::BN - 1) / TL::BN) * s, nk = (K + TL::KB - 1) / TL::KB;
    const int64_t slices = s > 1 ? (nk + s - 1) / s : nk;
    double slice_us = c.slice_us, rounds = 1.0, together = 1.0;
    if (tiles < cus) {
        slice_us *= 1.0 - c.idle_gain * (1.0 - (double)tiles / (double)cus);
    } else {
        int64_t wgs = 1;
        const int used = TL::lds(direct, slices);
        if (used < TL::lds(direct, TL::stages(direct))) {
            const int64_t per_cu = (tiles + cus - 1) / cus;
            wgs = LDS_CU / used < c.wgs ? LDS_CU / used : c.wgs;
            if (wgs > per_cu) wgs = per_cu;
        }
        rounds = (double)((tiles + cus * wgs - 1) / (cus * wgs));
        together += c.share * (double)(wgs - 1);
    }
    double t = 2.5 + rounds * ((double)slices * slice_us + c.tile_us) * together;
    if (s > 1) t += (parts ? 1.0 : 4.5) + (double)(s + 1) * (double)M * (double)N * 4.0 / 3e6;      // the second pass
    return t;
}

GemmF32Plan plan_gemm(int64_t M, int64_t N, int64_t K, int cus, int max_split, bool direct, bool parts)
{
    static const TileCost costs[2][NTILES] = {
        {{2.10, 6.5, 0.05, 0.0, 1}, {1.22, 5.0, 0.05, 0.5, 1}, {1.25, 4.7, 0.1, 0.3, 1}, {0.69, 3.5, 0.2, 0.2, 2}, {0.80, 3.0, 0.0, 0.3, 2}, {0.40, 1.2, 1.0, 0.35, 2}},
        {{1.82, 6.5, 0.05, 0.0, 1}, {1.01, 5.0, 0.05, 0.5, 2}, {1.03, 4.7, 0.1, 0.3, 2}, {0.55, 3.5, 0.2, 0.2, 3}, {0.55, 3.0, 0.0, 0.3, 3}, {0.38, 1.2, 1.0, 0.35, 4}}};
    const TileCost* const c = costs[direct ? 1 : 0];
    GemmF32Plan best = {false, 0, 1, direct, 1e30};
    for (int s = 1; s <= max_split; ++s) {
        const double t[NTILES] = {plan_time<T0>(M, N, K, cus, s, direct, parts, c[0]), plan_time<T1>(M, N, K, cus, s, direct, parts, c[1]),
                                  plan_time<T2>(M, N, K, cus, s, direct, parts, c[2]), plan_time<T3>(M, N, K, cus, s, direct, parts, c[3]),
                                  plan_time<T4>(M, N, K, cus, s, direct, parts, c[4]), plan_time<T5>(M, N, K, cus, s, direct, parts, c[5])};
        for (int i = 0; i < NTILES; ++i)
            if (t[i] < best.us) best = GemmF32Plan{false, i, s, direct, t[i]};
    }
    return best;
}

template <class TL, bool A_KS, bool B_KS, int EPI, bool DIRECT>
hipError_t launch_tile(Params p, DeviceInfo& dev, int slot, int split, hipStream_t stream)
{
    const int64_t tm = (p.M + TL::BM - 1) / TL::BM, tn = (p.N + TL::BN - 1) / TL::BN;
    if (tm * tn > 0x7fffffffLL) return hipErrorInvalidValue;
    if (!dev.gemm_f32_lds_set[slot]) {
        hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(&gemm_f32_kernel<TL, A_KS, B_KS, EPI, DIRECT>),
                                           hipFuncAttributeMaxDynamicSharedMemorySize, TL::lds(DIRECT, TL::stages(DIRECT)));
        if (e != hipSuccess) return e;
        dev.gemm_f32_lds_set[slot] = true;
    }
    const int64_t nk = (p.K + TL::KB - 1) / TL::KB;
    p.per_split = split > 1 ? (nk + split - 1) / split : nk;
    p.split_k = split > 1 ? (int)((nk + p.per_split - 1) / p.per_split) : 1;      // (no empty split)
    gemm_f32_raster(p, tm, tn, TL::BM, TL::BN, dev);
    hipLaunchKernelGGL((gemm_f32_kernel<TL, A_KS, B_KS, EPI, DIRECT>), dim3((unsigned)(tm * tn), (unsigned)p.split_k), dim3(NT),
                       TL::lds(DIRECT, p.per_split), stream, p);
    hipError_t e = hipGetLastError();
    if (p.parts) *p.parts = p.split_k;
    if (e != hipSuccess || p.split_k <= 1 || p.parts) return e;
    return launch_splitk_reduce(p, EPI, stream);
}

template <bool A_KS, bool B_KS, int EPI, bool DIRECT>
hipError_t launch_vec(const Params& p, DeviceInfo& dev, int combo, const GemmF32Plan& plan, hipStream_t stream)
{
    const int slot = (combo * 2 + (DIRECT ? 1 : 0)) * NTILES + plan.tile;
    switch (plan.tile) {
        case 0: return launch_tile<T0, A_KS, B_KS, EPI, DIRECT>(p, dev, slot, plan.split, stream);
        case 1: return launch_tile<T1, A_KS, B_KS, EPI, DIRECT>(p, dev, slot, plan.split, stream);
        case 2: return launch_tile<T2, A_KS, B_KS, EPI, DIRECT>(p, dev, slot, plan.split, stream);
        case 3: return launch_tile<T3, A_KS, B_KS, EPI, DIRECT>(p, dev, slot, plan.split, stream);
        case 4: return launch_tile<T4, A_KS, B_KS, EPI, DIRECT>(p, dev, slot, plan.split, stream);
        default: return launch_tile<T5, A_KS, B_KS, EPI, DIRECT>(p, dev, slot, plan.split, stream);
    }
}

// Direct loads: every operand row 16-byte aligned, 32-bit byte offsets between the rows of a load.
bool direct_loads(const GemmF32Args& a)
{
    auto rows16 = [](const float* P, int64_t ld, bool ks, int64_t rows) {
        return ld % 4 == 0 && reinterpret_cast<uintptr_t>(P) % 16 == 0 && (!ks || rows % 4 == 0) && ld < (1LL << 25);
    };
    return rows16(a.A, a.lda, a.a_kstrided, a.M) && rows16(a.B, a.ldb, a.b_kstrided, a.N);
}

template <bool A_KS, bool B_KS, int EPI>
hipError_t launch_any(const Params& p, DeviceInfo& dev, int combo, const GemmF32Plan& plan, hipStream_t stream)
{
    if (plan.direct) return launch_vec<A_KS, B_KS, EPI, true>(p, dev, combo, plan, stream);
    return launch_vec<A_KS, B_KS, EPI, false>(p, dev, combo, plan, stream);
}

// How many ways a contraction may be split along k at most: only when there are few output tiles and every
// split still gets at least 8 k-slices.  The scratch is sized for this bound; the launcher picks the split.
int gemm_f32_max_split(int64_t M, int64_t N, int64_t K)
{
    if (M <= 0 || N <= 0 || K <= 0) return 1;
    const int64_t t128 = ((M + 127) / 128) * ((N + 127) / 128), nk = (K + 31) / 32;
    if (t128 >= 256) return 1;
    int64_t s = nk / 8;
    if (s > 8) s = 8;
    return s < 2 ? 1 : (int)s;
}

}  // namespace

void gemm_f32_raster(Params& p, int64_t tiles_m, int64_t tiles_n, int BM, int BN, const DeviceInfo& dev)
{
    p.tiles_m = (int)tiles_m;
    p.tiles_n = (int)tiles_n;
    p.num_xcd = dev.xcds > 0 ? dev.xcds : 1;
    // block of tiles per XCD with the fewest operand rows: group_m ~ sqrt(tiles per XCD * BN / BM)
    const double per_xcd = (double)(tiles_m * tiles_n) / p.num_xcd;
    int gm = (int)(sqrt(per_xcd * BN / BM) + 0.5);
    if (gm < 1) gm = 1;
    if (gm > tiles_m) gm = (int)tiles_m;
    p.group_m = gm;
}

hipError_t launch_splitk_reduce(const Params& p, int epilogue, hipStream_t stream)
{
    int64_t g = (p.M * ((p.N + 3) / 4) + 255) / 256;
    if (g > 4096) g = 4096;
    const dim3 grid((unsigned)g), block(256);
    switch (epilogue) {
        case EPI_STORE: hipLaunchKernelGGL(splitk_reduce_kernel<EPI_STORE>, grid, block, 0, stream, p); break;
        case EPI_RMW: hipLaunchKernelGGL(splitk_reduce_kernel<EPI_RMW>, grid, block, 0, stream, p); break;
        case EPI_RESID: hipLaunchKernelGGL(splitk_reduce_kernel<EPI_RESID>, grid, block, 0, stream, p); break;
        default: hipLaunchKernelGGL(splitk_reduce_kernel<EPI_SHRINK>, grid, block, 0, stream, p); break;
    }
    return hipGetLastError();
}

int64_t gemm_f32_partial_bytes(int64_t M, int64_t N, int64_t K)
{
    const int s = gemm_f32_max_split(M, N, K);
    return s > 1 ? (int64_t)s * M * N * 4 : 0;
}

GemmF32Plan gemm_f32_plan(const GemmF32Args& a)
{
    const int max_split = a.partial ? gemm_f32_max_split(a.M, a.N, a.K) : 1;
    const GemmF32Plan plan = plan_gemm(a.M, a.N, a.K, a.dev->cus > 0 ? a.dev->cus : 256, max_split, direct_loads(a), a.parts != nullptr);
    if (plan.us <= gemm_f32x3_least_us()) return plan;      // (a small call does without the other model, 0.1 us of the host)
    const GemmF32Plan x3 = gemm_f32x3_plan(a, max_split);
    return x3.us < plan.us ? x3 : plan;
}

hipError_t launch_gemm_f32(const GemmF32Args& a, hipStream_t stream)
{
    if (a.M <= 0 || a.N <= 0) return hipSuccess;
    if (!a.dev || (a.parts && a.epilogue != EPI_STORE)) return hipErrorInvalidValue;
    Params p = {};
    p.A = a.A; p.B = a.B; p.C = a.C; p.aux = a.aux; p.L_ptr = a.L_ptr;
    p.lda = a.lda; p.ldb = a.ldb; p.ldc = a.ldc;
    p.M = a.M; p.N = a.N; p.K = a.K;
    p.eta = a.eta; p.lambda = a.lambda;
    p.partial = a.partial;
    p.parts = a.parts;
    const GemmF32Plan plan = gemm_f32_plan(a);
    if (plan.three_terms) return launch_gemm_f32x3(a, p, plan, stream);
    const bool aks = a.a_kstrided, bks = a.b_kstrided;
    if (!aks && !bks && a.epilogue == EPI_STORE) return launch_any<false, false, EPI_STORE>(p, *a.dev, 0, plan, stream);
    if (!aks && !bks && a.epilogue == EPI_SHRINK) return launch_any<false, false, EPI_SHRINK>(p, *a.dev, 1, plan, stream);
    if (!aks && bks && a.epilogue == EPI_RESID) return launch_any<false, true, EPI_RESID>(p, *a.dev, 2, plan, stream);
    if (aks && bks && a.epilogue == EPI_RMW) return launch_any<true, true, EPI_RMW>(p, *a.dev, 3, plan, stream);
    return hipErrorInvalidValue;
}

}  // namespace sfb
