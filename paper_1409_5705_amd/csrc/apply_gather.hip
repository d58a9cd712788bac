// The bf16 apply for sparse second factors: W -= eta * U^T V where few entries of V are stored.
//
// With hundreds of factor pairs every column of W is touched by some pair, so W is read and written whole whatever V
// holds; what can be left out is the multiplication by zeros.  Sixteen columns of V at half a per cent of non-zeros have
// entries in 79 of 1024 rows (1024 (1 - 0.995^16)): a contraction over those is three MFMA steps instead of 32.
// csr_lists_kernel writes, for every tile of sixteen columns, the rows that have entries there and V on those rows as MFMA
// operands (2 MB in all at 10000 columns); apply_gather_kernel keeps U of 64 classes and all pairs in LDS, [pair][class]
// as it is in memory, and gathers the listed pairs with LDS reads that transpose 16-bit elements (ds_read_b64_tr_b16:
// four pairs x sixteen classes), where the address of each pair is free.  U needs no transposed copy in memory.
//
// Bound: the stream of W, 20 GB on the planes at 325000 x 10000.  1024 pairs, 0.5 % stored: 4.36 ms with 10 us for the
// lists (4.6 TB/s; dense product 6.12 and 0.26 for U^T); every further step of 32 pairs a tile 0.3 ms.  A request of the
// list waits for an L2 hit, several times what a step's LDS reads and MFMAs take: one step at a time it was 0.48 ms a
// step.
// An infinite or NaN factor is NaN times the zeros that are left out, as in the dense product: a panel with one is gone over
// again at the end.  (Looking for them costs 0.5 % there, 3 to 4 % of 51344 x 696 with 1191 pairs; the second pass, where
// every factor is NaN, 100000 x 5000 with 512 pairs 0.67 -> 1.8 ms.)
#include "planes.h"

#include <type_traits>

namespace sfb {
namespace {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float floatx4 __attribute__((ext_vector_type(4)));
typedef short s16x4 __attribute__((ext_vector_type(4)));
typedef unsigned short u16x2 __attribute__((ext_vector_type(2)));

constexpr int PANEL = 64, CHUNK = 128, NT = 512;      // classes of a workgroup; columns of a wavefront's turn
constexpr int AHEAD = 4;                              // steps requested at a time (2 or 3: 1 % slower at three steps a tile)
constexpr int MAX_PAIRS = 1276;                       // (and four rows of zeros: 160 KB of LDS)

struct Params {
    const uint16_t* U;
    float* C;
    uint16_t* shadow;       // bf16 copy of C, or null; the high plane
    uint16_t* lo;           // the low plane, or null: C is fp32
    int64_t J, D, ldc, ld_shadow;
    int N, max_steps, chunks, panels, num_xcd;
    float eta;
    const uint32_t* steps;  // [tile] MFMA steps of 32 pairs
    const uint32_t* rows;   // [tile][max_steps][16]: pairs 8 q + r and 8 q + 4 + r of a step in word 4 q + r
    const u32x4* frags;     // [tile][max_steps][64]: V on them, as lane l multiplies it
};

// Column of element l16 of tile t (0 .. 7) of a chunk: a lane of the apply owns eight columns of its eight tiles, in a row
// (planes) or as two groups of four 64 apart (fp32 array), that 16-byte accesses cover.
__device__ __forceinline__ int tile_column(bool planes, int t, int l16) { return planes ? 8 * l16 + t : 4 * l16 + (t & 3) + 64 * (t >> 2); }
__device__ __forceinline__ int tile_of_column(bool planes, int c) { return planes ? c & 7 : (c & 3) + 4 * (c >> 6); }

// One workgroup per tile.  Vt: V^T as a bf16 operand of pitch Np (columns D .. of the last block of rows are zero).  The
// listed pairs of each residue modulo 4 take every fourth place of the list (the gaps of the shorter ones are rows of
// zeros): the sixteen pairs of an LDS read then meet every bank equally often.
__global__ __launch_bounds__(256) void csr_lists_kernel(const uint16_t* __restrict__ Vt, int64_t Np, int N, int planes, int max_steps,
                                                        uint32_t* __restrict__ steps, uint32_t* __restrict__ rows, u32x4* __restrict__ frags)
{
    __shared__ uint16_t list[4][MAX_PAIRS / 4 + 8];
    __shared__ int wave_count[4][4];
    const int tile = blockIdx.x, tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, c = tid & 3;
    const int64_t d0 = (int64_t)(tile / 8) * CHUNK;
    auto value = [&](int l16, int i) -> uint16_t {
        const int64_t d = d0 + tile_column(planes, tile % 8, l16);
        return Vt[((d / BM) * (Np / BK) + i / BK) * (BM * BK) + (d % BM) * BK + i % BK];
    };
    int total[4] = {0, 0, 0, 0};
    for (int i0 = 0; i0 < N; i0 += 256) {
        const int i = i0 + tid;
        uint32_t any = 0;
        if (i < N) {
#pragma unroll
            for (int l = 0; l < 16; ++l) any |= value(l, i) & 0x7fffu;
        }
        const uint64_t mask = __builtin_amdgcn_ballot_w64(any != 0), mine = 0x1111111111111111ull << c;
        if (lane < 4) wave_count[wave][c] = __builtin_popcountll(mask & mine);
        __syncthreads();
        int at = 0;
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            if (k == c) at = total[k];
#pragma unroll
            for (int w = 0; w < 4; ++w) {
                if (k == c && w < wave) at += wave_count[w][k];
                total[k] += wave_count[w][k];
            }
        }
        if (any) list[c][at + __builtin_popcountll(mask & mine & ((1ull << lane) - 1))] = (uint16_t)i;
        __syncthreads();
    }
    int most = 0;
#pragma unroll
    for (int k = 0; k < 4; ++k) most = total[k] > most ? total[k] : most;
    const int n = (most + 7) / 8, zero = (N + 3) / 4 * 4;
    for (int j = tid; j < 32 * n; j += 256)      // (U's rows of zeros)
        if (j / 4 >= (c == 0 ? total[0] : c == 1 ? total[1] : c == 2 ? total[2] : total[3])) list[c][j / 4] = (uint16_t)(zero + c);
    __syncthreads();
    auto pair = [&](int k) -> int { return list[k & 3][k >> 2]; };
    if (tid == 0) steps[tile] = (uint32_t)n;
    uint32_t* const my_rows = rows + (int64_t)tile * max_steps * 16;
    for (int j = tid; j < 16 * n; j += 256) {
        const int k = 32 * (j / 16) + 8 * (j % 16 / 4) + j % 4;
        my_rows[j] = (uint32_t)pair(k) | (uint32_t)pair(k + 4) << 16;
    }
    u32x4* const my_frags = frags + (int64_t)tile * max_steps * 64;
    for (int j = tid; j < 64 * n; j += 256) {
        const int k = 32 * (j / 64) + 8 * (j % 64 / 16), l16 = j % 16;
        u32x4 v;
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            const int a = pair(k + 2 * e), b = pair(k + 2 * e + 1);
            v[e] = (a < N ? (uint32_t)value(l16, a) : 0u) | (b < N ? (uint32_t)value(l16, b) : 0u) << 16;
        }
        my_frags[j] = v;
    }
}

// One workgroup of eight wavefronts per 64 classes; a wavefront takes every eighth chunk of 128 columns.  LDS: pair i is a
// row of 128 bytes, its 32-byte pieces (16 classes) swizzled by i & 3, so that the sixteen pairs of a read, four of each
// residue, spread over the banks although their rows all begin at bank 0.
template <bool PLANES>
__global__ __launch_bounds__(NT, 2) void apply_gather_kernel(Params p)
{
    extern __shared__ u32x4 gather_smem[];
    char* const lds = reinterpret_cast<char*>(gather_smem);
    typedef __attribute__((address_space(3))) s16x4* LdsWords;
    const uint32_t lds_base = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) char*)gather_smem;
    const int tid = threadIdx.x, lane = tid & 63, l16 = lane & 15, quad = lane >> 4;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    // each XCD a contiguous range of panels: neighbours share lines of U (rows of U are not aligned to lines)
    int64_t m0;
    {
        const uint32_t xcds = (uint32_t)p.num_xcd, x = blockIdx.x % xcds, q = (uint32_t)p.panels / xcds, r = (uint32_t)p.panels % xcds;
        m0 = (int64_t)(x * q + (x < r ? x : r) + blockIdx.x / xcds) * PANEL;
    }
    u16x2 largest = {0, 0};      // from 0x7f80 on: a value that is not finite
    for (int i = tid >> 3; i < (p.N + 3) / 4 * 4 + 4; i += NT / 8) {
        const int piece = tid & 7;
        u32x4 v = {0u, 0u, 0u, 0u};
        if (i < p.N && m0 + 8 * piece < p.J) v = *reinterpret_cast<const u32x4*>(p.U + (int64_t)i * p.J + m0 + 8 * piece);
#pragma unroll
        for (int k = 0; k < 4; ++k) largest = __builtin_elementwise_max(largest, __builtin_bit_cast(u16x2, v[k] & 0x7fff7fffu));
        *reinterpret_cast<u32x4*>(lds + i * 128 + (((piece >> 1) ^ (i & 3)) << 5) + ((piece & 1) << 4)) = v;
    }
    const bool wave_bad = __builtin_amdgcn_ballot_w64(largest[0] >= 0x7f80 || largest[1] >= 0x7f80) != 0;
    __syncthreads();

    const int last_m = (int)(p.J - m0 < PANEL ? p.J - m0 : PANEL) - 1;
    auto make_rsrc = [&](const void* base, uint64_t bytes) {
        return __builtin_amdgcn_make_buffer_rsrc(reinterpret_cast<void*>(uniform64(reinterpret_cast<uint64_t>(base))), 0,
                                                 bytes > 0xffffffffu ? 0xffffffffu : (uint32_t)bytes, 0x00020000);
    };
    const uint32_t row_c = (uint32_t)p.ldc * 4u;
    auto shadow_at = [](uint32_t c) { return (c / BK) * (uint32_t)(BM * BK * 2) + (c % BK) * 2u; };
    const bool has_shadow = p.shadow != nullptr;

    for (int chunk = wave; chunk < p.chunks; chunk += NT / 64) {
        const int64_t n0 = (int64_t)chunk * CHUNK;
        const int last_n = (int)(p.D - n0 < CHUNK ? p.D - n0 : CHUNK) - 1;
        // (rows past J are there in the blocks of the planes; past the fp32 array they read zeros)
        const auto crs = make_rsrc(PLANES ? p.C : p.C + m0 * p.ldc + n0, (uint64_t)((p.J - m0) * p.ldc - n0) * 4);
        const auto srs = make_rsrc(has_shadow ? p.shadow + ((m0 / BM) * (p.ld_shadow / BK) + n0 / BK) * (int64_t)(BM * BK) + (m0 % BM) * BK : p.shadow, 0xffffffffu);
        const auto lrs = make_rsrc(PLANES ? p.lo + ((m0 / BM) * ((p.D + BN - 1) / BN) + n0 / BN) * (int64_t)(BM * BN) + (m0 % BM) * BN + n0 % BN : p.lo, 0xffffffffu);
        const int c0 = (PLANES ? 8 : 4) * l16, c1 = 64 + 4 * l16;
        const bool ok0 = c0 <= last_n, ok1 = c1 <= last_n;              // D % 8 == 0: a whole group or none
        const uint32_t at0 = (uint32_t)(ok0 ? c0 : 0), at1 = (uint32_t)(ok1 ? c1 : 0);
        const uint32_t lane_s = shadow_at(at0) + 4u * quad * (BK * 2), lane_l = at0 * 2u + 4u * quad * (BN * 2);
        const uint32_t lane_c0 = at0 * 4u + 4u * quad * row_c, lane_c1 = at1 * 4u + 4u * quad * row_c;
        const uint32_t lane_s1 = shadow_at(at1) + 4u * quad * (BK * 2);
        // rows 16 ta + 4 quad + e; two of the four row tiles at a time
        auto load = [&](int ta, int e, u32x4(&w)[2]) {
            const uint32_t r = (uint32_t)(16 * ta + e);
            if (PLANES) {
                w[0] = __builtin_amdgcn_raw_buffer_load_b128(srs, lane_s, r * (BK * 2), C_POLICY);
                w[1] = __builtin_amdgcn_raw_buffer_load_b128(lrs, lane_l, r * (BN * 2), C_POLICY);
            } else {
                w[0] = __builtin_amdgcn_raw_buffer_load_b128(crs, lane_c0, r * row_c, C_POLICY);
                w[1] = __builtin_amdgcn_raw_buffer_load_b128(crs, lane_c1, r * row_c, C_POLICY);
            }
        };
        floatx4 acc[4][8];
#pragma unroll
        for (int ta = 0; ta < 4; ++ta)
#pragma unroll
            for (int t = 0; t < 8; ++t) acc[ta][t] = floatx4{0.f, 0.f, 0.f, 0.f};
        // Steps four at a time: those of the next tile are requested before those of this one are multiplied (the waits are
        // for L2 hits, as long as a step's eight LDS reads and four MFMAs several times over).  W is requested behind the
        // last of them, since loads are waited for in order.
        struct Batch {
            uint32_t pair[AHEAD];
            u32x4 v[AHEAD];
        };
        auto request = [&](int t, int s) {
            const uint32_t* rows = p.rows + ((int64_t)(8 * chunk + t) * p.max_steps + s) * 16 + 4 * quad + (l16 >> 2);
            const u32x4* frags = p.frags + ((int64_t)(8 * chunk + t) * p.max_steps + s) * 64 + lane;
            Batch b;
#pragma unroll
            for (int q = 0; q < AHEAD; ++q) {      // (past the tile's last step: some other words, not used)
                b.pair[q] = rows[16 * q];
                b.v[q] = frags[64 * q];
            }
            return b;
        };
        int n[8];
#pragma unroll
        for (int t = 0; t < 8; ++t) n[t] = (int)p.steps[8 * chunk + t];
        u32x4 w[2][4][2];
        Batch cur = request(0, 0);
        static_for<0, 8>([&](auto t_) {
            constexpr int t = decltype(t_)::value;
            Batch next;
            if constexpr (t < 7) {
                next = request(t + 1, 0);
            } else {
#pragma unroll
                for (int ta = 0; ta < 2; ++ta)
#pragma unroll
                    for (int e = 0; e < 4; ++e) load(ta, e, w[ta][e]);
            }
            for (int s = 0;;) {
#pragma unroll
                for (int q = 0; q < AHEAD; ++q) {
                    if (s + q >= n[t]) break;
                    const uint32_t i0 = cur.pair[q] & 0xffffu, i1 = cur.pair[q] >> 16;
                    const uint32_t a0 = lds_base + i0 * 128u + ((i0 & 3u) << 5) + 8u * (l16 & 3), a1 = lds_base + i1 * 128u + ((i1 & 3u) << 5) + 8u * (l16 & 3);
#pragma unroll
                    for (int ta = 0; ta < 4; ++ta) {
                        union {
                            s16x4 h[2];
                            bf16x8 v;
                        } u;
                        u.h[0] = __builtin_amdgcn_ds_read_tr16_b64_v4i16((LdsWords)(uintptr_t)(a0 ^ (32u * ta)));
                        u.h[1] = __builtin_amdgcn_ds_read_tr16_b64_v4i16((LdsWords)(uintptr_t)(a1 ^ (32u * ta)));
                        acc[ta][t] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(u.v, __builtin_bit_cast(bf16x8, cur.v[q]), acc[ta][t], 0, 0, 0);
                    }
                }
                s += AHEAD;
                if (s >= n[t]) break;
                cur = request(t, s);
            }
            if constexpr (t < 7) cur = next;
        });

        // ---- W - eta * acc.  Register e of lane (quad, l16) of MFMA tile (ta, t): row 16 ta + 4 quad + e, column t of the lane's
        auto store = [&](auto ta_, auto e_, const u32x4(&old)[2]) {
            constexpr int ta = decltype(ta_)::value, e = decltype(e_)::value;
            constexpr uint32_t r = 16 * ta + e;
            const bool row_ok = 4 * quad <= last_m - (int)r;
            if (PLANES) {
                uint32_t oh[4], ol[4];
                bool changed = false;
#pragma unroll
                for (int k = 0; k < 4; ++k) {
                    const uint32_t hk = old[0][k], lk = old[1][k];
                    const uint32_t w0 = split_word(split_value(join_pair0(hk, lk)) - p.eta * acc[ta][2 * k][e]);
                    const uint32_t w1 = split_word(split_value(join_pair1(hk, lk)) - p.eta * acc[ta][2 * k + 1][e]);
                    oh[k] = pack_hi(w0, w1);
                    ol[k] = pack_lo(w0, w1);
                    changed = changed || oh[k] != hk;
                }
                if (row_ok && ok0) {
                    if (any_in_line<8>(changed, lane))
                        __builtin_amdgcn_raw_buffer_store_b128(u32x4{oh[0], oh[1], oh[2], oh[3]}, srs, lane_s, r * (BK * 2), C_POLICY);
                    __builtin_amdgcn_raw_buffer_store_b128(u32x4{ol[0], ol[1], ol[2], ol[3]}, lrs, lane_l, r * (BN * 2), C_POLICY);
                }
            } else {
#pragma unroll
                for (int h = 0; h < 2; ++h) {       // the two groups of four columns
                    if (!(row_ok && (h ? ok1 : ok0))) continue;
                    float nf[4];
                    uint32_t sh[2];
                    bool changed = false;
#pragma unroll
                    for (int k = 0; k < 2; ++k) {
                        const uint32_t oa = old[h][2 * k], ob = old[h][2 * k + 1];
                        nf[2 * k] = __uint_as_float(oa) - p.eta * acc[ta][4 * h + 2 * k][e];
                        nf[2 * k + 1] = __uint_as_float(ob) - p.eta * acc[ta][4 * h + 2 * k + 1][e];
                        sh[k] = pack_bf16(nf[2 * k], nf[2 * k + 1]);
                        changed = changed || sh[k] != pack_bf16(__uint_as_float(oa), __uint_as_float(ob));
                    }
                    const u32x4 out = {__float_as_uint(nf[0]), __float_as_uint(nf[1]), __float_as_uint(nf[2]), __float_as_uint(nf[3])};
                    __builtin_amdgcn_raw_buffer_store_b128(out, crs, h ? lane_c1 : lane_c0, r * row_c, C_POLICY);
                    if (has_shadow && any_in_line<16>(changed, lane))
                        __builtin_amdgcn_raw_buffer_store_b64(u32x2{sh[0], sh[1]}, srs, h ? lane_s1 : lane_s, r * (BK * 2), C_POLICY);
                }
            }
        };
        static_for<0, 2>([&](auto ta_) {
            static_for<0, 4>([&](auto e_) {
                constexpr int ta = decltype(ta_)::value, e = decltype(e_)::value;
                store(ta_, e_, w[ta][e]);
                load(ta + 2, e, w[ta][e]);
            });
        });
        static_for<0, 2>([&](auto ta_) {
            static_for<0, 4>([&](auto e_) {
                constexpr int ta = decltype(ta_)::value, e = decltype(e_)::value;
                store(std::integral_constant<int, ta + 2>{}, e_, w[ta][e]);
            });
        });
    }

    // ---- a factor that is not finite is NaN times the zeros of V that were left out: each wavefront goes over its chunks
    // again, a lane a class, and makes NaN what belongs to a class and a tile with such a pair that is not listed there
    // (the arguments and the lane read again: kept since the start they would take registers from the loop above)
    uint64_t args = (uint64_t)__builtin_amdgcn_kernarg_segment_ptr();
    asm volatile("" : "+s"(args));
    const int cls = __builtin_amdgcn_mbcnt_hi(~0u, __builtin_amdgcn_mbcnt_lo(~0u, 0u));
    const auto* q = (const __attribute__((address_space(4))) Params*)args;
    const int N = q->N;
    __syncthreads();
    uint32_t* const flag = reinterpret_cast<uint32_t*>(lds + (N + 3) / 4 * 4 * 128);      // (in the rows of zeros)
    if (wave_bad && cls == 0) *flag = 1u;
    __syncthreads();
    if (*flag == 0u) return;
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    auto bad_of = [&](int i) -> int {
        return (*reinterpret_cast<const uint16_t*>(lds + i * 128 + (((cls >> 4) ^ (i & 3)) << 5) + 2 * (cls & 15)) & 0x7f80) == 0x7f80 ? 1 : 0;
    };
    int all = 0;
    for (int i = 0; i < N; ++i) all += bad_of(i);
    const int64_t D = q->D;
    const uint32_t nan_word = split_word(__builtin_nanf(""));
    for (int chunk = wave; chunk < q->chunks; chunk += NT / 64) {
        int unlisted = 0;      // bit t: tile t of the chunk lacks such a pair of this class
        for (int t = 0; t < 8; ++t) {
            const int64_t tile = 8 * (int64_t)chunk + t;
            const int n = (int)q->steps[tile];
            int listed = 0;
            if (__builtin_amdgcn_ballot_w64(all > 0 && all <= 32 * n) != 0)      // (more than can be listed: need not be counted)
                for (int j = 0; j < 16 * n; ++j) {
                    const uint32_t two = q->rows[tile * q->max_steps * 16 + j];
                    const int i0 = (int)(two & 0xffffu), i1 = (int)(two >> 16);
                    if (i0 < N) listed += bad_of(i0);
                    if (i1 < N) listed += bad_of(i1);
                }
            if (all > 32 * n || listed < all) unlisted |= 1 << t;
        }
        for (uint64_t rows = __builtin_amdgcn_ballot_w64(unlisted != 0 && m0 + cls < q->J); rows != 0; rows &= rows - 1) {
            const int r = __builtin_ctzll(rows), tiles = __builtin_amdgcn_readlane(unlisted, r);
            const int64_t m = m0 + r;
            for (int e = 0; e < 2; ++e) {
                const int c = 2 * cls + e;
                const int64_t d = (int64_t)chunk * CHUNK + c;
                if (d >= D || !(tiles >> tile_of_column(PLANES, c) & 1)) continue;
                if (q->shadow) q->shadow[((m / BM) * (q->ld_shadow / BK) + d / BK) * (int64_t)(BM * BK) + (m % BM) * BK + d % BK] = (uint16_t)(nan_word >> 16);
                if (PLANES)
                    q->lo[((m / BM) * ((D + BN - 1) / BN) + d / BN) * (int64_t)(BM * BN) + (m % BM) * BN + d % BN] = (uint16_t)nan_word;
                else
                    q->C[m * q->ldc + d] = __builtin_nanf("");
            }
        }
    }
}

int64_t tiles_of(int64_t D) { return (D + CHUNK - 1) / CHUNK * 8; }
int64_t round256(int64_t x) { return (x + 255) / 256 * 256; }

}  // namespace

bool apply_gather_supported(int64_t N, int64_t J, int64_t D)
{
    return N >= 1 && N <= MAX_PAIRS && (J + PANEL - 1) / PANEL <= 0x7fffffffLL && D < (1LL << 24) && tiles_of(D) <= 0x7fffffffLL;
}

int64_t apply_gather_workspace_bytes(int64_t N, int64_t D)
{
    const int64_t tiles = tiles_of(D), max_steps = (N + 31) / 32;
    return round256(tiles * 4) + round256((tiles * max_steps + 4) * 64) + (tiles * max_steps + 4) * 1024;      // (requests of four steps)
}

hipError_t launch_apply_gather(float* W, uint16_t* W_shadow, uint16_t* W_lo, const uint16_t* U, const uint16_t* Vt, int64_t N, int64_t J,
                               int64_t D, float eta, void* workspace, DeviceInfo& dev, hipStream_t stream)
{
    if (N <= 0 || J <= 0 || D <= 0) return hipSuccess;
    if (!apply_gather_supported(N, J, D)) return hipErrorInvalidValue;
    const int64_t tiles = tiles_of(D), max_steps = (N + 31) / 32;
    char* ws = static_cast<char*>(workspace);
    Params p = {};
    p.U = U; p.C = W; p.shadow = W_shadow; p.lo = W_lo;
    p.J = J; p.D = D; p.ldc = D; p.ld_shadow = bf16_pitch(D);
    p.N = (int)N; p.max_steps = (int)max_steps;
    p.chunks = (int)(tiles / 8);
    p.panels = (int)((J + PANEL - 1) / PANEL);
    p.num_xcd = dev.xcds > 0 ? dev.xcds : 1;
    p.eta = eta;
    uint32_t* const steps = reinterpret_cast<uint32_t*>(ws);
    uint32_t* const rows = reinterpret_cast<uint32_t*>(ws + round256(tiles * 4));
    u32x4* const frags = reinterpret_cast<u32x4*>(ws + round256(tiles * 4) + round256((tiles * max_steps + 4) * 64));
    p.steps = steps; p.rows = rows; p.frags = frags;
    hipLaunchKernelGGL(csr_lists_kernel, dim3((unsigned)tiles), dim3(256), 0, stream, Vt, bf16_pitch(N), (int)N, W_lo ? 1 : 0, (int)max_steps, steps, rows, frags);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    const int lds = (int)((N + 3) / 4 * 4 + 4) * 128, slot = W_lo ? 1 : 0;
    const void* f = W_lo ? reinterpret_cast<const void*>(&apply_gather_kernel<true>) : reinterpret_cast<const void*>(&apply_gather_kernel<false>);
    if (!dev.apply_gather_lds_set[slot]) {
        e = hipFuncSetAttribute(f, hipFuncAttributeMaxDynamicSharedMemorySize, (MAX_PAIRS + 4) * 128);
        if (e != hipSuccess) return e;
        dev.apply_gather_lds_set[slot] = true;
    }
    if (W_lo)
        hipLaunchKernelGGL(apply_gather_kernel<true>, dim3((unsigned)p.panels), dim3(NT), lds, stream, p);
    else
        hipLaunchKernelGGL(apply_gather_kernel<false>, dim3((unsigned)p.panels), dim3(NT), lds, stream, p);
    return hipGetLastError();
}

}  // namespace sfb
