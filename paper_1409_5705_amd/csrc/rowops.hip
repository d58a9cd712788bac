// Row-wise and elementwise kernels around the GEMMs: the softmax/label step of
// multiclass logistic regression, the pair difference and hinge coefficient of
// distance metric learning, the power iteration and the row projection of
// sparse coding.  Rows stay in registers where they fit; sums over the 64 lanes go
// through DPP, those of the softmax through shuffles.
#include "device.h"
#include "kernels.h"

namespace sfb {
namespace {

typedef float floatx4 __attribute__((ext_vector_type(4)));
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));

// Reductions over the 64 lanes (all active): four DPP steps inside rows of 16 lanes, then the four rows through scalar
// registers.  (The shuffles through the LDS unit that stood here cost six round trips of some 50 ns each.)
template <int CTRL>
__device__ __forceinline__ float dpp(float v)
{
    return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), CTRL, 0xf, 0xf, true));
}
__device__ __forceinline__ float lane_value(float v, int lane) { return __int_as_float(__builtin_amdgcn_readlane(__float_as_int(v), lane)); }
constexpr int DPP_XOR1 = 0xB1, DPP_XOR2 = 0x4E, DPP_HALF_MIRROR = 0x141, DPP_MIRROR = 0x140;
__device__ __forceinline__ float wave_sum(float v)
{
    v += dpp<DPP_XOR1>(v);
    v += dpp<DPP_XOR2>(v);
    v += dpp<DPP_HALF_MIRROR>(v);
    v += dpp<DPP_MIRROR>(v);
    return (lane_value(v, 0) + lane_value(v, 16)) + (lane_value(v, 32) + lane_value(v, 48));
}
__device__ __forceinline__ float wave_max(float v)
{
    v = fmaxf(v, dpp<DPP_XOR1>(v));
    v = fmaxf(v, dpp<DPP_XOR2>(v));
    v = fmaxf(v, dpp<DPP_HALF_MIRROR>(v));
    v = fmaxf(v, dpp<DPP_MIRROR>(v));
    return fmaxf(fmaxf(lane_value(v, 0), lane_value(v, 16)), fmaxf(lane_value(v, 32), lane_value(v, 48)));
}
// The sum as a butterfly over distances 32, 16, .. 1.  The multiclass-logistic softmax keeps this order: where a sample is
// classified with near certainty its factor is 1 / s - 1 with s close to 1, and which way the last bit of s falls is a
// few per cent of that factor (either order is as far from the exact sum).
__device__ __forceinline__ float wave_sum_butterfly(float v)
{
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) v += __shfl_xor(v, off, 64);
    return v;
}
// Block reductions; `sm` has NT/64 floats.  Every thread gets the result.
template <int NT, bool BUTTERFLY = false>
__device__ __forceinline__ float block_sum(float v, float* sm)
{
    v = BUTTERFLY ? wave_sum_butterfly(v) : wave_sum(v);
    __syncthreads();
    if ((threadIdx.x & 63) == 0) sm[threadIdx.x >> 6] = v;
    __syncthreads();
    float r = 0.f;
#pragma unroll
    for (int w = 0; w < NT / 64; ++w) r += sm[w];
    return r;
}
template <int NT>
__device__ __forceinline__ float block_max(float v, float* sm)
{
    v = wave_max(v);
    __syncthreads();
    if ((threadIdx.x & 63) == 0) sm[threadIdx.x >> 6] = v;
    __syncthreads();
    float r = sm[0];
#pragma unroll
    for (int w = 1; w < NT / 64; ++w) r = fmaxf(r, sm[w]);
    return r;
}

// ---------------------------------------------------------------------------
// MLR: u = softmax(z) - onehot(y).  One workgroup per sample; two passes over
// the row: (1) running maximum and sum of exponentials together (the sum is
// rescaled whenever the maximum grows), read from HBM; (2) normalise + label +
// store, re-read from L2 (a row of the headline size is 1.3 MB).  Four 16-byte
// loads per thread are in flight in both passes.
// ---------------------------------------------------------------------------
__device__ __forceinline__ void online_update(float& m, float& s, const floatx4 v)
{
    const float mn = fmaxf(fmaxf(m, fmaxf(v[0], v[1])), fmaxf(v[2], v[3]));
    s = s * expf(m - mn) + ((expf(v[0] - mn) + expf(v[1] - mn)) + (expf(v[2] - mn) + expf(v[3] - mn)));
    m = mn;
}

// tiles_m > 0: Z is not row-major but an array of 256 x 256 tiles, tile (row / 256, j / 256) at index
// (j / 256) * tiles_m + row / 256 (the layout the bf16 forward contraction writes: one piece per workgroup).
template <bool OUT_BF16>
__global__ __launch_bounds__(1024) void mlr_softmax_kernel(const float* __restrict__ Z, const int32_t* __restrict__ y,
                                                         void* __restrict__ Uv, int64_t J, int vec, int64_t tiles_m)
{
    constexpr int NT = 1024;
    __shared__ float sm[NT / 64];
    const int64_t row = blockIdx.x;
    const bool blocked = tiles_m > 0;
    const float* z = blocked ? Z + (row / 256) * 65536 + (row % 256) * 256 : Z + row * J;
    const int64_t tile_stride = tiles_m * 65536;          // floats from a tile to the next one along j
    struct View {   // logits of this row by class index (at1) or by group of four classes (at4)
        const float* z;
        int64_t ts;
        bool blocked;
        __device__ floatx4 at4(int64_t q) const
        {
            const int64_t o = blocked ? (q >> 6) * (ts >> 2) + (q & 63) : q;
            return reinterpret_cast<const floatx4*>(z)[o];
        }
        __device__ float at1(int64_t j) const { return z[blocked ? (j >> 8) * ts + (j & 255) : j]; }
    };
    const View zv = {z, tile_stride, blocked};
    const int tid = threadIdx.x;
    const int64_t J4 = vec ? J / 4 : 0;

    float m = -INFINITY, s = 0.f;
    int64_t q = tid;
    for (; q + 3 * NT < J4; q += 4 * NT) {
        const floatx4 a = zv.at4(q), b = zv.at4(q + NT), c = zv.at4(q + 2 * NT), d = zv.at4(q + 3 * NT);
        online_update(m, s, a);
        online_update(m, s, b);
        online_update(m, s, c);
        online_update(m, s, d);
    }
    for (; q < J4; q += NT) online_update(m, s, zv.at4(q));
    for (int64_t j = J4 * 4 + tid; j < J; j += NT) {
        const float v = zv.at1(j), mn = fmaxf(m, v);
        s = s * expf(m - mn) + expf(v - mn);
        m = mn;
    }
    // (a thread that saw no element has m = -inf, s = 0: its term is 0 * exp(-inf) = 0)
    const float M = block_max<NT>(m, sm);
    s = block_sum<NT, true>(s * expf(m - M), sm);
    const float inv = 1.0f / s;

    const int64_t lab = y[row];
    auto emit = [&](int64_t qq, const floatx4 v) {
        floatx4 p;
#pragma unroll
        for (int e = 0; e < 4; ++e) p[e] = expf(v[e] - M) * inv - ((qq * 4 + e == lab) ? 1.0f : 0.0f);
        if (OUT_BF16) {
            uint2 o;
            o.x = pack_bf16(p[0], p[1]);
            o.y = pack_bf16(p[2], p[3]);
            reinterpret_cast<uint2*>(reinterpret_cast<uint16_t*>(Uv) + row * J)[qq] = o;
        } else {
            reinterpret_cast<floatx4*>(reinterpret_cast<float*>(Uv) + row * J)[qq] = p;
        }
    };
    q = tid;
    for (; q + 3 * NT < J4; q += 4 * NT) {
        const floatx4 a = zv.at4(q), b = zv.at4(q + NT), c = zv.at4(q + 2 * NT), d = zv.at4(q + 3 * NT);
        emit(q, a);
        emit(q + NT, b);
        emit(q + 2 * NT, c);
        emit(q + 3 * NT, d);
    }
    for (; q < J4; q += NT) emit(q, zv.at4(q));
    for (int64_t j = J4 * 4 + tid; j < J; j += NT) {
        const float p = expf(zv.at1(j) - M) * inv - ((j == lab) ? 1.0f : 0.0f);
        if (OUT_BF16) {
            reinterpret_cast<uint16_t*>(Uv)[row * J + j] = (uint16_t)(pack_bf16(p, 0.f) & 0xffffu);
        } else {
            reinterpret_cast<float*>(Uv)[row * J + j] = p;
        }
    }
}

// Rows of at most PER floats per thread: the row stays in registers between the maximum, the exponentials and the
// output, every logit is read once and exponentiated once (the exponentials of a thread are added in groups of four, as in
// the kernel above).  PLANES: the logits are the sum of several partial arrays.  Workgroups past the B rows copy
// copy_bytes from copy_src to copy_dst (the samples that become the second factors): one launch less.
template <int PER, bool OUT_BF16, bool VEC, bool PLANES>
__global__ __launch_bounds__(256) void mlr_softmax_row_kernel(const float* __restrict__ Z, const int32_t* __restrict__ y,
                                                            void* __restrict__ Uv, int64_t B, int64_t J, int64_t tiles_m, int planes,
                                                            int64_t plane_floats, const u32x4* __restrict__ copy_src,
                                                            u32x4* __restrict__ copy_dst, int64_t copy_bytes)
{
    constexpr int NT = 256;
    __shared__ float sm[NT / 64];
    const int tid = threadIdx.x;
    const int64_t row = blockIdx.x;
    if (row >= B) {
        const int64_t n = copy_bytes / 16, stride = (int64_t)(gridDim.x - B) * NT, first = (row - B) * NT + tid;
        for (int64_t i = first; i < n; i += stride) copy_dst[i] = copy_src[i];
        if (first < (copy_bytes % 16) / 4)
            reinterpret_cast<uint32_t*>(copy_dst)[n * 4 + first] = reinterpret_cast<const uint32_t*>(copy_src)[n * 4 + first];
        return;
    }
    const bool blocked = tiles_m > 0;
    const float* z = blocked ? Z + (row / 256) * 65536 + (row % 256) * 256 : Z + row * J;
    constexpr int E = VEC ? 4 : 1, CH = PER / E;             // elements of a chunk; chunks of a thread
    float v[CH][E];
    auto load = [&](const float* at, float* dst) {
        if constexpr (VEC) {
            const floatx4 t = *reinterpret_cast<const floatx4*>(at);
            const float t0 = t[0], t1 = t[1], t2 = t[2], t3 = t[3];
            dst[0] = t0; dst[1] = t1; dst[2] = t2; dst[3] = t3;
        } else {
            dst[0] = at[0];
        }
    };
    float m = -INFINITY;
#pragma unroll
    for (int i = 0; i < CH; ++i) {
        const int64_t j = (int64_t)(tid + NT * i) * E;
#pragma unroll
        for (int e = 0; e < E; ++e) v[i][e] = -INFINITY;
        if (j < J) load(z + (blocked ? (j >> 8) * (tiles_m * 65536) + (j & 255) : j), v[i]);
    }
    if (PLANES) {
        constexpr int AHEAD = PER <= 4 ? 7 : (PER <= 16 ? 2 : 1);      // arrays in flight
        for (int k0 = 1; k0 < planes; k0 += AHEAD) {
            float t[AHEAD][CH][E];
#pragma unroll
            for (int a = 0; a < AHEAD; ++a)
#pragma unroll
                for (int i = 0; i < CH; ++i) {
                    const int64_t j = (int64_t)(tid + NT * i) * E;
                    if (k0 + a < planes && j < J)
                        load(z + (k0 + a) * plane_floats + (blocked ? (j >> 8) * (tiles_m * 65536) + (j & 255) : j), t[a][i]);
                }
#pragma unroll
            for (int a = 0; a < AHEAD; ++a)
#pragma unroll
                for (int i = 0; i < CH; ++i)
                    if (k0 + a < planes && (int64_t)(tid + NT * i) * E < J) {
#pragma unroll
                        for (int e = 0; e < E; ++e) v[i][e] += t[a][i][e];
                    }
        }
    }
#pragma unroll
    for (int i = 0; i < CH; ++i)
#pragma unroll
        for (int e = 0; e < E; ++e) m = fmaxf(m, v[i][e]);
    const float M = block_max<NT>(m, sm);
    float s = 0.f;
#pragma unroll
    for (int i = 0; i < CH; ++i) {
#pragma unroll
        for (int e = 0; e < E; ++e) v[i][e] = expf(v[i][e] - M);
        s += VEC ? (v[i][0] + v[i][E > 1 ? 1 : 0]) + (v[i][E > 2 ? 2 : 0] + v[i][E > 3 ? 3 : 0]) : v[i][0];
    }
    s = block_sum<NT, true>(s, sm);
    const float inv = 1.0f / s;
    const int64_t lab = y[row];
#pragma unroll
    for (int i = 0; i < CH; ++i) {
        const int64_t j = (int64_t)(tid + NT * i) * E;
        if (j >= J) continue;
        float p[E];
#pragma unroll
        for (int e = 0; e < E; ++e) p[e] = v[i][e] * inv - ((j + e == lab) ? 1.0f : 0.0f);
        if (OUT_BF16) {
            uint16_t* u = reinterpret_cast<uint16_t*>(Uv) + row * J + j;
            if constexpr (VEC)
                *reinterpret_cast<u32x2*>(u) = u32x2{pack_bf16(p[0], p[1]), pack_bf16(p[2], p[3])};
            else
                *u = (uint16_t)(pack_bf16(p[0], 0.f) & 0xffffu);
        } else {
            float* u = reinterpret_cast<float*>(Uv) + row * J + j;
            if constexpr (VEC)
                *reinterpret_cast<floatx4*>(u) = floatx4{p[0], p[1], p[2], p[3]};
            else
                *u = p[0];
        }
    }
}

// ---------------------------------------------------------------------------
// The same for long rows of tile-blocked logits, reading them once.  A row of
// the headline size (1.3 MB) outlives every cache between the two passes above,
// so the second pass is a second trip to memory.  Here CL workgroups share a
// row: each keeps its 1/CL of the row in registers (up to CHUNKS x 16 bytes a
// thread), reduces it to (max, sum of exponentials relative to that max),
// publishes the pair in one 64-bit word and collects the CL words of the row;
// the stored values become exp(z - max_own) and are rescaled on output.
//
// The grid is one workgroup per CU (1024 threads at no more than 128 registers), so
// the CL partners of a row normally run at the same time, and they execute the
// same number of row iterations.  Nothing depends on that, though: the wait for a
// partner's word is bounded (spin_limit polls), and a workgroup whose partner has
// not published in time (kernels of other streams can keep it off the chip)
// computes that partner's pair itself from the logits, and no longer waits for that
// partner in later rows.  So every workgroup finishes whatever the others do; the
// price of a missing partner is reading its part of the row a second time.
// `slots`: [B][CL] 64-bit words, all zero before the launch (a published word
// has a non-zero high half: the bits of a sum that is at least 1).
// ---------------------------------------------------------------------------
constexpr int CLUSTER_CHUNKS = 10;        // 16-byte chunks of a row per thread
// Cache policy of the logits read and of the factors written here: non-temporal, both are touched once (measured
// at the headline size, interleaved: 0.460 -> 0.434 ms; with only the loads non-temporal the transposes that read
// the factors next slow down by as much, with both they do not).
constexpr int STREAM_POLICY = 2;
// partner pairs computed by the waiting workgroup itself (one count per workgroup, row and partner)
__device__ unsigned long long g_softmax_fallbacks = 0;

__global__ __launch_bounds__(1024) void mlr_softmax_cluster_kernel(const float* __restrict__ Z,
                                                                  const int32_t* __restrict__ y,
                                                                  uint16_t* __restrict__ U, int64_t B, int64_t J,
                                                                  int64_t tiles_m, int CL, int tiles_per_wg,
                                                                  unsigned long long* __restrict__ slots, int spin_limit)
{
    constexpr int NT = 1024, R = CLUSTER_CHUNKS;
    __shared__ float sm[NT / 64];
    __shared__ float part_m[32], part_s[32];
    __shared__ int part_ok[32], gone[32];       // gone: partners this workgroup has stopped waiting for
    if (threadIdx.x < 32) gone[threadIdx.x] = 0;
    const int tid = threadIdx.x;
    const int groups = (int)gridDim.x / CL, grp = (int)blockIdx.x / CL, w = (int)blockIdx.x % CL;
    if (grp >= groups) return;                      // (a grid that is not a multiple of CL: the rest has no row)
    const int64_t tn = (J + 255) / 256;
    const int64_t t0 = (int64_t)w * tiles_per_wg;
    int64_t t1 = t0 + tiles_per_wg;
    if (t1 > tn) t1 = tn;
    const int64_t my_chunks = t1 > t0 ? (t1 - t0) * 64 : 0;      // 64 chunks of four classes per tile row

    // Chunk i of this thread: tile t0 + 16 i + tid / 64, classes 4 (tid % 64) .. + 3 of it.  Addresses are a
    // uniform part (row, i) plus a 32-bit part of the thread; which chunks exist does not depend on the row.
    const uint32_t t_tile = (uint32_t)tid >> 6, t_col = ((uint32_t)tid & 63u) * 4u;
    const uint32_t z_thread = t_tile * (uint32_t)(tiles_m * 65536) + t_col;        // floats; B <= 65536 (host check): < 2^28
    const uint32_t j_thread = t_tile * 256u + t_col;
    const int64_t z_step = 16 * tiles_m * 65536;                                   // floats from chunk i to i + 1
    uint32_t have = 0;
#pragma unroll
    for (int i = 0; i < R; ++i) {
        const int64_t c = (int64_t)i * NT + tid;
        if (c < my_chunks && (t0 + (c >> 6)) * 256 + (c & 63) * 4 < J) have |= 1u << i;
    }
    // (buffer accesses: a uniform 64-bit base in scalar registers plus one 32-bit offset register per thread,
    // instead of a 64-bit address pair per chunk)
    auto rsrc = [](const void* base) {
        return __builtin_amdgcn_make_buffer_rsrc(const_cast<void*>(base), 0, 0xffffffff, 0x00020000);
    };
    auto load_row = [&](int64_t row, floatx4* v) {
        const float* base = Z + (row / 256) * 65536 + (row % 256) * 256 + t0 * tiles_m * 65536;
#pragma unroll
        for (int i = 0; i < R; ++i) {
            v[i] = floatx4{-INFINITY, -INFINITY, -INFINITY, -INFINITY};
            if (have & (1u << i)) {
                const u32x4 r = __builtin_amdgcn_raw_buffer_load_b128(rsrc(base + i * z_step), z_thread * 4u, 0, STREAM_POLICY);
                const uint32_t r0 = r[0], r1 = r[1], r2 = r[2], r3 = r[3];
                v[i] = floatx4{__uint_as_float(r0), __uint_as_float(r1), __uint_as_float(r2), __uint_as_float(r3)};
            }
        }
    };

    floatx4 v[R], vn[R];
    int64_t row = grp;
    if (row < B) load_row(row, v);
    for (; row < B; row += groups) {
        // own part: maximum, then exponentials relative to it (kept in v) and their sum
        float m = -INFINITY;
#pragma unroll
        for (int i = 0; i < R; ++i) m = fmaxf(m, fmaxf(fmaxf(v[i][0], v[i][1]), fmaxf(v[i][2], v[i][3])));
        const float m_own = block_max<NT>(m, sm);
        // (2^(z log2 e - m log2 e) through the hardware exponential: one multiply-add and one v_exp per class instead
        // of the library routine's dozen instructions, which made this kernel ALU-bound; the result differs from
        // exp(z - m) by a few 1e-6 relative for |m| up to 60, far below the bf16 spacing of the output)
        const float LOG2E = 1.4426950408889634f;
        const float mb = -m_own * LOG2E;
        float s = 0.f;
#pragma unroll
        for (int i = 0; i < R; ++i) {
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                v[i][e] = m_own == -INFINITY ? 0.f : __builtin_amdgcn_exp2f(__builtin_fmaf(v[i][e], LOG2E, mb));
                s += v[i][e];
            }
        }
        float s_own = block_sum<NT, true>(s, sm);
        if (m_own == -INFINITY) s_own = 1.0f;       // no class at all in this part: counts as 1 * exp(-inf) = 0
        if (tid == 0) {
            const unsigned long long word = ((unsigned long long)__float_as_uint(s_own) << 32) | __float_as_uint(m_own);
            __hip_atomic_store(&slots[row * CL + w], word, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        }
        // the next row's loads travel while the partners' words are awaited and this row is written
        const int64_t next = row + groups;
        if (next < B) load_row(next, vn);
        if (tid < CL) {
            if (tid == w) {
                part_m[tid] = m_own;
                part_s[tid] = s_own;
                part_ok[tid] = 1;
            } else {
                unsigned long long word = 0;
                const int polls = gone[tid] ? 1 : spin_limit;
                for (int spin = 0; spin < polls; ++spin) {
                    word = __hip_atomic_load(&slots[row * CL + tid], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                    if (word >> 32) break;
                    __builtin_amdgcn_s_sleep(8);
                }
                const int ok = (word >> 32) != 0;
                part_m[tid] = __uint_as_float((uint32_t)word);
                part_s[tid] = __uint_as_float((uint32_t)(word >> 32));
                part_ok[tid] = ok;
                if (!ok) gone[tid] = 1;
            }
        }
        __syncthreads();
        for (int k = 0; k < CL; ++k) {
            if (part_ok[k]) continue;               // (the same for every thread: read from LDS after the barrier)
            // partner k has not published: its pair from the logits themselves
            const int64_t k0 = (int64_t)k * tiles_per_wg;
            int64_t k1 = k0 + tiles_per_wg;
            if (k1 > tn) k1 = tn;
            const float* base = Z + (row / 256) * 65536 + (row % 256) * 256;
            float mk = -INFINITY, sk = 0.f;
            for (int64_t c = tid; c < (k1 - k0) * 64; c += NT) {
                const int64_t tile = k0 + (c >> 6);
                if (tile * 256 + (c & 63) * 4 < J)
                    online_update(mk, sk, *reinterpret_cast<const floatx4*>(base + tile * tiles_m * 65536 + (c & 63) * 4));
            }
            const float Mk = block_max<NT>(mk, sm);
            float Sk = block_sum<NT, true>(mk == -INFINITY ? 0.f : sk * expf(mk - Mk), sm);
            if (Mk == -INFINITY) Sk = 1.0f;
            if (tid == 0) {
                part_m[k] = Mk;
                part_s[k] = Sk;
                atomicAdd(&g_softmax_fallbacks, 1ull);
            }
            __syncthreads();
        }
        float M = part_m[0];
        for (int k = 1; k < CL; ++k) M = fmaxf(M, part_m[k]);
        float S = 0.f;
        for (int k = 0; k < CL; ++k) S += part_s[k] * expf(part_m[k] - M);
        const float scale = expf(m_own - M) / S;

        const int64_t out0 = row * J + t0 * 256;          // U index of class t0 * 256 of this row
        // the label relative to this thread's first class of chunk 0 (|.| < 2^31: labels and J are 32-bit)
        const int32_t lab_t = (int32_t)((int64_t)y[row] - t0 * 256) - (int32_t)j_thread;
#pragma unroll
        for (int i = 0; i < R; ++i) {
            if (have & (1u << i)) {
                floatx4 p = v[i] * scale;
                const uint32_t at = (uint32_t)(lab_t - i * 4096);      // 0..3: the label is one of these four
                if (at < 4u) {
#pragma unroll
                    for (int e = 0; e < 4; ++e) p[e] -= (at == (uint32_t)e) ? 1.0f : 0.0f;
                }
                const u32x2 o = {pack_bf16(p[0], p[1]), pack_bf16(p[2], p[3])};
                __builtin_amdgcn_raw_buffer_store_b64(o, rsrc(U + out0 + i * 4096), j_thread * 2u, 0, STREAM_POLICY);
            }
        }
#pragma unroll
        for (int i = 0; i < R; ++i) v[i] = vn[i];
        __syncthreads();                            // part_m / part_s are rewritten in the next iteration
    }
}

// V = X - Y; also clears *counter (nullable): the count of active pairs a later kernel of the same call adds to.
// E floats an access.
template <int E>
__global__ __launch_bounds__(256) void diff_kernel(const float* __restrict__ X, const float* __restrict__ Y,
                                                   float* __restrict__ V, int64_t n, int32_t* __restrict__ counter)
{
    typedef float F __attribute__((ext_vector_type(E)));
    if (counter && blockIdx.x == 0 && threadIdx.x == 0) *counter = 0;
    const int64_t stride = (int64_t)gridDim.x * 256;
    for (int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x; i < n / E; i += stride)
        reinterpret_cast<F*>(V)[i] = reinterpret_cast<const F*>(X)[i] - reinterpret_cast<const F*>(Y)[i];
}

__global__ __launch_bounds__(256) void scale_rows_kernel(const float* __restrict__ V, const float* __restrict__ coef,
                                                         float* __restrict__ Vs, int64_t N, int64_t D)
{
    const int64_t total = N * D, stride = (int64_t)gridDim.x * 256;
    for (int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x; i < total; i += stride) Vs[i] = coef[i / D] * V[i];
}

__global__ __launch_bounds__(256) void fill_u32_kernel(uint32_t* __restrict__ p, uint32_t value, int64_t n)
{
    const int64_t stride = (int64_t)gridDim.x * 256;
    for (int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x; i < n; i += stride) p[i] = value;
}

// W = Z / lambda: the primal matrix from the auxiliary one for the squared l2
// regulariser (W = grad h^*(Z), Section 2.1, Stochastic DCA).
template <int E>
__global__ __launch_bounds__(256) void div_scalar_kernel(const float* __restrict__ Z, float* __restrict__ W,
                                                         float lambda, int64_t n)
{
    typedef float F __attribute__((ext_vector_type(E)));
    const int64_t stride = (int64_t)gridDim.x * 256;
    for (int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x; i < n / E; i += stride)
        reinterpret_cast<F*>(W)[i] = reinterpret_cast<const F*>(Z)[i] / lambda;
}

// w > 0 with w + log w = L (w = W0(e^L), the principal Lambert function).  The
// start is a lower bound of the root (e^L / (1 + e^L) for L < 1, L - log L
// otherwise), from which Newton's iteration on the concave left side rises
// monotonically; three steps reach fp32 accuracy over the whole range, four are
// taken.  Below L = -15 the series w = y - y^2 of y = e^L is exact in fp32.
__device__ __forceinline__ float lambert_w_exp(float L)
{
    if (L < -15.f) {
        const float y = expf(L);
        return y - y * y;
    }
    float w;
    if (L >= 1.f) {
        w = L - __logf(L);
    } else {
        const float y = __expf(L);
        w = y / (1.f + y);
    }
#pragma unroll
    for (int it = 0; it < 4; ++it) w = w * (1.f + L - logf(w)) / (1.f + w);
    return w;
}

// Dual coordinate step of l2-regularised multiclass logistic regression, one
// workgroup per sample.  With z = W a_i (the row of Zl), c = ||a_i||^2 / (lambda N)
// and the sample's dual point p_old in the simplex, the minimiser p of the dual
// over this sample's variable solves
//     log p_j + c p_j = z_j + c p_old_j - nu  (every class j),   sum_j p_j = 1.
// Each class equation is p_j = W0(c e^{t_j}) / c; sum_j p_j is decreasing in nu
// and the root lies in [lse(theta) - c, lse(theta)], theta = z + c p_old.  nu is
// found by Newton's iteration on log(sum p) kept inside that bracket (bisection
// when a step leaves it).  Outputs: dU = beta (p - p_old), P += dU.
//
// Rows of at most PER classes a thread: logits and dual point stay in registers for all the passes (seven on average),
// every pass takes one barrier (two sums reduced together, alternating LDS slots); what bounds it is the chain of
// exponentials and logarithms of a Newton step, hence few classes a thread while there are few samples (256 samples of 1000
// classes: 27.7 us re-reading the rows with four barriers a step, 16.0 now).  PER == 0: rows of any length, re-read
// from the cache.
template <int NT, int PER>
__global__ __launch_bounds__(NT) void sdca_mlr_kernel(const float* __restrict__ Zl, const float* __restrict__ X,
                                                      float* __restrict__ P, float* __restrict__ dU, int64_t J,
                                                      int64_t D, float inv_lambda_n, float beta)
{
    constexpr int NWV = NT / 64, R = PER > 0 ? PER : 1;
    __shared__ float sm[2][2][NWV];
    const int64_t i = blockIdx.x;
    const float* z = Zl + i * J;
    float* p_old = P + i * J;
    float* du = dU + i * J;
    const int tid = threadIdx.x, wave = tid >> 6;
    int turn = 0;
    auto sum2 = [&](float& a, float& b) {      // (a slot is rewritten two calls later: the barrier between has been passed)
        a = wave_sum(a);
        b = wave_sum(b);
        if ((tid & 63) == 0) {
            sm[turn][0][wave] = a;
            sm[turn][1][wave] = b;
        }
        __syncthreads();
        a = 0.f;
        b = 0.f;
#pragma unroll
        for (int w = 0; w < NWV; ++w) {
            a += sm[turn][0][w];
            b += sm[turn][1][w];
        }
        turn ^= 1;
    };
    auto max1 = [&](float v) {
        v = wave_max(v);
        if ((tid & 63) == 0) sm[turn][0][wave] = v;
        __syncthreads();
        v = sm[turn][0][0];
#pragma unroll
        for (int w = 1; w < NWV; ++w) v = fmaxf(v, sm[turn][0][w]);
        turn ^= 1;
        return v;
    };
    float rz[R], rp[R];
    if (PER > 0) {
#pragma unroll
        for (int k = 0; k < R; ++k) {
            const int64_t j = tid + (int64_t)NT * k;
            rz[k] = j < J ? z[j] : 0.f;
            rp[k] = j < J ? p_old[j] : 0.f;
        }
    }
    // f(class, logit, dual point) over the classes of this thread
    auto each = [&](auto&& f) {
        if (PER > 0) {
#pragma unroll
            for (int k = 0; k < R; ++k) {
                const int64_t j = tid + (int64_t)NT * k;
                if (j < J) f(j, rz[k], rp[k]);
            }
        } else {
            for (int64_t j = tid; j < J; j += NT) f(j, z[j], p_old[j]);
        }
    };

    float acc = 0.f, none = 0.f;
    for (int64_t d = tid; d < D; d += NT) {
        const float x = X[i * D + d];
        acc += x * x;
    }
    sum2(acc, none);
    const float c = acc * inv_lambda_n;

    float m = -INFINITY;
    each([&](int64_t, float zj, float pj) { m = fmaxf(m, zj + c * pj); });
    m = max1(m);
    float s = 0.f;
    each([&](int64_t, float zj, float pj) { s += expf(zj + c * pj - m); });
    sum2(s, none);
    const float lse = m + logf(s);

    if (!(c > 1e-30f)) {   // a zero sample: the class equations decouple, p = softmax(z)
        each([&](int64_t j, float zj, float po) {
            const float d = beta * (expf(zj - lse) - po);
            du[j] = d;
            p_old[j] = po + d;
        });
        return;
    }
    const float logc = logf(c), inv_c = 1.f / c;
    float lo = lse - c, hi = lse, nu = lo;
    for (int it = 0; it < 32; ++it) {
        float S = 0.f, T = 0.f;
        each([&](int64_t, float zj, float pj) {
            const float w = lambert_w_exp(logc + (zj + c * pj - nu));
            S += w;                 // c p_j
            T += w / (1.f + w);     // c p_j / (1 + c p_j)
        });
        sum2(S, T);
        S *= inv_c;
        T *= inv_c;
        if (fabsf(S - 1.f) <= 1e-6f) break;          // (every thread holds the same S: a uniform exit)
        if (S > 1.f) lo = nu; else hi = nu;
        float cand = nu + S * logf(S) / T;
        if (!(cand > lo && cand < hi)) cand = 0.5f * (lo + hi);
        if (cand == nu) break;                        // bracket exhausted at fp32 resolution
        nu = cand;
    }
    each([&](int64_t j, float zj, float po) {
        const float p = lambert_w_exp(logc + (zj + c * po - nu)) * inv_c;
        const float d = beta * (p - po);
        du[j] = d;
        p_old[j] = po + d;
    });
}

// DML: one workgroup per pair; PER > 0: rows of at most 256 PER floats, in registers between the norm and the product.
// Q is the sum of `parts` arrays, `part` floats apart (PER > 0), all of them in flight together.  With the sum as a launch of
// its own / here (us of the whole factor computation, pairs x rows of the metric x features): 100 x 601 x 5000 21.5 / 18.9,
// 1000 x 600 x 1000 26.8 / 25.0, 500 x 1001 x 5000 48.0 / 45.5; adding one array at a time 100 x 1000 x 21504 57.2 / 60.4
// (now 54.6).
template <int PER>
__global__ __launch_bounds__(256) void dml_scale_kernel(const float* __restrict__ Q, int parts, int64_t part, const int8_t* __restrict__ sim,
                                                        float* __restrict__ U, int32_t* __restrict__ n_active,
                                                        float margin, int64_t K)
{
    __shared__ float sm[4];
    constexpr int AHEAD = 7;      // arrays in flight beside the first
    const int64_t row = blockIdx.x;
    const float* q = Q + row * K;
    float* const u = U + row * K;
    const int s = sim[row];
    float d = 0.f, v[PER > 0 ? PER : 1];
    if (PER > 0) {
#pragma unroll
        for (int i = 0; i < PER; ++i) v[i] = threadIdx.x + 256 * i < K ? q[threadIdx.x + 256 * i] : 0.f;
        for (int z0 = 1; z0 < parts; z0 += AHEAD) {
            float t[AHEAD][PER > 0 ? PER : 1];
#pragma unroll
            for (int z = 0; z < AHEAD; ++z)
#pragma unroll
                for (int i = 0; i < PER; ++i)
                    t[z][i] = z0 + z < parts && threadIdx.x + 256 * i < K ? q[(z0 + z) * part + threadIdx.x + 256 * i] : 0.f;
#pragma unroll
            for (int z = 0; z < AHEAD; ++z)
#pragma unroll
                for (int i = 0; i < PER; ++i) v[i] = z0 + z < parts ? v[i] + t[z][i] : v[i];
        }
#pragma unroll
        for (int i = 0; i < PER; ++i) d += v[i] * v[i];
    } else {
        for (int64_t k = threadIdx.x; k < K; k += 256) d += q[k] * q[k];
    }
    d = block_sum<256>(d, sm);
    float c;
    if (s > 0)
        c = 2.0f;
    else
        c = (d < margin) ? -2.0f : 0.0f;
    if (PER > 0) {
#pragma unroll
        for (int i = 0; i < PER; ++i)
            if (threadIdx.x + 256 * i < K) u[threadIdx.x + 256 * i] = c * v[i];
    } else {
        for (int64_t k = threadIdx.x; k < K; k += 256) u[k] = c * q[k];
    }
    if (threadIdx.x == 0 && c != 0.0f && n_active) atomicAdd(n_active, 1);
}

// Prox of the unit-ball constraint on each row.
__global__ __launch_bounds__(256) void prox_rows_kernel(float* __restrict__ W, int64_t D, int mode)
{
    __shared__ float sm[4];
    float* w = W + (int64_t)blockIdx.x * D;
    float nn = 0.f;
    for (int64_t d = threadIdx.x; d < D; d += 256) nn += w[d] * w[d];
    nn = block_sum<256>(nn, sm);
    const float nrm = sqrtf(nn);
    const bool scale = (mode == 0) ? (nrm > 1.0f) : (nrm > 0.0f);
    if (scale)
        for (int64_t d = threadIdx.x; d < D; d += 256) w[d] = w[d] / nrm;
}
// The same for rows of at most 1024 floats: one wavefront a row, the row in its registers (4096 x 1024: 18.6 -> 15.7 us).
template <bool VEC>
__global__ __launch_bounds__(256) void prox_rows_wave_kernel(float* __restrict__ W, int64_t J, int64_t D, int mode)
{
    const int lane = threadIdx.x & 63, d_count = (int)D;
    const int64_t row = (int64_t)blockIdx.x * 4 + (threadIdx.x >> 6);
    if (row >= J) return;
    float* const w = W + row * D;
    constexpr int E = VEC ? 4 : 1, CH = 16 / E;
    typedef float V __attribute__((ext_vector_type(E)));
    V v[CH];
    float nn = 0.f;
#pragma unroll
    for (int i = 0; i < CH; ++i) {
        const int d = (lane + 64 * i) * E;
        v[i] = V(0.f);
        if (d < d_count) v[i] = *reinterpret_cast<const V*>(w + d);
#pragma unroll
        for (int e = 0; e < E; ++e) nn += v[i][e] * v[i][e];
    }
    const float nrm = sqrtf(wave_sum(nn));
    const bool scale = (mode == 0) ? (nrm > 1.0f) : (nrm > 0.0f);
    if (!scale) return;
#pragma unroll
    for (int i = 0; i < CH; ++i) {
        const int d = (lane + 64 * i) * E;
        if (d < d_count) *reinterpret_cast<V*>(w + d) = v[i] / nrm;
    }
}

// ---------------------------------------------------------------------------
// Power iteration on W^T W: two kernels per iteration, W read from memory once.
// ---------------------------------------------------------------------------
// One workgroup per chunk of `rows` rows of W.  With b = g / ||g|| (g the raw vector of the previous iteration;
// every workgroup takes the norm itself while it reads g anyway):
//   c_j = W_j . b  for its rows (one wavefront per row at a time), then
//   part[chunk][d] = sum over its rows of W[j][d] c_j   (the rows come from the cache the second time).
constexpr int POWER_MAX_ROWS = 1024;
__global__ __launch_bounds__(256) void power_step_kernel(const float* __restrict__ W, const float* __restrict__ g,
                                                         float* __restrict__ part, int64_t J, int64_t D, int rows)
{
    __shared__ float sm[16];
    __shared__ float c[POWER_MAX_ROWS];
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    float nn = 0.f;
    for (int64_t d = tid; d < D; d += 256) nn += g[d] * g[d];
    const float inv = 1.0f / sqrtf(block_sum<256>(nn, sm));
    const int64_t j0 = (int64_t)blockIdx.x * rows;
    for (int r = wave; r < rows; r += 4) {
        const int64_t j = j0 + r;
        float s = 0.f;
        if (j < J)
            for (int64_t d = lane; d < D; d += 64) s += W[j * D + d] * g[d];
        s = wave_sum(s);
        if (lane == 0) c[r] = s * inv;
    }
    __syncthreads();
    const int64_t j1 = j0 + rows < J ? j0 + rows : J;
    for (int64_t d = tid; d < D; d += 256) {
        float s = 0.f;
        for (int64_t j = j0; j < j1; ++j) s += W[j * D + d] * c[j - j0];
        part[(int64_t)blockIdx.x * D + d] = s;
    }
}
// The same for rows of at most 1024 floats: a workgroup keeps its 16 rows in registers, all loads in flight together, so W
// is read once and nothing waits on a chain of dependent loads.  VEC (rows 16-byte aligned): thread t holds columns
// 4 t .. 4 t + 3 of every row; otherwise columns t, t + 256, t + 512, t + 768.
// `g` is gchunks partial vectors of D floats; every workgroup adds them up itself (in the same order).  With few
// partials that costs less than the launch of power_reduce_kernel; with many the caller passes their sum (gchunks 1).
// One iteration: 1000 x 300 10.4 -> 7.3 us (in one launch), 4096 x 1024 12.1 -> 10.1 us (in two; the rest is the reductions).
template <bool VEC>
__global__ __launch_bounds__(256) void power_step16_kernel(const float* __restrict__ W, const float* __restrict__ g, int gchunks,
                                                           float* __restrict__ part, int64_t J, int64_t D)
{
    __shared__ float sm[16];
    __shared__ float cw[16][4];
    __shared__ float ps[1024];
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, d_count = (int)D;
    const int64_t j0 = (int64_t)blockIdx.x * 16;
    constexpr int CW = VEC ? 4 : 1;                                          // floats of an access
    auto column = [&](int e) { return VEC ? 4 * tid + e : tid + 256 * e; };
    auto load4 = [&](const float* row) {
        floatx4 v = {0.f, 0.f, 0.f, 0.f};
        if (VEC) {
            if (4 * tid < d_count) v = *reinterpret_cast<const floatx4*>(row + 4 * tid);
        } else {
#pragma unroll
            for (int e = 0; e < 4; ++e)
                if (tid + 256 * e < d_count) v[e] = row[tid + 256 * e];
        }
        return v;
    };
    floatx4 w[16];
#pragma unroll
    for (int r = 0; r < 16; ++r) {
        w[r] = floatx4{0.f, 0.f, 0.f, 0.f};
        if (j0 + r < J) w[r] = load4(W + (j0 + r) * D);
    }
    floatx4 g4 = {0.f, 0.f, 0.f, 0.f};
    if (gchunks == 1) {
        g4 = load4(g);
    } else {
        // the threads are `groups` times the columns (in units of CW): group k adds partials k, k + groups, ...
        typedef float V __attribute__((ext_vector_type(CW)));
        const int units = d_count / CW, groups = units < 256 ? 256 / units : 1;
        const int grp = units < 256 ? tid / units : 0;
        if (grp < groups)
            for (int u = units < 256 ? tid - grp * units : tid; u < units; u += 256) {      // (units < 256: once)
                V sum = V(0.f);
                int ch = grp;
                for (; ch + 7 * groups < gchunks; ch += 8 * groups) {
                    V v[8];
#pragma unroll
                    for (int q = 0; q < 8; ++q) v[q] = reinterpret_cast<const V*>(g + (int64_t)(ch + q * groups) * D)[u];
#pragma unroll
                    for (int q = 0; q < 8; ++q) sum += v[q];
                }
                for (; ch < gchunks; ch += groups) sum += reinterpret_cast<const V*>(g + (int64_t)ch * D)[u];
                reinterpret_cast<V*>(ps)[grp * units + u] = sum;
            }
        __syncthreads();
#pragma unroll
        for (int e = 0; e < 4; ++e)
            if (column(e) < d_count) {
                float t = ps[column(e)];
                for (int k = 1; k < groups; ++k) t += ps[k * d_count + column(e)];
                g4[e] = t;
            }
    }
    const float inv = 1.0f / sqrtf(block_sum<256>(g4[0] * g4[0] + g4[1] * g4[1] + g4[2] * g4[2] + g4[3] * g4[3], sm));
#pragma unroll
    for (int r = 0; r < 16; ++r) {
        const float s = wave_sum(w[r][0] * g4[0] + w[r][1] * g4[1] + w[r][2] * g4[2] + w[r][3] * g4[3]);
        if (lane == 0) cw[r][wave] = s;
    }
    __syncthreads();
    floatx4 out = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int r = 0; r < 16; ++r) {
        const float c = (((cw[r][0] + cw[r][1]) + cw[r][2]) + cw[r][3]) * inv;
        out += w[r] * c;
    }
    float* const to = part + (int64_t)blockIdx.x * D;
    if (VEC) {
        if (4 * tid < d_count) *reinterpret_cast<floatx4*>(to + 4 * tid) = out;
    } else {
#pragma unroll
        for (int e = 0; e < 4; ++e)
            if (column(e) < d_count) to[column(e)] = out[e];
    }
}
// g[d] = sum of the chunks' partials in a fixed order: 16 columns a workgroup, 16 interleaved groups of chunks
// per column (eight loads in flight per thread), combined in order.
__global__ __launch_bounds__(256) void power_reduce_kernel(const float* __restrict__ part, float* __restrict__ g,
                                                           int64_t D, int64_t chunks)
{
    __shared__ float sm[16][17];
    const int col = threadIdx.x & 15, grp = threadIdx.x >> 4;
    const int64_t d = (int64_t)blockIdx.x * 16 + col;
    float s = 0.f;
    if (d < D) {
        int64_t ch = grp;
        for (; ch + 7 * 16 < chunks; ch += 8 * 16) {
            float v[8];
#pragma unroll
            for (int u = 0; u < 8; ++u) v[u] = part[(ch + 16 * u) * D + d];
#pragma unroll
            for (int u = 0; u < 8; ++u) s += v[u];
        }
        for (; ch < chunks; ch += 16) s += part[ch * D + d];
    }
    sm[grp][col] = s;
    __syncthreads();
    if (grp == 0 && d < D) {
        float t = sm[0][col];
#pragma unroll
        for (int k = 1; k < 16; ++k) t += sm[k][col];
        g[d] = t;
    }
}
// L = ||sum of the partials||.  One workgroup.
__global__ __launch_bounds__(1024) void vec_norm_kernel(const float* __restrict__ g, int gchunks, float* __restrict__ L_out, int64_t D)
{
    __shared__ float sm[16];
    __shared__ float ps[1024];
    float nn = 0.f;
    if (gchunks == 1) {
        for (int64_t d = threadIdx.x; d < D; d += 1024) nn += g[d] * g[d];
    } else {                                        // (D <= 1024)
        const int d_count = (int)D, groups = 1024 / d_count, grp = (int)threadIdx.x / d_count, d = (int)threadIdx.x % d_count;
        float t = 0.f;
        if (grp < groups) {
            int ch = grp;
            for (; ch + 7 * groups < gchunks; ch += 8 * groups) {
                float v[8];
#pragma unroll
                for (int q = 0; q < 8; ++q) v[q] = g[(int64_t)(ch + q * groups) * D + d];
#pragma unroll
                for (int q = 0; q < 8; ++q) t += v[q];
            }
            for (; ch < gchunks; ch += groups) t += g[(int64_t)ch * D + d];
        }
        ps[threadIdx.x] = t;
        __syncthreads();
        if (grp == 0) {
            for (int k = 1; k < groups; ++k) t += ps[k * d_count + d];
            nn = t * t;
        }
    }
    nn = block_sum<1024>(nn, sm);
    if (threadIdx.x == 0) L_out[0] = sqrtf(nn);
}

unsigned grid_for(int64_t n)
{
    int64_t g = (n + 255) / 256;
    if (g > 65536) g = 65536;
    if (g < 1) g = 1;
    return (unsigned)g;
}

}  // namespace

// Cluster size of the one-read softmax for rows of J classes (tile-blocked logits), or 0 where the two-pass
// kernel is used: short rows (the second pass then comes from the L2), J not a multiple of 4, rows too long for
// 32 workgroups to hold.
static int softmax_cluster(int64_t J)
{
    if (J < 65536 || J % 4 != 0) return 0;
    const int64_t tn = (J + 255) / 256, per_wg = CLUSTER_CHUNKS * 1024 / 64;      // tile rows one workgroup holds
    for (int cl = 2; cl <= 32; cl *= 2)
        if ((tn + cl - 1) / cl <= per_wg) return cl;
    return 0;
}

hipError_t softmax_fallbacks(unsigned long long* count)
{
    return hipMemcpyFromSymbol(count, HIP_SYMBOL(g_softmax_fallbacks), sizeof(*count), 0, hipMemcpyDeviceToHost);
}

int64_t mlr_softmax_scratch_bytes(int64_t B, int64_t J) { return softmax_cluster(J) ? B * softmax_cluster(J) * 8 : 0; }

constexpr int64_t SOFTMAX_ADDS_MAX = 4096;
// The launch of its own (4.3 us and more) has as many workgroups as there are logits, the row kernel one a sample: it adds
// them up where a thread has at most four logits, so that all their parts are in flight together, or where the samples fill
// the chip.  Measured (us of the whole factor computation, with the launch / without; samples x classes x features):
// 100 x 191 x 20000 22.8 / 18.2, 100 x 1000 x 4000 19.0 / 16.8, 600 x 1001 x 1000 24.1 / 21.3, 256 x 2000 x 4000 36.3 / 34.9,
// 256 x 2001 x 2000 27.9 / 25.4; but 100 x 1300 x 4000 23.3 / 24.3, 100 x 2000 x 4000 26.2 / 27.0.
bool mlr_softmax_adds(int64_t B, int64_t J, int cus) { return J <= 1024 || (J <= SOFTMAX_ADDS_MAX && B >= cus); }

template <int PER, bool VEC>
static hipError_t launch_softmax_row(const MlrSoftmaxArgs& a, hipStream_t stream)
{
    constexpr int NT = 256;
    int64_t copies = a.copy_src ? (a.copy_bytes / 16 + NT * 4 - 1) / (NT * 4) : 0;       // (at least four 16-byte pieces a thread)
    if (a.copy_src && copies < 1) copies = 1;
    if (copies > 1024) copies = 1024;
    const dim3 grid((unsigned)(a.B + copies));
    const int64_t tiles_m = a.blocked ? (a.B + 255) / 256 : 0;
    auto go = [&](auto bf16, auto planes) {
        hipLaunchKernelGGL((mlr_softmax_row_kernel<PER, decltype(bf16)::value, VEC, decltype(planes)::value>), grid, dim3(NT), 0, stream, a.Z,
                           a.y, a.U, a.B, a.J, tiles_m, a.planes, a.plane_floats, static_cast<const u32x4*>(a.copy_src), static_cast<u32x4*>(a.copy_dst), a.copy_bytes);
        return hipGetLastError();
    };
    typedef std::true_type Y;
    typedef std::false_type N;
    if constexpr (VEC)
        if (a.planes > 1 && a.out_bf16) return go(Y{}, Y{});
    if (a.planes > 1 && a.out_bf16) return hipErrorInvalidValue;      // (its logits are tile-blocked)
    if constexpr (PER <= SOFTMAX_ADDS_MAX / 256)
        if (a.planes > 1) return go(N{}, Y{});
    if (a.planes > 1) return hipErrorInvalidValue;
    return a.out_bf16 ? go(Y{}, N{}) : go(N{}, N{});
}

hipError_t launch_mlr_softmax(const MlrSoftmaxArgs& a, hipStream_t stream)
{
    if (a.B <= 0 || a.J <= 0) return hipSuccess;
    // Vector path: rows of Z (and of U) must start 16-byte (8-byte for bf16 U) aligned.
    const bool vec = a.J % 4 == 0 && reinterpret_cast<uintptr_t>(a.Z) % 16 == 0 && reinterpret_cast<uintptr_t>(a.U) % 16 == 0 &&
                     a.plane_floats % 4 == 0;
    if (a.J <= MLR_SOFTMAX_ROW_MAX) {
        if (a.B > 0x7fff0000LL) return hipErrorInvalidValue;
        // No more registers than the row needs: a thread exponentiates all of them.  4096 rows of 191 classes take 12.3 us
        // with 16 a thread, 7.7 with one; 1024 rows of 4104 15.5 with 64, 12.0 with 32.
        if (a.J <= 256 && !vec) return launch_softmax_row<1, false>(a, stream);
        if (a.J <= 1024) return vec ? launch_softmax_row<4, true>(a, stream) : launch_softmax_row<4, false>(a, stream);
        if (a.J <= 4096) return vec ? launch_softmax_row<16, true>(a, stream) : launch_softmax_row<16, false>(a, stream);
        if (a.J <= 8192) return vec ? launch_softmax_row<32, true>(a, stream) : launch_softmax_row<32, false>(a, stream);
        return vec ? launch_softmax_row<64, true>(a, stream) : launch_softmax_row<64, false>(a, stream);
    }
    if (a.planes > 1) return hipErrorInvalidValue;
    if (a.copy_src) {
        hipError_t e = hipMemcpyAsync(a.copy_dst, a.copy_src, (size_t)a.copy_bytes, hipMemcpyDeviceToDevice, stream);
        if (e != hipSuccess) return e;
    }
    const int cl = (a.blocked && a.out_bf16 && a.B <= 65536) ? softmax_cluster(a.J) : 0;   // (32-bit offsets of a thread)
    if (cl && a.scratch && a.dev && vec) {
        // one workgroup per CU so that all are resident together; whole clusters only
        int grid = a.dev->cus / cl * cl;
        if (grid < cl) return hipErrorInvalidValue;
        if ((int64_t)grid / cl > a.B) grid = (int)a.B * cl;
        const int64_t tn = (a.J + 255) / 256;
        const int tiles_per_wg = (int)((tn + cl - 1) / cl);
        hipError_t e = launch_fill_u32(a.scratch, 0u, a.B * cl * 2, stream);
        if (e != hipSuccess) return e;
        unsigned long long* slots = static_cast<unsigned long long*>(a.scratch);
        hipLaunchKernelGGL(mlr_softmax_cluster_kernel, dim3((unsigned)grid), dim3(1024), 0, stream, a.Z, a.y, static_cast<uint16_t*>(a.U),
                           a.B, a.J, (a.B + 255) / 256, cl, tiles_per_wg, slots, a.dev->softmax_wait_polls);
        return hipGetLastError();
    }
    const dim3 grid((unsigned)a.B);
    const int64_t tiles_m = a.blocked ? (a.B + 255) / 256 : 0;
    if (a.out_bf16)
        hipLaunchKernelGGL((mlr_softmax_kernel<true>), grid, dim3(1024), 0, stream, a.Z, a.y, a.U, a.J, (int)vec, tiles_m);
    else
        hipLaunchKernelGGL((mlr_softmax_kernel<false>), grid, dim3(1024), 0, stream, a.Z, a.y, a.U, a.J, (int)vec, tiles_m);
    return hipGetLastError();
}

hipError_t launch_diff(const float* X, const float* Y, float* V, int64_t n, int32_t* counter, hipStream_t stream)
{
    if (n <= 0) return counter ? launch_fill_u32(counter, 0u, 1, stream) : hipSuccess;
    auto aligned = [](const void* p) { return reinterpret_cast<uintptr_t>(p) % 16 == 0; };
    if (n % 4 == 0 && aligned(X) && aligned(Y) && aligned(V))
        hipLaunchKernelGGL(diff_kernel<4>, dim3(grid_for(n / 4)), dim3(256), 0, stream, X, Y, V, n, counter);
    else
        hipLaunchKernelGGL(diff_kernel<1>, dim3(grid_for(n)), dim3(256), 0, stream, X, Y, V, n, counter);
    return hipGetLastError();
}

hipError_t launch_scale_rows(const float* V, const float* coef, float* Vs, int64_t N, int64_t D, hipStream_t stream)
{
    if (N <= 0 || D <= 0) return hipSuccess;
    hipLaunchKernelGGL(scale_rows_kernel, dim3(grid_for(N * D)), dim3(256), 0, stream, V, coef, Vs, N, D);
    return hipGetLastError();
}

hipError_t launch_div_scalar(const float* Z, float* W, float lambda, int64_t n, hipStream_t stream)
{
    if (n <= 0) return hipSuccess;
    if (n % 4 == 0 && reinterpret_cast<uintptr_t>(Z) % 16 == 0 && reinterpret_cast<uintptr_t>(W) % 16 == 0)
        hipLaunchKernelGGL(div_scalar_kernel<4>, dim3(grid_for(n / 4)), dim3(256), 0, stream, Z, W, lambda, n);
    else
        hipLaunchKernelGGL(div_scalar_kernel<1>, dim3(grid_for(n)), dim3(256), 0, stream, Z, W, lambda, n);
    return hipGetLastError();
}

hipError_t launch_sdca_mlr(const float* Zl, const float* X, float* P, float* dU, int64_t B, int64_t J, int64_t D,
                           float lambda, int64_t n_total, float beta, int cus, hipStream_t stream)
{
    if (B <= 0 || J <= 0) return hipSuccess;
    if (B > 0x7fffffffLL) return hipErrorInvalidValue;
    const float inv_lambda_n = (float)(1.0 / ((double)lambda * (double)n_total));
    auto go = [&](auto nt, auto per) {
        constexpr int NT = decltype(nt)::value, PER = decltype(per)::value;
        hipLaunchKernelGGL((sdca_mlr_kernel<NT, PER>), dim3((unsigned)B), dim3(NT), 0, stream, Zl, X, P, dU, J, D, inv_lambda_n, beta);
    };
    // Up to two samples a CU: few classes a thread, for the chain of exponentials of each.  More: workgroups of 256, of which
    // more share a CU (us, 512 or 1024 threads / 256, 16 features: 300 classes, 256 samples 11.4 / 12.2, 1024 17.4 / 15.2, 4096
    // 47.7 / 36.0; 1025 classes, 256 samples 14.8 / 17.2, 512 21.8 / 20.5, 4096 117 / 86; 4096 classes, 512 samples 44 / 48,
    // 4096 239 / 227).
    using std::integral_constant;
    const bool few = B <= 2 * (int64_t)cus;
    if (J <= 256)
        go(integral_constant<int, 256>{}, integral_constant<int, 1>{});
    else if (J <= 512)
        few ? go(integral_constant<int, 512>{}, integral_constant<int, 1>{}) : go(integral_constant<int, 256>{}, integral_constant<int, 2>{});
    else if (J <= 1024)
        few ? go(integral_constant<int, 512>{}, integral_constant<int, 2>{}) : go(integral_constant<int, 256>{}, integral_constant<int, 4>{});
    else if (J <= 4096 && few)
        go(integral_constant<int, 1024>{}, integral_constant<int, 4>{});
    else if (J <= 2048)
        go(integral_constant<int, 256>{}, integral_constant<int, 8>{});
    else if (J <= 4096)
        go(integral_constant<int, 256>{}, integral_constant<int, 16>{});
    else
        go(integral_constant<int, 256>{}, integral_constant<int, 0>{});
    return hipGetLastError();
}

hipError_t launch_fill_u32(void* p, uint32_t value, int64_t n, hipStream_t stream)
{
    if (n <= 0) return hipSuccess;
    hipLaunchKernelGGL(fill_u32_kernel, dim3(grid_for(n)), dim3(256), 0, stream, reinterpret_cast<uint32_t*>(p),
                       value, n);
    return hipGetLastError();
}

hipError_t launch_dml_scale(const float* Q, int parts, const int8_t* sim, float* U, int32_t* n_active, float margin, int64_t B,
                            int64_t K, hipStream_t stream)
{
    if (B <= 0) return hipSuccess;
    if (parts > 1 && !dml_scale_adds(K)) return hipErrorInvalidValue;
    if (K <= 1024)
        hipLaunchKernelGGL(dml_scale_kernel<4>, dim3((unsigned)B), dim3(256), 0, stream, Q, parts, B * K, sim, U, n_active, margin, K);
    else
        hipLaunchKernelGGL(dml_scale_kernel<0>, dim3((unsigned)B), dim3(256), 0, stream, Q, 1, B * K, sim, U, n_active, margin, K);
    return hipGetLastError();
}

hipError_t launch_prox_rows(float* W, int64_t J, int64_t D, int mode, hipStream_t stream)
{
    if (J <= 0 || D <= 0) return hipSuccess;
    if (D <= 1024) {
        const dim3 grid((unsigned)((J + 3) / 4));
        if (D % 4 == 0 && reinterpret_cast<uintptr_t>(W) % 16 == 0)
            hipLaunchKernelGGL(prox_rows_wave_kernel<true>, grid, dim3(256), 0, stream, W, J, D, mode);
        else
            hipLaunchKernelGGL(prox_rows_wave_kernel<false>, grid, dim3(256), 0, stream, W, J, D, mode);
    } else {
        hipLaunchKernelGGL(prox_rows_kernel, dim3((unsigned)J), dim3(256), 0, stream, W, D, mode);
    }
    return hipGetLastError();
}

// Rows of W per workgroup of the power iteration: 16, more where that would be over 1024 workgroups.
static int power_rows(int64_t J)
{
    int64_t r = (J + 1023) / 1024;
    if (r < 16) r = 16;
    return (int)r;
}

int64_t power_chunks(int64_t J)
{
    const int64_t ch = (J + power_rows(J) - 1) / power_rows(J);
    return ch < 1 ? 1 : ch;
}

hipError_t launch_power_iteration(const float* W, int64_t J, int64_t D, int iters, float* scratch, float* spare, int64_t spare_floats,
                                  float* L_out, hipStream_t stream)
{
    const int rows = power_rows(J);
    if (rows > POWER_MAX_ROWS) return hipErrorInvalidValue;
    const int64_t chunks = power_chunks(J);
    float* b = scratch;                     // the start vector, then unused
    float* part = b + D + J;
    float* g = part + chunks * D;
    const float b0 = 1.0f / sqrtf((float)D);
    hipError_t e = launch_fill_u32(b, __builtin_bit_cast(uint32_t, b0), D, stream);
    if (e != hipSuccess) return e;
    auto aligned = [](const void* p) { return reinterpret_cast<uintptr_t>(p) % 16 == 0; };
    const bool vec = rows == 16 && D <= 1024 && D % 4 == 0 && J % 4 == 0 && aligned(W) && aligned(scratch) && aligned(spare);
    // Unaligned rows of up to a float a thread: power_step_kernel waits for nothing longer (ten iterations, us, it / the rows in
    // registers: 1000 x 61 82 / 98, 1000 x 255 97 / 104, 1000 x 301 112 / 106, 1000 x 1023 209 / 109).
    const bool in_registers = vec || (rows == 16 && D <= 1024 && D > 256);
    // One launch per iteration where a workgroup adds up the partials faster than a launch of its own (3 us) does, and with a
    // second array for them to alternate with: up to 128 KB of them in 16-byte loads, of rows that are not so short that the
    // adders of a column meet in a long chain (152 x 8 117 / 70 in two launches, 152 x 64 69 / 73); up to 20 KB otherwise
    // (152 x 301 91 / 97, 1000 x 301 155 / 106).
    const bool one_launch = in_registers && chunks > 1 && spare_floats >= chunks * D && (vec ? D >= 32 && chunks * D <= 32768 : chunks * D <= 5120);
    const float* from = b;
    int from_chunks = 1;
    for (int it = 0; it < iters; ++it) {
        float* const to = one_launch && (it & 1) ? spare : part;
        if (vec)
            hipLaunchKernelGGL(power_step16_kernel<true>, dim3((unsigned)chunks), dim3(256), 0, stream, W, from, from_chunks, to, J, D);
        else if (in_registers)
            hipLaunchKernelGGL(power_step16_kernel<false>, dim3((unsigned)chunks), dim3(256), 0, stream, W, from, from_chunks, to, J, D);
        else
            hipLaunchKernelGGL(power_step_kernel, dim3((unsigned)chunks), dim3(256), 0, stream, W, from, to, J, D, rows);
        if (one_launch) {
            from = to;
            from_chunks = (int)chunks;
        } else {
            hipLaunchKernelGGL(power_reduce_kernel, dim3((unsigned)((D + 15) / 16)), dim3(256), 0, stream, to, g, D, chunks);
            from = g;
        }
        e = hipGetLastError();
        if (e != hipSuccess) return e;
    }
    hipLaunchKernelGGL(vec_norm_kernel, dim3(1), dim3(1024), 0, stream, from, from_chunks, L_out, D);
    return hipGetLastError();
}

}  // namespace sfb
