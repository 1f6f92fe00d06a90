// k_field.hip -- neural density field on gfx950 matrix cores.
//
// x -> 96 Fourier features [sin, cos](2 pi f_b x~_a) (f_b = 2^(0.6 b), b = 0..15) ->
// 4 x (64, ReLU) -> 1 -> softplus, trained by mean squared error on the
// normalised densities the method produces.  Every layer product is a chain of
// v_mfma_f32_32x32x16_bf16 (bf16 operands, fp32 accumulation) per wave of 32
// points, in the transposed form Z^T = W^T H^T: weights are the A operand (read
// from LDS), activations the B operand (registers).  The accumulator layout of
// one product (lane = point, rows 8q + 4h + r) is exactly the B-operand layout
// of the next one once the input features of each 16-wide k-step are visited
// in the slot order of slot_feature(); the packed weight image stores every
// matrix in that order, so activations never leave registers between layers.
// The backward pass reuses the same trick for dH = W dZ and takes the weight
// gradients dW = H dZ^T as MFMA products over the 32 points of a tile: the first kernel
// of a step leaves every tile's H and dZ in memory, transposed (features in rows) through
// per-wave LDS, and the second multiplies them tile by tile and adds the products in a
// fixed order (no atomics), so the gradient, and training, is the same bit for bit on every
// run.  The third adds the partial sums, takes the Adam step (Kingma and Ba 2015; fp32
// master weights and moments) and writes the BF16 image of the new weights.
#include <hip/hip_runtime.h>

#include <cstdint>

#include "gm_internal.h"
#include "gm_philox.h"

namespace gm {
namespace {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float f32x16 __attribute__((ext_vector_type(16)));
typedef short i16x8 __attribute__((ext_vector_type(8)));
typedef float f32x8 __attribute__((ext_vector_type(8)));
typedef unsigned u32x4 __attribute__((ext_vector_type(4)));

constexpr int kW = kFieldWidth;              // 64
constexpr int kS1 = 104;                     // LDS row stride (bf16) of the layer-1 weights, padded
constexpr int kSH = 72;                      // LDS row stride (bf16) of a 64-wide weight matrix, padded
constexpr int kOffF1 = 0;                    // forward operand of layer 1: [64 out][104]
constexpr int kMatH = kW * kSH * 2;          // bytes of one 64 x 64 operand
constexpr int kOffF2 = kOffF1 + kW * kS1 * 2;  // forward operands of layers 2..4: [64 out][72]
constexpr int kOffBias = kOffF2 + 3 * kMatH;   // fp32 b1..b4
constexpr int kOffW5 = kOffBias + 4 * kW * 4;  // fp32 w5
constexpr int kOffB5 = kOffW5 + kW * 4;        // fp32 b5 (+ padding)
constexpr int kInfer = kOffB5 + 16;
constexpr int kOffB2 = kInfer;                 // backward operands of layers 2..4: [64 in][72]
constexpr int kPack = kOffB2 + 3 * kMatH;
static_assert(kInfer % 16 == 0 && kPack % 16 == 0, "16-byte copies");

constexpr int kThreads = 256;
constexpr int kTileStride = 40;              // LDS row stride (bf16) of the per-wave 32-point tiles

// slot s of a 16-wide k-step -> feature offset inside the step (the accumulator
// rows 8q + 4h + r of one product, read as the operand of the next)
__host__ __device__ constexpr int slot_feature(int s)
{
    return (s & 7) < 4 ? 4 * (s >> 3) + (s & 7) : 8 + 4 * (s >> 3) + (s & 7) - 4;
}

// layer-1 input slot c = 16 ks + 8 h + j -> feature index 6 band + 2 axis + (sin 0 | cos 1)
__host__ __device__ constexpr int input_feature(int c)
{
    return 6 * ((8 * (c / 16) + c % 8) / 3) + 2 * ((8 * (c / 16) + c % 8) % 3) + (c % 16) / 8;
}

__device__ __forceinline__ f32x16 mfma(const bf16x8& a, const bf16x8& b, const f32x16& c)
{
    return __builtin_amdgcn_mfma_f32_32x32x16_bf16(a, b, c, 0, 0, 0);
}

__device__ __forceinline__ bf16x8 lds8(const unsigned char* base, int elem)
{
    return *reinterpret_cast<const bf16x8*>(base + 2 * elem);
}

struct Acts {
    bf16x8 x0[6];     // features, k-steps of layer 1
    bf16x8 h[4][4];   // hidden layers 1..4, k-steps of the next product
};

// log(1 + e) with e = exp(-|o|) in (0, 1], through the hardware exp2/log2: 1 + e rounds away
// at most 2^-24 of the sum, an absolute error below 1e-7 in the output
__device__ __forceinline__ float softplus(float o) { return fmaxf(o, 0.0f) + __logf(1.0f + __expf(-fabsf(o))); }

// The accumulators of a layer start from its bias (in the accumulator layout), so the
// products add onto it.
__device__ __forceinline__ void bias_init(const unsigned char* lds, int layer, int h, f32x16& a0, f32x16& a1)
{
    const float* bias = reinterpret_cast<const float*>(lds + kOffBias) + layer * kW;
#pragma unroll
    for (int v = 0; v < 16; ++v) {
        const int f = 8 * (v >> 2) + 4 * h + (v & 3);
        a0[v] = bias[f];
        a1[v] = bias[32 + f];
    }
}

// ReLU and BF16 rounding of a layer's accumulators into the next product's operand layout.
// The ReLU acts on the rounded values (the same bits as rounding after it: rounding keeps
// the sign), two at a time as 16-bit integers: a BF16 value is negative exactly when its
// sign bit is set, so max(bits, 0) zeroes the negative ones.
__device__ __forceinline__ bf16x8 relu_bf16x8(const f32x16& a, int v0)
{
    const f32x8 f = {a[v0], a[v0 + 1], a[v0 + 2], a[v0 + 3], a[v0 + 4], a[v0 + 5], a[v0 + 6], a[v0 + 7]};
    // the empty asm keeps the conversion and the max apart: combined, the compiler would
    // convert one value per instruction and repack the halves
    u32x4 u = __builtin_bit_cast(u32x4, __builtin_convertvector(f, bf16x8));
    asm("" : "+v"(u));
    return __builtin_bit_cast(bf16x8, __builtin_elementwise_max(__builtin_bit_cast(i16x8, u), i16x8{}));
}

__device__ __forceinline__ void relu_bf16(const f32x16& a0, const f32x16& a1, bf16x8 (&out)[4])
{
    out[0] = relu_bf16x8(a0, 0);
    out[1] = relu_bf16x8(a0, 8);
    out[2] = relu_bf16x8(a1, 0);
    out[3] = relu_bf16x8(a1, 8);
}

// Forward pass of the 32 points of a wave (lane & 31 = point, lane >> 5 = half).
// Returns the pre-softplus output o (same value in both halves).
__device__ __forceinline__ float field_forward(const unsigned char* lds, const FieldGeom& g, float x, float y,
                                               float z, int lane, Acts& A)
{
    const int n = lane & 31, h = lane >> 5;
    const float xt[3] = {(x - g.lo[0]) * g.inv_ext, (y - g.lo[1]) * g.inv_ext, (z - g.lo[2]) * g.inv_ext};
    // slot j of k-step ks: sin/cos pair p = 8 ks + j (band p / 3, axis p % 3); the lane
    // half picks sin (h = 0) or cos (h = 1), taken as sin of the phase + 1/4 revolution
    const float quarter = h ? 0.25f : 0.0f;
#pragma unroll
    for (int ks = 0; ks < 6; ++ks) {
#pragma unroll
        for (int j = 0; j < 8; ++j) {
            const int pr = 8 * ks + j;
            // revolutions, reduced to [0, 1) (the hardware sine takes a bounded range)
            const float rev = __builtin_amdgcn_fractf(__builtin_fmaf(g.freq[pr / 3], xt[pr % 3], quarter));
            A.x0[ks][j] = (__bf16)__builtin_amdgcn_sinf(rev);  // sin(2 pi rev)
        }
    }
    f32x16 c0, c1;
    bias_init(lds, 0, h, c0, c1);
#pragma unroll
    for (int ks = 0; ks < 6; ++ks) {
        c0 = mfma(lds8(lds + kOffF1, n * kS1 + 16 * ks + 8 * h), A.x0[ks], c0);
        c1 = mfma(lds8(lds + kOffF1, (32 + n) * kS1 + 16 * ks + 8 * h), A.x0[ks], c1);
    }
    relu_bf16(c0, c1, A.h[0]);
#pragma unroll
    for (int L = 1; L < 4; ++L) {
        const unsigned char* F = lds + kOffF2 + (L - 1) * kMatH;
        f32x16 d0, d1;
        bias_init(lds, L, h, d0, d1);
#pragma unroll
        for (int ks = 0; ks < 4; ++ks) {
            d0 = mfma(lds8(F, n * kSH + 16 * ks + 8 * h), A.h[L - 1][ks], d0);
            d1 = mfma(lds8(F, (32 + n) * kSH + 16 * ks + 8 * h), A.h[L - 1][ks], d1);
        }
        relu_bf16(d0, d1, A.h[L]);
    }
    const float* w5 = reinterpret_cast<const float*>(lds + kOffW5);
    float part = 0.0f;
#pragma unroll
    for (int ks = 0; ks < 4; ++ks)
#pragma unroll
        for (int j = 0; j < 8; ++j) part = __builtin_fmaf(w5[16 * ks + slot_feature(8 * h + j)], (float)A.h[3][ks][j], part);
    return part + __shfl_xor(part, 32, 64) + *reinterpret_cast<const float*>(lds + kOffB5);
}

// A workgroup's copy of the packed weights to LDS, ten 16-byte loads of a thread in flight
// before their stores (k_field_infer_routed 99 -> 97 us for 2,000,010 points; more of them
// cost registers that the caller needs).
template <int Threads, int Bytes>
__device__ __forceinline__ void stage(unsigned char* dst, const unsigned char* __restrict__ src)
{
    constexpr int kFull = Bytes / (16 * Threads);
    constexpr int kAtOnce = 10;
    const int t = 16 * (int)threadIdx.x;
    const int tail = 16 * kFull * Threads + t;
    uint4 last = make_uint4(0, 0, 0, 0);
    if (tail < Bytes) last = *reinterpret_cast<const uint4*>(src + tail);
#pragma unroll
    for (int g = 0; g < kFull; g += kAtOnce) {
        uint4 v[kAtOnce];
#pragma unroll
        for (int k = 0; k < kAtOnce; ++k)
            if (g + k < kFull) v[k] = *reinterpret_cast<const uint4*>(src + 16 * (g + k) * Threads + t);
#pragma unroll
        for (int k = 0; k < kAtOnce; ++k)
            if (g + k < kFull) *reinterpret_cast<uint4*>(dst + 16 * (g + k) * Threads + t) = v[k];
    }
    if (tail < Bytes) *reinterpret_cast<uint4*>(dst + tail) = last;
}

// ---------------------------------------------------------------------------
__global__ void k_field_pack(const float* __restrict__ p, unsigned char* __restrict__ blob, int64_t pack_stride)
{
    const int t = blockIdx.x * kThreads + threadIdx.x;
    p += (int64_t)blockIdx.y * kFieldParams;  // network blockIdx.y
    blob += (int64_t)blockIdx.y * pack_stride;
    __bf16* bf = reinterpret_cast<__bf16*>(blob);
    float* f32 = reinterpret_cast<float*>(blob);
    const int nF1 = kW * kS1, nH = kW * kSH;
    if (t < nF1) {  // layer 1: row = output, column = input slot
        const int i = t / kS1, c = t % kS1;
        bf[t] = (__bf16)(c < kFieldFeat ? p[kFieldOffW[1] + input_feature(c) * kW + i] : 0.0f);
        return;
    }
    int u = t - nF1;
    if (u < 3 * nH) {  // layers 2..4, forward: row = output, column slot -> input feature
        const int L = 2 + u / nH, r = u % nH, i = r / kSH, c = r % kSH;
        float v = 0.0f;
        if (c < kW) v = p[kFieldOffW[L] + (16 * (c / 16) + slot_feature(c % 16)) * kW + i];
        bf[kOffF2 / 2 + u] = (__bf16)v;
        return;
    }
    u -= 3 * nH;
    if (u < 3 * nH) {  // layers 2..4, backward: row = input, column slot -> output feature
        const int L = 2 + u / nH, r = u % nH, k = r / kSH, c = r % kSH;
        float v = 0.0f;
        if (c < kW) v = p[kFieldOffW[L] + k * kW + 16 * (c / 16) + slot_feature(c % 16)];
        bf[kOffB2 / 2 + u] = (__bf16)v;
        return;
    }
    u -= 3 * nH;
    if (u < 4 * kW) {
        f32[kOffBias / 4 + u] = p[kFieldOffB[1 + u / kW] + u % kW];
        return;
    }
    u -= 4 * kW;
    if (u < kW) {
        f32[kOffW5 / 4 + u] = p[kFieldOffW5 + u];
        return;
    }
    u -= kW;
    if (u < 4) f32[kOffB5 / 4 + u] = u == 0 ? p[kFieldOffB5] : 0.0f;
}
constexpr int kPackThreads = kW * kS1 + 6 * kW * kSH + 5 * kW + 4;

__global__ void __launch_bounds__(kThreads) k_field_infer(const unsigned char* __restrict__ blob, FieldGeom g,
                                                          const float* __restrict__ pos, int64_t q,
                                                          float* __restrict__ out, FieldRoute route)
{
    __shared__ __attribute__((aligned(16))) unsigned char s_blob[kInfer];
    stage<kThreads, kInfer>(s_blob, blob);
    __syncthreads();
    const int lane = __lane_id(), wave = threadIdx.x >> 6;
    const int64_t tiles = (q + 31) / 32;
    for (int64_t tile = (int64_t)blockIdx.x * (kThreads / 64) + wave; tile < tiles;
         tile += (int64_t)gridDim.x * (kThreads / 64)) {
        // keep the weights in LDS: without this the loop-invariant operand reads are
        // hoisted out of the tile loop and pin the whole weight set in registers
        asm volatile("" ::: "memory");
        const int64_t i = tile * 32 + (lane & 31);
        const bool ok = i < q;
        const int64_t ii = ok ? i : 0;
        Acts A;
        const float o = field_forward(s_blob, g, pos[3 * ii], pos[3 * ii + 1], pos[3 * ii + 2], lane, A);
        if (ok && lane < 32) {
            bool mine = route.m < 0;
            if (!mine) {
                int pm = -1;
                if (route.mesh) {
                    pm = route.mesh[i];
                } else if (route.tri) {
                    const int t = route.tri[i];
                    pm = t >= 0 && t < route.T ? route.tri_mesh[t] : -1;
                }
                mine = pm == route.m;
            }
            if (mine) out[i] = softplus(o);
        }
    }
}

// Routed inference: the points of every network are listed together, one segment per
// mesh in mesh order, each padded to a whole number of kGroup points, segment m starting
// at base[m] (route layout: base [M + 1], then start [M], then count [M]).  A mesh whose
// points already lie contiguously in the input (start[m] >= 0: they are
// start[m] .. start[m] + count[m] - 1, as for samples generated mesh by mesh) is read in
// place; the others through the index list ridx.  Every network evaluates only its own
// mesh's points, all networks in one launch.  A workgroup takes groups of kGroup points
// (one 32-point tile per wave) and stages the weights of the group's network, again only
// when the network changes (its groups run in mesh order).
constexpr int kGroup = 32 * (kThreads / 64);

__device__ __forceinline__ int group_mesh(const int64_t* __restrict__ base, int32_t M, int64_t first)
{
    int lo = 0, hi = M - 1;  // last m with base[m] <= first
    while (lo < hi) {
        const int mid = (lo + hi + 1) >> 1;
        if (base[mid] <= first) lo = mid; else hi = mid - 1;
    }
    return lo;
}

__global__ void __launch_bounds__(kThreads) k_field_infer_routed(const unsigned char* __restrict__ blobs,
                                                                 int64_t pack_stride,
                                                                 const FieldGeom* __restrict__ geoms,
                                                                 const float* __restrict__ pos,
                                                                 const int32_t* __restrict__ ridx,
                                                                 const int64_t* __restrict__ base, int32_t M,
                                                                 float* __restrict__ out)
{
    __shared__ __attribute__((aligned(16))) unsigned char s_blob[kInfer];
    const int lane = __lane_id(), wave = threadIdx.x >> 6;
    const int64_t groups = base[M] / kGroup;
    const int64_t* start = base + M + 1;
    const int64_t* count = base + 2 * M + 1;
    int staged = -1;
    FieldGeom g;
    // a contiguous run of groups per workgroup: it crosses at most a few mesh boundaries,
    // so the weights are staged about once per workgroup
    const int64_t g0 = groups * blockIdx.x / gridDim.x, g1 = groups * (blockIdx.x + 1) / gridDim.x;
    for (int64_t gi = g0; gi < g1; ++gi) {
        const int m = group_mesh(base, M, gi * kGroup);
        if (m != staged) {
            __syncthreads();
            stage<kThreads, kInfer>(s_blob, blobs + (int64_t)m * pack_stride);
            __syncthreads();
            staged = m;
            g = geoms[m];
        }
        asm volatile("" ::: "memory");  // weights stay in LDS (see k_field_infer)
        const int64_t slot = gi * kGroup + 32 * wave + (lane & 31);
        const int64_t off = slot - base[m];
        const int64_t s0 = start[m];
        const int64_t i = off >= count[m] ? -1 : s0 >= 0 ? s0 + off : (int64_t)ridx[slot];
        const int64_t ii = i >= 0 ? i : 0;
        Acts A;
        const float o = field_forward(s_blob, g, pos[3 * ii], pos[3 * ii + 1], pos[3 * ii + 2], lane, A);
        if (i >= 0 && lane < 32) out[i] = softplus(o);
    }
}

// point counts of the routed meshes: the point's mesh (mesh[i], or tri_mesh[tri[i]]), when
// it has a network and take[m] is set (NULL: every mesh)
__device__ __forceinline__ int route_mesh(const int32_t* __restrict__ mesh, const int32_t* __restrict__ tri,
                                          const int32_t* __restrict__ tri_mesh, int64_t T,
                                          const uint8_t* __restrict__ take, int32_t M, int64_t i)
{
    int m = -1;
    if (mesh) {
        m = mesh[i];
    } else if (tri) {
        const int t = tri[i];
        m = t >= 0 && t < T ? tri_mesh[t] : -1;
    }
    if (m < 0 || m >= M || (take && !take[m])) return -1;
    return m;
}

// Lanes of a wave that route to the same mesh take their slots with one atomic: the
// wave serves one mesh per round (the first pending lane's), so a wave of points of one
// mesh costs one atomic however many points share it.  Returns this lane's slot among
// the points of its mesh, counted from the value the atomic returned.
// With lo/hi set, the same round also keeps the smallest and largest point index of each
// mesh (lanes hold increasing indices i, so the first and last lane of a round have them).
__device__ __forceinline__ unsigned int wave_reserve(int m, unsigned int* __restrict__ ctr,
                                                     unsigned int* __restrict__ lo = nullptr,
                                                     unsigned int* __restrict__ hi = nullptr, int64_t i = 0)
{
    const int lane = __lane_id();
    uint64_t pending = __ballot(m >= 0);
    unsigned int mine = 0u;
    while (pending) {
        const int lead = __builtin_ctzll(pending);
        const int mm = __builtin_amdgcn_readlane(m, lead);
        const uint64_t same = __ballot(m == mm) & pending;
        if (lo) {
            if (lane == lead) atomicMin(&lo[mm], (unsigned int)i);
            if (lane == 63 - __builtin_clzll(same)) atomicMax(&hi[mm], (unsigned int)i);
        }
        unsigned int base = 0u;
        if (lane == lead) base = atomicAdd(&ctr[mm], (unsigned int)__popcll(same));
        base = __builtin_amdgcn_readlane(base, lead);
        if ((same >> lane) & 1ull) mine = base + (unsigned int)__popcll(same & ((1ull << lane) - 1ull));
        pending &= ~same;
    }
    return mine;
}

// Routing works on chunks of kRouteChunk points per workgroup: the chunk's per-mesh
// counts are gathered in LDS (one LDS atomic per wave and mesh) and added to the global
// ones with one atomic per mesh, so a few hundred global atomics route millions of points.
constexpr int kRouteChunk = 8 * kThreads;
constexpr int kRouteLds = 1024;  // meshes counted in LDS (more: one global atomic per wave and mesh)

__global__ void __launch_bounds__(kThreads) k_route_count(const int32_t* __restrict__ mesh,
                                                          const int32_t* __restrict__ tri,
                                                          const int32_t* __restrict__ tri_mesh, int64_t T,
                                                          const uint8_t* __restrict__ take, int32_t M, int64_t q,
                                                          unsigned int* __restrict__ cnt, unsigned int* __restrict__ part)
{
    // cnt: counts [M], then the smallest [M] and the largest [M] point index per mesh.  With
    // part set, the chunk stores its own three rows at part[chunk][3 M] instead (no two
    // chunks touch one address; k_route_reduce combines them)
    __shared__ unsigned int lc[3 * kRouteLds];
    const bool lds = M <= kRouteLds;
    unsigned int* c = lds ? lc : cnt;
    const int stride = lds ? kRouteLds : M;
    for (int m = threadIdx.x; lds && m < M; m += kThreads) {
        lc[m] = 0u;
        lc[kRouteLds + m] = 0xffffffffu;
        lc[2 * kRouteLds + m] = 0u;
    }
    __syncthreads();
    const int64_t c0 = (int64_t)blockIdx.x * kRouteChunk;
    constexpr int kPer = kRouteChunk / kThreads;
    int mm[kPer];
#pragma unroll
    for (int j = 0; j < kPer; ++j) {  // every load in flight before the first reservation
        const int64_t i = c0 + j * kThreads + threadIdx.x;
        mm[j] = i < q ? route_mesh(mesh, tri, tri_mesh, T, take, M, i) : -1;
    }
#pragma unroll
    for (int j = 0; j < kPer; ++j)
        (void)wave_reserve(mm[j], c, c + stride, c + 2 * stride, c0 + j * kThreads + threadIdx.x);
    __syncthreads();
    if (lds && part) {
        unsigned int* row = part + (int64_t)blockIdx.x * 3 * M;
        for (int m = threadIdx.x; m < M; m += kThreads) {
            row[m] = lc[m];
            row[M + m] = lc[kRouteLds + m];
            row[2 * M + m] = lc[2 * kRouteLds + m];
        }
        return;
    }
    for (int m = threadIdx.x; lds && m < M; m += kThreads)
        if (lc[m]) {
            atomicAdd(&cnt[m], lc[m]);
            atomicMin(&cnt[M + m], lc[kRouteLds + m]);
            atomicMax(&cnt[2 * M + m], lc[2 * kRouteLds + m]);
        }
}

__global__ void k_route_init(unsigned int* __restrict__ cnt, int32_t M)
{
    const int i = blockIdx.x * kThreads + threadIdx.x;
    if (i < 3 * M) cnt[i] = i >= M && i < 2 * M ? 0xffffffffu : 0u;
}

// one workgroup per mesh: its count, smallest and largest index over the chunks' rows
__global__ void __launch_bounds__(kThreads) k_route_reduce(const unsigned int* __restrict__ part, int64_t chunks,
                                                           int32_t M, unsigned int* __restrict__ cnt)
{
    __shared__ unsigned int rs[kThreads], rl[kThreads], rh[kThreads];
    const int m = blockIdx.x;
    unsigned int s = 0u, lo = 0xffffffffu, hi = 0u;
    for (int64_t c = threadIdx.x; c < chunks; c += kThreads) {
        const unsigned int* row = part + c * 3 * M;
        s += row[m];
        lo = min(lo, row[M + m]);
        hi = max(hi, row[2 * M + m]);
    }
    rs[threadIdx.x] = s; rl[threadIdx.x] = lo; rh[threadIdx.x] = hi;
    __syncthreads();
    for (int h = kThreads / 2; h > 0; h >>= 1) {
        if (threadIdx.x < h) {
            rs[threadIdx.x] += rs[threadIdx.x + h];
            rl[threadIdx.x] = min(rl[threadIdx.x], rl[threadIdx.x + h]);
            rh[threadIdx.x] = max(rh[threadIdx.x], rh[threadIdx.x + h]);
        }
        __syncthreads();
    }
    if (threadIdx.x == 0) {
        cnt[m] = rs[0];
        cnt[M + m] = rl[0];
        cnt[2 * M + m] = rh[0];
    }
}

// one thread: padded segment starts, the in-place start of every mesh whose points are
// contiguous in the input (largest - smallest index + 1 == count; else -1), the counts,
// and the per-mesh cursors cleared
__global__ void k_route_base(unsigned int* __restrict__ cnt, int32_t M, int64_t* __restrict__ base)
{
    if (blockIdx.x != 0 || threadIdx.x != 0) return;
    int64_t run = 0;
    for (int m = 0; m < M; ++m) {
        const int64_t c = cnt[m];
        base[m] = run;
        run += (c + kGroup - 1) / kGroup * kGroup;
        const bool contiguous = c > 0 && (int64_t)cnt[2 * M + m] - (int64_t)cnt[M + m] + 1 == c;
        base[M + 1 + m] = contiguous ? (int64_t)cnt[M + m] : -1;
        base[2 * M + 1 + m] = c;
        cnt[m] = 0u;
    }
    base[M] = run;
}

__global__ void __launch_bounds__(kThreads) k_route_scatter(const int32_t* __restrict__ mesh,
                                                            const int32_t* __restrict__ tri,
                                                            const int32_t* __restrict__ tri_mesh, int64_t T,
                                                            const uint8_t* __restrict__ take, int32_t M, int64_t q,
                                                            const int64_t* __restrict__ base,
                                                            unsigned int* __restrict__ cur,
                                                            int32_t* __restrict__ ridx)
{
    constexpr int kPer = kRouteChunk / kThreads;
    __shared__ unsigned int lc[kRouteLds];
    const bool lds = M <= kRouteLds;
    for (int m = threadIdx.x; lds && m < M; m += kThreads) lc[m] = 0u;
    __syncthreads();
    const int64_t c0 = (int64_t)blockIdx.x * kRouteChunk;
    int mm[kPer];
    unsigned int rank[kPer];
#pragma unroll
    for (int j = 0; j < kPer; ++j) {
        const int64_t i = c0 + j * kThreads + threadIdx.x;
        mm[j] = i < q ? route_mesh(mesh, tri, tri_mesh, T, take, M, i) : -1;
        if (mm[j] >= 0 && base[M + 1 + mm[j]] >= 0) mm[j] = -1;  // read in place: no list entry
        rank[j] = wave_reserve(mm[j], lds ? lc : cur);  // rank in the chunk (LDS) or the mesh (global)
    }
    __syncthreads();
    // the chunk's range of each mesh: one global atomic per mesh
    for (int m = threadIdx.x; lds && m < M; m += kThreads)
        lc[m] = lc[m] ? atomicAdd(&cur[m], lc[m]) : 0u;
    __syncthreads();
#pragma unroll
    for (int j = 0; j < kPer; ++j) {
        const int64_t i = c0 + j * kThreads + threadIdx.x;
        if (mm[j] >= 0) ridx[base[mm[j]] + (lds ? lc[mm[j]] : 0u) + rank[j]] = (int32_t)i;
    }
}

// ---------------------------------------------------------------------------
// One training step.  The batch is cut into tiles of 32 points, `slots` of them at a time:
// tile w + k slots is the k-th of slot w (usually there is one per slot).  The gradient of a
// parameter is the sum over the slots, each the sum of its tiles' in order, taken in eight
// rows of consecutive slots: every row in slot order, then the rows in order.  That order is
// fixed by (batch, networks) alone.
//
//   k_field_tiles  a wave per tile: forward, dZ of every layer, and to memory the features
//                  and hidden activations H and the dZ, BF16, features in rows (what the
//                  products below read), and the tile's sums for the biases and the output
//                  layer (kAux floats);
//   k_field_dw     a workgroup per (network, row, half layer), a wave per 32 x 32 block of
//                  the layer's weights: H dZ^T of each tile by two matrix products, added to
//                  the row's sum in slot order;
//   k_field_step   a thread per parameter: the rows, Adam, the new BF16 images.
//
// Only activations go through memory (35 KB a tile) instead of a whole gradient (75 KB a
// tile, written and read again): 4 networks x 16,384 points take 118 -> 43 us a step, one
// network 51 -> 38 us.
// ---------------------------------------------------------------------------
constexpr int kRows = 8;
// a workgroup stages a network's 70 KB image once for this many tiles (512 tiles on 256 CUs:
// 19.9 us with eight, 27.5 with four, 27.0 with two; 33 tiles: 15.0, 21.9, 22.0)
constexpr int kTileWaves = 8;
constexpr int kDzBytes = kW * 64;                  // one dZ or H of 64 features x 32 points
constexpr int kX0Bytes = kFieldFeat * 64;          // the 96 input features
constexpr int kOffDz = 0;                          // dZ of layers 1..4
constexpr int kOffX0 = 4 * kDzBytes;               // input features (slot order)
constexpr int kOffH = kOffX0 + kX0Bytes;           // hidden layers 1..3
constexpr int kOffAux = kOffH + 3 * kDzBytes;      // biases of layers 1..4, w5, b5
constexpr int kAux = 4 * kW + kW + 1;
constexpr int kTileBytes = kOffAux + (kAux + 3) / 4 * 16;

// row r, position q of a network: the tile, or -1; positions run through the row's slots,
// `rounds` tiles each; rows: those that hold slots
struct TileOrder {
    int32_t tiles, slots, used, per, rounds, rows;
};

__device__ __forceinline__ int tile_at(const TileOrder& o, int r, int q)
{
    const int w = r * o.per + q / o.rounds, k = q % o.rounds;
    if (w >= min(o.used, (r + 1) * o.per)) return -1;
    const int64_t tile = (int64_t)w + (int64_t)k * o.slots;
    return tile < o.tiles ? (int)tile : -1;
}

// A lane holds two neighbouring features of its point n, as packed BF16 (the even one low);
// it gets the two points n & ~1 and n | 1 of one feature, the even one in even lanes and the
// odd one in odd lanes: transposed rows are then written four bytes at a time.
__device__ __forceinline__ unsigned pair_points(unsigned x, unsigned sel)
{
    const unsigned y = __builtin_amdgcn_update_dpp(0, x, 0xB1, 0xf, 0xf, true);  // the neighbour's (quad_perm 1, 0, 3, 2)
    return __builtin_amdgcn_perm(y, x, sel);
}

// the pairs of a run of 8 features in registers, feature row0 + 0 .. 7 (row0 + 4 after every
// four when `split`: the accumulator's row order), put(row of the pair, value)
template <bool Split, class Put>
__device__ __forceinline__ void pairs8(const bf16x8& f, int row0, unsigned sel, const Put& put)
{
    const u32x4 u = __builtin_bit_cast(u32x4, f);
#pragma unroll
    for (int k = 0; k < 4; ++k) put(row0 + 2 * k + (Split && k >= 2 ? 4 : 0), pair_points(u[k], sel));
}

// 32 R feature rows of 32 points from LDS to memory, in the operand order of the products:
// per 32 rows 2 KB, [half of the points][half of those][row][8 points], so that both this
// wave's stores and the next kernel's loads are whole kilobytes
template <int R>
__device__ __forceinline__ void rows_out(const __bf16 (*tr)[kTileStride], unsigned char* dst, int lane)
{
#pragma unroll
    for (int c = 0; c < 2 * R; ++c) {
        const int row = 32 * (c >> 1) + (lane & 31), part = 2 * (c & 1) + (lane >> 5);
        *reinterpret_cast<uint4*>(dst + 1024 * c + 16 * lane) = *reinterpret_cast<const uint4*>(&tr[row][8 * part]);
    }
}

__global__ void __launch_bounds__(64 * kTileWaves) k_field_tiles(const unsigned char* __restrict__ blob, FieldGeom g,
                                                              FieldTrain t, FieldNets nets, TileOrder ord,
                                                              int q0, int Q, unsigned char* __restrict__ buf)
{
    const int net = blockIdx.y;
    if (nets.off) {
        // network blockIdx.y of several trained in one launch
        const int64_t c = nets.cnt[net];
        if (c == 0) return;
        blob += (int64_t)net * nets.pack_stride;
        g = nets.geom[net];
        t.idx += nets.off[net];
        t.n_idx = c;
        t.key0 ^= (uint32_t)(nets.first + net);
    }
    __shared__ __attribute__((aligned(16))) unsigned char s_blob[kPack];
    __shared__ __attribute__((aligned(16))) __bf16 s_tr[kTileWaves][kW][kTileStride];
    stage<64 * kTileWaves, kPack>(s_blob, blob);
    __syncthreads();
    const int lane = __lane_id(), wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int n = lane & 31, h = lane >> 5;
    const int b = blockIdx.x * kTileWaves + wave;  // row-major over (row, position)
    if (b >= ord.rows * Q) return;
    const int tile = tile_at(ord, b / Q, q0 + b % Q);
    if (tile < 0) return;
    unsigned char* out = buf + ((int64_t)net * ord.rows * Q + b) * kTileBytes;
    float* aux = reinterpret_cast<float*>(out + kOffAux);
    __bf16(*tr)[kTileStride] = s_tr[wave];
    const float* w5 = reinterpret_cast<const float*>(s_blob + kOffW5);
    const int64_t j = (int64_t)tile * 32 + n;
    const bool ok = j < t.batch;
    int64_t i = ok ? j : 0;
    if (t.idx) {
        uint32_t c0 = (uint32_t)j, c1 = t.step, c2 = 0u, c3 = 4u;
        philox4x32_10(c0, c1, c2, c3, t.key0, t.key1);
        i = t.idx[(int64_t)(((uint64_t)c0 * (uint64_t)t.n_idx) >> 32)];
    }
    Acts A;
    const float o = field_forward(s_blob, g, t.pos[3 * i], t.pos[3 * i + 1], t.pos[3 * i + 2], lane, A);
    const float y = softplus(o);
    const float diff = ok ? y - t.target[i] : 0.0f;
    const float dO = __fdividef(2.0f * diff * t.inv_batch, 1.0f + __expf(-o));  // d loss / d o
    // loss and the output bias' gradient, reduced over the 32 points of the wave
    float se = h == 0 ? diff * diff : 0.0f, sb = h == 0 ? dO : 0.0f;
#pragma unroll
    for (int d = 1; d < 32; d <<= 1) {
        se += __shfl_xor(se, d, 64);
        sb += __shfl_xor(sb, d, 64);
    }
    if (lane == 0) {
        t.se[(int64_t)net * ord.tiles + tile] = se;
        aux[5 * kW] = sb;
    }
    {
        // the output weights' gradients: 32 sums over the 32 points, the pairwise tree over
        // the lanes' bits; each step halves the values a lane still carries, so lane n ends
        // with the sum of the value whose index is n's bits reversed
        float v[32];
#pragma unroll
        for (int ks = 0; ks < 4; ++ks)
#pragma unroll
            for (int jj = 0; jj < 8; ++jj) v[8 * ks + jj] = (float)A.h[3][ks][jj] * dO;
#pragma unroll
        for (int d = 0; d < 5; ++d) {
            const int half = 16 >> d;
            const bool up = (n >> d) & 1;
#pragma unroll
            for (int k = 0; k < half; ++k) {
                const float keep = up ? v[half + k] : v[k], give = up ? v[k] : v[half + k];
                v[k] = keep + __shfl_xor(give, 1 << d, 64);
            }
        }
        const int idx = ((n & 1) << 4) | ((n & 2) << 2) | (n & 4) | ((n & 8) >> 2) | ((n & 16) >> 4);
        // value idx = 8 ks + jj is feature 16 ks + slot_feature(8 h + jj)
        const int sl = 8 * h + (idx & 7);
        aux[4 * kW + 16 * (idx >> 3) + ((sl & 7) < 4 ? 4 * (sl >> 3) + (sl & 7) : 8 + 4 * (sl >> 3) + (sl & 7) - 4)] = v[0];
    }
    // input features and hidden layers 1..3, transposed through the wave's LDS rows
    const unsigned sel = (n & 1) ? 0x03020706u : 0x05040100u;
    unsigned char* pt = reinterpret_cast<unsigned char*>(&tr[n & 1][n & 30]);
    const auto put8 = [pt, h](int row, unsigned v) { *reinterpret_cast<unsigned*>(pt + 2 * kTileStride * (row + 8 * h)) = v; };
    const auto put4 = [pt, h](int row, unsigned v) { *reinterpret_cast<unsigned*>(pt + 2 * kTileStride * (row + 4 * h)) = v; };
#pragma unroll
    for (int ks = 0; ks < 4; ++ks) pairs8<false>(A.x0[ks], 16 * ks, sel, put8);
    asm volatile("" ::: "memory");
    rows_out<2>(tr, out + kOffX0, lane);
    asm volatile("" ::: "memory");
#pragma unroll
    for (int ks = 4; ks < 6; ++ks) pairs8<false>(A.x0[ks], 16 * (ks - 4), sel, put8);
    asm volatile("" ::: "memory");
    rows_out<1>(tr, out + kOffX0 + kDzBytes, lane);
#pragma unroll
    for (int L = 0; L < 3; ++L) {
        asm volatile("" ::: "memory");
#pragma unroll
        for (int ks = 0; ks < 4; ++ks) pairs8<true>(A.h[L][ks], 16 * ks, sel, put4);
        asm volatile("" ::: "memory");
        rows_out<2>(tr, out + kOffH + L * kDzBytes, lane);
    }
    // dZ of layer 4 in the accumulator layout
    f32x16 dz0, dz1;
#pragma unroll
    for (int v = 0; v < 16; ++v) {
        const int f = 8 * (v >> 2) + 4 * h + (v & 3);
        dz0[v] = (float)A.h[3][v >> 3][v & 7] > 0.0f ? w5[f] * dO : 0.0f;
        dz1[v] = (float)A.h[3][2 + (v >> 3)][v & 7] > 0.0f ? w5[32 + f] * dO : 0.0f;
    }
#pragma unroll
    for (int L = 4; L >= 1; --L) {
        asm volatile("" ::: "memory");  // one layer at a time (bounds register pressure)
        bf16x8 dzb[4];
#pragma unroll
        for (int v = 0; v < 16; ++v) {
            dzb[v >> 3][v & 7] = (__bf16)dz0[v];
            dzb[2 + (v >> 3)][v & 7] = (__bf16)dz1[v];
        }
#pragma unroll
        for (int k = 0; k < 4; ++k) pairs8<true>(dzb[k], 16 * k, sel, put4);
        asm volatile("" ::: "memory");
        rows_out<2>(tr, out + kOffDz + (L - 1) * kDzBytes, lane);
        {
            // bias gradient: row sums of dZ over the points in order (lane = output feature)
            float sbias = 0.0f;
#pragma unroll
            for (int c = 0; c < 4; ++c) {
                const bf16x8 d8 = *reinterpret_cast<const bf16x8*>(&tr[lane][8 * c]);
#pragma unroll
                for (int k = 0; k < 8; ++k) sbias += (float)d8[k];
            }
            aux[(L - 1) * kW + lane] = sbias;
        }
        if (L >= 2) {
            const unsigned char* Bm = s_blob + kOffB2 + (L - 2) * kMatH;
            f32x16 e0 = {}, e1 = {};
#pragma unroll
            for (int ks = 0; ks < 4; ++ks) {
                e0 = mfma(lds8(Bm, n * kSH + 16 * ks + 8 * h), dzb[ks], e0);
                e1 = mfma(lds8(Bm, (32 + n) * kSH + 16 * ks + 8 * h), dzb[ks], e1);
            }
#pragma unroll
            for (int v = 0; v < 16; ++v) {
                dz0[v] = (float)A.h[L - 2][v >> 3][v & 7] > 0.0f ? e0[v] : 0.0f;
                dz1[v] = (float)A.h[L - 2][2 + (v >> 3)][v & 7] > 0.0f ? e1[v] : 0.0f;
            }
        }
    }
}

// Row sums of the gradients over positions [q0, q0 + Q) of every row, continuing from
// sums / part (the slot in progress; NULL: one pass or one tile a slot) when q0 > 0: the two halves of layers 1..4's outputs in
// blockIdx.z 0..7 (a wave per 32 of the layer's inputs), the biases and the output layer in 8
// and 9.
constexpr int kDwThreads = 192;

__global__ void __launch_bounds__(kDwThreads) k_field_dw(const unsigned char* __restrict__ buf, const int64_t* __restrict__ cnt,
                                                         TileOrder ord, int q0, int Q, float* __restrict__ sums,
                                                         float* __restrict__ part)
{
    const int r = blockIdx.x, net = blockIdx.y, layer = blockIdx.z >> 1, mb = blockIdx.z & 1;
    if (cnt && cnt[net] == 0) return;
    const unsigned char* tiles = buf + ((int64_t)net * ord.rows + r) * Q * kTileBytes;
    sums += ((int64_t)net * ord.rows + r) * kFieldParams;
    if (part) part += ((int64_t)net * ord.rows + r) * kFieldParams;
    const int lane = __lane_id(), wave = threadIdx.x >> 6;
    // positions of this pass in the row, where a slot is one tile
    const int m = max(0, min(Q, min(ord.used, (r + 1) * ord.per) - r * ord.per - q0));
    if (layer == 4) {
        const int p = mb * kDwThreads + threadIdx.x;
        if (p >= kAux) return;
        const int to = p < kW       ? kFieldOffB[1] + p
                       : p < 4 * kW ? kFieldOffB[2] + (p / kW - 1) * (kFieldOffB[3] - kFieldOffB[2]) + p % kW
                                    : kFieldOffW5 + p - 4 * kW;
        float sum = q0 > 0 ? sums[to] : 0.0f, v = q0 > 0 && part ? part[to] : 0.0f;
        const float* src = reinterpret_cast<const float*>(tiles + kOffAux) + p;
        if (ord.rounds == 1) {
            int q = 0;
            for (; q + 16 <= m; q += 16) {  // sixteen loads in flight, added in slot order
                float c[16];
#pragma unroll
                for (int k = 0; k < 16; ++k) c[k] = src[(int64_t)(q + k) * (kTileBytes / 4)];
#pragma unroll
                for (int k = 0; k < 16; ++k) sum += c[k];
            }
            for (; q < m; ++q) sum += src[(int64_t)q * (kTileBytes / 4)];
            sums[to] = sum;
            return;
        }
        for (int q = 0; q < Q; ++q) {
            const int tile = tile_at(ord, r, q0 + q);
            if (tile < 0) continue;
            const float c = src[(int64_t)q * (kTileBytes / 4)];
            v = (q0 + q) % ord.rounds == 0 ? c : v + c;
            if (tile_at(ord, r, q0 + q + 1) < 0 || (q0 + q + 1) % ord.rounds == 0) sum += v;
        }
        sums[to] = sum;
        if (part) part[to] = v;
        return;
    }
    const int nk = layer == 0 ? 3 : 2;
    const int nb = wave;
    if (nb >= nk) return;
    const int n = lane & 31, h = lane >> 5;
    const int krow = layer == 0 ? input_feature(nb * 32 + n) : nb * 32 + n;
    const int to = (layer == 0 ? kFieldOffW[1] : kFieldOffW[2] + (layer - 1) * (kFieldOffW[3] - kFieldOffW[2])) + krow * kW +
                   mb * 32 + 4 * h;
    const unsigned char* pa = tiles + kOffDz + layer * kDzBytes + mb * 2048 + 16 * lane;
    const unsigned char* pb = tiles + (layer == 0 ? kOffX0 : kOffH + (layer - 1) * kDzBytes) + nb * 2048 + 16 * lane;
    f32x16 sum = {}, v = {};
    if (q0 > 0) {
#pragma unroll
        for (int k = 0; k < 16; ++k) {
            sum[k] = sums[to + 8 * (k >> 2) + (k & 3)];
            if (part) v[k] = part[to + 8 * (k >> 2) + (k & 3)];
        }
    }
    if (ord.rounds == 1) {
        // one tile a slot: the operands of the next eight tiles are in flight
        constexpr int kAhead = 8;
        bf16x8 a[kAhead][2], b[kAhead][2];
#pragma unroll
        for (int u = 0; u < kAhead; ++u) {
            const int64_t at = (int64_t)min(u, max(m - 1, 0)) * kTileBytes;
#pragma unroll
            for (int kp = 0; kp < 2; ++kp) {
                a[u][kp] = *reinterpret_cast<const bf16x8*>(pa + at + 1024 * kp);
                b[u][kp] = *reinterpret_cast<const bf16x8*>(pb + at + 1024 * kp);
            }
        }
        for (int q = 0; q < m; q += kAhead) {
#pragma unroll
            for (int u = 0; u < kAhead; ++u) {
                f32x16 c = {};
                c = mfma(a[u][0], b[u][0], c);
                c = mfma(a[u][1], b[u][1], c);
                const int64_t at = (int64_t)min(q + u + kAhead, m - 1) * kTileBytes;
#pragma unroll
                for (int kp = 0; kp < 2; ++kp) {
                    a[u][kp] = *reinterpret_cast<const bf16x8*>(pa + at + 1024 * kp);
                    b[u][kp] = *reinterpret_cast<const bf16x8*>(pb + at + 1024 * kp);
                }
                if (q + u < m) {
#pragma unroll
                    for (int k = 0; k < 16; ++k) sum[k] += c[k];
                }
            }
        }
    } else {
        for (int q = 0; q < Q; ++q) {
            if (tile_at(ord, r, q0 + q) < 0) continue;
            const int64_t at = (int64_t)q * kTileBytes;
            f32x16 c = {};
#pragma unroll
            for (int kp = 0; kp < 2; ++kp)
                c = mfma(*reinterpret_cast<const bf16x8*>(pa + at + 1024 * kp), *reinterpret_cast<const bf16x8*>(pb + at + 1024 * kp), c);
            const bool first = (q0 + q) % ord.rounds == 0;
            const bool last = (q0 + q + 1) % ord.rounds == 0 || tile_at(ord, r, q0 + q + 1) < 0;
#pragma unroll
            for (int k = 0; k < 16; ++k) {
                v[k] = first ? c[k] : v[k] + c[k];
                if (last) sum[k] += v[k];
            }
        }
    }
#pragma unroll
    for (int k = 0; k < 16; ++k) {
        sums[to + 8 * (k >> 2) + (k & 3)] = sum[k];
        if (part) part[to + 8 * (k >> 2) + (k & 3)] = v[k];
    }
}

// the rows of a parameter in row order (0 for a row without slots)
__device__ __forceinline__ float row_total(const float* __restrict__ sums, int rows, int net, int p)
{
    const float* s = sums + (int64_t)net * rows * kFieldParams + p;
    float v[kRows];
#pragma unroll
    for (int r = 0; r < kRows; ++r) v[r] = r < rows ? s[(int64_t)r * kFieldParams] : 0.0f;
    float g = v[0];
#pragma unroll
    for (int r = 1; r < kRows; ++r) g += v[r];
    return g;
}

// loss[net]: every slot the sum of its tiles in order, thread i of the workgroup the slots i,
// i + kThreads, ... in order, then a fixed pairwise tree
__device__ __forceinline__ void total_loss(const float* __restrict__ se, const TileOrder& ord, bool live, double* __restrict__ loss)
{
    __shared__ double lrows[kThreads];
    double l = 0.0;
    for (int w = threadIdx.x; live && w < ord.used; w += kThreads) {
        double v = (double)se[w];
        for (int64_t tile = (int64_t)w + ord.slots; tile < ord.tiles; tile += ord.slots) v += (double)se[tile];
        l += v;
    }
    lrows[threadIdx.x] = l;
    __syncthreads();
    for (int h = kThreads / 2; h > 0; h >>= 1) {
        if (threadIdx.x < h) lrows[threadIdx.x] += lrows[threadIdx.x + h];
        __syncthreads();
    }
    if (threadIdx.x == 0) *loss = lrows[0];
}

__global__ void __launch_bounds__(kThreads) k_field_grad(const float* __restrict__ sums, const float* __restrict__ se, TileOrder ord,
                                                         float* __restrict__ grad, double* __restrict__ loss)
{
    const int p = blockIdx.x * kThreads + threadIdx.x;
    if (p < kFieldParams) grad[p] = row_total(sums, ord.rows, 0, p);
    if (blockIdx.x == 0) total_loss(se, ord, true, loss);
}

struct AdamStep {
    float lr, b1, b2, eps, c1, c2;
};

__device__ __forceinline__ float adam(float& p, float& m, float& v, float g, const AdamStep& a)
{
    const float mi = a.b1 * m + (1.0f - a.b1) * g;
    const float vi = a.b2 * v + (1.0f - a.b2) * g * g;
    m = mi;
    v = vi;
    p -= a.lr * (mi * a.c1) / (sqrtf(vi * a.c2) + a.eps);
    return p;
}

// where parameter p lies in the packed image: k_field_pack's inverse
__device__ __forceinline__ void pack_param(unsigned char* blob, int p, float x)
{
    __bf16* bf = reinterpret_cast<__bf16*>(blob);
    float* f32 = reinterpret_cast<float*>(blob);
    // feature -> slot of a 16-wide step (slot_feature's inverse)
    auto slot = [](int f) { return (f & 3) | ((f >> 3) << 2) | (((f >> 2) & 1) << 3); };
    if (p < kFieldOffB[1]) {
        const int k = p / kW, i = p % kW;  // feature index 6 band + 2 axis + (sin 0 | cos 1)
        const int pr = k / 2;              // 3 band + axis = 8 (c / 16) + c % 8
        bf[i * kS1 + 16 * (pr / 8) + 8 * (k & 1) + pr % 8] = (__bf16)x;
        return;
    }
    if (p >= kFieldOffW5) {
        if (p < kFieldOffB5) f32[kOffW5 / 4 + p - kFieldOffW5] = x;
        else f32[kOffB5 / 4] = x;
        return;
    }
    if (p < kFieldOffW[2]) {
        f32[kOffBias / 4 + p - kFieldOffB[1]] = x;
        return;
    }
    const int L = (p - kFieldOffW[2]) / (kFieldOffW[3] - kFieldOffW[2]), o = p - kFieldOffW[2] - L * (kFieldOffW[3] - kFieldOffW[2]);
    if (o >= kW * kW) {
        f32[kOffBias / 4 + (L + 1) * kW + o - kW * kW] = x;
        return;
    }
    const int k = o / kW, i = o % kW;
    bf[kOffF2 / 2 + L * kW * kSH + i * kSH + 16 * (k / 16) + slot(k % 16)] = (__bf16)x;
    bf[kOffB2 / 2 + L * kW * kSH + k * kSH + 16 * (i / 16) + slot(i % 16)] = (__bf16)x;
}

__global__ void __launch_bounds__(kThreads) k_field_step(const float* __restrict__ sums, const float* __restrict__ se,
                                                         const int64_t* __restrict__ cnt, TileOrder ord, AdamStep a,
                                                         float* __restrict__ master, float* __restrict__ m1,
                                                         float* __restrict__ m2, unsigned char* __restrict__ blob,
                                                         int64_t pack_stride, double* __restrict__ loss)
{
    const int net = blockIdx.y;
    const bool live = cnt[net] > 0;
    const int p = blockIdx.x * kThreads + threadIdx.x;
    if (p < kFieldParams) {
        const int64_t i = (int64_t)net * kFieldParams + p;
        float x = master[i], m = m1[i], v = m2[i];
        const float g = live ? row_total(sums, ord.rows, net, p) : 0.0f;
        x = adam(x, m, v, g, a);
        master[i] = x;
        m1[i] = m;
        m2[i] = v;
        pack_param(blob + (int64_t)net * pack_stride, p, x);
    }
    if (blockIdx.x == 0) total_loss(se + (int64_t)net * ord.tiles, ord, live, loss + net);
}

__global__ void k_field_adam(float* __restrict__ p, float* __restrict__ m, float* __restrict__ v,
                             float* __restrict__ grad, int64_t count, AdamStep a)
{
    const int64_t i = (int64_t)blockIdx.x * kThreads + threadIdx.x;
    if (i >= count) return;
    (void)adam(p[i], m[i], v[i], grad[i], a);
    grad[i] = 0.0f;
}

__global__ void k_field_split(int64_t n, uint32_t key0, uint32_t key1, uint32_t threshold, uint32_t* __restrict__ flag)
{
    const int64_t i = (int64_t)blockIdx.x * kThreads + threadIdx.x;
    if (i >= n) return;
    uint32_t c0 = (uint32_t)i, c1 = (uint32_t)(i >> 32), c2 = 0u, c3 = 3u;
    philox4x32_10(c0, c1, c2, c3, key0, key1);
    flag[i] = c0 >= threshold ? 1u : 0u;  // 1 = training, 0 = held out
}

__global__ void k_field_select(const uint32_t* __restrict__ flag, const int32_t* __restrict__ mesh, int32_t m,
                               int64_t n, uint32_t* __restrict__ sel)
{
    const int64_t i = (int64_t)blockIdx.x * kThreads + threadIdx.x;
    if (i < n) sel[i] = flag[i] && mesh[i] == m ? 1u : 0u;
}

__global__ void k_field_compact(const uint32_t* __restrict__ flag, const uint32_t* __restrict__ offs, int64_t n,
                                int32_t* __restrict__ idx)
{
    const int64_t i = (int64_t)blockIdx.x * kThreads + threadIdx.x;
    if (i < n && flag[i]) idx[offs[i]] = (int32_t)i;
}

// Held-out error sums per mesh, in a fixed order: workgroup (chunk, m) adds the squared
// error and squared target of the held-out points of mesh m in its chunk of kL2Chunk points
// (each thread its points in index order, then a fixed pairwise tree) into part[m][chunk];
// k_field_l2_sum adds the chunks of each mesh the same way.  No atomics: the gate decision
// is the same on every run.
constexpr int kL2Chunk = 16 * kThreads;

__device__ __forceinline__ void tree_sum2(double* a, double* b)
{
    for (int h = kThreads / 2; h > 0; h >>= 1) {
        if (threadIdx.x < h) {
            a[threadIdx.x] += a[threadIdx.x + h];
            b[threadIdx.x] += b[threadIdx.x + h];
        }
        __syncthreads();
    }
}

__global__ void __launch_bounds__(kThreads) k_field_l2(const float* __restrict__ pred, const float* __restrict__ target,
                                                       const int32_t* __restrict__ mesh,
                                                       const uint32_t* __restrict__ flag, int64_t n, int32_t M,
                                                       double* __restrict__ part)
{
    __shared__ double se[kThreads], st[kThreads];
    const int m = blockIdx.y;
    const int64_t c0 = (int64_t)blockIdx.x * kL2Chunk;
    double e = 0.0, s = 0.0;
#pragma unroll 4
    for (int j = 0; j < kL2Chunk / kThreads; ++j) {
        const int64_t i = c0 + j * kThreads + threadIdx.x;
        if (i < n && !flag[i] && mesh[i] == m) {
            const double d = (double)pred[i] - (double)target[i];
            e += d * d;
            s += (double)target[i] * (double)target[i];
        }
    }
    se[threadIdx.x] = e;
    st[threadIdx.x] = s;
    __syncthreads();
    tree_sum2(se, st);
    if (threadIdx.x == 0) {
        part[2 * ((int64_t)m * gridDim.x + blockIdx.x)] = se[0];
        part[2 * ((int64_t)m * gridDim.x + blockIdx.x) + 1] = st[0];
    }
}

__global__ void __launch_bounds__(kThreads) k_field_l2_sum(const double* __restrict__ part, int64_t chunks,
                                                           double* __restrict__ sums)
{
    __shared__ double se[kThreads], st[kThreads];
    const int m = blockIdx.x;
    double e = 0.0, s = 0.0;
    for (int64_t c = threadIdx.x; c < chunks; c += kThreads) {
        e += part[2 * (m * chunks + c)];
        s += part[2 * (m * chunks + c) + 1];
    }
    se[threadIdx.x] = e;
    st[threadIdx.x] = s;
    __syncthreads();
    tree_sum2(se, st);
    if (threadIdx.x == 0) {
        sums[2 * m] = se[0];
        sums[2 * m + 1] = st[0];
    }
}

__global__ void k_gate_flags(const int32_t* __restrict__ mesh, const int32_t* __restrict__ tri,
                             const int32_t* __restrict__ tri_mesh, int64_t T, const uint8_t* __restrict__ gate,
                             int32_t M, int64_t q, uint32_t* __restrict__ need)
{
    const int64_t i = (int64_t)blockIdx.x * kThreads + threadIdx.x;
    if (i >= q) return;
    int m = -1;
    if (mesh) m = mesh[i];
    else if (tri) {
        const int t = tri[i];
        if (t >= 0 && t < T) m = tri_mesh[t];
    }
    need[i] = (gate == nullptr || m < 0 || m >= M || gate[m] == 0) ? 1u : 0u;
}

__global__ void k_gather_points(const float* __restrict__ pos, const int32_t* __restrict__ tri,
                                const int32_t* __restrict__ mesh, const uint32_t* __restrict__ need,
                                const uint32_t* __restrict__ offs, int64_t q, float* __restrict__ gpos,
                                int32_t* __restrict__ gtri, int32_t* __restrict__ gmesh, int32_t* __restrict__ gidx)
{
    const int64_t i = (int64_t)blockIdx.x * kThreads + threadIdx.x;
    if (i >= q || !need[i]) return;
    const uint32_t j = offs[i];
    gpos[3 * j] = pos[3 * i];
    gpos[3 * j + 1] = pos[3 * i + 1];
    gpos[3 * j + 2] = pos[3 * i + 2];
    gtri[j] = tri ? tri[i] : -1;
    gmesh[j] = mesh ? mesh[i] : -1;
    gidx[j] = (int32_t)i;
}

__global__ void k_scatter_fallback(const float* __restrict__ rho, const int32_t* __restrict__ gidx, int64_t m,
                                   const float* __restrict__ norm, float* __restrict__ out)
{
    const int64_t j = (int64_t)blockIdx.x * kThreads + threadIdx.x;
    if (j >= m) return;
    const float d = *norm;
    out[gidx[j]] = d > 0.0f ? rho[j] / d : 0.0f;
}

__global__ void k_used_flags(const uint32_t* __restrict__ need, int64_t q, uint8_t* __restrict__ used)
{
    const int64_t i = (int64_t)blockIdx.x * kThreads + threadIdx.x;
    if (i < q) used[i] = (uint8_t)need[i];
}

inline unsigned blocks(int64_t n) { return (unsigned)((n + kThreads - 1) / kThreads); }

}  // namespace

size_t field_pack_bytes() { return kPack; }
size_t field_infer_bytes() { return kInfer; }

void launch_field_pack_nets(const float* master, unsigned char* blob, int32_t M, hipStream_t s)
{
    if (M > 0) k_field_pack<<<dim3(blocks(kPackThreads), (unsigned)M), kThreads, 0, s>>>(master, blob, kPack);
}

void launch_field_infer(const unsigned char* blob, const FieldGeom& g, const float* pos, int64_t q, float* out,
                        const FieldRoute& route, hipStream_t s)
{
    if (q <= 0) return;
    const int64_t tiles = (q + 31) / 32;
    const unsigned grid = (unsigned)std::min<int64_t>((tiles + 3) / 4, 2048);
    k_field_infer<<<grid, kThreads, 0, s>>>(blob, g, pos, q, out, route);
}

int64_t field_route_slots(int64_t q, int32_t M) { return q + (int64_t)kGroup * M; }

int64_t field_route_part_bytes(int64_t q, int32_t M)
{
    const int64_t chunks = (q + kRouteChunk - 1) / kRouteChunk;
    const int64_t b = chunks * 3 * (int64_t)M * 4;
    return M <= kRouteLds && b <= ((int64_t)64 << 20) ? b : 0;
}

void launch_field_infer_routed(const unsigned char* blobs, int64_t pack_stride, const FieldGeom* geoms,
                               const float* pos, int64_t q, float* out, const FieldRoute& route,
                               const uint8_t* take, int32_t M, unsigned int* cnt, unsigned int* part, int64_t* base,
                               int32_t* ridx, hipStream_t s)
{
    if (q <= 0 || M <= 0) return;
    const int64_t slots = field_route_slots(q, M);
    const unsigned chunks = (unsigned)((q + kRouteChunk - 1) / kRouteChunk);
    if (!part) k_route_init<<<blocks(3 * (int64_t)M), kThreads, 0, s>>>(cnt, M);
    k_route_count<<<chunks, kThreads, 0, s>>>(route.mesh, route.tri, route.tri_mesh, route.T, take, M, q, cnt, part);
    if (part) k_route_reduce<<<(unsigned)M, kThreads, 0, s>>>(part, chunks, M, cnt);
    k_route_base<<<1, 1, 0, s>>>(cnt, M, base);
    k_route_scatter<<<chunks, kThreads, 0, s>>>(route.mesh, route.tri, route.tri_mesh, route.T, take, M, q, base,
                                                   cnt, ridx);
    const unsigned grid = (unsigned)std::min<int64_t>(slots / kGroup + 1, 2048);
    k_field_infer_routed<<<grid, kThreads, 0, s>>>(blobs, pack_stride, geoms, pos, ridx, base, M, out);
}

void launch_field_select(const uint32_t* flag, const int32_t* mesh, int32_t m, int64_t n, uint32_t* sel, hipStream_t s)
{
    if (n > 0) k_field_select<<<blocks(n), kThreads, 0, s>>>(flag, mesh, m, n, sel);
}

namespace {

int64_t tiles_of(int32_t batch) { return ((int64_t)batch + 31) / 32; }

// The slots of a step (they set the order of its sums): one per tile up to 4,096 and to 1 /
// networks of 3,576 (a multiple of four, at least four).
int32_t train_slots(int32_t batch, int32_t M)
{
    const int64_t waves = kThreads / 64;
    const int64_t cap = std::max<int64_t>(1, ((int64_t)256 << 20) / ((int64_t)M * waves * kFieldParams * 4));
    const int64_t grid = std::min<int64_t>(std::min<int64_t>((tiles_of(batch) + waves - 1) / waves, 1024), cap);
    return (int32_t)(std::max<int64_t>(grid, 1) * waves);
}

TileOrder tile_order(int32_t batch, int32_t M)
{
    TileOrder o;
    o.tiles = (int32_t)tiles_of(batch);
    o.slots = train_slots(batch, M);
    o.used = std::min(o.tiles, o.slots);
    o.per = (o.used + kRows - 1) / kRows;
    o.rounds = (o.tiles + o.slots - 1) / o.slots;
    o.rows = (o.used + o.per - 1) / o.per;
    return o;
}

// How a step is cut: `nets` networks at a time, `positions` of each of their rows in a pass of the
// two kernels, so that a pass holds at most 8,192 tiles (285 MB) and 2,048 rows (154 MB of sums),
// or one position of one network's rows.  Whole networks come first: cut by positions alone, a
// pass of many networks holds a few tiles of each, and each stages its 70 KB image for them.  A
// step of 30 networks x 16,384 points 0.47 -> 0.42 ms, 300 x 1,024 0.98 -> 0.46, 1,000 x 256 2.72
// -> 0.67, 1,000 x 16,384 170 -> 13.7 (with 1.5 GB -> 0.3 GB of scratch).
struct TrainCut {
    int32_t nets, positions;
    int64_t all;  // positions of a row
    bool parts;   // a slot may be cut by a pass
};

TrainCut train_cut(const TileOrder& o, int32_t M)
{
    constexpr int64_t kPassTiles = 8192, kPassRows = 2048;
    TrainCut c;
    c.all = (int64_t)o.per * o.rounds;
    const int64_t most = std::min(kPassTiles / std::max<int64_t>(1, c.all * o.rows), kPassRows / o.rows);
    const int64_t groups = most > 0 ? (M + most - 1) / most : M;
    c.nets = (int32_t)((M + groups - 1) / groups);
    c.positions = (int32_t)std::min<int64_t>(c.all, std::max<int64_t>(1, kPassTiles / ((int64_t)o.rows * c.nets)));
    c.parts = c.positions < c.all && o.rounds > 1;
    return c;
}

// row sums of one step over M <= cut.nets networks
void launch_field_sums(const unsigned char* blob, const FieldGeom& g, const FieldTrain& t, const FieldNets& nets, int32_t M,
                       const TileOrder& o, const TrainCut& c, hipStream_t s)
{
    const int Q = c.positions;
    for (int64_t q0 = 0; q0 < c.all; q0 += Q) {
        const dim3 grid((unsigned)((o.rows * Q + kTileWaves - 1) / kTileWaves), (unsigned)M);
        k_field_tiles<<<grid, 64 * kTileWaves, 0, s>>>(blob, g, t, nets, o, (int)q0, Q, t.buf);
        k_field_dw<<<dim3((unsigned)o.rows, (unsigned)M, 10), kDwThreads, 0, s>>>(t.buf, nets.cnt, o, (int)q0, Q, t.sums,
                                                                                  c.parts ? t.part : nullptr);
    }
}

}  // namespace

void field_train_bytes(int32_t batch, int32_t M, size_t& buf, size_t& sums, size_t& part, size_t& se)
{
    const TileOrder o = tile_order(batch, M);
    const TrainCut c = train_cut(o, M);
    buf = (size_t)c.nets * (size_t)o.rows * (size_t)c.positions * kTileBytes;
    sums = (size_t)c.nets * (size_t)o.rows * kFieldParams * sizeof(float);
    part = c.parts ? sums : 0;
    se = (size_t)c.nets * (size_t)o.tiles * sizeof(float);
}

void launch_field_gradient(const unsigned char* blob, const FieldGeom& g, const FieldTrain& t, float* grad, double* loss,
                           hipStream_t s)
{
    if (t.batch <= 0) return;
    const TileOrder o = tile_order(t.batch, 1);
    launch_field_sums(blob, g, t, FieldNets{}, 1, o, train_cut(o, 1), s);
    k_field_grad<<<blocks(kFieldParams), kThreads, 0, s>>>(t.sums, t.se, o, grad, loss);
}

void launch_field_step(unsigned char* blob, const FieldNets& nets, int32_t M, const FieldTrain& t, float* master, float* m,
                       float* v, float lr, float b1, float b2, float eps, float c1, float c2, double* loss, hipStream_t s)
{
    if (t.batch <= 0 || M <= 0) return;
    const TileOrder o = tile_order(t.batch, M);
    const TrainCut c = train_cut(o, M);
    for (int32_t n0 = 0; n0 < M; n0 += c.nets) {
        const int32_t n = std::min(c.nets, M - n0);
        const int64_t p0 = (int64_t)n0 * kFieldParams;
        FieldNets some = nets;
        some.geom += n0;
        some.off += n0;
        some.cnt += n0;
        some.first = n0;
        unsigned char* image = blob + (int64_t)n0 * nets.pack_stride;
        launch_field_sums(image, FieldGeom{}, t, some, n, o, c, s);
        k_field_step<<<dim3(blocks(kFieldParams), (unsigned)n), kThreads, 0, s>>>(
            t.sums, t.se, some.cnt, o, AdamStep{lr, b1, b2, eps, c1, c2}, master + p0, m + p0, v + p0, image,
            nets.pack_stride, loss + n0);
    }
}

void launch_field_adam(float* master, float* m, float* v, float* grad, int64_t count, float lr, float b1, float b2,
                       float eps, float c1, float c2, hipStream_t s)
{
    if (count > 0)
        k_field_adam<<<blocks(count), kThreads, 0, s>>>(master, m, v, grad, count, AdamStep{lr, b1, b2, eps, c1, c2});
}

void launch_field_split(int64_t n, uint32_t key0, uint32_t key1, uint32_t threshold, uint32_t* flag, hipStream_t s)
{
    if (n > 0) k_field_split<<<blocks(n), kThreads, 0, s>>>(n, key0, key1, threshold, flag);
}

void launch_field_compact(const uint32_t* flag, const uint32_t* offs, int64_t n, int32_t* idx, hipStream_t s)
{
    if (n > 0) k_field_compact<<<blocks(n), kThreads, 0, s>>>(flag, offs, n, idx);
}

int64_t field_l2_part_bytes(int64_t n, int32_t M) { return 16 * ((n + kL2Chunk - 1) / kL2Chunk) * (int64_t)M; }

void launch_field_l2(const float* pred, const float* target, const int32_t* mesh, const uint32_t* flag, int64_t n,
                     int32_t M, double* part, double* sums, hipStream_t s)
{
    if (M <= 0) return;
    const int64_t chunks = (n + kL2Chunk - 1) / kL2Chunk;
    if (chunks > 0)
        k_field_l2<<<dim3((unsigned)chunks, (unsigned)M), kThreads, 0, s>>>(pred, target, mesh, flag, n, M, part);
    k_field_l2_sum<<<(unsigned)M, kThreads, 0, s>>>(part, chunks, sums);
}

void launch_gate_flags(const int32_t* mesh, const int32_t* tri, const int32_t* tri_mesh, int64_t T,
                       const uint8_t* gate, int32_t M, int64_t q, uint32_t* need, hipStream_t s)
{
    if (q > 0) k_gate_flags<<<blocks(q), kThreads, 0, s>>>(mesh, tri, tri_mesh, T, gate, M, q, need);
}

void launch_gather_points(const float* pos, const int32_t* tri, const int32_t* mesh, const uint32_t* need,
                          const uint32_t* offs, int64_t q, float* gpos, int32_t* gtri, int32_t* gmesh, int32_t* gidx,
                          hipStream_t s)
{
    if (q > 0) k_gather_points<<<blocks(q), kThreads, 0, s>>>(pos, tri, mesh, need, offs, q, gpos, gtri, gmesh, gidx);
}

void launch_scatter_fallback(const float* rho, const int32_t* gidx, int64_t m, const float* norm, float* out,
                             hipStream_t s)
{
    if (m > 0) k_scatter_fallback<<<blocks(m), kThreads, 0, s>>>(rho, gidx, m, norm, out);
}

void launch_used_flags(const uint32_t* need, int64_t q, uint8_t* used, hipStream_t s)
{
    if (q > 0) k_used_flags<<<blocks(q), kThreads, 0, s>>>(need, q, used);
}

}  // namespace gm
