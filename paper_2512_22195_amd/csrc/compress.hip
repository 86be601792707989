// Compressed form of a materialized chunk blob (the paper names KV compression as its lever on
// storage cost and load time, Section III-C; the scheme is this library's): per (layer, K or V,
// KV head) one power-of-two scale s - the smallest with max|x| <= 448 s - and per element the
// E4M3 code (OCP FP8: 4 exponent bits of bias 7, 3 mantissa bits, no infinities, largest value
// 448) of x / s, rounded to nearest even by the hardware conversion.  x / s is exact in fp32, so
// the codes depend on nothing but the format.  HBM bound.  A head of up to 1024 tokens (256 KB)
// is held in the registers of its workgroup between the two passes - every load of the launch is
// requested before anything is consumed, and the blob is read once; longer heads are read twice
// (the second time from the last-level cache).  Written once at half the size.
#include <algorithm>

#include "matkv_internal.h"

namespace matkv {
namespace {

__device__ __forceinline__ uint32_t max_mag2(uint32_t acc, uint32_t w) {
    // two bf16 per word: magnitudes order like their bit patterns
    return max(acc, max(w & 0x7fffu, (w >> 16) & 0x7fffu));
}

// Scale exponent k of a head whose largest magnitude has the bf16 pattern amax (s = 2^k).
__device__ __forceinline__ int scale_exponent(uint32_t amax) {
    // amax = f 2^E, f in [1, 2): 448 = 1.75 * 2^8, so s = 2^(E - 8) if f <= 1.75, else 2^(E - 7)
    if (amax == 0) return 0;
    const int E = (int)(amax >> 7) - 127, m7 = (int)(amax & 0x7f);
    return max(m7 <= 96 ? E - 8 : E - 7, -60);            // floor 2^-60 (a subnormal amax lands there too)
}
__device__ __forceinline__ uint2 encode8(const uint4& v, float inv) {
    const uint32_t w[4] = {v.x, v.y, v.z, v.w};
    int lo = 0, hi = 0;
    lo = __builtin_amdgcn_cvt_pk_fp8_f32(__uint_as_float(w[0] << 16) * inv, __uint_as_float(w[0] & 0xffff0000u) * inv, lo, false);
    lo = __builtin_amdgcn_cvt_pk_fp8_f32(__uint_as_float(w[1] << 16) * inv, __uint_as_float(w[1] & 0xffff0000u) * inv, lo, true);
    hi = __builtin_amdgcn_cvt_pk_fp8_f32(__uint_as_float(w[2] << 16) * inv, __uint_as_float(w[2] & 0xffff0000u) * inv, hi, false);
    hi = __builtin_amdgcn_cvt_pk_fp8_f32(__uint_as_float(w[3] << 16) * inv, __uint_as_float(w[3] & 0xffff0000u) * inv, hi, true);
    return make_uint2((uint32_t)lo, (uint32_t)hi);
}

// Heads of more than 1024 tokens, in two launches: the largest magnitude of every piece of a head, then, from those of its head,
// a piece's codes.  A workgroup per head, which read it twice, left most of the chip idle and had one load per thread in flight:
// four layers of the 8B shape 164 us of a 3501-token chunk's pass, 64 of a 2000-token one's, 37 of a 1030-token one's; now 22, 11 and
// 7.  (Heads that fit the registers stay there: eight layers of 1000 tokens 14.6 us against 16.6 this way, 32 layers 45 against 58;
// up to four layers the two are equal.  These are blobs from HBM; one that the last-level cache still holds takes 10.3 and 32.1.)
// A piece is 4096 vectors of eight values (64 KB); a workgroup takes every gridDim.x-th.
constexpr int NTP = 512, NVP = 8;
__device__ __forceinline__ void load_piece(const uint4* src, size_t first, size_t n_vec, uint4 (&v)[NVP]) {
#pragma unroll
    for (int u = 0; u < NVP; ++u) v[u] = src[min(first + u * NTP + threadIdx.x, n_vec - 1)];      // past the end: the last vector again
}
__global__ __launch_bounds__(NTP) void compress_max_kernel(const uint16_t* __restrict__ blob, uint32_t* __restrict__ maxima, size_t head_elems) {
    const size_t head = (size_t)blockIdx.z * gridDim.y + blockIdx.y, n_vec = head_elems / 8;
    const uint4* const src = reinterpret_cast<const uint4*>(blob + head * head_elems);
    uint32_t amax = 0;
    for (size_t first = (size_t)blockIdx.x * (NTP * NVP); first < n_vec; first += (size_t)gridDim.x * (NTP * NVP)) {
        uint4 v[NVP];
        load_piece(src, first, n_vec, v);
#pragma unroll
        for (int u = 0; u < NVP; ++u) amax = max_mag2(max_mag2(max_mag2(max_mag2(amax, v[u].x), v[u].y), v[u].z), v[u].w);
    }
#pragma unroll
    for (int off = 32; off >= 1; off >>= 1) amax = max(amax, (uint32_t)__shfl_xor((int)amax, off));
    __shared__ uint32_t sm[NTP / 64];
    if ((threadIdx.x & 63) == 0) sm[threadIdx.x >> 6] = amax;
    __syncthreads();
    if (threadIdx.x == 0) {
#pragma unroll
        for (int w = 1; w < NTP / 64; ++w) amax = max(amax, sm[w]);
        maxima[head * gridDim.x + blockIdx.x] = amax;
    }
}
// out, scales: of the launch's first head.
__global__ __launch_bounds__(NTP) void compress_codes_kernel(const uint16_t* __restrict__ blob, const uint32_t* __restrict__ maxima, uint8_t* __restrict__ out,
                                                             float* __restrict__ scales, size_t head_elems) {
    const size_t head = (size_t)blockIdx.z * gridDim.y + blockIdx.y, n_vec = head_elems / 8;
    const uint4* const src = reinterpret_cast<const uint4*>(blob + head * head_elems);
    uint2* const dst = reinterpret_cast<uint2*>(out + head * head_elems);
    uint4 v[NVP];
    size_t first = (size_t)blockIdx.x * (NTP * NVP);
    load_piece(src, first, n_vec, v);
    uint32_t amax = 0;
    for (unsigned p = threadIdx.x & 63; p < gridDim.x; p += 64) amax = max(amax, maxima[head * gridDim.x + p]);
#pragma unroll
    for (int off = 32; off >= 1; off >>= 1) amax = max(amax, (uint32_t)__shfl_xor((int)amax, off));
    const int k = scale_exponent(amax);
    const float inv = __uint_as_float((uint32_t)(127 - k) << 23);
    if (blockIdx.x == 0 && threadIdx.x == 0) scales[head] = __uint_as_float((uint32_t)(127 + k) << 23);
    for (;;) {
#pragma unroll
        for (int u = 0; u < NVP; ++u) {
            const size_t i = first + u * NTP + threadIdx.x;
            if (i < n_vec) dst[i] = encode8(v[u], inv);
        }
        first += (size_t)gridDim.x * (NTP * NVP);
        if (first >= n_vec) break;
        load_piece(src, first, n_vec, v);
    }
}

// Heads of at most NV * 512 vectors of eight values: the whole head in registers.
constexpr int NTR = 512, NV = 32;
__global__ __launch_bounds__(NTR) void compress_resident_kernel(const uint16_t* __restrict__ blob, uint8_t* __restrict__ out,
                                                                size_t head_elems, size_t scales_off) {
    const int kvh = blockIdx.x, kv = blockIdx.y, layer = blockIdx.z;
    const size_t head = ((size_t)layer * 2 + kv) * gridDim.x + kvh;
    const uint4* src = reinterpret_cast<const uint4*>(blob + head * head_elems);
    uint2* dst = reinterpret_cast<uint2*>(out + head * head_elems);
    const int n_vec = (int)(head_elems / 8);              // at most NV * NTR (checked by the launcher)

    uint4 v[NV];
#pragma unroll
    for (int u = 0; u < NV; ++u) v[u] = src[min(u * NTR + (int)threadIdx.x, n_vec - 1)];   // past the end: the last vector again
    uint32_t amax = 0;
#pragma unroll
    for (int u = 0; u < NV; ++u) amax = max_mag2(max_mag2(max_mag2(max_mag2(amax, v[u].x), v[u].y), v[u].z), v[u].w);
#pragma unroll
    for (int off = 32; off >= 1; off >>= 1) amax = max(amax, (uint32_t)__shfl_xor((int)amax, off));
    __shared__ uint32_t sm[NTR / 64];
    if ((threadIdx.x & 63) == 0) sm[threadIdx.x >> 6] = amax;
    __syncthreads();
    amax = sm[0];
#pragma unroll
    for (int w = 1; w < NTR / 64; ++w) amax = max(amax, sm[w]);

    const int k = scale_exponent(amax);
    const float inv = __uint_as_float((uint32_t)(127 - k) << 23);
    if (threadIdx.x == 0)
        reinterpret_cast<float*>(out + scales_off)[head] = __uint_as_float((uint32_t)(127 + k) << 23);
#pragma unroll
    for (int u = 0; u < NV; ++u) {
        const int i = u * NTR + (int)threadIdx.x;
        if (i < n_vec) dst[i] = encode8(v[u], inv);
    }
}

}  // namespace

hipError_t launch_compress(const void* blob, void* out, int n_layers, int Hkv, int n_tokens, int D, float* scratch, size_t scratch_floats, hipStream_t s) {
    const size_t head_elems = (size_t)n_tokens * D, n_vec = head_elems / 8;
    const size_t scales_off = ((size_t)n_layers * 2 * Hkv * head_elems + 15) & ~(size_t)15;
    const uint16_t* const from = reinterpret_cast<const uint16_t*>(blob);
    uint8_t* const to = reinterpret_cast<uint8_t*>(out);
    if (n_vec <= (size_t)NV * NTR) {
        hipLaunchKernelGGL(compress_resident_kernel, dim3(Hkv, 2, n_layers), dim3(NTR), 0, s, from, to, head_elems, scales_off);
        return hipGetLastError();
    }
    // As many layers at a time as half of the last-level cache holds, so that the second launch finds there what the first one read
    // (and as scratch has places for the maxima).
    const size_t heads = 2 * (size_t)Hkv, layer_bytes = heads * head_elems * 2;
    const size_t pieces = std::max<size_t>(std::min({(n_vec + NTP * NVP - 1) / (NTP * NVP), scratch_floats / heads, (size_t)65535}), 1);
    const size_t group = std::max<size_t>(std::min({kLastLevelCacheBytes / 2 / layer_bytes, scratch_floats / (heads * pieces), (size_t)n_layers}), 1);
    uint32_t* const maxima = reinterpret_cast<uint32_t*>(scratch);
    for (size_t l = 0; l < (size_t)n_layers; l += group) {
        const dim3 grid((unsigned)pieces, (unsigned)heads, (unsigned)std::min(group, n_layers - l));
        const size_t first = l * heads;
        hipLaunchKernelGGL(compress_max_kernel, grid, dim3(NTP), 0, s, from + first * head_elems, maxima, head_elems);
        hipLaunchKernelGGL(compress_codes_kernel, grid, dim3(NTP), 0, s, from + first * head_elems, maxima, to + first * head_elems,
                           reinterpret_cast<float*>(to + scales_off) + first, head_elems);
    }
    return hipGetLastError();
}

}  // namespace matkv
