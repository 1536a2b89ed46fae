// Frame stack: the last D observations of every env, resident in HBM.
//
// What it computes (paper, Section 5, "Memory limitations"): agents consume
// each env's last four 84x84 observations; the paper keeps them uncompressed
// and names compression as future work.  Here the ring of D observations per
// env lives in device memory, optionally packed to 4 bits per pixel (the
// gray level's top nibble, two pixels per byte).  A push after a step writes
// the step's observation into the env's ring -- into every slot when the
// env's episode ended (the new episode starts with D copies of its first
// observation) -- and writes the stacked observation [D][84][84], oldest
// first, each pixel the stored value widened back to 8 bits (identity for
// 8-bit storage, q * 17 for a 4-bit q).
#include "vcs_device.h"

namespace vcs {

struct StackArgs {
    uint8_t* ring;            // [num_envs][D][slot_bytes]
    uint8_t* head;            // [num_envs]: slot of the newest observation
    const int32_t* ids;       // NULL = position i is env i
    uint32_t n, num_envs, depth, bits;
    const uint8_t* obs;       // [n][84][84]
    const uint8_t* done;      // [n] or NULL
    uint8_t* out;             // [n][D][84][84] or NULL
};

// 4 pixels -> 4 nibbles (16 bits): pixel k's top nibble at bits 4k..4k+3
__device__ __forceinline__ uint32_t pack4(uint32_t w) {
    return ((w >> 4) & 0xF) | ((w >> 8) & 0xF0) | ((w >> 12) & 0xF00) | ((w >> 16) & 0xF000);
}
// 16 bits of nibbles -> 4 pixels, each q * 17
__device__ __forceinline__ uint32_t unpack4(uint32_t h) {
    const uint32_t w = (h & 0xF) | ((h & 0xF0) << 4) | ((h & 0xF00) << 8) | ((h & 0xF000) << 12);
    return w * 17u;   // 17 * q <= 255: no carry between bytes
}

// Pixels as a thread moves them (V, 16 or 4) and as a slot holds them (S).
__device__ __forceinline__ void store_form(uint4& d, const uint4 v) { d = v; }
__device__ __forceinline__ void store_form(uint2& d, const uint4 v) {
    d = make_uint2(pack4(v.x) | (pack4(v.y) << 16), pack4(v.z) | (pack4(v.w) << 16));
}
__device__ __forceinline__ void store_form(uint32_t& d, const uint32_t v) { d = v; }
__device__ __forceinline__ void store_form(uint16_t& d, const uint32_t v) { d = (uint16_t)pack4(v); }
__device__ __forceinline__ void pixels(uint4& v, const uint4 d) { v = d; }
__device__ __forceinline__ void pixels(uint4& v, const uint2 d) {
    v = make_uint4(unpack4(d.x & 0xFFFF), unpack4(d.x >> 16), unpack4(d.y & 0xFFFF), unpack4(d.y >> 16));
}
__device__ __forceinline__ void pixels(uint32_t& v, const uint32_t d) { v = d; }
__device__ __forceinline__ void pixels(uint32_t& v, const uint16_t d) { v = unpack4(d); }

// One workgroup per listed position; every thread moves its pixels of the
// observation and of all older slots, which it loads together.  Bound: HBM.
// An observation is 441 16-byte words, one per thread of 7 waves.  A push of
// 16,384 envs (8 bits, depth 4): 201 us, 5.2 TB/s, what a large copy reaches;
// by 4-byte words, with the newest slot read back from the ring, 266 us.
template <class V, class S>
__global__ void __launch_bounds__(448) k_stack(StackArgs A) {
    const uint32_t i = blockIdx.x;
    if (i >= A.n) return;
    const int32_t e = A.ids ? A.ids[i] : (int32_t)i;
    if (e < 0 || (uint32_t)e >= A.num_envs) return;      // invalid ids are left alone
    constexpr uint32_t kItems = kObsBytes / sizeof(V);
    const uint32_t D = A.depth;
    S* ring = reinterpret_cast<S*>(A.ring) + (size_t)e * D * kItems;
    const V* ob = reinterpret_cast<const V*>(A.obs + (size_t)i * kObsBytes);
    V* out = A.out ? reinterpret_cast<V*>(A.out + (size_t)i * D * kObsBytes) : nullptr;
    const bool fresh = A.done && A.done[i];
    const uint32_t old = A.head[e];
    const uint32_t h = fresh ? 0u : (old + 1 == D ? 0u : old + 1);
    __syncthreads();   // every thread has read the head before thread 0 moves it
    if (threadIdx.x == 0) A.head[e] = (uint8_t)h;
    for (uint32_t j = threadIdx.x; j < kItems; j += blockDim.x) {
        S held;
        store_form(held, ob[j]);
        V newest;
        pixels(newest, held);
        if (fresh) {                           // a new episode: its first observation in every slot
            for (uint32_t d = 0; d < D; ++d) {
                ring[d * kItems + j] = held;
                if (out) out[d * kItems + j] = newest;
            }
            continue;
        }
        if (out) {                             // oldest first: the slot after the newest
            for (uint32_t d0 = 0; d0 + 1 < D; d0 += 3) {
                S q[3];
#pragma unroll
                for (uint32_t k = 0; k < 3; ++k) {
                    uint32_t s = h + 1 + d0 + k;
                    s = s >= D ? s - D : s;
                    if (d0 + k + 1 < D) q[k] = ring[s * kItems + j];
                }
#pragma unroll
                for (uint32_t k = 0; k < 3; ++k) {
                    if (d0 + k + 1 >= D) continue;
                    V v;
                    pixels(v, q[k]);
                    out[(d0 + k) * kItems + j] = v;
                }
            }
            out[(D - 1) * kItems + j] = newest;
        }
        ring[h * kItems + j] = held;
    }
}

// 16-byte words where the caller's buffers allow them (the ring does: a slot
// is 441 x 16 or x 8 bytes), else 4-byte ones.
void launch_stack(uint8_t* ring, uint8_t* head, const int32_t* ids, uint32_t n, uint32_t num_envs, uint32_t depth,
                  uint32_t bits, const uint8_t* obs, const uint8_t* done, uint8_t* out, hipStream_t s) {
    StackArgs a{ring, head, ids, n, num_envs, depth, bits, obs, done, out};
    const bool wide = (((uintptr_t)obs | (uintptr_t)out) & 15) == 0;
    const dim3 grid(n), block(448);
    if (wide) {
        if (bits == 4) hipLaunchKernelGGL((k_stack<uint4, uint2>), grid, block, 0, s, a);
        else hipLaunchKernelGGL((k_stack<uint4, uint4>), grid, block, 0, s, a);
    } else {
        if (bits == 4) hipLaunchKernelGGL((k_stack<uint32_t, uint16_t>), grid, block, 0, s, a);
        else hipLaunchKernelGGL((k_stack<uint32_t, uint32_t>), grid, block, 0, s, a);
    }
}

}  // namespace vcs
