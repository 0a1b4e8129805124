// Non-temporal 16-byte accesses to the logits and the mask rows, shared by the kernels that stream them.
#pragma once
#include <hip/hip_runtime.h>

#include <cstdint>

namespace pre3 {

// 16-byte accesses marked non-temporal: the logits pass through once, and lines marked this way
// are the first to leave L2, so the automaton's tables survive the pass for the next kernel.
typedef unsigned int NativeUint4 __attribute__((ext_vector_type(4)));
// Accesses may start at any logit (rows of an odd vocabulary do): the memory system takes 16-byte accesses at any
// address, and a wave's loads stay one contiguous 1 KiB (8 top-20 steps on 300 x 100,003: 393 us against 948 us
// with one load per logit; 8 greedy steps on 100 x 100,003: 170 against 254 us).
typedef NativeUint4 __attribute__((aligned(2))) NativeUint4AtLogit;
__device__ __forceinline__ uint4 stream_load(const uint16_t *p) {
    const NativeUint4 x = __builtin_nontemporal_load(reinterpret_cast<const NativeUint4AtLogit *>(p));
    return make_uint4(x.x, x.y, x.z, x.w);
}
// The same at a wave-uniform row plus a 32-bit byte offset per lane (no 64-bit address register per load).
__device__ __forceinline__ uint4 stream_load_at(const uint16_t *row, uint32_t byte_offset) {
    return stream_load(reinterpret_cast<const uint16_t *>(reinterpret_cast<const char *>(row) + byte_offset));
}
__device__ __forceinline__ void stream_store(uint4 v, uint16_t *p) {
    const NativeUint4 x = {v.x, v.y, v.z, v.w};
    __builtin_nontemporal_store(x, reinterpret_cast<NativeUint4AtLogit *>(p));
}

// The same store for a mask row: the row is read once, by the kernel that masks the logits, and
// lines that linger dirty in the writer's L2 slow that kernel down (B = 2,048: 232 us per step with
// plain stores of the mask rows against 209 us; B = 256: 35.0 against 34.6 us).
__device__ __forceinline__ void stream_store(uint4 v, uint4 *p) {
    const NativeUint4 x = {v.x, v.y, v.z, v.w};
    __builtin_nontemporal_store(x, reinterpret_cast<NativeUint4 *>(p));
}

// A row of logits (16-byte aligned) as a buffer of so many bytes: a load at an offset beyond it (kNowhere) reads nothing and
// returns zeros.  A load that only some lanes need is then one instruction without a branch, and the wave knows how many
// loads are in flight behind the one it waits for.
typedef __amdgpu_buffer_rsrc_t RowBuffer;
constexpr uint32_t kNowhere = 0xFFFFFFF0u;
__device__ __forceinline__ RowBuffer row_buffer(const uint16_t *row, uint32_t bytes) {
    constexpr int kRaw32Bit = 0x00020000, kNoStride = 0;
    return __builtin_amdgcn_make_buffer_rsrc(const_cast<uint16_t *>(row), kNoStride, (int)bytes, kRaw32Bit);
}
__device__ __forceinline__ uint4 buffer_load(RowBuffer row, uint32_t byte_offset) {
    constexpr int kNonTemporal = 2;
    const NativeUint4 x = __builtin_amdgcn_raw_buffer_load_b128(row, (int)byte_offset, 0, kNonTemporal);
    return make_uint4(x.x, x.y, x.z, x.w);
}

constexpr uint32_t kNegInfPair = 0xFF80FF80u;   // two bf16 -inf

}  // namespace pre3
