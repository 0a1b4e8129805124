// gfx950 kernel that masks the logits in place: one pass over the [batch, vocab] bf16 logits,
// bound by HBM bandwidth.
#include <hip/hip_runtime.h>

#include <cstdint>

#include "launch.hpp"
#include "stream_access.hpp"

namespace pre3 {

namespace {

constexpr int kApplyBlock = 256;
constexpr int kApplySpan = kApplyBlock * 8;            // logits per block
constexpr int64_t kMaskBytesInL2 = 16 << 20;            // masks up to this size are read where they were written (half of the L2s)

// One block per span of kApplySpan logits of one row.  kRowsByXcd = false: blockIdx.y = row,
// blockIdx.x = span.  kRowsByXcd = true (one-dimensional grid): workgroups go round-robin to the
// chip's eight XCDs in the order of their linear id, and the kernels that write the mask run row b
// in block b, that is on XCD b % 8 -- so block L takes a row of XCD L % 8's, and the mask bytes it
// reads are still in that XCD's L2 (B = 256: 34.8 -> 33.7 us per step, B = 1,024: 111.5 -> 109.0;
// a mask beyond the L2s gains nothing and the scattered rows cost 2 %, so large batches keep the
// two-dimensional grid).  A lane owns one group of 8 consecutive
// logits (16 bytes), so that every access of a wave is one contiguous 1 KiB.  Fully allowed groups
// are not touched, fully masked groups are overwritten without being read, mixed groups are read,
// patched and written back: the mask byte's bits become the AND masks of the group's four registers
// (sign-extending bit extracts, a byte permute), and one bit-select per register puts -inf where a
// bit is clear.  The kernel is bound by the turnover of its waves (a mask byte, then the logits,
// then the store) as much as by HBM: the fewer instructions a wave issues, the faster it runs, and
// variants that give a lane several groups -- 4 KiB apart or side by side -- were slower (26.6 us
// and 52.8 us against 23.6 us at B = 256, V = 128,256).
// kShifted: rows that do not all start on a 128-byte line (an odd vocabulary without padding starts every row at
// another 2-byte offset).  The lanes' groups are then counted from the line the row begins in, so that accesses stay
// 16-byte aligned and a line is still the groups of eight consecutive lanes; a group's mask bits straddle two
// mask bytes, and the row's first and last groups, which it shares with what lies around it, store their masked
// logits one by one.  96 rows of 100,003 logits: 10.2 us against 19.2 us with one lane per logit.
constexpr int kXcds = 8;
constexpr int kLineLogits = 64;
template <bool kRowsByXcd, bool kShifted>
__global__ __launch_bounds__(kApplyBlock) void apply_mask_vec8_kernel(uint16_t *__restrict__ logits,
                                                                     const uint32_t *__restrict__ bitmask,
                                                                     int vocab, int64_t row_stride, int n_words,
                                                                     int batch, int spans) {
    int b = blockIdx.y, span = blockIdx.x;
    if (kRowsByXcd) {
        const int xcd = blockIdx.x % kXcds, at = blockIdx.x / kXcds;
        b = (at / spans) * kXcds + xcd;
        span = at % spans;
        if (b >= batch) return;
    }
    const uint8_t *mask_bytes = reinterpret_cast<const uint8_t *>(bitmask + (size_t)b * n_words);   // little endian: byte g of the row = bits of group g
    uint16_t *row = logits + (size_t)b * row_stride;
    const int g = span * kApplyBlock + threadIdx.x;
    int t0 = g * 8;                                     // the group's first token
    if (kShifted) t0 -= (int)((reinterpret_cast<uintptr_t>(row) / 2) % kLineLogits);
    const bool inside = t0 >= 0 && t0 < vocab, whole = t0 >= 0 && t0 <= vocab - 8;
    uint32_t mu = 0xFFu;
    if (!kShifted) {
        if (inside) mu = mask_bytes[g];
    } else if (whole) {
        const int at = t0 >> 3, sh = t0 & 7;
        mu = mask_bytes[at];
        if (sh) mu = ((mu | (uint32_t)mask_bytes[at + 1] << 8) >> sh) & 0xFFu;   // token t0 + 7 lies in the second byte
    } else if (t0 > -8 && t0 < vocab) {                 // one end of the row
        for (int k = 0; k < 8; ++k) {
            const int t = t0 + k;
            if (t >= 0 && t < vocab && !((mask_bytes[t >> 3] >> (t & 7)) & 1u)) row[t] = 0xFF80;
        }
    }
    // a 128-byte line (the groups of eight consecutive lanes) is written whole or not at all: lines
    // written in part cost the memory system far more than the bytes saved
    const unsigned long long changed = __ballot(mu != 0xFFu);
    if (!(kShifted ? whole : inside) || !((changed >> (threadIdx.x & 56)) & 0xFFull)) return;
    uint16_t *p = row + t0;
    if (kShifted || whole) {
        uint4 v = make_uint4(0u, 0u, 0u, 0u);
        if (mu != 0u) v = stream_load(p);
        uint32_t *x = reinterpret_cast<uint32_t *>(&v);
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            const uint32_t lo = (uint32_t)__builtin_amdgcn_sbfe((int)mu, 2 * k, 1);        // all ones if the token is allowed
            const uint32_t hi = (uint32_t)__builtin_amdgcn_sbfe((int)mu, 2 * k + 1, 1);
            const uint32_t allow = __builtin_amdgcn_perm(hi, lo, 0x05040100u);              // low half from lo, high half from hi
            x[k] = (x[k] & allow) | (~allow & kNegInfPair);
        }
        stream_store(v, p);
    } else {
        for (int k = 0; t0 + k < vocab; ++k)
            if (!((mu >> k) & 1u)) p[k] = 0xFF80;
    }
}

__global__ void timestamp_kernel(int64_t *out) { *out = (int64_t)wall_clock64(); }

}  // namespace

hipError_t launch_timestamp(int64_t *out, hipStream_t stream) {
    hipLaunchKernelGGL(timestamp_kernel, dim3(1), dim3(1), 0, stream, out);
    return hipGetLastError();
}

template <bool kShifted>
static void launch_apply_rows(uint16_t *logits, const uint32_t *bitmask, int batch, int vocab, int64_t row_stride, int n_words,
                              hipStream_t stream) {
    const int spans = (vocab + (kShifted ? kLineLogits - 1 : 0) + kApplySpan - 1) / kApplySpan;
    const int64_t by_xcd = (int64_t)spans * kXcds * ((batch + kXcds - 1) / kXcds);
    if ((int64_t)batch * n_words * 4 <= kMaskBytesInL2)
        hipLaunchKernelGGL((apply_mask_vec8_kernel<true, kShifted>), dim3((unsigned)by_xcd), dim3(kApplyBlock), 0, stream, logits,
                           bitmask, vocab, row_stride, n_words, batch, spans);
    else
        hipLaunchKernelGGL((apply_mask_vec8_kernel<false, kShifted>), dim3(spans, batch), dim3(kApplyBlock), 0, stream, logits,
                           bitmask, vocab, row_stride, n_words, batch, spans);
}

hipError_t launch_apply_mask(uint16_t *logits, const uint32_t *bitmask, int batch, int vocab, int64_t row_stride,
                             hipStream_t stream) {
    if (batch == 0 || vocab == 0) return hipSuccess;
    const int n_words = (vocab + 31) / 32;
    const bool on_lines = (reinterpret_cast<uintptr_t>(logits) % (2 * kLineLogits) == 0) && (row_stride % kLineLogits == 0);
    constexpr int kRowsPerLaunch = 65528;               // the grid's second dimension ends at 65,535; a multiple of 8 keeps rows on their XCD
    for (int first = 0; first < batch; first += kRowsPerLaunch) {
        const int rows = batch - first < kRowsPerLaunch ? batch - first : kRowsPerLaunch;
        uint16_t *lo = logits + (size_t)first * row_stride;
        const uint32_t *mo = bitmask + (size_t)first * n_words;
        if (on_lines) launch_apply_rows<false>(lo, mo, rows, vocab, row_stride, n_words, stream);
        else launch_apply_rows<true>(lo, mo, rows, vocab, row_stride, n_words, stream);
    }
    return hipGetLastError();
}

}  // namespace pre3
