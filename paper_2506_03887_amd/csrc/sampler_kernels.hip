// gfx950 kernels that sample behind the mask: the greedy choice and the k best among the allowed
// tokens.  Both read the [batch, vocab] bf16 logits once and write nothing back.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cstdint>

#include "argmax.hpp"
#include "launch.hpp"
#include "stream_access.hpp"

namespace pre3 {

namespace {

// ------------------------------------------------------------------- masked argmax

constexpr int kArgUnroll = 4;

// Greedy choice among the allowed tokens without writing the masked logits back: a row's logits
// are read once (groups of 8 whose mask byte is zero are not read at all).  blockIdx.x = row,
// blockIdx.y = segment of the row.  The stream is bound by instruction issue as much as by HBM, so
// the inner loop does as little as it can per token: the two bf16 patterns of a register become
// two signed 16-bit order keys with packed arithmetic (masked halves get the lowest key; the mask
// byte of a group expands to its four AND masks through a 4 KB table in LDS), packed maxima fold a
// group of 8 into its largest key, and only when that beats the lane's best so far (strictly: the
// first of equal values stays) the lane keeps the key, the group's index, registers and mask byte.
// At the end a lane finds its winner's position inside the kept group; lanes, waves and segments
// are combined through argmax_word.  Two cases the keys cannot decide are left to
// argmax_segment_by_compare, for the whole segment: a positive NaN pattern has a key above +inf's
// (the block's best key shows it), and -0 and +0 have different keys but are equal values (the
// block's best value is zero).  With one segment per row the block writes out[b] itself; otherwise
// it stores its word in partial[b][segment] and masked_argmax_finish_kernel combines the segments.
// (Combining them inside this kernel with device-scope atomics and a last-arrival counter was
// measured: rows that finish early then cost tens of microseconds per launch.)  The mask bytes of
// the next pass are fetched while the logits of the current one are in flight.
__global__ __launch_bounds__(kArgBlock) void masked_argmax_kernel(
    const uint16_t *__restrict__ logits, const uint32_t *__restrict__ bitmask, int vocab, int64_t row_stride,
    int n_words, int groups_per_seg, unsigned long long *__restrict__ partial, int32_t *__restrict__ out) {
    __shared__ unsigned long long s_part[kArgBlock / 64 + 1];
    __shared__ uint2 s_expand[16];                      // half a mask byte -> AND masks of two of the group's registers
    const int b = blockIdx.x, seg = blockIdx.y, n_seg = gridDim.y, tid = threadIdx.x;
    const int groups = (vocab + 7) >> 3;
    const int g_lo = seg * groups_per_seg, g_hi = min(groups, g_lo + groups_per_seg);
    const uint8_t *mrow = reinterpret_cast<const uint8_t *>(bitmask + (size_t)b * n_words);
    const uint16_t *lrow = logits + (size_t)b * row_stride;
    mask_nibble_table_init(s_expand, tid);
    int best = kOrderNegInf - 1, best_g = -1;           // only a valid value (or a positive NaN pattern) beats the start
    uint4 best_x = make_uint4(0, 0, 0, 0);
    uint32_t best_m = 0u;
    uint32_t m[kArgUnroll], m_next[kArgUnroll];
#pragma unroll
    for (int u = 0; u < kArgUnroll; ++u) {
        const int g = g_lo + tid + u * kArgBlock;
        m[u] = g < g_hi ? mrow[g] : 0u;
    }
    __syncthreads();                                    // s_expand
    for (int g0 = g_lo + tid; g0 < g_hi; g0 += kArgBlock * kArgUnroll) {
        uint4 v[kArgUnroll];
#pragma unroll
        for (int u = 0; u < kArgUnroll; ++u) {
            const int g = g0 + u * kArgBlock;
            if (m[u] != 0u && g * 8 + 8 <= vocab) v[u] = stream_load(lrow + (size_t)g * 8);
        }
#pragma unroll
        for (int u = 0; u < kArgUnroll; ++u) {
            const int g = g0 + kArgBlock * kArgUnroll + u * kArgBlock;
            m_next[u] = g < g_hi ? mrow[g] : 0u;
        }
#pragma unroll
        for (int u = 0; u < kArgUnroll; ++u) {
            uint32_t mu = m[u];
            if (mu == 0u) continue;
            const int g = g0 + u * kArgBlock, t0 = g * 8;
            if (t0 + 8 > vocab) {                      // ragged tail: one logit at a time
                uint32_t x[4] = {0u, 0u, 0u, 0u};
                mu &= (1u << (vocab - t0)) - 1u;
                for (int k = 0; k < 8 && t0 + k < vocab; ++k) x[k >> 1] |= (uint32_t)lrow[t0 + k] << (16 * (k & 1));
                v[u] = make_uint4(x[0], x[1], x[2], x[3]);
                if (mu == 0u) continue;
            }
            const uint4 allow = expand_mask_byte(s_expand, mu);
            const uint32_t k01 = packed_max_s16(bf16_order_pair(v[u].x, allow.x), bf16_order_pair(v[u].y, allow.y));
            const uint32_t k23 = packed_max_s16(bf16_order_pair(v[u].z, allow.z), bf16_order_pair(v[u].w, allow.w));
            const uint32_t k = packed_max_s16(k01, k23);
            const int group_best = max((int)(int16_t)(k & 0xFFFFu), (int)k >> 16);
            if (group_best > best) {
                best = group_best;
                best_g = g;
                best_x = v[u];
                best_m = mu;
            }
        }
#pragma unroll
        for (int u = 0; u < kArgUnroll; ++u) m[u] = m_next[u];
    }
    unsigned long long mine = 0ull;
    if (best_g >= 0) {
        const uint32_t x[4] = {best_x.x, best_x.y, best_x.z, best_x.w};
        int first = 0;
#pragma unroll
        for (int k = 7; k >= 0; --k) {                  // descending: the smallest k is assigned last
            const uint32_t h = (k & 1) ? (x[k >> 1] >> 16) : (x[k >> 1] & 0xFFFFu);
            if (((best_m >> k) & 1u) && bf16_order(h) == best) first = k;
        }
        mine = argmax_word(best, best_g * 8 + first);
    }
    mine = argmax_block_max(mine, s_part, tid);
    const int order = (int)(uint32_t)(mine >> 32) - 32768;
    if (mine != 0ull && (order > kOrderPosInf || order == 0))
        mine = argmax_block_max(argmax_segment_by_compare(lrow, mrow, g_lo, g_hi, vocab, tid), s_part, tid);
    if (n_seg > 1) {
        if (tid == 0) partial[(size_t)b * n_seg + seg] = mine;
        return;
    }
    if (tid == 0) out[b] = mine != 0ull ? (int32_t)(0xFFFFFFFFu - (uint32_t)mine) : -1;
}

// One wave per row: combines the row's segments.
constexpr int kArgFinishRows = 4;
__global__ __launch_bounds__(64 * kArgFinishRows) void masked_argmax_finish_kernel(
    int batch, int n_seg, const unsigned long long *__restrict__ partial, int32_t *__restrict__ out) {
    const int lane = threadIdx.x & 63, b = blockIdx.x * kArgFinishRows + (threadIdx.x >> 6);
    if (b >= batch) return;
    unsigned long long mine = 0ull;
    for (int i = lane; i < n_seg; i += 64) {
        const unsigned long long p = partial[(size_t)b * n_seg + i];
        mine = p > mine ? p : mine;
    }
    mine = wave_max_u64(mine);
    if (lane == 0) out[b] = mine != 0ull ? (int32_t)(0xFFFFFFFFu - (uint32_t)mine) : -1;
}


// ------------------------------------------------------------------- masked top-k

// Order-preserving 16-bit key of a non-NaN bf16 pattern: a negative value's pattern is negated
// (two's complement), a non-negative one gets its top bit set (so -0 and +0 share a key), and 0x7F
// is subtracted with saturation.  Valid values map to 0x0001 (-inf) .. 0xFF01 (+inf); negative NaN
// patterns map to 0 (no candidate), positive NaN patterns to keys above 0xFF01.
constexpr uint32_t kTopkKeyMax = 0xFF01u;
__device__ __forceinline__ uint32_t bf16_key(uint32_t h) {
    const uint32_t folded = (h & 0x8000u) ? ((0u - h) & 0xFFFFu) : (h | 0x8000u);
    return folded > 0x7Fu ? folded - 0x7Fu : 0u;
}

// The same for two patterns in one register, with packed 16-bit arithmetic.
typedef unsigned short PackedU16 __attribute__((ext_vector_type(2)));
typedef short PackedI16 __attribute__((ext_vector_type(2)));
__device__ __forceinline__ uint32_t packed_sub_sat_u16(uint32_t a, uint32_t b) {
    return __builtin_bit_cast(uint32_t, __builtin_elementwise_sub_sat(__builtin_bit_cast(PackedU16, a), __builtin_bit_cast(PackedU16, b)));
}
__device__ __forceinline__ uint32_t bf16_key_pair(uint32_t x) {
    const PackedU16 h = __builtin_bit_cast(PackedU16, x);
    const uint32_t negative = __builtin_bit_cast(uint32_t, __builtin_bit_cast(PackedI16, x) >> 15);   // 0xFFFF per negative half
    const uint32_t neg = __builtin_bit_cast(uint32_t, (PackedU16)(PackedU16{0, 0} - h));
    const uint32_t pos = x | 0x80008000u;
    return packed_sub_sat_u16((neg & negative) | (pos & ~negative), 0x007F007Fu);
}
__device__ __forceinline__ uint32_t packed_max_u16(uint32_t a, uint32_t b) {
    return __builtin_bit_cast(uint32_t, __builtin_elementwise_max(__builtin_bit_cast(PackedU16, a), __builtin_bit_cast(PackedU16, b)));
}
__device__ __forceinline__ uint32_t packed_min_u16(uint32_t a, uint32_t b) {
    return __builtin_bit_cast(uint32_t, __builtin_elementwise_min(__builtin_bit_cast(PackedU16, a), __builtin_bit_cast(PackedU16, b)));
}

// A candidate travels between the stages as the word  key << 21 | (0x1FFFFF - id)  (id < 2^21):
// distinct words, larger = better value, then smaller id; 0 = no candidate.
constexpr int kTopkIdBits = 21;
constexpr uint32_t kTopkIdMask = (1u << kTopkIdBits) - 1u;
__device__ __forceinline__ unsigned long long topk_word(uint32_t key, uint32_t id) {
    return ((unsigned long long)key << kTopkIdBits) | (unsigned long long)(kTopkIdMask - id);
}

constexpr int kTopkBlock = 512, kTopkBlockWide = 1024;        // threads per block
constexpr int kTopkChunk = 4 * 8 * kTopkBlock;                // tokens of a narrow block

// Eight logits from t0 on, one 2-byte load each (the group that straddles the end of the vocabulary);
// tokens beyond the vocabulary read as NaN.  A loop that
// is not unrolled: the path is rare and must not cost the kernel registers.
__device__ __forceinline__ uint4 topk_load_last_group(const uint16_t *__restrict__ lrow, int t0, int vocab) {
    unsigned long long lo = 0x7FC07FC07FC07FC0ull, hi = lo;
#pragma unroll 1
    for (int j = 0; j < 8; ++j) {
        if (t0 + j >= vocab) break;
        const unsigned long long h = lrow[t0 + j];
        const int sh = (j & 3) * 16;
        if (j < 4) lo = (lo & ~(0xFFFFull << sh)) | (h << sh);
        else hi = (hi & ~(0xFFFFull << sh)) | (h << sh);
    }
    return make_uint4((uint32_t)lo, (uint32_t)(lo >> 32), (uint32_t)hi, (uint32_t)(hi >> 32));
}

// Block barrier for data exchanged through LDS: waits for the wave's own LDS operations only, so
// that global loads issued ahead stay in flight across it (__syncthreads would wait for them).
__device__ __forceinline__ void lds_barrier() {
    asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
}

// What the blocks of a row hand to the one that merges them: kTopkMax words a block (512 bytes, lines of its own), of which those
// behind its last candidate are zero.  Stored and loaded past the L2s: the blocks run on different XCDs.
__device__ __forceinline__ void topk_hand_over(unsigned long long *workspace, int b, int seg, int n_seg, int i, unsigned long long word) {
    __hip_atomic_store(workspace + ((size_t)b * n_seg + seg) * kTopkMax + i, word, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// The stored bf16 pattern behind a key of bf16_key, or -1 for the key of zero, which -0 and +0 share.
__device__ __forceinline__ int bf16_pattern_of_key(uint32_t key) {
    const uint32_t folded = key + 0x7Fu;
    if (folded == 0x8000u) return -1;
    return (folded & 0x8000u) ? (int)(folded & 0x7FFFu) : (int)((0x10000u - folded) & 0xFFFFu);
}

// The k best of a whole row (blockIdx.x), or of a segment of kBlock * kG * 8 tokens of a longer one (blockIdx.y), by one
// block that keeps it in registers.  The mask row goes to LDS with a few loads per thread, and every
// thread loads its kG groups of logits, kAhead of them in flight, whatever their mask bytes say and without a branch
// (groups beyond the row's end load the last one), and works on a group as it arrives.  The block is then bound by what
// its waves do after the stream, so what is done to every token is two packed instructions under the stream: its half is
// set to 0xFFFF if it is masked, and the maximum of the patterns as signed 16-bit numbers is taken.  For
// patterns above zero that order is the order of the values, and the k best of most rows are such.  Then
//   (1) a lower bound M of the k-th largest value: the k-th largest of 128 maxima of neighbouring threads, ranked
//       by all threads together between two barriers: 64 of 128,256 random values reach the bound for k = 50;
//   (2) the few groups whose maximum reaches M are copied to a list in LDS (one atomic per wave), and behind a barrier
//       eight threads per listed group pick the tokens that reach M out of it, as words;
//   (3) the words (little more than k) are ranked by all threads together -- a word's rank is the
//       number of larger words -- and the k best write their id and pattern (rebuilt from the key, read back only
//       for a zero) in order.
// A row where fewer than k of the 128 hold a value (few tokens allowed, or few above zero) or an allowed NaN of
// positive sign takes the maxima and (1) again on the keys of bf16_key (0xFFFF, the pattern of a negative NaN, becomes
// 0 = no candidate) of the groups that have an allowed token; the registers keep the patterns.
// Lists that would run full (hundreds of ties with the bound, or a dense row where the threads' maxima do not
// say enough) are given up: the block then counts (topk_by_counts), which has no such limit.
// Twenty groups per thread (163,840 tokens) is what the 128 vector registers hold without spills.
// (14.6 us per launch at 256 x 128,256, k = 50, 4.8 TB/s; 15.4 us per call in a graph: 9.4 us until the row has arrived and is worked on, 0.8 for
// the bound, 1.4 for the list, 0.7 for the ranks.  24.9 us before, with keys computed for every token, all sixteen
// loads issued first -- behind branches, so that nothing was worked on before the last had arrived: a wave that wants
// to issue its sixteenth load waits for it until 8 us --, a bound from quotas per wave (147 words listed) and one
// returning atomic per listed token.  Copying all sixteen groups of a thread to the list without a branch per group
// costs 1 us more: a 16-byte LDS store takes its time whatever the number of lanes.
// Measured and dropped: taking the bound from half of the row while the other half is still in
// flight, with the second half filtered as it arrives -- the waves of a block finish their halves
// microseconds apart, so the barrier gains nothing, and the looser bound doubles the list.)
__device__ __forceinline__ uint32_t packed_max_i16(uint32_t a, uint32_t b) {
    return __builtin_bit_cast(uint32_t, __builtin_elementwise_max(__builtin_bit_cast(PackedI16, a), __builtin_bit_cast(PackedI16, b)));
}
constexpr int kTopkRowTokens = 20 * 8 * kTopkBlockWide;        // longest row that one block keeps in registers
constexpr int kTopkRowList = 512;
constexpr int kTopkMaxima = 128;                   // thread maxima that give the bound
static_assert(kTopkMax <= kTopkMaxima, "the k-th of them has to exist");

// The sum, or the maximum, over kLanes (2, 4 or 8) neighbouring lanes.
template <int kLanes, class Op>
__device__ __forceinline__ int lanes_reduce(int x, Op op) {
    x = op(x, __builtin_amdgcn_mov_dpp(x, 0xB1, 0xF, 0xF, true));                        // lane ^ 1
    if (kLanes > 2) x = op(x, __builtin_amdgcn_mov_dpp(x, 0x4E, 0xF, 0xF, true));        // lane ^ 2
    if (kLanes > 4) x = op(x, __builtin_amdgcn_mov_dpp(x, 0x141, 0xF, 0xF, true));       // the other four of eight
    return x;
}

// Step (1): the k-th largest of the kTopkMaxima maxima of the block's threads (kLanes threads each) in *kth, the largest
// in *first; 0 where there are fewer.  s_pub: a word per maximum, s_out: two words that start at zero; every
// call of a block takes others.  Two barriers.
template <int kBlock>
__device__ __forceinline__ void topk_bound(uint32_t best, int k, uint32_t *s_pub, uint32_t *s_out, int tid, uint32_t *first, uint32_t *kth) {
    constexpr int kLanes = kBlock / kTopkMaxima;
    auto largest = [](int a, int b) { return max(a, b); };
    auto sum = [](int a, int b) { return a + b; };
    const uint32_t top = (uint32_t)lanes_reduce<kLanes>((int)best, largest);
    const int at = tid / kLanes, part = tid % kLanes;
    if (part == 0) s_pub[at] = top << 7 | (uint32_t)(kTopkMaxima - 1 - at);      // distinct
    lds_barrier();
    // the threads of one maximum count the larger ones
    const uint32_t mine = s_pub[at];
    int larger = 0;
#pragma unroll
    for (int i = 0; i < kTopkMaxima / kLanes / 4; ++i) {
        const uint4 x = reinterpret_cast<const uint4 *>(s_pub)[i * kLanes + part];
        larger += (x.x > mine ? 1 : 0) + (x.y > mine ? 1 : 0) + (x.z > mine ? 1 : 0) + (x.w > mine ? 1 : 0);
    }
    larger = lanes_reduce<kLanes>(larger, sum);
    if (part == 0 && larger == 0) s_out[0] = mine >> 7;
    if (part == 0 && larger == k - 1) s_out[1] = mine >> 7;
    lds_barrier();
    *first = s_out[0];
    *kth = s_out[1];
}

// Step (3): ranks the n words of the list (kBlock / kTopkMaxima lanes to a word) and hands out those below k.
template <int kBlock, class Emit>
__device__ __forceinline__ void topk_rank(const unsigned long long *s_cand, int n, int k, int tid, Emit emit) {
    constexpr int kLanes = kBlock / kTopkMaxima;
    auto sum = [](int a, int b) { return a + b; };
    for (int at0 = 0; at0 < n; at0 += kTopkMaxima) {
        const int at = at0 + tid / kLanes;
        const unsigned long long mine = at < n ? s_cand[at] : ~0ull;
        int larger = 0;
#pragma unroll 4
        for (int j = tid % kLanes; j < n; j += kLanes) larger += s_cand[j] > mine ? 1 : 0;
        larger = lanes_reduce<kLanes>(larger, sum);
        if (tid % kLanes == 0 && at < n && larger < k) emit(larger, mine);
    }
}

// One of a row's results: the id and the pattern of `word`, or the padding.
__device__ __forceinline__ void topk_put(int rank, unsigned long long word, int k, int b, const uint16_t *__restrict__ row,
                                         int32_t *__restrict__ out_ids, uint16_t *__restrict__ out_vals) {
    int32_t id = -1;
    uint16_t value = 0xFF80u;
    if (word != 0ull) {
        id = (int32_t)(kTopkIdMask - ((uint32_t)word & kTopkIdMask));
        const int pattern = bf16_pattern_of_key((uint32_t)(word >> kTopkIdBits));
        if (out_vals) value = pattern >= 0 ? (uint16_t)pattern : row[id];
    }
    out_ids[(size_t)b * k + rank] = id;
    if (out_vals) out_vals[(size_t)b * k + rank] = value;
}

// Of the threads' words (distinct, 0: none) those that reach the k-th largest of 128 maxima of neighbouring threads, to s_words;
// returns how many.  The bound of topk_bound, of whole words, ids among them, for what that left: hundreds of words that tie
// take longer to rank (a block's 365, 6 us) than to bound again.  s_words may be where the words came from.  Three barriers.
template <int kBlock, int kPer>
__device__ __forceinline__ int topk_cut(const unsigned long long (&c)[kPer], int k, unsigned long long *s_words, int tid) {
    constexpr int kLanes = kBlock / kTopkMaxima;
    __shared__ unsigned long long s_top[kTopkMaxima], s_least;
    __shared__ int s_few;
    const int lane = tid & 63, at = tid / kLanes, part = tid % kLanes;
    unsigned long long top = 0ull;
#pragma unroll
    for (int i = 0; i < kPer; ++i) top = c[i] > top ? c[i] : top;
#pragma unroll
    for (int step = 1; step < kLanes; step *= 2) {
        const unsigned long long other = shfl_xor_u64(top, step);
        top = other > top ? other : top;
    }
    if (part == 0) s_top[at] = top;
    if (tid == 0) { s_least = 0ull; s_few = 0; }
    lds_barrier();
    int larger = 0;
#pragma unroll 4
    for (int i = part; i < kTopkMaxima; i += kLanes) larger += s_top[i] > top ? 1 : 0;
    larger = lanes_reduce<kLanes>(larger, [](int x, int y) { return x + y; });
    if (part == 0 && larger == k - 1 && top != 0ull) s_least = top;      // (fewer than k maxima: every word stays)
    lds_barrier();
    const unsigned long long least = s_least;
#pragma unroll
    for (int i = 0; i < kPer; ++i) {
        const bool keep = c[i] != 0ull && c[i] >= least;
        const unsigned long long m = __ballot(keep);
        if (m == 0ull) continue;
        int base = 0;
        if (lane == 0) base = atomicAdd(&s_few, __popcll(m));
        base = __builtin_amdgcn_readfirstlane(base);
        if (keep) s_words[base + __popcll(m & ((1ull << lane) - 1ull))] = c[i];
    }
    lds_barrier();
    return s_few;
}

// A segment's n listed words, the k best among them (behind a barrier): ranked to out_ids and out_vals, or, where the row has
// several segments, to the workspace (topk_hand_over), unranked where they fit there; the block that merges ranks them.
template <int kBlock, bool kSeveral>
__device__ __forceinline__ void topk_hand_out(unsigned long long *s_cand, int n, int k, const uint16_t *__restrict__ row,
                                              unsigned long long *__restrict__ workspace, int32_t *__restrict__ out_ids,
                                              uint16_t *__restrict__ out_vals, int b, int seg, int n_seg, int width, int tid) {
    auto emit = [&](int rank, unsigned long long word) {
        if (kSeveral) topk_hand_over(workspace, b, seg, n_seg, rank, word);
        else topk_put(rank, word, k, b, row, out_ids, out_vals);
    };
    auto nothing_behind = [&](int at) {                       // no candidates beyond those that are handed over
        if (kSeveral && tid >= at && tid < width) topk_hand_over(workspace, b, seg, n_seg, tid, 0ull);
    };
    if (n > 2 * kTopkMaxima) {                                // (below that the ranking is the shorter: 200 words of 128,256 tokens 13.0 us, 14.2 cut first)
        constexpr int kApart = kBlock / kTopkRowList;
        const unsigned long long c[1] = {tid % kApart == 0 && tid / kApart < n ? s_cand[tid / kApart] : 0ull};
        n = topk_cut<kBlock, 1>(c, k, s_cand, tid);
    }
    if (kSeveral && n <= width) {
        if (tid < n) topk_hand_over(workspace, b, seg, n_seg, tid, s_cand[tid]);
        nothing_behind(n);
        return;
    }
    if (tid >= n && tid < k) emit(tid, 0ull);
    topk_rank<kBlock>(s_cand, n, k, tid, emit);
    nothing_behind(k);
}

// The k best of a segment in which more tokens reach `bound` (a key of bf16_key, 1 or more) than the lists hold: nearly always
// ties with the bound, because a row has few values, or few that are not -inf.  The segment is read again, its keys stay in
// registers, and the block counts how many reach a key: the bound, the next key, and by bisection from there, until they are
// few enough to list or the k-th largest key is found.  Then the larger ones are listed and, because ids ascend by group, then by
// thread, the first of its ties.  A call of its own: its registers stay apart from the row kernel's
// (one to each kernel, which then knows where its LDS lies).
// Bound by the latency of its rounds: the loads, two counts and one round of ties for the rows above.  It replaces a pass with lists
// per wave that were cut to their k best whenever they ran full, a cut being 37 counts.  us per call, that pass and this: 16 x
// 152,064 equal logits, k = 50, in narrow blocks 111 and 15.1 (in one block a row 100), k = 1 89 and 11.8; 20 tokens finite and the rest -inf, k = 1,
// which one block a row need not come here for and takes 10.1, 86 and 12.8; 64 x 128,256 equal, one block a row, k = 50, 100 and
// 29.4; 200 x 152,064 111 and 46.7.  Also the way of vocabularies below eight tokens.
template <int kBlock, int kG, bool kSeveral>
__device__ __noinline__ void topk_by_counts(const uint16_t *logits, const uint32_t *bitmask, int vocab, int64_t row_stride, int n_words, int k,
                                            uint32_t bound, unsigned long long *workspace, int32_t *out_ids,
                                            uint16_t *out_vals, int b, int seg, int n_seg, int width) {
    constexpr int kWaves = kBlock / 64, kSegTokens = kBlock * kG * 8, kAhead = kG < 8 ? kG : 8;
    constexpr int kCounts = 18;                               // the bound, the next key, sixteen halvings
    __shared__ uint2 s_expand[16];
    __shared__ int s_reach[kCounts], s_tied[kG][kWaves], s_n;
    __shared__ unsigned long long s_cand[kTopkRowList];
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const unsigned long long lanes_below = (1ull << lane) - 1ull;
    const uint16_t *whole_row = logits + (size_t)b * row_stride;
    const int first_token = seg * kSegTokens, n_tokens = min(vocab - first_token, kSegTokens), whole = n_tokens >> 3;
    const uint8_t *mask_bytes = reinterpret_cast<const uint8_t *>(bitmask + (size_t)b * n_words + first_token / 32);
    // (as in topk_segment; a row below eight tokens: sixteen bytes that are there, none of them looked at)
    const uint16_t *lrow = vocab < 8 ? reinterpret_cast<const uint16_t *>(workspace) : whole_row + (whole > 0 ? first_token : max(first_token - 8, 0));
    const uint32_t last_group = (uint32_t)max(whole - 1, 0) * 16u;
    mask_nibble_table_init(s_expand, tid);
    if (tid < kCounts) s_reach[tid] = 0;
    if (tid == 0) s_n = 0;
    lds_barrier();
    // the keys, two to a register; 0: masked, NaN, behind the row
    uint32_t kp[kG * 4], m[kG], packed[kG / 4];
    auto keys = [](uint32_t x, uint32_t allow) {
        const uint32_t key = bf16_key_pair(x), nan = packed_min_u16(packed_sub_sat_u16(key, kTopkKeyMax * 0x10001u), 0x00010001u);
        return allow & packed_sub_sat_u16(key, nan * 0xFFFFu);                                             // (a positive NaN's key goes)
    };
#pragma unroll
    for (int u = 0; u < kG; ++u) m[u] = mask_bytes[min(u * kBlock + tid, max(whole - 1, 0))];
#pragma unroll
    for (int i = 0; i < kG / 4; ++i) {
        packed[i] = m[i * 4] | m[i * 4 + 1] << 8 | m[i * 4 + 2] << 16 | m[i * 4 + 3] << 24;
        asm volatile("" : "+v"(packed[i]));
    }
    uint4 v[kG];
    auto load_group = [&](int u) { v[u] = stream_load_at(lrow, min((uint32_t)tid * 16u + (uint32_t)(u * kBlock * 16), last_group)); };
#pragma unroll
    for (int u = 0; u < kAhead; ++u) load_group(u);
#pragma unroll
    for (int u = 0; u < kG; ++u) {
        if (u + kAhead < kG) load_group(u + kAhead);
        __builtin_amdgcn_sched_barrier(0);
        const uint4 allow = expand_mask_byte(s_expand, u * kBlock + tid < whole ? (packed[u / 4] >> (8 * (u & 3))) & 0xFFu : 0u);
        kp[u * 4] = keys(v[u].x, allow.x);
        kp[u * 4 + 1] = keys(v[u].y, allow.y);
        kp[u * 4 + 2] = keys(v[u].z, allow.z);
        kp[u * 4 + 3] = keys(v[u].w, allow.w);
        asm volatile("" : "+v"(kp[u * 4]), "+v"(kp[u * 4 + 1]), "+v"(kp[u * 4 + 2]), "+v"(kp[u * 4 + 3]));
    }
    if ((n_tokens & 7) != 0 && whole % kBlock == tid) {         // the last, partial group
        const uint4 x = topk_load_last_group(whole_row, first_token + whole * 8, vocab), allow = expand_mask_byte(s_expand, mask_bytes[whole]);
#pragma unroll
        for (int u = 0; u < kG; ++u) {
            if (u != whole / kBlock) continue;
            kp[u * 4] = keys(x.x, allow.x);
            kp[u * 4 + 1] = keys(x.y, allow.y);
            kp[u * 4 + 2] = keys(x.z, allow.z);
            kp[u * 4 + 3] = keys(x.w, allow.w);
        }
    }
    auto count = [&](uint32_t key, int at) {                  // the segment's keys of at least `key`
        const uint32_t below = (key - 1u) * 0x10001u;
        uint32_t two = 0u;
#pragma unroll
        for (int i = 0; i < kG * 4; ++i) two += packed_min_u16(packed_sub_sat_u16(kp[i], below), 0x00010001u);
        int sum = (int)((two & 0xFFFFu) + (two >> 16));
        for (int step = 32; step > 0; step >>= 1) sum += __shfl_xor(sum, step);
        if (lane == 0) atomicAdd(&s_reach[at], sum);
        lds_barrier();
        return __builtin_amdgcn_readfirstlane(s_reach[at]);
    };
    // lo: reached by `few` or more (unknown before the first count), hi: by n_hi, fewer than k
    constexpr int kUnknown = 0x7FFFFFFF;
    uint32_t lo = bound - 1u, hi = kTopkKeyMax + 1u, mid = bound;
    int n_lo = kUnknown, n_hi = 0;
    for (int at = 0; at < kCounts && n_lo > kTopkRowList && hi - lo > 1u; ++at) {
        const int c = count(mid, at);
        if (c >= k) { lo = mid; n_lo = c; }
        else { hi = mid; n_hi = c; }
        mid = at == 0 ? lo + 1u : lo + (hi - lo) / 2u;
    }
    const bool fits = n_lo <= kTopkRowList;
    // (one token of a group at a time, in a loop: the code is fetched for the one call)
    auto four = [&](int at) { return (unsigned long long)kp[at + 1] << 32 | kp[at]; };
    const uint32_t least = fits ? lo : hi, below = (least - 1u) * 0x10001u;
#pragma unroll
    for (int u = 0; u < kG; ++u) {
        uint32_t any = 0u;
#pragma unroll
        for (int j = 0; j < 4; ++j) any |= packed_sub_sat_u16(kp[u * 4 + j], below);
        if (any != 0u) {
            const unsigned long long low = four(u * 4), high = four(u * 4 + 2);
#pragma unroll 1
            for (int e = 0; e < 8; ++e) {
                const uint32_t key = (uint32_t)((e < 4 ? low : high) >> (16 * (e & 3))) & 0xFFFFu;
                if (key >= least) s_cand[atomicAdd(&s_n, 1)] = topk_word(key, (uint32_t)(first_token + (u * kBlock + tid) * 8 + e));
            }
        }
    }
    int n = fits ? n_lo : n_hi;
    if (!fits && n_lo != kUnknown) {                           // ties of the k-th, group by group of all threads
        const int want = k - n_hi;
        int taken = 0;
#pragma unroll
        for (int u = 0; u < kG; ++u) {
            if (taken >= want) continue;                       // (the same in every thread)
            uint32_t others = 0u;
#pragma unroll
            for (int j = 0; j < 4; ++j) others += packed_min_u16(kp[u * 4 + j] ^ (lo * 0x10001u), 0x00010001u);
            const int mine = 8 - (int)((others & 0xFFFFu) + (others >> 16));
            int slot = taken, sum = 0;                         // ties of the lanes before, of the wave
#pragma unroll
            for (int bit = 0; bit < 4; ++bit) {
                const unsigned long long has = __ballot((mine >> bit) & 1);
                slot += __popcll(has & lanes_below) << bit;
                sum += __popcll(has) << bit;
            }
            if (lane == 0) s_tied[u][wave] = sum;
            lds_barrier();
            int upto = lane < kWaves ? s_tied[u][lane] : 0;       // lane w: ties of the waves 0 .. w
            upto += __builtin_amdgcn_mov_dpp(upto, 0x111, 0xF, 0xF, true);       // (row shifts by 1, 2, 4, 8)
            upto += __builtin_amdgcn_mov_dpp(upto, 0x112, 0xF, 0xF, true);
            upto += __builtin_amdgcn_mov_dpp(upto, 0x114, 0xF, 0xF, true);
            upto += __builtin_amdgcn_mov_dpp(upto, 0x118, 0xF, 0xF, true);
            if (wave > 0) slot += __builtin_amdgcn_readlane(upto, wave - 1);
            taken += __builtin_amdgcn_readlane(upto, kWaves - 1);
            if (mine != 0 && slot < want) {
                const unsigned long long low = four(u * 4), high = four(u * 4 + 2);
#pragma unroll 1
                for (int e = 0; e < 8; ++e) {
                    const uint32_t key = (uint32_t)((e < 4 ? low : high) >> (16 * (e & 3))) & 0xFFFFu;
                    if (key == lo && slot < want) s_cand[n_hi + slot++] = topk_word(lo, (uint32_t)(first_token + (u * kBlock + tid) * 8 + e));
                }
            }
        }
        n = k;
    }
    lds_barrier();
    topk_hand_out<kBlock, kSeveral>(s_cand, n, k, whole_row, workspace, out_ids, out_vals, b, seg, n_seg, width, tid);
}

// A row's segment: its k best to out_ids and out_vals, or, where the row has several, its candidates to the workspace
// (topk_hand_over: `width` words, the k best of the segment among them).
template <int kBlock, int kG, bool kSeveral>
__device__ __forceinline__ void topk_segment(
    const uint16_t *__restrict__ logits, const uint32_t *__restrict__ bitmask, int vocab, int64_t row_stride,
    int n_words, int k, unsigned long long *__restrict__ workspace, int32_t *__restrict__ out_ids,
    uint16_t *__restrict__ out_vals, int b, int seg, int n_seg, int width, int tid) {
    constexpr int kWaves = kBlock / 64, kSegTokens = kBlock * kG * 8;
    constexpr int kAhead = kG < 8 ? kG : 8;                   // groups a thread has in flight
    static_assert(kG % 4 == 0, "mask words of four rounds at a time");
    // Groups listed.  A narrow block, whose part of a row holds fewer different values, lists as many as tokens: with 256, half-integers
    // on 16 x 128,256, k = 64, were counted although the list holds them (19.2 us, 13.8).  The wide ones lose 0.3 % by it (top-50 steps
    // of 256 x 128,256).
    constexpr int kGroupList = kBlock == kTopkBlock ? kTopkRowList : kTopkRowList / 2;
    __shared__ uint32_t s_mask[kBlock * kG / 4];              // the mask row, for every wave the bytes of its groups
    __shared__ uint2 s_expand[16];                            // half a mask byte -> AND masks of two of the group's registers
    __shared__ __align__(16) uint32_t s_pub[2][kTopkMaxima];
    __shared__ uint32_t s_bound[2][2];
    __shared__ uint4 s_group[kGroupList];
    __shared__ int s_group_at[kGroupList];
    __shared__ unsigned long long s_cand[kTopkRowList];
    __shared__ int s_count, s_groups;
    const int lane = tid & 63, wave = tid >> 6;
    if (kBlock == kTopkBlock && vocab < 8) {                  // not one group of eight logits that the loads below could take
        topk_by_counts<kBlock, kG, kSeveral>(logits, bitmask, vocab, row_stride, n_words, k, 1u, workspace, out_ids, out_vals, b, 0, 1, width);
        return;
    }
    const unsigned long long lanes_below = (1ull << lane) - 1ull;
    const uint16_t *whole_row = logits + (size_t)b * row_stride;
    const int first_token = seg * kSegTokens, n_tokens = min(vocab - first_token, kSegTokens);
    const uint32_t *mrow = bitmask + (size_t)b * n_words + first_token / 32;
    const int seg_words = (n_tokens + 31) / 32, whole = n_tokens >> 3;
    // (a last segment of less than a group loads the eight tokens before it and looks at none)
    const uint16_t *lrow = whole_row + (whole > 0 ? first_token : max(first_token - 8, 0));
    const uint32_t last_group = (uint32_t)max(whole - 1, 0) * 16u;
    // the mask words of the wave's own groups: its 64 groups of round u are the words u * kBlock / 4 + wave * 16 + (0 .. 15)
    uint32_t mw[kG / 4];
    auto mask_word = [&](int i) { return (i * 4 + (lane >> 4)) * (kBlock / 4) + wave * 16 + (lane & 15); };
#pragma unroll
    for (int i = 0; i < kG / 4; ++i) mw[i] = mrow[min(mask_word(i), seg_words - 1)];
    uint4 v[kG];
    auto load_group = [&](int u) { v[u] = stream_load_at(lrow, min((uint32_t)tid * 16u + (uint32_t)(u * kBlock * 16), last_group)); };
#pragma unroll
    for (int u = 0; u < kAhead; ++u) load_group(u);
    mask_nibble_table_init(s_expand, tid);
    if (tid == 0) { s_count = 0; s_groups = 0; s_bound[0][0] = s_bound[0][1] = s_bound[1][0] = s_bound[1][1] = 0u; }
    lds_barrier();                                            // s_expand and what starts at zero (the loads are on their way)
#pragma unroll
    for (int i = 0; i < kG / 4; ++i) {
        const int w = mask_word(i);
        // bits of groups that are not whole count as masked: their tokens are taken one by one below
        uint32_t x = w * 4 + 4 <= whole ? mw[i] : 0u;
        if (w * 4 < whole && w * 4 + 4 > whole) x = mw[i] & ((1u << ((whole & 3) * 8)) - 1u);
        s_mask[wave * (kG * 16) + i * 64 + lane] = x;
    }
    wave_exchange();                          // (written and read by the same wave)
    const uint8_t *mask_bytes = reinterpret_cast<const uint8_t *>(s_mask) + wave * (kG * 64);
    uint32_t kp[kG * 4], mu[kG];
    int gmax[kG], best_i = 0;                                 // the largest pattern of a group, of the thread (as signed numbers)
#pragma unroll
    for (int u = 0; u < kG; ++u) mu[u] = mask_bytes[u * 64 + lane];
#pragma unroll
    for (int u = 0; u < kG; ++u) {
        if (u + kAhead < kG) load_group(u + kAhead);
        __builtin_amdgcn_sched_barrier(0);
        const uint4 allow = expand_mask_byte(s_expand, mu[u]);
        kp[u * 4] = v[u].x | ~allow.x;
        kp[u * 4 + 1] = v[u].y | ~allow.y;
        kp[u * 4 + 2] = v[u].z | ~allow.z;
        kp[u * 4 + 3] = v[u].w | ~allow.w;
        const uint32_t top2 = packed_max_i16(packed_max_i16(kp[u * 4], kp[u * 4 + 1]), packed_max_i16(kp[u * 4 + 2], kp[u * 4 + 3]));
        gmax[u] = max((int)(int16_t)(top2 & 0xFFFFu), (int)top2 >> 16);
        best_i = max(best_i, gmax[u]);
        // (worked on here, as it arrives: the compiler would otherwise read the table for all groups first, which does
        // not fit the registers, and do the rest behind the barrier below)
        asm volatile("" : "+v"(kp[u * 4]), "+v"(kp[u * 4 + 1]), "+v"(kp[u * 4 + 2]), "+v"(kp[u * 4 + 3]), "+v"(gmax[u]), "+v"(best_i));
    }
    // the tokens behind the last whole group, one thread each
    uint32_t tail = 0xFFFFu;
    const int tail_t = whole * 8 + tid;                       // (within the segment)
    if (tail_t < n_tokens && ((mrow[tail_t >> 5] >> (tail_t & 31)) & 1u)) tail = whole_row[first_token + tail_t];
    // (1) the bound
    uint32_t first, kth;
    uint32_t best = (uint32_t)max(best_i, (int)(int16_t)tail);
    topk_bound<kBlock>(best, k, s_pub[0], s_bound[0], tid, &first, &kth);
    const bool nan = first > 0x7F80u;
    const bool positive = !nan && kth != 0u;                  // the same in every thread
    if (!positive) {
        best = 0u;
#pragma unroll
        for (int u = 0; u < kG; ++u) {
            const bool empty = (kp[u * 4] & kp[u * 4 + 1] & kp[u * 4 + 2] & kp[u * 4 + 3]) == 0xFFFFFFFFu;
            gmax[u] = 0;
            if (!__any(!empty)) continue;
            uint32_t top2 = 0u;
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                uint32_t key = bf16_key_pair(kp[u * 4 + j]);
                if (nan) {                                    // a positive NaN's key goes
                    const uint32_t lo = key & 0xFFFFu, hi = key >> 16;
                    key = (lo > kTopkKeyMax ? 0u : lo) | ((hi > kTopkKeyMax ? 0u : hi) << 16);
                }
                top2 = packed_max_u16(top2, key);
            }
            gmax[u] = (int)max(top2 & 0xFFFFu, top2 >> 16);
            best = max(best, (uint32_t)gmax[u]);
        }
        tail = bf16_key(tail);
        if (tail > kTopkKeyMax) tail = 0u;
        best = max(best, tail);
        topk_bound<kBlock>(best, k, s_pub[1], s_bound[1], tid, &first, &kth);
    } else {
        if ((int)(int16_t)tail < 0) tail = 0u;
    }
    const uint32_t bound = kth != 0u ? kth : first != 0u ? 1u : 0u;      // fewer than k: every candidate
    if (bound == 0u) {                                        // nothing is allowed (or only NaN)
        topk_hand_out<kBlock, kSeveral>(s_cand, 0, k, whole_row, workspace, out_ids, out_vals, b, seg, n_seg, width, tid);
        return;
    }
    // (2) the groups that hold a value of at least `bound`, then the tokens
    const uint32_t to_key = positive ? bf16_key(0u) : 0u;     // a positive pattern's key is the pattern plus that of zero
    if (__any(best >= bound)) {
        unsigned long long reach[kG];
        int total = 0;
#pragma unroll
        for (int u = 0; u < kG; ++u) {
            reach[u] = __ballot(gmax[u] >= (int)bound);
            total += __popcll(reach[u]);
        }
        int slot0 = 0;
        if (lane == 0) slot0 = atomicAdd(&s_groups, total);
        slot0 = __builtin_amdgcn_readfirstlane(slot0);
#pragma unroll
        for (int u = 0; u < kG; ++u) {
            if (reach[u] == 0ull) continue;
            const int slot = slot0 + __popcll(reach[u] & lanes_below);
            if (gmax[u] >= (int)bound && slot < kGroupList) {
                s_group[slot] = make_uint4(kp[u * 4], kp[u * 4 + 1], kp[u * 4 + 2], kp[u * 4 + 3]);
                s_group_at[slot] = tid + u * kBlock;
            }
            slot0 += __popcll(reach[u]);
        }
        if (tail >= bound) {                                  // at most seven tokens, all in the first wave
            const int slot = atomicAdd(&s_count, 1);
            s_cand[slot] = topk_word(tail + to_key, (uint32_t)(first_token + tail_t));
        }
    }
    lds_barrier();
    const int n_groups = s_groups;                            // the same in every thread
    if (n_groups <= kGroupList) {
        const uint16_t *halves = reinterpret_cast<const uint16_t *>(s_group);
        for (int at0 = wave * 64; at0 < n_groups * 8; at0 += kBlock) {
            const int at = at0 + lane;
            uint32_t x = at < n_groups * 8 ? halves[at] : 0xFFFFu;
            if (positive) {
                if (x & 0x8000u) x = 0u;
            } else {
                x = bf16_key(x);
                if (x > kTopkKeyMax) x = 0u;                  // a positive NaN
            }
            const bool take = x >= bound;
            const unsigned long long mm = __ballot(take);
            if (mm == 0ull) continue;
            int base = 0;
            if (lane == 0) base = atomicAdd(&s_count, __popcll(mm));
            const int slot = __builtin_amdgcn_readfirstlane(base) + __popcll(mm & lanes_below);
            if (take && slot < kTopkRowList) s_cand[slot] = topk_word(x + to_key, (uint32_t)(first_token + s_group_at[at >> 3] * 8 + (at & 7)));
        }
    }
    lds_barrier();
    const int n = s_count;
    if (n > kTopkRowList || n_groups > kGroupList) {   // same in every thread
        topk_by_counts<kBlock, kG, kSeveral>(logits, bitmask, vocab, row_stride, n_words, k, bound + to_key, workspace, out_ids, out_vals, b, seg,
                                             n_seg, width);
        return;
    }
    // (3) ranks
    topk_hand_out<kBlock, kSeveral>(s_cand, n, k, whole_row, workspace, out_ids, out_vals, b, seg, n_seg, width, tid);
}

// The k best of a row out of what its blocks handed over (n_cand <= kTopkMergeMax words, 0 = empty), by the last of them.  As
// above, the k-th largest of 128 thread maxima bounds the k-th largest key from below, and the words that reach it are ranked.
constexpr int kTopkMergeMax = 1024;
template <int kBlock>
__device__ __forceinline__ void topk_merge(const unsigned long long *__restrict__ workspace, int n_seg, int width, int k,
                                           const uint16_t *__restrict__ row, int32_t *__restrict__ out_ids,
                                           uint16_t *__restrict__ out_vals, int b, int tid) {
    constexpr int kPer = kTopkMergeMax / kBlock;
    __shared__ __align__(16) uint32_t s_pub[kTopkMaxima];
    __shared__ uint32_t s_bound[2];
    __shared__ unsigned long long s_words[kTopkMergeMax];
    __shared__ int s_count;
    const int lane = tid & 63, n_cand = n_seg * width;
    unsigned long long c[kPer], top = 0ull;
#pragma unroll
    for (int i = 0; i < kPer; ++i) {
        // The threads of one maximum take words far apart in a block's list (a wave one block's 512 bytes), or of different blocks: where a
        // block has ranked its words first, neighbours under one maximum left four times k words to rank (16 x 200,000, k = 64: 15.9 us,
        // 11.3 with neighbours of different blocks, so 9.6; k = 50 10.3, 9.3, 9.1; 40 and fewer lose 2 % by it).
        constexpr int kLanes = kBlock / kTopkMaxima;
        const int at = i * kBlock + tid;
        int from = at / kTopkMax, nth = at % kTopkMax;
        if (k > kTopkMax * 3 / 4) nth = nth % kLanes * (kTopkMax / kLanes) + nth / kLanes;
        if (width != kTopkMax) { nth = at / n_seg; from = at - nth * n_seg; }
        c[i] = 0ull;
        if (at < n_cand)
            c[i] = __hip_atomic_load(workspace + ((size_t)b * n_seg + from) * kTopkMax + nth, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        top = c[i] > top ? c[i] : top;
    }
    if (tid == 0) { s_count = 0; s_bound[0] = s_bound[1] = 0u; }
    uint32_t first, kth;
    topk_bound<kBlock>((uint32_t)(top >> kTopkIdBits), k, s_pub, s_bound, tid, &first, &kth);
#pragma unroll
    for (int i = 0; i < kPer; ++i) {
        const bool keep = c[i] != 0ull && (uint32_t)(c[i] >> kTopkIdBits) >= kth;
        const unsigned long long m = __ballot(keep);
        if (m == 0ull) continue;
        int base = 0;
        if (lane == 0) base = atomicAdd(&s_count, __popcll(m));
        base = __builtin_amdgcn_readfirstlane(base);
        if (keep) s_words[base + __popcll(m & ((1ull << lane) - 1ull))] = c[i];
    }
    lds_barrier();
    int n = s_count;
    if (n > kTopkMaxima) n = topk_cut<kBlock, kPer>(c, k, s_words, tid);
    auto put = [&](int rank, unsigned long long word) { topk_put(rank, word, k, b, row, out_ids, out_vals); };
    if (tid >= n && tid < k) put(tid, 0ull);
    topk_rank<kBlock>(s_words, n, k, tid, put);
}

__device__ __forceinline__ int topk_width(int n_seg, int k) { return n_seg * kTopkMax <= kTopkMergeMax ? kTopkMax : k; }

// A row per blockIdx.x, a segment per blockIdx.y (kSeveral: of more than one).  The blocks of a row that has several count
// themselves in when what they hand over has arrived; the last one merges, and sets the count back to zero for the next
// launch.  No block waits for another.  (arrivals null: masked_topk_merge_kernel merges, in a launch of its own.)
template <int kBlock, int kG, bool kSeveral>
__global__ __launch_bounds__(kBlock) __attribute__((amdgpu_waves_per_eu(4))) void masked_topk_row_kernel(
    const uint16_t *__restrict__ logits, const uint32_t *__restrict__ bitmask, int vocab, int64_t row_stride,
    int n_words, int k, unsigned long long *__restrict__ workspace, int32_t *__restrict__ out_ids,
    uint16_t *__restrict__ out_vals, StepArrivals *__restrict__ arrivals) {
    const int b = blockIdx.x, seg = kSeveral ? blockIdx.y : 0, n_seg = kSeveral ? gridDim.y : 1, tid = threadIdx.x;
    const int width = topk_width(n_seg, k);
    topk_segment<kBlock, kG, kSeveral>(logits, bitmask, vocab, row_stride, n_words, k, workspace, out_ids, out_vals, b, seg, n_seg, width, tid);
    if constexpr (kSeveral) {
        if (arrivals == nullptr) return;
        __shared__ int s_last;
        asm volatile("s_waitcnt vmcnt(0)" ::: "memory");           // this wave's candidates are where the other XCDs see them ...
        __syncthreads();                                           // ... and those of the block's other waves
        if (tid == 0) s_last = atomicAdd(&arrivals[b].listed, 1u) == (uint32_t)(n_seg - 1);
        __syncthreads();
        if (!s_last) return;
        if (tid == 0) atomicExch(&arrivals[b].listed, 0u);
        topk_merge<kBlock>(workspace, n_seg, width, k, logits + (size_t)b * row_stride, out_ids, out_vals, b, tid);
    }
}
__global__ __launch_bounds__(kTopkBlock) void masked_topk_merge_kernel(
    const unsigned long long *__restrict__ workspace, int n_seg, int k, const uint16_t *__restrict__ logits, int64_t row_stride,
    int32_t *__restrict__ out_ids, uint16_t *__restrict__ out_vals) {
    const int b = blockIdx.x;
    topk_merge<kTopkBlock>(workspace, n_seg, topk_width(n_seg, k), k, logits + (size_t)b * row_stride, out_ids, out_vals, b, threadIdx.x);
}

}  // namespace

// blocks per row of the argmax kernel: enough blocks to fill the chip, and every block at least
// one full pass wide
static int masked_argmax_segments(int batch, int vocab, int n_compute_units) {
    const int groups = (vocab + 7) / 8;
    const int max_seg = (groups + kArgBlock * kArgUnroll - 1) / (kArgBlock * kArgUnroll);
    int n_seg = batch > 0 ? (n_compute_units + batch - 1) / batch : 1;
    n_seg = n_seg > max_seg ? max_seg : n_seg;
    return n_seg < 1 ? 1 : n_seg;
}

// (for a batch of `batch` rows or fewer: fewer rows are split into more segments, at most units + rows in all)
size_t masked_argmax_workspace_bytes(int batch, int vocab, int n_compute_units) {
    const size_t split = (size_t)batch * masked_argmax_segments(1, vocab, n_compute_units);
    return std::min(split, (size_t)batch + n_compute_units) * sizeof(unsigned long long);
}

hipError_t launch_masked_argmax(const uint16_t *logits, const uint32_t *bitmask, int batch, int vocab, int64_t row_stride,
                                int n_compute_units, unsigned long long *workspace, int32_t *out, hipStream_t stream) {
    if (batch == 0) return hipSuccess;
    const int n_words = (vocab + 31) / 32, groups = (vocab + 7) / 8;
    const int n_seg = masked_argmax_segments(batch, vocab, n_compute_units);
    const int groups_per_seg = (groups + n_seg - 1) / n_seg;
    hipLaunchKernelGGL(masked_argmax_kernel, dim3(batch, n_seg), dim3(kArgBlock), 0, stream, logits, bitmask, vocab,
                       row_stride, n_words, groups_per_seg, workspace, out);
    if (n_seg > 1)
        hipLaunchKernelGGL(masked_argmax_finish_kernel, dim3((batch + kArgFinishRows - 1) / kArgFinishRows),
                           dim3(64 * kArgFinishRows), 0, stream, batch, n_seg, workspace, out);
    return hipGetLastError();
}

static int masked_topk_chunks(int vocab, int chunk = kTopkChunk) { return (vocab + chunk - 1) / chunk; }

bool masked_topk_fits(int vocab, int k) {
    return k >= 1 && k <= kTopkMax && vocab >= 1 && vocab <= (1 << kTopkIdBits) &&
           masked_topk_chunks(vocab) * k <= kTopkMergeMax;
}

size_t masked_topk_workspace_bytes(int batch, int vocab) {
    return (size_t)batch * masked_topk_chunks(vocab) * kTopkMax * sizeof(unsigned long long);
}

// Groups of eight logits per thread of the blocks that a row is cut into (4: the narrow block, 16,384 tokens; else the wide
// one).  A row that fits the registers of a block is one block's, the smallest that holds it (128,256 tokens, k = 50: 8.0 us
// for one row, 10.7 for 64, 15.4 for 256), except
//   * small batches of the rows that one block streams longest, which go over narrow blocks that hand over in one launch.  That costs
//     the exchange (a store, a count and a load past the L2s, about 2.5 us) and saves the stream of one compute unit and, where few
//     tokens are allowed, the ranking of all of them by one block.  us, narrow blocks and one block, k = 50 (64; k = 50 with 1 in 1,024 tokens
//     allowed): 8 x 131,073 8.1 and 10.7 (8.5 and 11.0; 8.3 and 14.5), 28 x 131,073 9.0 and 11.3 (9.2 and 11.6; 9.2 and 15.2), 1 x 152,064 7.9
//     and 9.4 (8.3 and 12.6; 8.1 and 9.7), 25 x 152,064 9.3 and 11.1 (9.6 and 11.4; 9.5 and 14.9), 25 x 163,840 9.3 and 11.3 (9.8 and 11.6; 9.5
//     and 14.1); 1 x 128,256 7.6 and 8.9 (8.0 and 9.2; 7.9 and 9.0), 16 x 128,256 8.4 and 9.8 (8.7 and 10.0; 8.6 and 13.3), 16 x 114,689 8.4 and 9.9.
//     Rows of more than sixteen groups take them while their blocks fit the compute units once (with a few more, 31 x 163,840 with k = 64,
//     12.8 and 11.7), rows of more than fourteen for half of the units (24 x 128,256 9.4 and 9.8).  On shorter rows they lose (16 x
//     65,000 10.0 and 7.8);
//   * rows of more than sixteen groups off 16-byte boundaries, whose loads a block gets through more slowly: twenty groups only where
//     two blocks a row are more than one round of the chip (160,003 tokens: 200 rows 20.8 and 28.3, 300 38.0 and 39.9; but 128 19.8 and
//     17.8, 32 18.3 and 16.1, and, against narrow blocks, 16 17.8 and 12.4, 2 16.9 and 10.9); on 16-byte boundaries they win (64 x
//     152,064 11.8 and 12.6, 200 14.5 and 21.7, 512 31.8 and 42.0).
// A longer row is cut into wide blocks unless the batch is too small to fill the chip with them (at the line, 31 rows
// of 200,000 tokens take 13.8 to 14.4 us in narrow blocks and 13.7 in wide ones), of twenty groups where those come to
// fewer rounds (280,000 tokens: 128 rows 19.4 us, 27.3 in blocks of sixteen; 256 33.5 and 40.6; but 500,000 x 32 15.9 and 14.3,
// 400,000 x 64 16.3 and 15.4).  (This and the line before: measured with a second launch that merged the blocks' lists; merged by
// the last of the blocks they take 0.6 to 1.9 us less: 2 x 160,003 10.6 -> 9.4, 31 x 160,003 13.0 -> 11.9, 16 x 200,000 11.2 -> 10.3,
// 40 x 200,000 13.6 -> 13.0.)
int masked_topk_groups(int vocab, int batch, bool aligned, int n_compute_units) {
    constexpr int kPerGroup = 8 * kTopkBlockWide;
    if (vocab <= kTopkChunk) return 4;
    const int most = vocab > 8 * kTopkChunk ? n_compute_units : vocab > 7 * kTopkChunk ? n_compute_units / 2 : 0;
    if (batch * masked_topk_chunks(vocab) <= most) return 4;
    for (int g : {8, 12, 16})
        if (vocab <= g * kPerGroup) return g;
    if (vocab <= kTopkRowTokens && aligned) return 20;
    if (batch * 8 < n_compute_units) return 4;
    const int shorter = vocab <= 24 * kPerGroup ? 12 : 16;
    auto rounds = [&](int g) { return (batch * masked_topk_chunks(vocab, g * kPerGroup) + n_compute_units - 1) / n_compute_units; };
    return rounds(20) < rounds(shorter) ? 20 : shorter;
}

// A row's blocks are merged by a launch of their own where they are more than two rounds of the chip: the exchange is paid with every
// round, a launch (2 to 3 us) once.  us per call, k = 50, merged by the last block and apart: 128 x 200,000 18.8 and 19.5, 256 x 200,000 32.3
// and 32.6, 256 x 300,000 39.3 and 40.0, but 300 x 200,000 41.5 and 40.5, 400 x 200,000 51.7 and 49.6, 640 x 200,000 68.6 and 64.5, 400 x 300,000
// 65.2 and 63.0, 300 x 500,000 71.7 and 67.8 (k = 33); 16 x 900,000 in narrow blocks 16.0 and 15.7, 16 x 500,000 10.8 and 11.2.
bool masked_topk_merged_apart(int batch, int n_seg, int n_compute_units) { return batch * n_seg > 2 * n_compute_units; }

hipError_t launch_masked_topk(const uint16_t *logits, const uint32_t *bitmask, int batch, int vocab, int64_t row_stride,
                              int k, int n_compute_units, unsigned long long *workspace, StepArrivals *arrivals, int32_t *out_ids,
                              uint16_t *out_vals, hipStream_t stream) {
    if (batch == 0) return hipSuccess;
    if (!masked_topk_fits(vocab, k)) return hipErrorInvalidValue;
    const int n_words = (vocab + 31) / 32;
    const bool aligned = (reinterpret_cast<uintptr_t>(logits) & 15) == 0 && (row_stride & 7) == 0;
#define PRE3_TOPK_ROW(BLOCK, GROUPS)                                                                                         \
    n_seg = masked_topk_chunks(vocab, BLOCK * GROUPS * 8);                                                                   \
    apart = n_seg > 1 && masked_topk_merged_apart(batch, n_seg, n_compute_units);                                              \
    if (n_seg > 1) PRE3_TOPK_BLOCKS(BLOCK, GROUPS, true);                                                                    \
    else PRE3_TOPK_BLOCKS(BLOCK, GROUPS, false)
#define PRE3_TOPK_BLOCKS(BLOCK, GROUPS, SEVERAL)                                                                             \
    hipLaunchKernelGGL((masked_topk_row_kernel<BLOCK, GROUPS, SEVERAL>), dim3(batch, n_seg), dim3(BLOCK), 0, stream, logits, bitmask, \
                       vocab, row_stride, n_words, k, workspace, out_ids, out_vals, apart ? nullptr : arrivals)
    int n_seg = 1;
    bool apart = false;
    switch (masked_topk_groups(vocab, batch, aligned, n_compute_units)) {
        case 4: PRE3_TOPK_ROW(kTopkBlock, 4); break;
        case 8: PRE3_TOPK_BLOCKS(kTopkBlockWide, 8, false); break;          // (always one block)
        case 12: PRE3_TOPK_ROW(kTopkBlockWide, 12); break;
        case 16: PRE3_TOPK_ROW(kTopkBlockWide, 16); break;
        default: PRE3_TOPK_ROW(kTopkBlockWide, 20);
    }
#undef PRE3_TOPK_BLOCKS
#undef PRE3_TOPK_ROW
    if (apart)
        hipLaunchKernelGGL(masked_topk_merge_kernel, dim3(batch), dim3(kTopkBlock), 0, stream, workspace, n_seg, k, logits, row_stride, out_ids,
                           out_vals);
    return hipGetLastError();
}

}  // namespace pre3
