// gfx950 kernels of the stack advance: one sampled token per sequence walked on the sequence's
// own stack, alone or followed by the next step's mask row in the same launch.
#include <hip/hip_runtime.h>

#include <mutex>

#include "argmax.hpp"
#include "launch.hpp"
#include "row_plan.hpp"

// Spill area of the private stacks for pre3_advance_static, the entry point that allocates
// nothing: device memory that belongs to the loaded library itself (every GPU the library runs
// on holds its own copy until the process ends).  Host code never passes this name to a kernel:
// the device address is taken once per device with hipGetSymbolAddress (static_advance_scratch).
static __device__ __align__(256) int32_t pre3_static_scratch[pre3::kStaticScratchEntries];

namespace pre3 {

namespace {

// -------------------------------------------------------------------------- advance

// The bytes of a sampled token as the walk needs them: lane i holds the class/offset word of byte i (of the first 64;
// later ones are read through the id-ordered vocabulary at lo + i).
struct StagedToken {
    int32_t infos;
    int lo, n_bytes;
};

// The token's line (length, then 31 byte words) as one load that waits for nothing: lane i gets byte i's word, lane 31
// the length.  finish_token makes a staged token of it (tokens longer than the line are fetched there).
__device__ __forceinline__ int32_t fetch_token_line(const DevTables &T, int t, int lane) {
    static_assert(kTokInfoBytes == 31, "a line is the length and 31 bytes");
    return T.tok_info[(size_t)t * 32 + ((lane + 1) & 31)];
}
__device__ __forceinline__ StagedToken finish_token(const DevTables &T, int t, int32_t line, int lane) {
    StagedToken tok{line, 0, __builtin_amdgcn_readlane(line, 31)};
    if (tok.n_bytes < 0) {
        tok.lo = T.voffsets[t];
        tok.n_bytes = T.voffsets[t + 1] - tok.lo;
        tok.infos = lane < tok.n_bytes ? T.byte_info[T.vbytes[tok.lo + lane]] : 0;
    }
    return tok;
}

// Lanes kLane0 .. kLane0 + kCount of `w` replaced by the wave-uniform words v[kSrc0 ..] (one v_writelane
// each; the lane is an immediate, the instruction takes one scalar register only).
template <int kLane0, int kSrc0, int kCount, int kI = 0>
__device__ __forceinline__ int32_t deal_to_lanes(int32_t w, const NativeInt16 &v) {
    if constexpr (kI < kCount) {
        asm("v_writelane_b32 %0, %1, %2" : "+v"(w) : "s"(v[kSrc0 + kI]), "n"(kLane0 + kI));
        return deal_to_lanes<kLane0, kSrc0, kCount, kI + 1>(w, v);
    } else {
        return w;
    }
}

// The words of a token's line, in two scalar loads' registers, dealt out to the lanes as fetch_token_line has them.
__device__ __forceinline__ int32_t deal_token_line(const NativeInt16 &a, const NativeInt16 &b) {
    int32_t w = 0;
    w = deal_to_lanes<0, 1, 15>(w, a);
    w = deal_to_lanes<15, 0, 16>(w, b);
    return deal_to_lanes<31, 0, 1>(w, a);
}

// The top 64 entries of a stack of 1 <= n <= cap entries (lane k: entry k below the top, -1 beyond the bottom) through
// the scalar cache: four 16-entry loads that end at the top -- each moved to where it lies wholly inside the row's
// cap entries, cap >= 16 --, dealt out to the lanes and put in order with one lane permute.  The first load is the
// caller's (`first`, at window_chunk(n, cap, 0)): it stands with the other loads that depend on the inputs alone.
__device__ __forceinline__ int window_chunk(int n, int cap, int c) {
    int lo = n - 16 * (c + 1);
    lo = lo < 0 ? 0 : lo;
    return lo > cap - 16 ? cap - 16 : lo;
}
__device__ __forceinline__ int32_t deal_window(const int32_t *row, const NativeInt16 &first, int n, int cap, int lane) {
    int32_t w = deal_to_lanes<0, 0, 16>(0, first);
    int my_lo = window_chunk(n, cap, 0);                // first entry of the chunk that holds this lane's entry
    // one chunk at a time, and only the chunks the stack reaches (few scalar registers live; the later loads
    // find their cache lines where the first one brought them)
    if (n > 16) {
        const int lo1 = window_chunk(n, cap, 1);
        w = deal_to_lanes<16, 0, 16>(w, scalar_load16(row + lo1));
        if (lane >= 16) my_lo = lo1;
        if (n > 32) {
            const int lo2 = window_chunk(n, cap, 2);
            w = deal_to_lanes<32, 0, 16>(w, scalar_load16(row + lo2));
            if (lane >= 32) my_lo = lo2;
            if (n > 48) {
                const int lo3 = window_chunk(n, cap, 3);
                w = deal_to_lanes<48, 0, 16>(w, scalar_load16(row + lo3));
                if (lane >= 48) my_lo = lo3;
            }
        }
    }
    // entry k below the top is entry n - 1 - k, in the chunk k / 16 (whose begin the lanes of that chunk hold)
    const int idx = n - 1 - lane;
    const int32_t x = __shfl(w, (lane & 48) + ((idx - my_lo) & 15));
    return idx >= 0 ? x : -1;
}

// The first min(d, 64) >= 1 entries of a table's list through the scalar cache: lane i holds entry i (lanes from d on hold
// what follows the list).  One vector load in its place waits behind the row loads of the block's other waves: one-kernel
// steps with cycle-aware stacks, whose tokens push a state per character, 100,000 tokens, 130 rows 17.6 us per step that way and 17.0
// this way, 200,000 x 64 20.3 and 19.6, greedy 128,256 x 128 16.3 and 15.6.
__device__ __forceinline__ int32_t fetch_list_scalar(const int32_t *list, int d) {
    int32_t w = deal_to_lanes<0, 0, 16>(0, scalar_load16(list));
    if (d > 16) {
        w = deal_to_lanes<16, 0, 16>(w, scalar_load16(list + 16));
        if (d > 32) {
            w = deal_to_lanes<32, 0, 16>(w, scalar_load16(list + 32));
            if (d > 48) w = deal_to_lanes<48, 0, 16>(w, scalar_load16(list + 48));
        }
    }
    return w;
}

constexpr int kScalarRunMin = 8;       // bytes left in a token before a scalar-only walk looks for a run

// Walks a staged token from the configuration  row[0..base) ++ pushed[0..d)  with capacity checks.  Runs on
// all 64 lanes with identical values (scalar table loads, single lanes of the wave's registers); a run of
// self-similar edges is applied in one step.  Returns kFed, kRejected or kOverflow.
template <bool kScalar = false>
__device__ __forceinline__ int walk_staged_token(const DevTables &T, WaveStack &ws, const StagedToken &tok, int cap, int &base,
                                                 int &d, int &top, int &kind) {
    int rc = tok.n_bytes > 0 ? kFed : kRejected;
    for (int i = 0; i < tok.n_bytes && rc == kFed; ++i) {
        int info = __builtin_amdgcn_readlane(tok.infos, i < 64 ? i : 63);
        if (i >= 64) info = __builtin_amdgcn_readfirstlane(T.byte_info[T.vbytes[tok.lo + i]]);
        int run_node = -1;
        rc = feed<true, true, kScalar>(T, ws, info, base, d, top, kind, ws, cap, &run_node);
        // (a run is examined with one vector load per lane: a wave that keeps to scalar loads takes short tails byte by byte)
        if (rc == kFed && run_node >= 0 && i + 1 < tok.n_bytes && (!kScalar || tok.n_bytes - (i + 1) >= kScalarRunMin))
            i += apply_run<true>(T, ws, tok.infos, i + 1, tok.n_bytes, run_node, kind, base, d, top, cap);
    }
    return rc;
}

// Writes the d pushed states of a finished walk above row[0..base): the first 64 by one lane each, states that
// spilled to global memory by lane 0.
__device__ __forceinline__ void commit_pushed(int32_t *row, const WaveStack &ws, int base, int d, int lane) {
    if (lane < d) row[base + lane] = ws.pushed;
    if (lane == 0)
        for (int i = kWindow; i < d; ++i) row[base + i] = global_read(ws.spill + (size_t)(i - kWindow) * ws.spill_stride);
}

// Cycle-aware stack compaction (Sec. 3.2.3; Alg. 1 step 1) of a stack staged in LDS, s[0 .. n): a
// complete traversal v1..vn of a registered reduction cycle that lies right below another v1 carries
// no information and is taken out.  The stack is rebuilt entry by entry from the bottom; after each
// entry that is the head of a cycle, the n entries under it are compared with the cycle's states
// and dropped on a match (then the check repeats).  Run by the 64 lanes of one wave in lockstep:
// lanes look up cycle_head for 64 entries at a time, a ballot finds the heads, lane i compares
// entry i of a traversal, segments between heads are moved down as blocks.  `pool` = the cycle
// records in their device layout (states last first, kCyclePoolPad entries of padding at the end),
// in LDS or global memory.  Returns the new length; *first_moved = lowest index whose
// content changed (= the new length if only the top was cut, n if nothing changed).
__device__ __forceinline__ int fold_cycles(int32_t *s, int n, const int32_t *cycle_head, const int32_t *pool,
                                           int n_states, int lane, int *first_moved) {
    // Where can the first traversal end?  Until one is dropped the stack has its original layout, and
    // a traversal of length k under the entry at position p needs s[p - k] == s[p] (both are the
    // cycle's first state): every lane tests that for one position and the cycles of its state, and
    // the rebuilding starts at the lowest position that passes -- in a stack that was compacted
    // before the call, that is inside the entries the call added.
    int start = n;
    for (int r0 = 0; r0 < n && start == n; r0 += 64) {
        const int p = r0 + lane;
        bool candidate = false;
        if (p < n) {
            const int x = s[p];
            for (int at = (unsigned)x < (unsigned)n_states ? cycle_head[x] : -1; at >= 0 && !candidate; at = pool[at + 1]) {
                const int k = pool[at];
                candidate = p - k >= 0 && s[p - k] == x;
            }
        }
        const unsigned long long c = __ballot(candidate);
        if (c) start = r0 + __ffsll((long long)c) - 1;
    }
    if (start == n) { *first_moved = n; return n; }
    int w = start, moved = n;
    for (int r0 = start; r0 < n; r0 += 64) {
        const int cnt = n - r0 < 64 ? n - r0 : 64;
        const int x = lane < cnt ? s[r0 + lane] : -1;
        const int hd = (unsigned)x < (unsigned)n_states ? cycle_head[x] : -1;
        unsigned long long heads = __ballot(hd >= 0);
        if (heads == 0 && w == r0) { w += cnt; continue; }
        int prev = 0;                                   // entries of this chunk already moved
        for (;;) {
            const int j = heads ? __ffsll((long long)heads) - 1 : cnt - 1;   // the segment prev..j ends at a head or at the chunk's end
            const int seg = j - prev + 1;
            if (seg > 0) {
                if (w != r0 + prev) {                   // all lanes read, then all lanes write: the ranges may overlap
                    const int v = lane < seg ? s[r0 + prev + lane] : 0;
                    wave_exchange();
                    if (lane < seg) s[w + lane] = v;
                    wave_exchange();
                    moved = w < moved ? w : moved;
                }
                w += seg;
            }
            if (!heads) break;
            heads &= heads - 1;
            prev = j + 1;
            const int first = __builtin_amdgcn_readlane(hd, j);   // s[w - 1] is the head of these cycles
            int h = first;
            while (h >= 0) {
                // one round of loads per record: its header, its states (stored last first and
                // padded, so no address depends on the length) and the entries under the head
                const int header = pool[h + (lane & 1)];
                const int want = pool[h + 2 + lane];
                const int have = w - 2 - lane >= 0 ? s[w - 2 - lane] : -1;
                const int k = __builtin_amdgcn_readlane(header, 0), next = __builtin_amdgcn_readlane(header, 1);
                const bool match = __all(lane >= k || have == want);   // an entry below the bottom (-1) matches no state
                if (match) {
                    w -= k;                             // the top stays: s[w - 1] held the same state
                    moved = w < moved ? w : moved;
                    // The new top failed every check when it was put there, over the same entries:
                    // no need to try its records again.  And the k entries just dropped, s[w .. w + k),
                    // took the stack from this very content back to it without any drop on the way, so
                    // every further copy of them that follows in the input does the same: skip those
                    // copies (as far as they lie in this chunk) at once.
                    const int left = cnt - prev;
                    if (left >= k) {
                        const bool same = lane < left && s[r0 + prev + lane] == s[w + lane % k];
                        const unsigned long long differs = ~__ballot(same);
                        const int run = differs ? __ffsll((long long)differs) - 1 : 64;
                        prev += run / k * k;
                        heads = prev >= 64 ? 0ull : heads & (~0ull << prev);
                    }
                    h = -1;
                } else {
                    h = next;
                }
            }
        }
    }
    *first_moved = moved;
    return w;
}

// The cycle tables (cycle_head[n_states], then the records) are small for most grammars: the threads
// given here copy them into LDS (`lds`, n_states + pool_n entries) so that fold_cycles, whose look-ups
// depend on one another, does not go to global memory for each.  The caller puts a block barrier
// between this copy and the first use.
constexpr int kStageCycleStates = 4096, kStageCyclePool = 1024;
__host__ __device__ inline bool cycles_fit_lds(int n_states, int pool_n) {
    return n_states <= kStageCycleStates && pool_n <= kStageCyclePool;
}
__device__ __forceinline__ void copy_cycle_tables(int32_t *lds, int n_states, int pool_n, const int32_t *head,
                                                  const int32_t *pool, int first, int step) {
    for (int i = first; i < n_states; i += step) lds[i] = head[i];
    for (int i = first; i < pool_n; i += step) lds[n_states + i] = pool[i];
}

// What an advance leaves to be stored: the new stack is  row[0 .. base) ++ pushed[0 .. d)  (or, compacted, the first
// nl entries staged in LDS, of which those from `from` on changed; just its bottom entry after a restart).
struct Advanced {
    int base, d, nl, from, n, token, out_err, out_state;
    bool shape_ok, restarted;
};

// What a launch advances from: the sampled token, the stack's length, its top state.  The first loads of a kernel, or of its
// branch that advances (the waves that fetch logits do not wait for them: greedy 256 x 128,256 127.9 us, 131.6 when they did).
struct StepInputs { int t, n, st; };
__device__ __forceinline__ StepInputs read_inputs(const int32_t *tokens, const int32_t *len, const int32_t *states, int b) {
    const StepInputs in{table<true>(tokens, b), table<true>(len, b), table<true>(states, b)};
    __builtin_amdgcn_sched_barrier(0);
    return in;
}

// Walks one sequence's sampled token on its stack (or applies the token's stack-effect record): the work of one
// wave, all 64 lanes with identical values, the stack in the wave's registers (ws).  Only a walk that succeeds changes the
// stack; nothing is stored: commit_advance does that.  `meet` is called once, when the inputs' loads are under way.
// The launches that wait for it are bound by this chain of dependent look-ups, and what a link costs is as much its
// instructions as its load.  The window, the token's bytes and the pushed states are in registers instead of LDS (one lane
// read looks at an entry), a child's record comes out of its lane with lane reads instead of permutes, and the token's
// line and the state's kind do not wait for the stack's top: bursts of 8 steps of 64 x 32,000 in a graph
// 76.8 -> 68.6 us, 1 x 128,256 57.9 -> 54.2, fill + mask + advance of 96 x 100,003 168 -> 158, advance + fill before a top-k
// of 256 x 128,256 187 -> 181, greedy steps of 320 x 128,256 with cycle-aware stacks 265 -> 255.
// With vector loads the chain begins with two rounds, the inputs with the tables' pointers, then all that depends on the inputs
// alone.  Behind a condition each of these loads was a round of its own wherever the compiler waited at the condition's end (three
// rounds, five in the spread step): 1 x 128,256 54.2 -> 52.8 us, 64 x 32,000 67.9 -> 67.1, fill + mask + advance of 96 x 100,003
// 153.1 -> 151.4, advance + fill before a top-k of 256 x 128,256 179.4 -> 178.2.  The wave that keeps to scalar loads is not held
// to that order: it has not the registers for all of them at once (greedy 320 x 128,256, cycle-aware, 202.4 us and 203.7 held to it).
// kWindowFirst: the window is in its lanes before the token's line is asked for (sixteen and thirty-two scalar registers together pass
// what the wave has where the block's other waves need the registers most: two rows to a unit, 368 scalars in lanes against 188;
// cycle-aware stacks on 256 x 150,000 161.5 against 159.1 us; the other forms lose by it: 256 x 128,256 130.7 against 134.5).
template <bool kScalar, bool kWindowFirst, class Meet>
__device__ __forceinline__ Advanced advance_stack(const DevTables &T, const DevTokenEdges &E, const StepInputs &in, int cap,
                                                  int restart_on_eos, WaveStack &ws, int lane, Meet meet) {
    const int32_t *row = ws.row;
    const int t = in.t, n = in.n, st = in.st;
    if (!kScalar) {
        // (the asm statements here and below: the loads of what they name are issued before this point and waited for together)
        asm volatile("" :: "s"(t), "s"(n), "s"(st), "s"(T.n_tokens), "s"(T.n_states), "s"(T.eos_id), "s"(T.ncol), "s"(T.state_kind),
                     "s"(T.tok_info), "s"(T.sym_nodes), "s"(T.sym_cell), "s"(E.root_id), "s"(E.root_nodes), "s"(E.fx_slots),
                     "s"(E.nodes), "s"(E.child_state), "s"(E.fx_mask), "s"(E.fx_min_len));
        __builtin_amdgcn_sched_barrier(0);
    }
    const bool shape_ok = n >= 1 && n <= cap;
    const bool live = t >= 0 && t < T.n_tokens && st >= 0 && shape_ok;
    // What depends on the inputs alone, one round of loads without a branch: the stack window, the token's line, and --
    // states[b] names the stack's top -- that state's kind and the root of its condition tree, from which the look-up of the
    // token's stack operations starts.  An input out of range, a table that was not built: the load is of something that is there
    // (token 0, state 0, the bottom entry, the tables' own copy), and what it brings is not looked at.
    const bool st_ok = (unsigned)st < (unsigned)T.n_states, look_up = live && st_ok && E.fx_slots && t != T.eos_id;
    const int tc = (unsigned)t < (unsigned)T.n_tokens ? t : 0, sc = st_ok ? st : 0, nc = shape_ok ? n : 1;
    const int32_t *spare = reinterpret_cast<const int32_t *>(T.pack);
    const int32_t *kind_at = T.state_kind ? T.state_kind + sc : spare, *root_at = E.fx_slots ? E.root_id + sc : spare;
    const DevConditionNode *nd_at = E.fx_slots ? E.root_nodes + sc : reinterpret_cast<const DevConditionNode *>(spare);
    int kind = table<true>(kind_at, 0), fx_root = table<true>(root_at, 0);
    const DevConditionNode fx_nd = scalar_node(nd_at);
    int32_t line;
    if (kScalar) {
        const int32_t *rec = T.tok_info + (size_t)tc * 32;
        if (kWindowFirst) {
            if (cap >= 16) ws.win = deal_window(row, scalar_load16(row + window_chunk(nc, cap, 0)), nc, cap, lane);
            else ws.win = nc - 1 - lane >= 0 ? row[nc - 1 - lane] : -1;
            __builtin_amdgcn_sched_barrier(0);
        }
        const NativeInt16 line0 = scalar_load16(rec), line1 = scalar_load16(rec + 16);
        if (!kWindowFirst && cap >= 16) {
            const NativeInt16 first = scalar_load16(row + window_chunk(nc, cap, 0));
            line = deal_token_line(line0, line1);
            ws.win = deal_window(row, first, nc, cap, lane);
        } else {
            line = deal_token_line(line0, line1);
            if (!kWindowFirst) ws.win = nc - 1 - lane >= 0 ? row[nc - 1 - lane] : -1;
        }
    } else {
        const int at = nc - 1 - lane;
        const int32_t entry = row[at >= 0 ? at : 0];
        line = fetch_token_line(T, tc, lane);
        asm volatile("" :: "v"(entry), "v"(line), "s"(kind), "s"(fx_root), "s"(fx_nd.known), "s"(fx_nd.child_count), "s"(fx_nd.a),
                     "s"(fx_nd.b));
        __builtin_amdgcn_sched_barrier(0);
        ws.win = at >= 0 ? entry : -1;
    }
    if (!shape_ok) ws.win = -1;
    if (!T.state_kind) kind = 0;
    if (!look_up) fx_root = -1;
    ws.pushed = 0;
    ws.n = n;
    meet();
    int out_err = 0, out_state = st, out_len = n, base = n, d = 0;
    bool restarted = false;
    if (t >= 0) {
        int top = live ? __builtin_amdgcn_readlane(ws.win, 0) : -1;
        if (!live || (unsigned)top >= (unsigned)T.n_states) {
            out_err = 1;
        } else {
            if (top != st && T.state_kind) kind = table<true>(T.state_kind, top);
            if (t == T.eos_id) {
                if (feed<false, true, kScalar>(T, ws, T.end_col, base, d, top, kind, ws, 0) == kAccepted) {
                    out_state = -1;
                    if (restart_on_eos) {               // slot reuse: back to the initial state, the stack's bottom entry
                        out_state = ws.at(0);
                        out_len = 1;
                        restarted = true;
                    }
                } else {
                    out_err = 1;
                }
                base = n;
                d = 0;                               // the '$' walk never changes the stack
            } else {
                // a longer token whose merged edge carries its stack operations is applied in one
                // step (look-up, truncate, push); every other token is walked byte by byte
                const StagedToken tok = finish_token(T, t, line, lane);
                EffectHit fx{0, 0, 0, 0, 0, 0, 0};
                if (fx_root >= 0 && top == st && tok.n_bytes >= E.fx_min_len) {
                    auto deeper = [&](int k2) { return global_read(row + (n - 1 - k2)); };
                    fx = kScalar ? find_effect_scalar(E, fx_root, fx_nd, ws.win, n, deeper, t)
                                 : find_effect(E, fx_root, fx_nd, ws.win, n, deeper, t, lane);
                }
                int rc;
                if (fx.found && fx.k <= n && fx.np <= T.max_depth) {
                    if (n + fx.peak >= cap) {
                        rc = kOverflow;
                    } else {
                        base = n - fx.k + 1;
                        d = fx.np;
                        if (fx.inline_count > 0) {
                            top = fx.inline_count == 2 ? fx.x1 : fx.x0;
                            ws.pushed = lane == 0 ? fx.x0 : fx.x1;
                        } else {
                            if (kScalar) {
                                ws.pushed = fetch_list_scalar(E.fx_pool + fx.x0, d);
                                top = __builtin_amdgcn_readlane(ws.pushed, min(d, kWindow) - 1);
                            }
                            for (int i0 = kScalar ? kWindow : 0; i0 < d; i0 += 64) {     // (64 states at a time, one load)
                                const int32_t v = i0 + lane < d ? E.fx_pool[fx.x0 + i0 + lane] : 0;
                                if (i0 == 0) ws.pushed = v;
                                else if (i0 + lane < d) ws.spill[(size_t)(i0 - kWindow + lane) * ws.spill_stride] = v;
                                if (d - i0 <= 64) top = __builtin_amdgcn_readlane(v, d - 1 - i0);
                            }
                            if (d > kWindow) __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup");   // other lanes read them back
                        }
                        rc = kFed;
                    }
                } else {
                    rc = walk_staged_token<kScalar>(T, ws, tok, cap, base, d, top, kind);
                }
                if (rc != kFed) {
                    out_err = rc == kOverflow ? 2 : 1;
                    base = n;
                    d = 0;
                } else {
                    out_len = base + d;
                    out_state = top;
                }
            }
        }
    }
    return Advanced{base, d, out_len, 0, n, t, out_err, out_state, shape_ok, restarted};
}

// The entries 0 .. 63 below the top of  row[0 .. base) ++ pushed[0 .. d), one per lane (-1 beyond the bottom).
__device__ __forceinline__ int32_t new_window(const WaveStack &ws, int base, int d, int lane) {
    const int i = d - 1 - lane, idx = base + i, k = ws.n - 1 - idx;      // pushed[i] if i >= 0, else row[idx], k below the old top
    int32_t pushed = __shfl(ws.pushed, i & 63), old = __shfl(ws.win, k & 63);
    if (i >= kWindow) pushed = global_read(ws.spill + (size_t)(i - kWindow) * ws.spill_stride);
    if (i < 0 && idx >= 0 && k >= kWindow && ws.n >= 1) old = global_read(ws.row + idx);
    return i >= 0 ? pushed : idx >= 0 ? old : -1;
}

// Cycle-aware stacks: puts the new stack together at `stack` (LDS, cap entries), takes complete traversals of
// reduction cycles out of it and notes in `r` what is left and what of it changed.
__device__ __forceinline__ void fold_new_stack(Advanced &r, const WaveStack &ws, int32_t *stack, const int32_t *cycle_head,
                                               const int32_t *cycle_pool, int n_states, int lane) {
    for (int i0 = 0; i0 < r.nl; i0 += 64) {
        const int i = i0 + lane, k = ws.n - 1 - i, p = i - r.base;
        int32_t old = __shfl(ws.win, k & 63), pushed = __shfl(ws.pushed, p & 63);
        if (i < r.nl) {
            if (p < 0 && k >= kWindow) old = global_read(ws.row + i);
            if (p >= kWindow) pushed = global_read(ws.spill + (size_t)(p - kWindow) * ws.spill_stride);
            stack[i] = p < 0 ? old : pushed;
        }
    }
    wave_exchange();
    int nl = r.nl, first_moved = nl;                    // (1 after a restart: only the bottom entry stays)
    if (nl >= 2) nl = fold_cycles(stack, nl, cycle_head, cycle_pool, n_states, lane, &first_moved);
    r.from = r.restarted ? nl : (first_moved < r.base ? first_moved : r.base);
    r.nl = nl;
}

// Stores what an advance found: the entries of the new stack that changed, states, len and err.
template <bool kCompact>
__device__ __forceinline__ void commit_advance(const Advanced &r, const WaveStack &ws, const int32_t *after_row, int32_t *states,
                                               int32_t *row, int32_t *len, int32_t *err, int cap, int b, int lane) {
    if (kCompact && r.shape_ok) {
        for (int i = r.from + lane; i < r.nl; i += 64) row[i] = after_row[i];
        if (lane == 0) {
            err[b] = r.out_err;
            if ((r.out_err == 0 && r.token >= 0) || r.nl != r.n) { states[b] = r.out_state; len[b] = r.nl; }
        }
    } else {
        commit_pushed(row, ws, r.base, r.d, lane);
        if (lane == 0) {
            err[b] = r.out_err;
            if (r.out_err == 0 && r.token >= 0) { states[b] = r.out_state; len[b] = r.nl; }
        }
    }
}

// One wave per sequence: the walk of a single token is a chain of dependent table look-ups, so
// giving every sequence its own wave keeps control flow uniform (lanes of a shared wave would
// serialise each other's reduction chains) and lets the chip overlap the chains of all
// sequences.
// kCompact (cycle-aware stacks): instead of storing the pushed states, the wave puts the new
// stack together in LDS (cap entries per sequence), takes complete traversals of reduction cycles
// out of it (fold_cycles) and writes back what changed.
constexpr int kAdvSeqPerBlock = 4;
template <bool kCompact>
__global__ __launch_bounds__(64 * kAdvSeqPerBlock) void advance_kernel(
    const int32_t *__restrict__ tokens, int32_t *__restrict__ len, int32_t *__restrict__ states,
    int32_t *__restrict__ data, int cap, int batch, const DevPack *pack, int32_t *__restrict__ err, int32_t *scratch,
    int restart_on_eos, const int32_t *cycle_head, const int32_t *cycle_pool, int stage_cycles) {
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63;
    const int b = blockIdx.x * kAdvSeqPerBlock + wave;
    const StepInputs in = read_inputs(tokens, len, states, b < batch ? b : 0);
    DevTables T;
    DevTokenEdges E;
    load_tables(pack, T, E);
    extern __shared__ int32_t adv_stage[];             // kCompact: kAdvSeqPerBlock x (cap stack entries [+ cycle tables])
    // kCompact with small cycle tables: the block copies them into LDS behind the staged stacks; every
    // wave passes exactly one block barrier (a wave without a sequence right here, the others once
    // their own input loads are under way)
    int32_t *cycle_lds = adv_stage + kAdvSeqPerBlock * cap;
    if (kCompact && stage_cycles) {
        copy_cycle_tables(cycle_lds, T.n_states, T.cycle_pool_n, cycle_head, cycle_pool, threadIdx.x, 64 * kAdvSeqPerBlock);
        cycle_head = cycle_lds;
        cycle_pool = cycle_lds + T.n_states;
    }
    if (b >= batch) {
        if (kCompact && stage_cycles) __syncthreads();
        return;
    }
    int32_t *row = data + (size_t)b * cap, *stack = adv_stage + wave * cap;
    WaveStack ws{row, scratch + b, (size_t)batch, 0, 0, 0};
    Advanced r = advance_stack<false, false>(T, E, in, cap, restart_on_eos, ws, lane,
                                      [&] { if (kCompact && stage_cycles) __syncthreads(); });
    if (kCompact && r.shape_ok) fold_new_stack(r, ws, stack, cycle_head, cycle_pool, T.n_states, lane);
    commit_advance<kCompact>(r, ws, stack, states, row, len, err, cap, b, lane);
}

// The work of the wave that advances one sequence and looks up its next mask row: walks the sampled token
// (advance_stack), then descends the condition tree of the token-level edges with the new stack; the result is
// `plan`.  kCompact: the new stack is put together at after_row (LDS, cap
// entries), folded and only then looked up; stage_cycles: the block's other waves copy the cycle tables to
// after_row + cap meanwhile and meet this wave at one block barrier.
// The tree is descended BEFORE anything is stored: a wave that has stores in flight waits for them wherever it next waits
// for a load, and in the one-launch step kernel they complete only behind the row loads of the block's other waves.
template <bool kCompact, bool kScalar = false, bool kWindowFirst = false>
__device__ __forceinline__ Advanced advance_and_plan(const DevTables &T, const DevTokenEdges &E, const StepInputs &in, int cap,
                                                 int restart_on_eos, WaveStack &ws, const int32_t *cycle_head,
                                                 const int32_t *cycle_pool, int stage_cycles, int32_t *after_row, RowPlan &plan,
                                                 int lane) {
    Advanced r = advance_stack<kScalar, kWindowFirst>(T, E, in, cap, restart_on_eos, ws, lane, [&] {
        if (kCompact && stage_cycles) {                 // the other waves have copied the cycle tables meanwhile
            __syncthreads();
            int32_t *cycle_lds = after_row + cap;
            cycle_head = cycle_lds;
            cycle_pool = cycle_lds + T.n_states;
        }
    });
    // the root of the new top's condition tree is under way while the new window is put together (taking cycles out keeps the top)
    const DevConditionNode root = scalar_node(E.root_nodes + ((unsigned)r.out_state < (unsigned)T.n_states ? r.out_state : 0));
    int32_t win;                                        // the top of the new stack
    if (kCompact && r.shape_ok) {
        fold_new_stack(r, ws, after_row, cycle_head, cycle_pool, T.n_states, lane);
        win = lane < r.nl ? after_row[r.nl - 1 - lane] : -1;
    } else {
        win = r.restarted ? (lane == 0 ? r.out_state : -1) : new_window(ws, r.base, r.d, lane);
    }
    auto deeper = [&](int k) -> int32_t {               // entry k >= 64 below the new top
        if (kCompact && r.shape_ok) return after_row[r.nl - 1 - k];
        return k < r.d ? ws.get(r.d - 1 - k) : ws.at(r.base - 1 - (k - r.d));
    };
    // ---- descent of the condition tree with the new stack
    const int top = __builtin_amdgcn_readlane(win, 0);
    if (r.out_state < 0) {
        if (lane == 0) plan.mode = kRowDone;
    } else if (!r.shape_ok || (unsigned)top >= (unsigned)T.n_states) {
        if (lane == 0) plan.mode = kRowEmpty;
    } else {
        const DevConditionNode nd = top == r.out_state ? root : scalar_node(E.root_nodes + top);    // (states[b] and the stack's top may differ)
        if (kScalar) plan_row_scalar(E, nd, win, r.nl, deeper, &plan, lane);
        else plan_row(E, nd, win, r.nl, deeper, &plan, lane);
    }
    if (lane == 0) { plan.top = top; plan.len = r.nl; }
    return r;
}

// Advance and next mask in one launch: one block per sequence.  Wave 0 walks the sampled token
// exactly like advance_kernel, descends
// the condition tree of the token-level edges with the NEW top of the stack and commits the new stack; then the
// whole block builds the sequence's next mask row (dense row copy, delta lists, leftover walks)
// and stores it.  The sequence's inputs are loaded once, no kernel boundary separates the two
// halves, and the long walks of a few sequences overlap the mask building of all others.
// kCompact (cycle-aware stacks): the new stack is put together in LDS, complete traversals of reduction
// cycles are taken out of it (fold_cycles) and only then is it written back and looked up, so the call
// leaves compacted stacks and the mask of exactly those stacks.
// Threads per block: 512 while two blocks of that size per compute unit hold the batch, half of that for larger ones (more
// of their blocks are on the chip at once: 1,024 x 128,256 tokens 10.4 against 14.2 us, 2,048 16.2 against 20.0; 256 x 128,256
// 8.8 against 8.6 us), and two waves for large batches of short rows (2,048 x 8,000: 10.3 us; 13.7 with 256 threads, 18.9
// with 512; 2,048 x 32,000 10.1 us with two waves, 2,048 x 33,000 13.6 with 256 threads, 18.5 and 18.7 with 512).
constexpr int kAfBlock = 512, kAfBlockMany = 256, kAfBlockShort = 128;
constexpr int kAfShortWords = 1024;                    // mask words of a short row (32,768 tokens)
// LDS kept for what the kernel declares statically (private stacks, the row plan): what is left of the 64 KB is for the
// dynamic part (mask row, staged stack)
constexpr size_t kAfStaticLdsBytes = 6144;
static_assert(sizeof(int32_t) * kLdsDepth * 64 + sizeof(RowPlan) <= kAfStaticLdsBytes, "the static part fits");
constexpr size_t kAfDynamicLdsMax = 65536 - kAfStaticLdsBytes;
template <bool kCompact, int kThreads>
__global__ __launch_bounds__(kThreads) void advance_fill_kernel(
    const int32_t *__restrict__ tokens, int32_t *__restrict__ len, int32_t *__restrict__ states,
    int32_t *__restrict__ data, int cap, int batch, const DevPack *pack, int32_t *__restrict__ err,
    uint32_t *__restrict__ bitmask, int restart_on_eos, int32_t *adv_scratch, int32_t *walk_spill,
    size_t walk_spill_stride, const int32_t *cycle_head, const int32_t *cycle_pool, int stage_cycles) {
    const StepInputs in = read_inputs(tokens, len, states, blockIdx.x);
    DevTables T;
    DevTokenEdges E;
    load_tables(pack, T, E);
    extern __shared__ uint4 bits4[];                   // whole row: n_words rounded up to a multiple of 4;
                                                       // kCompact: followed by cap stack entries [+ cycle tables]
    __shared__ int32_t s_walk_stack[kLdsDepth * 64];
    __shared__ RowPlan plan;
    const int tid = threadIdx.x, lane = tid & 63;
    const int b = blockIdx.x;
    const int n_vec = (T.n_words + 3) >> 2;
    int32_t *row = data + (size_t)b * cap;

    if (tid >= 64) {
        // The waves that wait for the walk pull the small tables it reads into this XCD's L2 (a
        // streaming kernel that ran in between has evicted them): one 128-byte line per lane,
        // the lines dealt out over the blocks of the XCD (blocks go round-robin to the 8 XCDs).
        const int64_t per_xcd = (gridDim.x + 7) >> 3, idle = kThreads - 64;
        int acc = 0;
        for (int64_t off = ((int64_t)(blockIdx.x >> 3) * idle + (tid - 64)) * 128; off < T.hot_bytes; off += per_xcd * idle * 128)
            acc |= *(const volatile __attribute__((address_space(1))) int *)(T.hot_begin + off);
        if (acc == 0x7ff1234f && T.fault) atomicAdd(T.fault, 0);   // keeps the loads alive; no effect
        if (kCompact && stage_cycles) {                 // ... and copy the cycle tables into LDS for wave 0
            int32_t *cycle_lds = reinterpret_cast<int32_t *>(bits4 + ((T.n_words + 3) >> 2)) + cap;
            copy_cycle_tables(cycle_lds, T.n_states, T.cycle_pool_n, cycle_head, cycle_pool, tid - 64, kThreads - 64);
            __syncthreads();
        }
    }
    if (tid < 64) {
        WaveStack ws{row, adv_scratch + b, (size_t)batch, 0, 0, 0};
        int32_t *after_row = reinterpret_cast<int32_t *>(bits4 + n_vec);
        const Advanced r = advance_and_plan<kCompact>(T, E, in, cap, restart_on_eos, ws, cycle_head, cycle_pool,
                                                      stage_cycles, after_row, plan, lane);
        commit_advance<kCompact>(r, ws, after_row, states, row, len, err, cap, b, lane);
    }
    __syncthreads();
    // ---- the next mask row, by the whole block
    PrivateStack wp;                                    // leftovers are walked on the committed stack
    wp.lds = s_walk_stack + lane;
    wp.lds_stride = 64;
    wp.spill = walk_spill + (size_t)b * 64 + lane;
    wp.spill_stride = walk_spill_stride;
    const bool vector_ok = (T.n_words & 3) == 0 && (reinterpret_cast<uintptr_t>(bitmask) & 15) == 0;
    build_and_store_row<kThreads, true, true>(T, E, plan, bits4, 0, n_vec, row, wp, bitmask + (size_t)b * T.n_words, vector_ok, tid);
}

// The part of advance_and_plan that is left when there is no token: the top of the stack as it stands is
// fetched and the condition tree descended with it, through scalar loads (the step kernel's
// wave 0 when the kernel is asked for mask + masking only).
__device__ __forceinline__ void plan_only_scalar(const DevTables &T, const DevTokenEdges &E, const StepInputs &in,
                                                 const int32_t *row, int cap, RowPlan &plan, int lane) {
    const int n = in.n, st = in.st;
    const bool shape_ok = n >= 1 && n <= cap;
    int32_t win = -1;
    if (shape_ok) {
        if (cap >= 16) win = deal_window(row, scalar_load16(row + window_chunk(n, cap, 0)), n, cap, lane);
        else if (n - 1 - lane >= 0) win = row[n - 1 - lane];
    }
    const int top = __builtin_amdgcn_readlane(win, 0);
    if (st < 0) {
        if (lane == 0) plan.mode = kRowDone;
    } else if (!shape_ok || (unsigned)top >= (unsigned)T.n_states) {
        if (lane == 0) plan.mode = kRowEmpty;
    } else {
        plan_row_scalar(E, scalar_node(E.root_nodes + top), win, n,
                        [&](int k) { return global_read(row + (n - 1 - k)); }, &plan, lane);
    }
    if (lane == 0) { plan.top = top; plan.len = n; }
}

// All ones in the halves of a register whose mask bits (the lowest two of `bits`) are set.
__device__ __forceinline__ uint32_t allow_pair(uint32_t bits) {
    const uint32_t lo = (uint32_t)__builtin_amdgcn_sbfe((int)bits, 0, 1), hi = (uint32_t)__builtin_amdgcn_sbfe((int)bits, 1, 1);
    return __builtin_amdgcn_perm(hi, lo, 0x05040100u);
}
// A group of 8 logits with -inf where its mask byte has a zero.
__device__ __forceinline__ uint4 mask_group(uint4 v, uint32_t mu) {
    const uint4 a = make_uint4(allow_pair(mu), allow_pair(mu >> 2), allow_pair(mu >> 4), allow_pair(mu >> 6));
    return make_uint4((v.x & a.x) | (~a.x & kNegInfPair), (v.y & a.y) | (~a.y & kNegInfPair), (v.z & a.z) | (~a.z & kNegInfPair),
                      (v.w & a.w) | (~a.w & kNegInfPair));
}

// The plan is a materialised row as it stands.
__device__ __forceinline__ bool plan_is_a_row(const RowPlan &plan) {
    return plan.mode == kRowFast && plan.dense >= 0 && plan.nseg == 0 && plan.walk_count == 0;
}
// A materialised row to the mask, by one wave: sixteen bytes per lane, whatever the row's alignment.
__device__ __forceinline__ void copy_mask_row(const uint32_t *src, uint32_t *dst, int n_words, int lane) {
    typedef NativeUint4 __attribute__((aligned(4))) NativeUint4AtWord;
    constexpr int kInFlight = 8;
    const int n_vec = n_words >> 2;
    for (int v0 = lane; v0 < n_vec; v0 += 64 * kInFlight) {
        NativeUint4 x[kInFlight];
#pragma unroll
        for (int u = 0; u < kInFlight; ++u) x[u] = reinterpret_cast<const NativeUint4 *>(src)[min(v0 + u * 64, n_vec - 1)];
#pragma unroll
        for (int u = 0; u < kInFlight; ++u)
            if (v0 + u * 64 < n_vec) __builtin_nontemporal_store(x[u], reinterpret_cast<NativeUint4AtWord *>(dst) + v0 + u * 64);
    }
    if (lane < (n_words & 3)) dst[n_vec * 4 + lane] = src[n_vec * 4 + lane];
}

// The largest of all threads' keys, in every thread of a block of 1,024 (s_key: a word per wave).
__device__ __forceinline__ int step_block_best(int key, int *s_key, int tid) {
    auto row_max = [](int v) {                          // of sixteen lanes
        v = max(v, __builtin_amdgcn_mov_dpp(v, 0xB1, 0xF, 0xF, true));     // lane ^ 1
        v = max(v, __builtin_amdgcn_mov_dpp(v, 0x4E, 0xF, 0xF, true));     // lane ^ 2
        v = max(v, __builtin_amdgcn_mov_dpp(v, 0x141, 0xF, 0xF, true));    // the other four of eight
        return max(v, __builtin_amdgcn_mov_dpp(v, 0x140, 0xF, 0xF, true)); // the other eight of sixteen
    };
    key = row_max(key);
    const int wave = max(max(__builtin_amdgcn_readlane(key, 0), __builtin_amdgcn_readlane(key, 16)),
                         max(__builtin_amdgcn_readlane(key, 32), __builtin_amdgcn_readlane(key, 48)));
    if ((tid & 63) == 0) s_key[tid >> 6] = wave;
    lds_barrier();
    return row_max(s_key[tid & 15]);
}
// Keys that do not decide by themselves: positive NaN patterns, and zeros (-0 and +0 are equal values).
__device__ __forceinline__ bool order_undecided(int key) { return key > kOrderPosInf || key == 0 || key == -1; }

// The whole decode step in one launch: advance, next mask row, and that row applied to the
// sequence's logits.  One 1,024-thread block per sequence.  Wave 0 advances and descends the
// condition tree as in advance_fill_kernel, but through scalar loads only (vector loads return in order
// per compute unit: behind the row loads of this block each of them would wait microseconds).  The
// other fifteen waves meanwhile fetch the
// sequence's whole row of logits -- the fetch does not depend on the mask -- into registers (kHeld
// groups of 8 bf16 per lane, lane j of the 960 holding groups j, j + 960, ...), so the read half of
// the masking pass runs under the advance instead of after it; once the plan is there they put the
// mask row together in LDS (materialised row, id lists; wave 0 walks what the tree left open),
// store it, and patch and store the logits they hold.  The two halves are separate branches of the
// kernel with the same number of block barriers, so the registers that hold the logits are not live
// in wave 0's code.  Masked logits are exactly those of apply_mask_vec8_kernel (-inf where a bit is
// clear, 128-byte lines written whole or not at all).
// kArgmax: the greedy decode step.  The logits are not written back; instead every lane takes the arg max
// of the allowed logits among the groups it holds (the order keys of masked_argmax_kernel, the same rules:
// largest value, first of equal values, +0 = -0, NaN never), the block combines the lanes, and out_tokens[b]
// is the sequence's next token (-1 if nothing is allowed).  out_tokens may be the tokens buffer: block b
// reads tokens[b] before anything else and writes out_tokens[b] last.
// With one row to a unit and ten to seventeen groups per lane (kByLane) the waves do not meet before the mask: a block's row loads
// are served one wave after the other (the first wave has its groups at 5,800 cycles, the last at 20,100), and a wave that has
// issued all of its loads waits for nothing but the plan, a flag in LDS.  Where the plan is a materialised row, every lane then
// fetches the mask bytes of its own groups and folds, and the wave that advances copies the mask row out; other rows are put
// together in LDS.  8 greedy steps of 256 x 128,256 126.3 -> 118.1 us on JSON, 136.6 -> 130.9 with cycle-aware stacks.  Twenty groups
// leave no registers for the mask words.  Up to nine, the logits are there before the plan is, and waves that look for it one by one
// gain nothing on what meets once: 256 x 52,000 97.1 and 99.9 us, cycle-aware 111.4 and 115.8, 256 x 69,000 115.2 and 117.6.  (The
// masking step loses too: stores that begin while other waves fetch, 191 against 215 us per 8 steps.)
// kRows = 2 (greedy, batches of more rows than compute units): two blocks share a unit, so a lane has half the registers; a block
// holds the first kHeld groups per lane, fetched under the advance, and streams what follows once it knows the mask,
// reading nothing that is masked as a whole.  Neither the advance as a launch of its own nor the second round of a grid of
// whole-row blocks stands in front of the stream.  us per step in a graph, against the two launches: 257 x 128,256 JSON 21.6
// (26.8), 320 24.0 (29.2), cycle-aware stacks 25.8 (32.3), 512 27.6 (34.2); schema 300 x 152,064 23.0 (27.9), 512 27.9 (32.6);
// 400 x 80,000 cycle-aware 21.5 (26.5); 1,024 x 128,256 50.1 (57.8), 2,048 95.1 (102.7).  Blocks of 512 threads with 16 groups
// per lane: the same.  (The masking step in this form loses: a block's loads and stores wait for one another, 512 x 128,256
// 52.2 against 51.2 us, a schema at 300 x 152,064 43.2 against 35.4.)
// tokens == nullptr: no advance -- the mask of the stacks as they are, and the masking (states, data and
// len are then only read).
constexpr int kStepBlock = 1024, kStepData = kStepBlock - 64;
constexpr int kStepAhead = 8, kRestAhead = 4;          // greedy: groups of logits a lane has in flight (the rest of a longer row)
static_assert(kStepBlock == kArgBlock && kStepBlock == 16 * 64, "the step kernel combines its lanes with argmax_block_max and step_block_best");
template <bool kCompact, int kHeld, bool kArgmax, int kRows>
__global__ __launch_bounds__(kStepBlock) __attribute__((amdgpu_waves_per_eu(4 * kRows))) void advance_fill_apply_kernel(
    const int32_t *tokens, int32_t *__restrict__ len, int32_t *__restrict__ states, int32_t *__restrict__ data, const DevPack *pack,
    int cap, int first_row, uint16_t *__restrict__ logits, int64_t row_stride, int batch, int32_t *__restrict__ err,
    uint32_t *__restrict__ bitmask, int restart_on_eos, int32_t *adv_scratch, int32_t *walk_spill,
    size_t walk_spill_stride, const int32_t *cycle_head, const int32_t *cycle_pool, int stage_cycles, int32_t *out_tokens) {
    DevTables T;
    DevTokenEdges E;
    load_tables(pack, T, E);
    static_assert(kRows == 1 || (kRows == 2 && kArgmax), "the masking form fills a unit's registers with one row");
    extern __shared__ uint4 bits4[];                   // the mask row; kCompact: then cap stack entries [+ cycle tables]
    __shared__ __align__(16) int32_t s_walk_stack[kLdsDepth * 64];
    __shared__ RowPlan plan;
    const int tid = threadIdx.x, lane = tid & 63;
    const int b = first_row + blockIdx.x;          // (a large batch comes as several launches of one row per compute unit)
    const int n_vec = (T.n_words + 3) >> 2;
    int32_t *row = data + (size_t)b * cap;
    uint32_t *bits = reinterpret_cast<uint32_t *>(bits4);
    uint32_t *dst_row = bitmask + (size_t)b * T.n_words;
    const bool vector_ok = (T.n_words & 3) == 0 && (reinterpret_cast<uintptr_t>(bitmask) & 15) == 0;
    uint16_t *lrow = logits + (size_t)b * row_stride;
    int top = -32768;                                  // kArgmax: the block's best order key
    constexpr bool kByLane = kArgmax && kRows == 1 && kHeld > 9 && kHeld <= 17;
    constexpr bool kWindowFirst = kArgmax && (kRows == 2 || kHeld > 17);
    bool by_lane = false;                              // kByLane: every lane fetches the mask bytes of its groups, the row is not in LDS
    __shared__ int s_key[kArgmax ? kStepBlock / 64 : 1], s_token;
    if (kArgmax && tid == 0) s_token = 0x7FFFFFFF;     // (lowered and read behind the block's barriers)
    // kArgmax: half a mask byte -> AND masks of two registers.  Sixteen entries: lanes that read the same entry are
    // served together and different entries lie in different banks (a 256-entry table of whole bytes cost 4-way
    // bank conflicts on every read: 5.1 us for the arg max of a block instead of the 3.3 us it takes now)
    __shared__ uint2 s_expand[kArgmax ? 16 : 1];
    __shared__ unsigned long long s_part[kArgmax ? kStepBlock / 64 + 1 : 1];

    // kByLane: a wave goes on when the plan is there, whether the others have their logits or not (their loads are served one wave
    // after the other: the first has its row at a third of the fetch, the last at its end).  The wave that advances sets the flag,
    // whatever it finds, so every wait ends.
    __shared__ int s_ready;
    auto plan_ready = [&] {
        if (!kByLane) { lds_barrier(); return; }
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup", "local");
        if (lane == 0) __hip_atomic_store(&s_ready, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
    };
    auto plan_is_there = [&] {
        const bool there = __hip_atomic_load(&s_ready, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP) != 0;
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup", "local");
        return __builtin_amdgcn_readfirstlane(there) != 0;
    };
    auto plan_awaited = [&] {
        if (!kByLane) lds_barrier();
        else while (!plan_is_there()) __builtin_amdgcn_s_sleep(1);
    };
    if (kArgmax) mask_nibble_table_init(s_expand, tid);
    if (kByLane) {
        if (tid == 0) s_ready = 0;
        lds_barrier();
    }
    if (__builtin_amdgcn_readfirstlane(tid >> 6) == 0) {
        const StepInputs in = read_inputs(tokens ? tokens : len, len, states, b);
        if (tokens) {
            WaveStack ws{row, adv_scratch + b, (size_t)batch, 0, 0, 0};
            int32_t *after_row = reinterpret_cast<int32_t *>(bits4 + n_vec);
            const Advanced r = advance_and_plan<kCompact, true, kWindowFirst>(T, E, in, cap, restart_on_eos, ws, cycle_head, cycle_pool,
                                                                stage_cycles, after_row, plan, lane);
            if (kArgmax) plan_ready();
            commit_advance<kCompact>(r, ws, after_row, states, row, len, err, cap, b, lane);
            if (!kArgmax) plan_ready();
        } else {
            plan_only_scalar(T, E, in, row, cap, plan, lane);
            plan_ready();
        }
        // (barriers that order LDS only: this wave's stores of the new stack are still on their way, and
        // nothing in this block reads them before the launch ends -- except the walks below, which wait)
        by_lane = kByLane && plan_is_a_row(plan);
        if (by_lane) {
            // the mask row goes out as it lies there, while the other waves apply it
            copy_mask_row(E.dense_rows + (size_t)plan.dense * n_vec * 4, dst_row, T.n_words, lane);
            if (kArgmax) top = step_block_best(-32768, s_key, tid);
        } else {
            lds_barrier();                                 // the materialised row (or zeros) is in LDS
            // tokens the tree leaves undetermined are walked on the committed stack, one lane per token
            PrivateStack wp;
            wp.lds = s_walk_stack + lane;
            wp.lds_stride = 64;
            wp.spill = walk_spill + (size_t)b * 64 + lane;
            wp.spill_stride = walk_spill_stride;
            const int mode = plan.mode, n = plan.len, top0 = plan.top;
            if (mode == kRowWalkAll || (mode == kRowFast && plan.walk_count > 0))
                __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup");      // the walks read the committed stack
            if (mode == kRowFast) {
                const int wc = plan.walk_count;
                for (int k = lane; k < wc; k += 64) {
                    const int t = E.walk_ids[plan.walk_begin + k];
                    if (walk_token_id(T, wp, t, row, n, top0)) atomicOr(&bits[t >> 5], 1u << (t & 31));
                }
            } else if (mode == kRowWalkAll) {
                for (int t = lane; t < T.n_tokens; t += 64)
                    if (walk_token_id(T, wp, t, row, n, top0)) atomicOr(&bits[t >> 5], 1u << (t & 31));
            } else if (mode == kRowDone && lane == 0) {
                bits[T.eos_id >> 5] = 1u << (T.eos_id & 31);
            }
            lds_barrier();                                 // the row is complete
            if (kArgmax) top = step_block_best(-32768, s_key, tid);
        }
    } else {
        const int j = tid - 64;
        if (kCompact && stage_cycles) {
            int32_t *cycle_lds = reinterpret_cast<int32_t *>(bits4 + n_vec) + cap;
            copy_cycle_tables(cycle_lds, T.n_states, T.cycle_pool_n, cycle_head, cycle_pool, j, kStepData);
            __syncthreads();
        }
        // the row of logits: every group of 8 that lies wholly inside the vocabulary
        const int whole = T.n_tokens >> 3;
        uint4 held[kHeld];
        auto group_keys = [](uint4 &v) {
            v = make_uint4(bf16_order_keys(v.x), bf16_order_keys(v.y), bf16_order_keys(v.z), bf16_order_keys(v.w));
            asm volatile("" : "+v"(v.x), "+v"(v.y), "+v"(v.z), "+v"(v.w));
        };
        auto half_max = [](uint32_t x) { return max((int)(int16_t)(x & 0xFFFFu), (int)x >> 16); };
        auto fold = [](const uint4 &v) { return packed_max_s16(packed_max_s16(v.x, v.y), packed_max_s16(v.z, v.w)); };
        auto mask_keys = [&](uint4 &v, uint32_t mu) {   // v: the group's order keys
            const uint4 allow = expand_mask_byte(s_expand, mu);
            v = make_uint4(mask_order_keys(v.x, allow.x), mask_order_keys(v.y, allow.y), mask_order_keys(v.z, allow.z), mask_order_keys(v.w, allow.w));
        };
        // the mask row put together in LDS, and stored
        auto row_in_lds = [&] {
            const int mode = plan.mode;
            if (mode == kRowFast && plan.dense >= 0) {
                const uint4 *src = reinterpret_cast<const uint4 *>(E.dense_rows) + (size_t)plan.dense * n_vec;
                for (int w = j; w < n_vec; w += kStepData) bits4[w] = src[w];
            } else {
                for (int w = j; w < n_vec; w += kStepData) bits4[w] = make_uint4(0, 0, 0, 0);
            }
            lds_barrier();                             // the materialised row (or zeros) is in LDS
            if (mode == kRowFast) {
                const int nseg = plan.nseg;
                for (int i = 0; i < nseg; ++i) {
                    const int32_t *ids = E.delta_ids + plan.seg_begin[i];
                    const int cnt = plan.seg_count[i];
                    for (int k = j; k < cnt; k += kStepData) {
                        const int t = ids[k];
                        atomicOr(&bits[t >> 5], 1u << (t & 31));
                    }
                }
            }
            lds_barrier();                             // the row is complete
            if (vector_ok) {
                uint4 *dst4 = reinterpret_cast<uint4 *>(dst_row);
                for (int w = j; w < n_vec; w += kStepData) stream_store(bits4[w], dst4 + w);
            } else {
                for (int w = j; w < T.n_words; w += kStepData) dst_row[w] = bits[w];
            }
        };
        auto group_fold = [&](uint4 v, uint32_t mu) { mask_keys(v, mu); return fold(v); };
        // kArgmax, one row to a unit: the lane's best keys and those of each of its groups, in the halves of a register
        uint32_t best2 = 0x80008000u, folded[kArgmax && kRows == 1 ? kHeld : 1];
        const uint8_t *mask_bytes = reinterpret_cast<const uint8_t *>(bits4);     // byte g = bits of group g
        auto masked = [&](int i, uint32_t mu) {
            folded[i] = group_fold(held[i], mu);
            best2 = packed_max_s16(best2, folded[i]);
        };
        auto masked_from_lds = [&] {
#pragma unroll
            for (int i = 0; i < kHeld; ++i) {
                // no branches: a group outside the row or without an allowed token gets the lowest key in every half, and the
                // LDS reads of the groups can overlap (the row's LDS area is at least kHeld * kStepData bytes, so the byte
                // is read at a fixed offset)
                const int g = i * kStepData + j;
                const uint32_t mu = mask_bytes[g];
                masked(i, g < whole ? mu : 0u);
            }
        };
        const int tail = T.n_tokens & 7;               // tokens of the last, partial group
        if (kArgmax) {
            // The patterns become order keys as the groups arrive: kStepAhead groups in flight, the loads without a branch
            // (a slot beyond the row loads its last group and is not looked at), each group worked on when it is its turn
            // (the compiler would otherwise leave all of that to the fold behind the barriers).  With the fold below that keeps
            // one register per group and looks for the token only where the block's best key is: 16.4 against 18.5 us per
            // greedy step in a graph at 256 x 128,256, 13.4 against 15.6 us at 128.
            const uint32_t last_group = (uint32_t)(whole - 1) * 16u;         // (advance_fill_apply_fits: a whole group at least)
            auto load_group = [&](int i) { held[i] = stream_load_at(lrow, min((uint32_t)j * 16u + (uint32_t)(i * kStepData * 16), last_group)); };
#pragma unroll
            for (int i = 0; i < (kStepAhead < kHeld ? kStepAhead : kHeld); ++i) load_group(i);
            auto arrived = [&](int i) {                 // group i's keys, with the load that follows
                if (i + kStepAhead < kHeld) load_group(i + kStepAhead);
                __builtin_amdgcn_sched_barrier(0);
                group_keys(held[i]);
            };
            if constexpr (kByLane) {
                // Where the row is a materialised one nobody puts it together: a lane fetches the mask bytes of its groups, which
                // return behind the logits then in flight.
                constexpr int kEarly = kHeld > kStepAhead ? kHeld - kStepAhead : 0;
#pragma unroll
                for (int i = 0; i < kEarly; ++i) arrived(i);
                plan_awaited();
                by_lane = plan_is_a_row(plan);
                if (by_lane) {
                    const uint8_t *bytes = reinterpret_cast<const uint8_t *>(E.dense_rows + (size_t)__builtin_amdgcn_readfirstlane(plan.dense) * n_vec * 4);
                    uint32_t mu[kHeld];
#pragma unroll
                    for (int i = 0; i < kHeld; ++i) mu[i] = bytes[min(i * kStepData + j, whole - 1)];
                    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
                    for (int i = kEarly; i < kHeld; ++i) arrived(i);
#pragma unroll
                    for (int i = 0; i < kHeld; ++i) masked(i, i * kStepData + j < whole ? mu[i] : 0u);
                } else {
#pragma unroll
                    for (int i = kEarly; i < kHeld; ++i) arrived(i);
                    row_in_lds();
                    masked_from_lds();
                }
            } else {
#pragma unroll
                for (int i = 0; i < kHeld; ++i) arrived(i);
            }
        } else {
#pragma unroll
            for (int i = 0; i < kHeld; ++i) {
                const int g = i * kStepData + j;
                held[i] = make_uint4(0u, 0u, 0u, 0u);
                // (a wave-uniform base per i plus one 32-bit lane offset: no 64-bit address register per group)
                if (g < whole) held[i] = stream_load(lrow + (size_t)i * (kStepData * 8) + (uint32_t)(j * 8));
            }
        }
        if (!kByLane) { plan_awaited(); row_in_lds(); }
        if (kArgmax) {
            // Per group: the AND masks of the two halves of the mask byte come from the LDS table, masked halves
            // get the lowest key and three packed maxima fold the group; what is left of it (one register) stays, and
            // one more packed maximum is the lane's best.  The block's best key is found first (step_block_best);
            // only the waves that hold it then look for the group, and in the group for the token.
            auto mask_byte_of = [&](int g) -> uint32_t {
                if (by_lane) return (E.dense_rows[(size_t)plan.dense * n_vec * 4 + (g >> 2)] >> ((g & 3) * 8)) & 0xFFu;
                return mask_bytes[g];
            };
            uint4 tail_keys = make_uint4(0, 0, 0, 0);
            uint32_t tail_m = 0u;
            int tail_fold = -32768;
            if (tail > 0 && j == 0) {                   // the last, partial group: its logits one at a time
                uint32_t x[4] = {0u, 0u, 0u, 0u};
#pragma unroll
                for (int k = 0; k < 7; ++k)
                    if (k < tail) x[k >> 1] |= (uint32_t)lrow[whole * 8 + k] << (16 * (k & 1));
                tail_m = mask_byte_of(whole) & ((1u << tail) - 1u);
                tail_keys = make_uint4(bf16_order_keys(x[0]), bf16_order_keys(x[1]), bf16_order_keys(x[2]), bf16_order_keys(x[3]));
                tail_fold = half_max(group_fold(tail_keys, tail_m));
            }
            int best, at = -1, first = 0;               // the lane's best key, and (once it is the block's) where it is
            uint4 keys = make_uint4(0, 0, 0, 0);
            uint32_t m = 0u;
            if constexpr (kRows == 1) {
                if (!kByLane) masked_from_lds();
                best = max(half_max(best2), tail_fold);
                top = step_block_best(best, s_key, tid);
                const unsigned long long holders = __ballot(best == top);
                if constexpr (!kByLane) {
                    if (best == top) {
                        // the first of a lane's groups that holds the value (its groups ascend, the partial one is the last)
                        at = whole;
#pragma unroll
                        for (int i = kHeld - 1; i >= 0; --i)
                            if (half_max(folded[i]) == top) { keys = held[i]; at = i * kStepData + j; }
                    }
                } else if (holders != 0ull && top >= kOrderNegInf && !order_undecided(top)) {
                    // Where: a lane that holds the value lays the best keys of its groups in LDS (the walks' private stacks, which
                    // nobody uses any more), every lane looks at one of them; then the keys of that group, in the same way.
                    const int wave = __builtin_amdgcn_readfirstlane(j >> 6);
                    constexpr int kSpot = kLdsDepth * 64 / (kStepData / 64) & ~3;  // words per wave
                    static_assert(kHeld * 4 <= kSpot, "a lane's groups in the wave's part of the stacks");
                    uint32_t *spot = reinterpret_cast<uint32_t *>(s_walk_stack) + wave * kSpot;
                    auto has = [&](uint32_t x) {
                        return (int)(int16_t)(x & 0xFFFFu) == top || (int)x >> 16 == top;
                    };
                    int who = __ffsll((long long)holders) - 1, i = -1;                     // the lane, its group (-1: the partial one)
                    if ((holders & (holders - 1ull)) == 0ull) {
                        wave_exchange();
                        if (lane == who) {
#pragma unroll
                            for (int u = 0; u < kHeld; ++u) spot[u] = folded[u];
                        }
                        wave_exchange();
                        const uint32_t f = spot[lane < kHeld ? lane : 0];
                        const unsigned long long here = __ballot(lane < kHeld && has(f));
                        i = here != 0ull ? __ffsll((long long)here) - 1 : -1;
                    } else {
                        // Several lanes: ids ascend by group, then by lane, so the first lane of the first group that holds the value
                        // has it (no lane beside the first one of the row has the partial group).  8 steps of 256 x 128,256 equal logits
                        // 131 us, 1,218 with one lane after the other (152 with a select over all groups in every lane).
#pragma unroll
                        for (int u = kHeld - 1; u >= 0; --u) {
                            const unsigned long long in = __ballot(has(folded[u]));
                            if (in != 0ull) { i = u; who = __ffsll((long long)in) - 1; }
                        }
                    }
                    at = i >= 0 ? i * kStepData + wave * 64 + who : whole;
                    wave_exchange();
                    if (lane == who) {
                        if (i < 0) {
                            __builtin_memcpy(__builtin_assume_aligned(spot, 16), &tail_keys, 16);
                        } else {
#pragma unroll
                            for (int u = 0; u < kHeld; ++u) __builtin_memcpy(__builtin_assume_aligned(spot + u * 4, 16), &held[u], 16);
                        }
                    }
                    wave_exchange();
                    const uint32_t pair = spot[(i > 0 ? i * 4 : 0) + ((lane & 7) >> 1)];
                    const int key = (int16_t)(pair >> (16 * (lane & 1)));
                    uint32_t hold = (uint32_t)__ballot(lane < 8 && key == top);            // tokens with that key, masked ones among them
                    if ((hold & (hold - 1u)) != 0u) hold &= i < 0 ? (uint32_t)__builtin_amdgcn_readfirstlane(tail_m) : mask_byte_of(at);
                    const int token = at * 8 + __builtin_ctz(hold | 0x80u);
                    if (lane == 0) atomicMin(&s_token, token);
                }
            } else {
                // What the block does not hold is streamed now that the mask is known: nothing of a group without an
                // allowed token is read, and the loads are issued without a branch, kStepAhead ahead, the first of them
                // before the groups that are held are worked on.
                const RowBuffer buffer = row_buffer(lrow, (uint32_t)whole * 16u);
                auto mask_of = [&](int g) { const uint32_t mu = mask_bytes[min(g, whole - 1)]; return g < whole ? mu : 0u; };
                auto load_rest = [&](int g) { return buffer_load(buffer, mask_of(g) != 0u ? (uint32_t)g * 16u : kNowhere); };
                best = kOrderNegInf - 1;                // (only a valid value or a positive NaN pattern beats the start)
                auto work_on = [&](uint4 v, int g) {    // no branch: the LDS reads of several groups overlap
                    const uint32_t mu = mask_of(g);
                    const int group_best = half_max(group_fold(v, mu));
                    const bool better = group_best > best;                       // strictly: the first of equals stays
                    best = better ? group_best : best;
                    at = better ? g : at;
                    keys.x = better ? v.x : keys.x; keys.y = better ? v.y : keys.y; keys.z = better ? v.z : keys.z; keys.w = better ? v.w : keys.w;
                };
                constexpr int kBatch = kRestAhead / 2;  // groups a lane works on together, while as many are in flight
                uint4 v[kRestAhead];
                int g = kHeld * kStepData + j;
#pragma unroll
                for (int u = 0; u < kRestAhead; ++u) v[u] = load_rest(g + u * kStepData);
                __builtin_amdgcn_sched_barrier(0);
#pragma unroll
                for (int i = 0; i < kHeld; ++i) work_on(held[i], i * kStepData + j);
                for (int r = kHeld * kStepData; r < whole; r += kRestAhead * kStepData) {
#pragma unroll
                    for (int u0 = 0; u0 < kRestAhead; u0 += kBatch) {
                        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
                        for (int u = u0; u < u0 + kBatch; ++u)
                            work_on(make_uint4(bf16_order_keys(v[u].x), bf16_order_keys(v[u].y), bf16_order_keys(v[u].z), bf16_order_keys(v[u].w)),
                                    g + u * kStepData);
#pragma unroll
                        for (int u = u0; u < u0 + kBatch; ++u) v[u] = load_rest(g + (u + kRestAhead) * kStepData);
                    }
                    g += kRestAhead * kStepData;
                }
                if (tail_fold > best) { best = tail_fold; at = whole; }
                top = step_block_best(best, s_key, tid);
            }
            if (!kByLane && best == top && top >= kOrderNegInf && !order_undecided(top)) {
                if (at == whole) { keys = tail_keys; m = tail_m; }
                else m = mask_bytes[at];
                const uint32_t x[4] = {keys.x, keys.y, keys.z, keys.w};
#pragma unroll
                for (int k = 7; k >= 0; --k) {          // descending: the smallest k is assigned last
                    const int key = (k & 1) ? ((int)x[k >> 1] >> 16) : (int)(int16_t)(x[k >> 1] & 0xFFFFu);
                    if (((m >> k) & 1u) && key == top) first = k;
                }
                atomicMin(&s_token, at * 8 + first);
            }
        } else {
#pragma unroll
        for (int i = 0; i < kHeld; ++i) {
            const int g = i * kStepData + j;
            // a group that needs no change is still written if one of the eight groups of its 128-byte line
            // does: lines written in part cost the memory system far more than the bytes saved
            const uint32_t mu = g < whole ? mask_bytes[g] : 0xFFu;
            const unsigned long long changed = __ballot(mu != 0xFFu);
            if (g < whole) {
                if ((changed >> (lane & 56)) & 0xFFull) {
                    uint4 v = held[i];
                    uint32_t *x = reinterpret_cast<uint32_t *>(&v);
#pragma unroll
                    for (int k = 0; k < 4; ++k) {
                        const uint32_t lo = (uint32_t)__builtin_amdgcn_sbfe((int)mu, 2 * k, 1);
                        const uint32_t hi = (uint32_t)__builtin_amdgcn_sbfe((int)mu, 2 * k + 1, 1);
                        const uint32_t allow = __builtin_amdgcn_perm(hi, lo, 0x05040100u);
                        x[k] = (x[k] & allow) | (~allow & kNegInfPair);
                    }
                    stream_store(v, lrow + (size_t)i * (kStepData * 8) + (uint32_t)(j * 8));
                }
            }
        }
        // the last, partial group of a vocabulary that is not a multiple of 8
        if (j < tail) {
            const int t = whole * 8 + j;
            if (!((bits[t >> 5] >> (t & 31)) & 1u)) lrow[t] = 0xFF80;
        }
        }
    }
    if (kArgmax) {
        // `top` is the block's best key in every thread, s_token the smallest id that holds it -- unless the keys cannot
        // decide: a positive NaN pattern or a zero on top are compared as numbers
        lds_barrier();
        if (top < kOrderNegInf) {
            if (tid == 0) out_tokens[b] = -1;
        } else if (!order_undecided(top)) {
            if (tid == 0) out_tokens[b] = s_token;
        } else {
            if (by_lane) {                             // (the row a second time, in order: its mask from LDS: 8 steps of 256 x 128,256 zeros 625 us, 687 from memory)
                const uint4 *src = reinterpret_cast<const uint4 *>(E.dense_rows) + (size_t)plan.dense * n_vec;
                for (int w = tid; w < n_vec; w += kStepBlock) bits4[w] = src[w];
                lds_barrier();
            }
            const unsigned long long mine = argmax_block_max(
                argmax_by_compare<kArgBlock>(lrow, [&](int g) { return (uint32_t)reinterpret_cast<const uint8_t *>(bits4)[g]; }, 0,
                                          (T.n_tokens + 7) >> 3, T.n_tokens, tid), s_part, tid);
            if (tid == 0) out_tokens[b] = mine != 0ull ? (int32_t)(0xFFFFFFFFu - (uint32_t)mine) : -1;
        }
    }
}

// The stack an advance leaves, as the wave that made it sees it before it is stored, for walks that look at other entries
// in every lane: `staged` (LDS) holds it as a whole (kCompact) or the first 64 of the states pushed above row[0 .. base).
template <bool kCompact>
struct NewStack {
    const int32_t *row, *staged, *spill;
    size_t spill_stride;
    int base;
    __device__ int32_t at(int idx) const {
        if (kCompact) return lds_read(staged + idx);
        if (idx < base) return global_read(row + idx);
        const int i = idx - base;
        int32_t v = lds_read(staged + (i < kWindow ? i : kWindow - 1));
        if (i >= kWindow) v = global_read(spill + (size_t)(i - kWindow) * spill_stride);
        return v;
    }
};

// The whole decode step of a small batch in one launch: every row of logits is spread over n_seg blocks, so that a few
// sequences fill the chip.  Each block of a row advances the sequence for itself (wave 0, as in advance_fill_kernel, on
// private stacks of its own) while its other four waves load the block's kSpreadGroups groups of 8 logits; the plan
// of the new row is the same in all of them, so each masks its groups and stores its part of the mask row by itself.
// Only one may store the advance, and none before all have read what it overwrites: the blocks of a row count
// themselves in when their plan is done, and the last to arrive stores (and sets the count back to zero for the next
// launch).  No block waits for another.  Where the condition tree leaves tokens of a row open, the advancing wave of each
// block walks those of the block's own groups, on the new stack as it has it (the stored one may not be there yet; what
// of it lies in memory, the entries below the advance's, is not what the last block stores): 16 x 128,256 of which some
// rows are walked whole 0.83 ms per step, 11.7 as two launches with a wave per row, 11.9 when the last block did such a
// row by itself; 4 x 32,000 with short lists 34 us (37, 39).
// kArgmax: the greedy step; the blocks' best words meet in best[row] through an atomic maximum, and the last block to
// count itself in on a second counter takes the result.  A block whose best the keys cannot decide (zeros of both signs, a
// NaN pattern) compares its own groups as numbers first: 1 x 128,256 with zeros on top 15.6 us per step, 71 when
// the last block did that for the whole row.
// A launch is bound by the chain of dependent loads of the advance (about 5 us) where the two-launch form pays for a
// second launch and for reading the mask row back.  us per step inside a graph, against the two calls: 1 x 128,256
// 6.8 (8.9), 16 x 128,256 8.2 (10.5), 60 x 128,256 11.2 (14.6), 4 x 513 7.3 (10.3), 64 x 32,000 8.6 (10.6); greedy
// 1 x 128,256 9.1 (13.6), 16 x 128,256 10.6 (14.3).  Four groups per lane and 256 lanes: when 1 and 16 x 128,256 took 7.6 and
// 9.1 us, eight groups took 8.2 and 10.0, 512 lanes 7.8 and 9.6, and the advance through scalar loads (as in the kernel above,
// where vector loads wait behind a whole row's) 8.8 and 10.5.
constexpr int kSpreadLanes = 256, kSpreadBlock = kSpreadLanes + 64, kSpreadHeld = 4;
constexpr int kSpreadGroups = kSpreadLanes * kSpreadHeld;
template <bool kCompact, bool kArgmax>
__global__ __launch_bounds__(kSpreadBlock) void step_spread_kernel(
    const int32_t *tokens, int32_t *len, int32_t *states, int32_t *data, int cap, int n_seg, uint16_t *__restrict__ logits,
    int64_t row_stride, size_t columns, DevTables T, DevTokenEdges E, int32_t *__restrict__ err, uint32_t *__restrict__ bitmask,
    int restart_on_eos, int32_t *adv_spill, int32_t *walk_spill, const int32_t *cycle_head, const int32_t *cycle_pool, int stage_cycles,
    int32_t *out_tokens, StepArrivals *arrivals) {
    const int b = blockIdx.y, seg = blockIdx.x, column = b * n_seg + seg;      // (columns: one spill column per block)
    extern __shared__ int32_t after_row[];             // kCompact: cap stack entries [+ cycle tables]
    __shared__ int32_t s_pushed[kWindow], s_walk_stack[kLdsDepth * 64];   // of an open row
    __shared__ uint32_t s_bits[kSpreadGroups / 4];     // an open row: this block's mask words
    __shared__ RowPlan plan;
    __shared__ unsigned long long s_part[kArgmax ? kSpreadBlock / 64 + 1 : 1];
    const int tid = threadIdx.x, lane = tid & 63, j = tid - 64;
    const int n_vec = (T.n_words + 3) >> 2, g0 = seg * kSpreadGroups;
    const int whole = T.n_tokens >> 3, tail = T.n_tokens & 7, groups = (T.n_tokens + 7) >> 3;
    int32_t *row = data + (size_t)b * cap;
    uint32_t *dst_row = bitmask + (size_t)b * T.n_words;
    uint16_t *lrow = logits + (size_t)b * row_stride;
    StepArrivals *mine = arrivals + b;
    WaveStack ws{row, adv_spill + column, columns, 0, 0, 0};
    Advanced r{};
    uint4 held[kSpreadHeld];
    if (__builtin_amdgcn_readfirstlane(tid >> 6) == 0) {
        const StepInputs in = read_inputs(tokens, len, states, b);
        r = advance_and_plan<kCompact>(T, E, in, cap, restart_on_eos, ws, cycle_head, cycle_pool, stage_cycles, after_row, plan, lane);
    } else {
#pragma unroll
        for (int i = 0; i < kSpreadHeld; ++i) {
            const int g = g0 + i * kSpreadLanes + j;
            held[i] = make_uint4(0u, 0u, 0u, 0u);
            if (g < whole) held[i] = stream_load(lrow + (size_t)g * 8);
        }
        if (kCompact && stage_cycles) {
            int32_t *cycle_lds = after_row + cap;
            copy_cycle_tables(cycle_lds, T.n_states, T.cycle_pool_n, cycle_head, cycle_pool, j, kSpreadLanes);
            __syncthreads();
        }
    }
    lds_barrier();                                     // the plan is there
    const int mode = plan.mode;
    // (the form is only chosen for tables without id lists: a row is a materialised row and tokens left to the walk)
    const bool open = mode == kRowWalkAll || (mode == kRowFast && plan.walk_count > 0);        // the same in every block of the row
    if (tid < 64) {
        uint32_t before = 0;
        loads_returned();                              // of the stack: the block that counts last overwrites it
        if (lane == 0) before = atomicAdd(&mine->planned, 1u);
        const bool last = (uint32_t)__builtin_amdgcn_readfirstlane((int)before) == (uint32_t)(n_seg - 1);
        if (last) {
            commit_advance<kCompact>(r, ws, after_row, states, row, len, err, cap, b, lane);
            if (lane == 0) atomicExch(&mine->planned, 0u);
        }
    }
    // the mask byte of a group: from the materialised row, else nothing (a finished sequence: the EOS bit) is allowed
    const uint32_t *dense = mode == kRowFast && plan.dense >= 0 ? E.dense_rows + (size_t)plan.dense * n_vec * 4 : nullptr;
    const int eos_group = mode == kRowDone ? T.eos_id >> 3 : -1;
    const int w0 = seg * (kSpreadGroups / 4);          // the block's first mask word
    if (open) {
        static_assert(kSpreadGroups / 4 == kSpreadLanes, "a mask word per lane");
        if (tid >= 64) s_bits[j] = dense && w0 + j < T.n_words ? dense[w0 + j] : 0u;
        else if (!kCompact) s_pushed[lane] = ws.pushed;
        lds_barrier();
        if (tid < 64) {
            const NewStack<kCompact> stack{row, kCompact ? after_row : s_pushed, ws.spill, ws.spill_stride, r.base};
            PrivateStack wp;
            wp.lds = s_walk_stack + lane;
            wp.lds_stride = 64;
            wp.spill = walk_spill + (size_t)column * 64 + lane;
            wp.spill_stride = columns * 64;
            const int n = plan.len, top0 = plan.top;
            const int t_lo = mode == kRowWalkAll ? w0 * 32 : 0;
            const int count = mode == kRowWalkAll ? min(T.n_tokens - t_lo, kSpreadGroups * 8) : plan.walk_count;
            for (int k = lane; k < count; k += 64) {
                const int t = mode == kRowWalkAll ? t_lo + k : E.walk_ids[plan.walk_begin + k], w = (t >> 5) - w0;
                if ((unsigned)w < (unsigned)(kSpreadGroups / 4) && walk_token_id_on(T, wp, t, stack, n, top0))
                    atomicOr(&s_bits[w], 1u << (t & 31));
            }
        }
        lds_barrier();
    }
    auto mask_byte = [&](int g) {
        uint32_t mu = g == eos_group ? 1u << (T.eos_id & 7) : 0u;
        if (dense) mu = reinterpret_cast<const uint8_t *>(dense)[g];
        if (open) mu = reinterpret_cast<const uint8_t *>(s_bits)[g - g0];
        return mu;
    };
    unsigned long long word = 0ull;                    // kArgmax: this lane's candidate
    if (tid >= 64) {
        uint32_t m[kSpreadHeld];
#pragma unroll
        for (int i = 0; i < kSpreadHeld; ++i) {
            const int g = g0 + i * kSpreadLanes + j;
            m[i] = g < groups ? mask_byte(g) : 0u;
        }
        const int w = w0 + j;                          // this block's part of the mask row: a word per lane
        if (w < T.n_words) dst_row[w] = open ? s_bits[j] : dense ? dense[w] : (w == (eos_group >> 2) && eos_group >= 0) ? 1u << (T.eos_id & 31) : 0u;
        uint32_t tail_x[4] = {0u, 0u, 0u, 0u};         // the last, partial group: in the lane whose group it is
        if (kArgmax) {
            int best = kOrderNegInf - 1, best_g = -1;
            uint4 best_x = make_uint4(0, 0, 0, 0);
            uint32_t best_m = 0u;
#pragma unroll
            for (int i = 0; i < kSpreadHeld; ++i) {
                const int g = g0 + i * kSpreadLanes + j;
                if (g >= groups) continue;
                uint32_t mu = m[i];
                if (g == whole) {
                    for (int k = 0; k < tail; ++k) tail_x[k >> 1] |= (uint32_t)lrow[whole * 8 + k] << (16 * (k & 1));
                    held[i] = make_uint4(tail_x[0], tail_x[1], tail_x[2], tail_x[3]);
                    mu &= (1u << tail) - 1u;
                }
                if (mu == 0u) continue;
                const uint4 allow = make_uint4(allow_pair(mu), allow_pair(mu >> 2), allow_pair(mu >> 4), allow_pair(mu >> 6));
                const uint32_t k01 = packed_max_s16(bf16_order_pair(held[i].x, allow.x), bf16_order_pair(held[i].y, allow.y));
                const uint32_t k23 = packed_max_s16(bf16_order_pair(held[i].z, allow.z), bf16_order_pair(held[i].w, allow.w));
                const uint32_t k = packed_max_s16(k01, k23);
                const int group_best = max((int)(int16_t)(k & 0xFFFFu), (int)k >> 16);
                if (group_best > best) { best = group_best; best_g = g; best_x = held[i]; best_m = mu; }
            }
            if (best_g >= 0) {
                const uint32_t x[4] = {best_x.x, best_x.y, best_x.z, best_x.w};
                int first = 0;
#pragma unroll
                for (int k = 7; k >= 0; --k) {          // descending: the smallest k is assigned last
                    const uint32_t h = (k & 1) ? (x[k >> 1] >> 16) : (x[k >> 1] & 0xFFFFu);
                    if (((best_m >> k) & 1u) && bf16_order(h) == best) first = k;
                }
                word = argmax_word(best, best_g * 8 + first);
            }
        } else {
#pragma unroll
            for (int i = 0; i < kSpreadHeld; ++i) {
                const int g = g0 + i * kSpreadLanes + j;
                const uint32_t mu = g < whole ? m[i] : 0xFFu;
                // (groups of a 128-byte line are written together or not at all, as in the other masking kernels)
                const unsigned long long changed = __ballot(mu != 0xFFu);
                if (g < whole && ((changed >> (lane & 56)) & 0xFFull)) stream_store(mask_group(held[i], mu), lrow + (size_t)g * 8);
                if (g == whole) {
                    for (int k = 0; k < tail; ++k)
                        if (!((m[i] >> k) & 1u)) lrow[whole * 8 + k] = 0xFF80;
                }
            }
        }
    }
    if (kArgmax) {
        word = argmax_block_max<kSpreadBlock>(word, s_part, tid);
        const int top = (int)(uint32_t)(word >> 32) - 32768;
        if (word != 0ull && (top > kOrderPosInf || top == 0))        // a NaN pattern or a zero on top: this block's groups compared as numbers
            word = argmax_block_max<kSpreadBlock>(
                argmax_by_compare<kSpreadBlock>(lrow, mask_byte, g0, min(g0 + kSpreadGroups, groups), T.n_tokens, tid), s_part, tid);
        if (tid == 0) {
            bool last = true;
            if (n_seg > 1) {
                // the count comes after the maximum has been taken (its result is waited for), so the last block finds all of them
                unsigned long long old = atomicMax(&mine->best, word);
                asm volatile("" : "+v"(old) : : "memory");
                last = atomicAdd(&mine->sampled, 1u + (uint32_t)(old & 0ull)) == (uint32_t)(n_seg - 1);
                if (last) {
                    word = atomicExch(&mine->best, 0ull);
                    atomicExch(&mine->sampled, 0u);
                }
            }
            if (last) out_tokens[b] = word != 0ull ? (int32_t)(0xFFFFFFFFu - (uint32_t)word) : -1;
        }
    }
}

// What input symbol `c` of each lane (one byte class each, or the end of input; c >= T.ncol: none) does to the stack
// row[0 .. n): kFed, kRejected or kAccepted, as feed() with nothing pushed yet would say.  The condition tree names the
// entries it tests whatever the symbol, so all lanes go down it together: one round per level in which lane j fetches
// condition j with child j's record and a ballot picks the child, while every lane looks at its own symbol's
// cell.  (Left to feed(), each lane scans the children by itself, one dependent load after the other: 12.7 us per
// jump_forward launch on 128 sequences of eight schemas, 5.6 us this way.)  Symbols whose merged edge was not
// precomputed are walked by feed().
__device__ __forceinline__ int try_symbols(const DevTables &T, PrivateStack &trial, int c, int n, int top, int kind, const WaveStack &ws,
                                           const StackView &view) {
    const int lane = threadIdx.x & 63;
    bool open = c < T.ncol, walk = false;
    int res = kRejected;
    if (T.sym_cell) {
        int node = kind;
        int4 nd = table<true>(T.sym_nodes, node);
        for (int level = 0; level < 64; ++level) {
            if (open) {
                const int code = T.sym_cell[node * T.ncol + c].x;
                if (code >= 0) {
                    // an edge: refused only where feed() refuses it, on a corrupted stack or beyond the depth bound
                    int known = code & 0xFF, np = (code >> 16) & 3;
                    if (!(code & kCellInline)) {
                        const int4 hdr = *reinterpret_cast<const int4 *>(T.sym_pool + code);
                        known = hdr.x;
                        np = hdr.z & kEffPushMask;
                    }
                    if (n - (known - 1) >= 1) {
                        if (np > T.max_depth) atomicAdd(T.fault, 1);
                        else res = kFed;
                    }
                    open = false;
                } else if (code == kEffNone || code == kEffAccept) {
                    if (code == kEffAccept) res = kAccepted;
                    open = false;
                } else if (code == kEffStepwise) {
                    walk = true;
                    open = false;
                }
            }
            if (!__any(open)) break;
            const int idx = n - 1 - nd.x;
            int next = -1;
            if (idx >= 0) {
                const int x = ws.at(idx);
                int4 cnd = make_int4(0, 0, 0, 0);
                for (int c0 = 0; c0 < nd.z && next < 0; c0 += 64) {
                    const int j = c0 + lane;
                    int cstate = -2;
                    if (j < nd.z) {
                        cstate = T.sym_pairs[nd.y + j].x;
                        cnd = T.sym_nodes[nd.w + j];
                    }
                    const unsigned long long m = __ballot(j < nd.z && cstate == x);
                    if (m) {
                        const int src = __ffsll((long long)m) - 1;
                        next = nd.w + c0 + src;
                        nd = make_int4(__builtin_amdgcn_readlane(cnd.x, src), __builtin_amdgcn_readlane(cnd.y, src),
                                       __builtin_amdgcn_readlane(cnd.z, src), __builtin_amdgcn_readlane(cnd.w, src));
                    }
                }
            }
            if (next < 0) break;
            node = next;
        }
    }
    walk |= open;
    if (__any(walk) && walk) {
        int base = n, d = 0, tp = top, tr = kind;
        res = feed<false, false>(T, trial, c, base, d, tp, tr, view, 0);
    }
    return res;
}

// Jump-forward: while a sequence's text is not a sentence and exactly one byte keeps it a viable
// prefix, that byte is forced; it is emitted and the stack is advanced by it.  One wave per
// sequence.  At every position lane c tries byte class c (and one lane the end-of-input symbol)
// from the current stack on a private overlay of its own -- the walk of a one-byte token --, the
// wave adds up the BYTES of the viable classes, and if that is one (and '$' is not accepted) the
// forced byte is walked on the real stack by all lanes together, exactly like in advance_kernel.
// kCompact (cycle-aware stacks): at the end the wave stages its stack in LDS (cap entries per
// sequence), takes complete traversals of reduction cycles out of it and writes back what changed.
constexpr int kJfSeqPerBlock = 4;
template <bool kCompact>
__global__ __launch_bounds__(64 * kJfSeqPerBlock) void jump_forward_kernel(
    int32_t *__restrict__ len, int32_t *__restrict__ states, int32_t *__restrict__ data, int cap, int batch, const DevPack *pack,
    uint8_t *__restrict__ out_bytes, int32_t *__restrict__ out_len, int max_bytes, int32_t *adv_scratch,
    int32_t *lane_spill, size_t lane_spill_stride, const int32_t *cycle_head, const int32_t *cycle_pool,
    int stage_cycles) {
    DevTables T;
    DevTokenEdges E;
    load_tables(pack, T, E);
    extern __shared__ int32_t jf_stage[];              // kCompact: kJfSeqPerBlock x (cap stack entries [+ cycle tables])
    __shared__ int32_t s_trial[kJfSeqPerBlock][kLdsDepth * 64];
    __shared__ int32_t s_win[kJfSeqPerBlock][kWindow];
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63;
    const int b = blockIdx.x * kJfSeqPerBlock + wave;
    if (kCompact && stage_cycles) {                     // small cycle tables: copied into LDS by the whole block
        int32_t *cycle_lds = jf_stage + kJfSeqPerBlock * cap;
        copy_cycle_tables(cycle_lds, T.n_states, T.cycle_pool_n, cycle_head, cycle_pool, threadIdx.x, 64 * kJfSeqPerBlock);
        cycle_head = cycle_lds;
        cycle_pool = cycle_lds + T.n_states;
        __syncthreads();
    }
    if (b >= batch) return;
    int32_t *row = data + (size_t)b * cap;
    int n = table<true>(len, b);
    const int st = table<true>(states, b);
    int count = 0;
    if (st >= 0 && n >= 1 && n <= cap && max_bytes > 0) {
        // the stack's top and what a forced byte's walk pushes, in the wave's registers; the lanes' own walks of byte classes
        // whose merged edge was not precomputed read the window in LDS
        WaveStack ws{row, adv_scratch + b, (size_t)batch, n, n - 1 - lane >= 0 ? row[n - 1 - lane] : -1, 0};
        s_win[wave][lane] = ws.win;
        int top = __builtin_amdgcn_readlane(ws.win, 0);
        if ((unsigned)top < (unsigned)T.n_states) {
            int kind = T.state_kind ? table<true>(T.state_kind, top) : 0;
            PrivateStack trial;                        // one column per lane
            trial.lds = s_trial[wave] + lane;
            trial.lds_stride = 64;
            trial.spill = lane_spill + (size_t)b * 64 + lane;
            trial.spill_stride = lane_spill_stride;
            int new_top = top;
            while (count < max_bytes) {
                // a state whose only edge shifts one byte starts a run of forced bytes known since the
                // tables were compiled: emitted and pushed in one step (the byte-by-byte search below
                // would find the same bytes one at a time)
                const int run = T.run_off ? table<true>(T.run_off, top) : -1;
                if (run >= 0) {
                    int take = table<true>(T.run_pool, run);
                    take = take < max_bytes - count ? take : max_bytes - count;
                    take = take < cap - n ? take : cap - n;
                    if (take <= 0) break;                  // the stack is full
                    const int word = lane < take ? T.run_pool[run + 1 + lane] : 0;
                    if (lane < take) {
                        row[n + lane] = word >> 8;
                        out_bytes[(size_t)b * max_bytes + count + lane] = (uint8_t)(word & 0xFF);
                    }
                    // the new top of the stack: the run's states, then what was the top before
                    const int from_run = __shfl(word, take - 1 - lane < 0 ? 0 : take - 1 - lane) >> 8;
                    const int below = __shfl(ws.win, lane >= take ? lane - take : 0);
                    ws.win = lane < take ? from_run : below;
                    s_win[wave][lane] = ws.win;
                    n += take;
                    ws.n = n;
                    top = __builtin_amdgcn_readlane(ws.win, 0);
                    kind = T.state_kind ? table<true>(T.state_kind, top) : 0;
                    count += take;
                    continue;
                }
                const StackView view{row, s_win[wave], n};
                int viable_bytes = 0, only = -1;
                bool at_end = false;
                for (int c0 = 0; c0 < T.ncol; c0 += 64) {
                    const int c = c0 + lane;
                    const int res = try_symbols(T, trial, c, n, top, kind, ws, view);
                    if (__ballot(c == T.end_col && res == kAccepted)) at_end = true;
                    int bytes_here = (c < T.end_col && res == kFed) ? (T.class_info[c] & 0xFFFF) : 0;
                    const unsigned long long m = __ballot(bytes_here > 0);
                    if (m) only = c0 + __ffsll((long long)m) - 1;
#pragma unroll
                    for (int off = 32; off >= 1; off >>= 1) bytes_here += __shfl_xor(bytes_here, off);
                    viable_bytes += bytes_here;
                }
                if (at_end || viable_bytes != 1) break;
                const int byte = __builtin_amdgcn_readfirstlane(T.class_info[only] >> 16);
                const int info = __builtin_amdgcn_readfirstlane(T.byte_info[byte]);
                int base = n, d = 0;
                new_top = top;
                int new_kind = kind;
                if (feed<true, true>(T, ws, info, base, d, new_top, new_kind, ws, cap) != kFed) break;   // would exceed cap
                // commit: stage the new top of the stack, then write the pushed entries
                const int32_t win = new_window(ws, base, d, lane);
                commit_pushed(row, ws, base, d, lane);
                if (lane == 0) out_bytes[(size_t)b * max_bytes + count] = (uint8_t)byte;
                ws.win = win;
                s_win[wave][lane] = win;
                n = base + d;
                ws.n = n;
                top = new_top;
                kind = new_kind;
                ++count;
            }
            if (lane == 0 && count > 0) {
                len[b] = n;
                states[b] = top;
            }
        }
    }
    if (lane == 0) out_len[b] = count;
    if (kCompact && n >= 2 && n <= cap) {
        // n is the current length (the entries committed above are this wave's own stores)
        __threadfence_block();
        int32_t *stack = jf_stage + wave * cap;
        for (int i = lane; i < n; i += 64) stack[i] = row[i];
        wave_exchange();
        int first_moved = n;
        const int w = fold_cycles(stack, n, cycle_head, cycle_pool, T.n_states, lane, &first_moved);
        if (w != n) {
            for (int i = first_moved + lane; i < w; i += 64) row[i] = stack[i];
            if (lane == 0) len[b] = w;
        }
    }
}


// Stack compaction as a kernel of its own (after advance_kernel and jump_forward_kernel): one wave
// per sequence, the stack staged in LDS (cap entries per wave) next to a copy of the cycle records
// (pool_n entries; 0 = read them from global memory).  A stack without any cycle head costs one
// pass over its entries and writes nothing.
__global__ __launch_bounds__(256) void compact_stacks_kernel(const int32_t *__restrict__ cycle_head,
                                                             const int32_t *__restrict__ cycle_pool, int pool_n,
                                                             int n_states, int32_t *__restrict__ data,
                                                             int32_t *__restrict__ len, int cap, int batch) {
    extern __shared__ int32_t compact_lds[];
    for (int i = threadIdx.x; i < pool_n; i += blockDim.x) compact_lds[i] = cycle_pool[i];
    __syncthreads();
    const int32_t *pool = pool_n > 0 ? compact_lds : cycle_pool;
    const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
    const int b = blockIdx.x * (blockDim.x >> 6) + wave;
    if (b >= batch) return;
    const int n = len[b];
    if (n < 2 || n > cap) return;
    int32_t *s = compact_lds + pool_n + wave * cap;
    int32_t *row = data + (size_t)b * cap;
    bool any = false;
    for (int i = lane; i < n; i += 64) {
        const int x = row[i];
        s[i] = x;
        any |= (unsigned)x < (unsigned)n_states && cycle_head[x] >= 0;
    }
    if (!__any(any)) return;
    wave_exchange();
    int first_moved;
    const int w = fold_cycles(s, n, cycle_head, pool, n_states, lane, &first_moved);
    if (w != n) {
        for (int i = first_moved + lane; i < w; i += 64) row[i] = s[i];
        if (lane == 0) len[b] = w;
    }
}

}  // namespace

hipError_t static_advance_scratch(int32_t **out) {
    constexpr int kMaxDevices = 64;
    static std::mutex lock;
    static int32_t *address[kMaxDevices] = {};
    int device = -1;
    hipError_t e = hipGetDevice(&device);
    if (e != hipSuccess) return e;
    if (device < 0 || device >= kMaxDevices) return hipErrorInvalidDevice;
    std::lock_guard<std::mutex> guard(lock);
    if (!address[device]) {
        void *p = nullptr;
        e = hipGetSymbolAddress(&p, HIP_SYMBOL(pre3_static_scratch));
        if (e != hipSuccess) return e;
        if (!p) return hipErrorInvalidSymbol;
        address[device] = static_cast<int32_t *>(p);
    }
    *out = address[device];
    return hipSuccess;
}

// (The header states this size, and pre3_advance_static refuses batches by it.  Since the stack of an advance lies in the
// wave's registers its pushed states spill from the 65th on, so the last 48 of the columns' entries stay untouched.)
size_t advance_scratch_entries(int batch, int max_depth) {
    const int deep = max_depth > kLdsDepth ? max_depth - kLdsDepth : 0;
    return (size_t)batch * (size_t)deep;
}

size_t advance_fill_walk_spill_entries(int batch, int max_depth) {
    const int deep = max_depth > kLdsDepth ? max_depth - kLdsDepth : 0;
    return (size_t)batch * 64 * (size_t)deep;
}

hipError_t launch_advance_fill(const DevTables &T, const int32_t *tokens, int32_t *states,
                               int32_t *data, int32_t *len, int cap, int batch, int32_t *err, uint32_t *bitmask,
                               int restart_on_eos, int32_t *adv_scratch, int32_t *walk_spill,
                               const int32_t *cycle_head, const int32_t *cycle_pool, int n_compute_units, hipStream_t stream) {
    if (batch == 0) return hipSuccess;
    size_t lds = (size_t)edge_row_stride_words(T.n_words) * sizeof(uint32_t);
    int stage = 0;
    if (cycle_head) {                                  // cycle-aware stacks: the new stack is staged in LDS too
        lds += (size_t)cap * sizeof(int32_t);
        if (cap > kCompactMaxLen || lds > kAfDynamicLdsMax) return hipErrorInvalidValue;
        const size_t tables = (size_t)(T.n_states + T.cycle_pool_n) * sizeof(int32_t);
        stage = cycles_fit_lds(T.n_states, T.cycle_pool_n) && lds + tables <= kAfDynamicLdsMax;
        if (stage) lds += tables;
    } else if (lds > kAfDynamicLdsMax) {
        return hipErrorInvalidValue;
    }
#define PRE3_AF(C, THREADS)                                                                                                 \
    hipLaunchKernelGGL((advance_fill_kernel<C, THREADS>), dim3(batch), dim3(THREADS), lds, stream, tokens, len, states, data,   \
                       cap, batch, T.pack, err, bitmask, restart_on_eos, adv_scratch, walk_spill, (size_t)batch * 64, cycle_head,  \
                       cycle_pool, stage)
#define PRE3_AF_SIZES(C)                                                                    \
    if (batch <= 2 * n_compute_units) PRE3_AF(C, kAfBlock);                                  \
    else if (batch > 4 * n_compute_units && T.n_words <= kAfShortWords) PRE3_AF(C, kAfBlockShort); \
    else PRE3_AF(C, kAfBlockMany)
    if (cycle_head) { PRE3_AF_SIZES(true); }
    else { PRE3_AF_SIZES(false); }
#undef PRE3_AF_SIZES
#undef PRE3_AF
    return hipGetLastError();
}

// (27 groups per lane, 207,360 tokens, is what fits the 128 vector registers of a 1,024-thread block beside the
// masking code; the greedy fold needs more registers and stops at 20 groups, 153,600 tokens)
constexpr int kStepHeldShort = 9, kStepHeldMax = 27, kStepHeldMaxGreedy = 20;
constexpr int kStepHeldTwoRows = 8, kTwoRowsPerUnit = -1;   // the greedy form with two rows to a unit
// Largest vocabulary the fused step kernel can hold in registers, and the choice of its variant.
bool advance_fill_apply_fits(int n_tokens, int n_words, int cap, bool cycles, bool greedy) {
    const size_t row_bytes = (size_t)edge_row_stride_words(n_words) * sizeof(uint32_t);
    // (the greedy form loads without a branch, slots beyond the row load its last whole group: there has to be one)
    if (greedy && n_tokens < 8) return false;
    if ((n_tokens >> 3) > (greedy ? kStepHeldMaxGreedy : kStepHeldMax) * kStepData) return false;
    if (cycles) return cap <= kCompactMaxLen && row_bytes + (size_t)cap * sizeof(int32_t) <= kAfDynamicLdsMax;
    return row_bytes <= kAfDynamicLdsMax;
}

bool greedy_two_rows_fit(int n_tokens, int n_words, int cap, bool cycles) {
    const size_t row_bytes = (size_t)edge_row_stride_words(n_words) * sizeof(uint32_t);
    if ((n_tokens >> 3) < kStepHeldTwoRows * kStepData) return false;        // (whole registers of groups; shorter rows take other forms)
    return cycles ? cap <= kCompactMaxLen && row_bytes + (size_t)cap * sizeof(int32_t) <= kAfDynamicLdsMax : row_bytes <= kAfDynamicLdsMax;
}

bool greedy_any_offset_rows(int n_tokens, int batch, int n_compute_units) {
    const int groups = n_tokens >> 3;
    return groups > 10 * kStepData && (groups <= 17 * kStepData || 3 * batch >= n_compute_units);
}

bool greedy_two_rows_long_row(int n_tokens) { return (n_tokens >> 3) >= 2 * kStepHeldTwoRows * kStepData; }

bool advance_fill_apply_short_row(int n_tokens) { return (n_tokens >> 3) <= kStepHeldShort * kStepData; }

template <bool kCompact, bool kArgmax>
static void launch_step_variant(int held, dim3 grid, size_t lds, hipStream_t stream, const DevTables &T,
                                const int32_t *tokens, int32_t *states, int32_t *data, int32_t *len, int cap, int batch,
                                int32_t *err, uint32_t *bitmask, int restart_on_eos, int32_t *adv_scratch, int32_t *walk_spill,
                                const int32_t *cycle_head, const int32_t *cycle_pool, int stage, uint16_t *logits,
                                int64_t row_stride, int32_t *out_tokens, int first_row) {
#define PRE3_STEP(H, ROWS)                                                                                                  \
    hipLaunchKernelGGL((advance_fill_apply_kernel<kCompact, H, kArgmax, ROWS>), grid, dim3(kStepBlock), lds, stream, tokens, len,   \
                       states, data, T.pack, cap, first_row, logits, row_stride, batch, err, bitmask, restart_on_eos,          \
                       adv_scratch, walk_spill, (size_t)batch * 64, cycle_head, cycle_pool, stage, out_tokens)
    if (held == kTwoRowsPerUnit) {
        if constexpr (kArgmax) PRE3_STEP(kStepHeldTwoRows, 2);
    } else if (held <= kStepHeldShort) PRE3_STEP(kStepHeldShort, 1);
    else if (held <= 17) PRE3_STEP(17, 1);
    else if (held <= kStepHeldMaxGreedy || kArgmax) PRE3_STEP(20, 1);
    else if constexpr (!kArgmax) PRE3_STEP(27, 1);
#undef PRE3_STEP
}

// A block holds its row in the registers of a whole compute unit, so a grid of more blocks than units runs in
// rounds whose blocks start as others end, out of step with each other (62.5 us per step at 512 x 152,064).  A
// large batch goes as several launches of at most rows_per_launch rows instead, in equal shares (320 rows on
// 256 units as 160 + 160: 32.2 us against 36.7 us as 256 + 64), each launch a front of its own (47.2 us at 512).
static int step_rows_per_launch(int batch, int rows_per_launch) {
    if (rows_per_launch <= 0 || rows_per_launch >= batch) return batch;
    const int launches = (batch + rows_per_launch - 1) / rows_per_launch;
    return (batch + launches - 1) / launches;
}

hipError_t launch_advance_fill_apply(const DevTables &T, const int32_t *tokens, int32_t *states,
                                     int32_t *data, int32_t *len, int cap, int batch, int32_t *err, uint32_t *bitmask,
                                     int restart_on_eos, int32_t *adv_scratch, int32_t *walk_spill,
                                     const int32_t *cycle_head, const int32_t *cycle_pool, uint16_t *logits,
                                     int64_t row_stride, int32_t *out_tokens, int rows_per_launch, hipStream_t stream) {
    if (batch == 0) return hipSuccess;
    const bool two_rows = rows_per_launch == kRowsTwoPerUnit;
    if (two_rows ? !out_tokens || !greedy_two_rows_fit(T.n_tokens, T.n_words, cap, cycle_head != nullptr)
                 : !advance_fill_apply_fits(T.n_tokens, T.n_words, cap, cycle_head != nullptr, out_tokens != nullptr))
        return hipErrorInvalidValue;
    const bool aligned = (reinterpret_cast<uintptr_t>(logits) & 15) == 0 && (row_stride & 7) == 0;
    if ((!aligned && (!out_tokens || two_rows)) || row_stride < T.n_tokens) return hipErrorInvalidValue;
    const int held = two_rows ? kTwoRowsPerUnit : ((T.n_tokens >> 3) + kStepData - 1) / kStepData;
    const int held_variant = held <= 9 ? 9 : held <= 17 ? 17 : kStepHeldMaxGreedy;
    size_t lds = (size_t)edge_row_stride_words(T.n_words) * sizeof(uint32_t);
    int stage = 0;
    if (cycle_head) {
        lds += (size_t)cap * sizeof(int32_t);
        const size_t tables = (size_t)(T.n_states + T.cycle_pool_n) * sizeof(int32_t);
        stage = cycles_fit_lds(T.n_states, T.cycle_pool_n) && lds + tables <= kAfDynamicLdsMax;
        if (stage) lds += tables;
    }
    // the greedy fold reads a mask byte for every group slot of a lane, also those past the row's end
    if (out_tokens && !two_rows && lds < (size_t)held_variant * kStepData + 16) lds = (size_t)held_variant * kStepData + 16;
#define PRE3_STEP_ARGS held, dim3(rows), lds, stream, T, tokens, states, data, len, cap, batch, err, bitmask, restart_on_eos, \
                       adv_scratch, walk_spill, cycle_head, cycle_pool, stage, logits, row_stride, out_tokens, first
    const int share = two_rows ? batch : step_rows_per_launch(batch, rows_per_launch);
    for (int first = 0; first < batch; first += share) {
        const int rows = batch - first < share ? batch - first : share;
        if (cycle_head) {
            if (out_tokens) launch_step_variant<true, true>(PRE3_STEP_ARGS);
            else launch_step_variant<true, false>(PRE3_STEP_ARGS);
        } else {
            if (out_tokens) launch_step_variant<false, true>(PRE3_STEP_ARGS);
            else launch_step_variant<false, false>(PRE3_STEP_ARGS);
        }
    }
#undef PRE3_STEP_ARGS
    return hipGetLastError();
}

hipError_t launch_fill_apply_rows(const DevTables &T, const int32_t *states, const int32_t *data,
                                  const int32_t *len, int cap, int batch, uint32_t *bitmask, int32_t *walk_spill,
                                  uint16_t *logits, int64_t row_stride, int rows_per_launch, hipStream_t stream) {
    if (batch == 0) return hipSuccess;
    if (!advance_fill_apply_fits(T.n_tokens, T.n_words, cap, false, false)) return hipErrorInvalidValue;
    if ((reinterpret_cast<uintptr_t>(logits) & 15) != 0 || (row_stride & 7) != 0 || row_stride < T.n_tokens)
        return hipErrorInvalidValue;
    const int held = ((T.n_tokens >> 3) + kStepData - 1) / kStepData;
    const size_t lds = (size_t)edge_row_stride_words(T.n_words) * sizeof(uint32_t);
    const int share = step_rows_per_launch(batch, rows_per_launch);
    // no tokens: the kernel only reads the states and the stacks
    for (int first = 0; first < batch; first += share)
        launch_step_variant<false, false>(held, dim3(batch - first < share ? batch - first : share), lds, stream, T, nullptr,
                                          const_cast<int32_t *>(states), const_cast<int32_t *>(data), const_cast<int32_t *>(len),
                                          cap, batch, nullptr, bitmask, 0, nullptr, walk_spill, nullptr, nullptr, 0, logits,
                                          row_stride, nullptr, first);
    return hipGetLastError();
}

int step_spread_segments(int n_tokens) { return ((n_tokens + 7) / 8 + kSpreadGroups - 1) / kSpreadGroups; }

hipError_t launch_step_spread(const DevTables &T, const DevTokenEdges &E, const int32_t *tokens, int32_t *states, int32_t *data,
                              int32_t *len, int cap, int batch, int32_t *err, uint32_t *bitmask, int restart_on_eos,
                              int32_t *adv_spill, int32_t *walk_spill, const int32_t *cycle_head, const int32_t *cycle_pool,
                              uint16_t *logits, int64_t row_stride, int32_t *out_tokens, StepArrivals *arrivals, hipStream_t stream) {
    if (batch == 0) return hipSuccess;
    size_t lds = 0;
    int stage = 0;
    if (cycle_head) {
        lds = (size_t)cap * sizeof(int32_t);
        if (cap > kCompactMaxLen || lds > kAfDynamicLdsMax) return hipErrorInvalidValue;
        const size_t tables = (size_t)(T.n_states + T.cycle_pool_n) * sizeof(int32_t);
        stage = cycles_fit_lds(T.n_states, T.cycle_pool_n) && lds + tables <= kAfDynamicLdsMax;
        if (stage) lds += tables;
    }
    const int n_seg = step_spread_segments(T.n_tokens);
#define PRE3_SPREAD(C, A)                                                                                                   \
    hipLaunchKernelGGL((step_spread_kernel<C, A>), dim3(n_seg, batch), dim3(kSpreadBlock), lds, stream, tokens, len, states, data, cap, \
                       n_seg, logits, row_stride, (size_t)batch * n_seg, T, E, err, bitmask, restart_on_eos, adv_spill, walk_spill,  \
                       cycle_head, cycle_pool, stage, out_tokens, arrivals)
    if (cycle_head) {
        if (out_tokens) PRE3_SPREAD(true, true);
        else PRE3_SPREAD(true, false);
    } else {
        if (out_tokens) PRE3_SPREAD(false, true);
        else PRE3_SPREAD(false, false);
    }
#undef PRE3_SPREAD
    return hipGetLastError();
}

bool advance_fill_fits_compact(int n_words, int cap) {
    return cap <= kCompactMaxLen &&
           (size_t)edge_row_stride_words(n_words) * sizeof(uint32_t) + (size_t)cap * sizeof(int32_t) <= kAfDynamicLdsMax;
}

bool advance_fits_compact(int cap) {
    return cap <= kCompactMaxLen && (size_t)kAdvSeqPerBlock * cap * sizeof(int32_t) + 4096 <= 65536;
}

hipError_t launch_advance(const DevTables &T, const int32_t *tokens, int32_t *states, int32_t *data,
                          int32_t *len, int cap, int batch, int32_t *err, int32_t *scratch, int restart_on_eos,
                          const int32_t *cycle_head, const int32_t *cycle_pool, hipStream_t stream) {
    if (batch == 0) return hipSuccess;
    const dim3 grid((batch + kAdvSeqPerBlock - 1) / kAdvSeqPerBlock), block(64 * kAdvSeqPerBlock);
    if (cycle_head) {                                  // cycle-aware stacks: the new stack is staged in LDS
        if (!advance_fits_compact(cap)) return hipErrorInvalidValue;
        const size_t tables = (size_t)(T.n_states + T.cycle_pool_n) * sizeof(int32_t);
        const int stage = cycles_fit_lds(T.n_states, T.cycle_pool_n) &&
                          (size_t)kAdvSeqPerBlock * cap * sizeof(int32_t) + tables + 4096 <= 65536;
        const size_t lds = (size_t)kAdvSeqPerBlock * cap * sizeof(int32_t) + (stage ? tables : 0);
        hipLaunchKernelGGL(advance_kernel<true>, grid, block, lds, stream, tokens, len, states, data, cap, batch, T.pack, err,
                           scratch, restart_on_eos, cycle_head, cycle_pool, stage);
    } else {
        hipLaunchKernelGGL(advance_kernel<false>, grid, block, 0, stream, tokens, len, states, data, cap, batch, T.pack, err,
                           scratch, restart_on_eos, nullptr, nullptr, 0);
    }
    return hipGetLastError();
}

bool jump_forward_fits_compact(int cap) {
    return cap <= kCompactMaxLen && (size_t)kJfSeqPerBlock * cap * sizeof(int32_t) + 20480 <= 65536;
}

hipError_t launch_jump_forward(const DevTables &T, int32_t *states, int32_t *data, int32_t *len, int cap, int batch,
                               uint8_t *out_bytes, int32_t *out_len, int max_bytes, int32_t *adv_scratch,
                               int32_t *lane_spill, const int32_t *cycle_head, const int32_t *cycle_pool,
                               hipStream_t stream) {
    if (batch == 0) return hipSuccess;
    const dim3 grid((batch + kJfSeqPerBlock - 1) / kJfSeqPerBlock), block(64 * kJfSeqPerBlock);
    if (cycle_head) {                                  // cycle-aware stacks: compacted before the kernel ends
        if (!jump_forward_fits_compact(cap)) return hipErrorInvalidValue;
        const size_t tables = (size_t)(T.n_states + T.cycle_pool_n) * sizeof(int32_t);
        const int stage = cycles_fit_lds(T.n_states, T.cycle_pool_n) &&
                          (size_t)kJfSeqPerBlock * cap * sizeof(int32_t) + tables + 20480 <= 65536;
        const size_t lds = (size_t)kJfSeqPerBlock * cap * sizeof(int32_t) + (stage ? tables : 0);
        hipLaunchKernelGGL(jump_forward_kernel<true>, grid, block, lds, stream, len, states, data, cap, batch, T.pack, out_bytes,
                           out_len, max_bytes, adv_scratch, lane_spill, (size_t)batch * 64, cycle_head, cycle_pool, stage);
    } else {
        hipLaunchKernelGGL(jump_forward_kernel<false>, grid, block, 0, stream, len, states, data, cap, batch, T.pack, out_bytes,
                           out_len, max_bytes, adv_scratch, lane_spill, (size_t)batch * 64, nullptr, nullptr, 0);
    }
    return hipGetLastError();
}

hipError_t launch_compact_stacks(const int32_t *cycle_head, const int32_t *cycle_pool, int pool_entries, int n_states,
                                 int32_t *data, int32_t *len, int cap, int batch, hipStream_t stream) {
    if (batch == 0) return hipSuccess;
    if (cap > kCompactMaxLen) return hipErrorInvalidValue;
    const int pool_n = pool_entries <= 1024 ? pool_entries : 0;         // small record pools are staged in LDS
    int waves = 4;                                                      // sequences per block, within 64 KB of LDS
    while (waves > 1 && (size_t)(pool_n + waves * cap) * sizeof(int32_t) > 65536) waves >>= 1;
    const size_t lds = (size_t)(pool_n + waves * cap) * sizeof(int32_t);
    hipLaunchKernelGGL(compact_stacks_kernel, dim3((batch + waves - 1) / waves), dim3(64 * waves), lds, stream, cycle_head,
                       cycle_pool, pool_n, n_states, data, len, cap, batch);
    return hipGetLastError();
}

}  // namespace pre3
