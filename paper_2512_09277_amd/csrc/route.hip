// Routing kernels for gfx950: the METRO greedy solve (Alg. 1, Sec. 4.3 of arxiv 2512.09277)
// and the token-balanced baseline (Sec. 2.3 / Sec. 6.1).  A workgroup solves one layer, every table in LDS; where pairs
// have to be numbered, several workgroups solve the same layer and share the numbering.
//
// The paper's kernel runs Alg. 1 with one thread per expert and test-and-set locks on one
// SM; the order in which experts are served is whatever the lock races give.  Here the order
// is fixed (ascending expert id, ties to the lowest rank), which removes the locks and lets
// most of the serial chain collapse:
//   - an active expert with a single replica has no choice; its effect on the load L[g] seen
//     by a later expert e is a prefix popcount of a per-rank bitmap of such experts below e;
//   - only active experts with >= 2 replicas (at most S - N of them) form a serial chain, and
//     each step is an argmin over <= G lanes, in registers.
#include <hip/hip_runtime.h>
#include <stdint.h>

#include <algorithm>

#include "device_utils.h"
#include "metro.h"

namespace metro {
namespace {

constexpr int kMaxN = 512;
constexpr int kMaxG = 64;
constexpr int kMaxSpr = 64;
constexpr int kMaxS = 2048;   // G*spr
constexpr int kWords = kMaxN / 64;
constexpr int kThreads = 1024;
constexpr int kWaves = kThreads / 64;
constexpr int kNoSlot = 0x7fffffff;
constexpr int kChain = 64, kChainRow = kChain + 4;   // chain steps prepared at a time; the row ends off a bank period
constexpr int kRunPairs = 2048;   // pairs a workgroup numbers at least: two 64-item chunks per wave

struct RouteArgs {
    const int32_t* ids;
    const int32_t* slot_to_expert;
    int T, k, N, G, spr;
    int vec4;  // 1 when every layer's id and pair_slot run is 16-byte aligned and T*k % 4 == 0
    int32_t* pair_slot;
    int32_t* expert_slot;
    int32_t* rank_active;
    uint64_t* rank_bitmap;
    int32_t* err_flag;
    int split;                // workgroups per layer, each numbers and emits its own run of pairs
    // token lists of one rank (single-layer calls only), each workgroup emits the rows of its run
    int list_rank;            // < 0: no lists
    int32_t* group_offsets;
    int32_t* perm_pair;
    int32_t* pair_row;
    int32_t* n_pairs;
};

__device__ __forceinline__ uint64_t join64(uint32_t lo, uint32_t hi) { return ((uint64_t)hi << 32) | lo; }

__device__ __forceinline__ void set_bit64(uint32_t* lo, uint32_t* hi, int idx, int bit) {
    if (bit < 32) atomicOr(&lo[idx], 1u << bit);
    else atomicOr(&hi[idx], 1u << (bit - 32));
}

// ------------------------------------------------------------------------------------------ shared pieces
// Smallest value over the wave, in every lane's scalar view.
__device__ __forceinline__ uint32_t wave_min(uint32_t v) {
    constexpr int kNone = -1;                        // identity of the unsigned minimum
    v = min(v, (uint32_t)__builtin_amdgcn_update_dpp(kNone, (int)v, 0x111, 0xf, 0xf, false));      // row_shr:1
    v = min(v, (uint32_t)__builtin_amdgcn_update_dpp(kNone, (int)v, 0x112, 0xf, 0xf, false));
    v = min(v, (uint32_t)__builtin_amdgcn_update_dpp(kNone, (int)v, 0x114, 0xf, 0xf, false));
    v = min(v, (uint32_t)__builtin_amdgcn_update_dpp(kNone, (int)v, 0x118, 0xf, 0xf, false));
    v = min(v, (uint32_t)__builtin_amdgcn_update_dpp(kNone, (int)v, 0x142, 0xa, 0xf, false));      // row_bcast:15
    v = min(v, (uint32_t)__builtin_amdgcn_update_dpp(kNone, (int)v, 0x143, 0xc, 0xf, false));      // row_bcast:31
    return __builtin_amdgcn_readlane(v, kWave - 1);
}

// Smallest value over this lane's aligned group of 8 or 16 lanes, in every lane of it.
template <int kGroup>
__device__ __forceinline__ uint32_t group_min(uint32_t v) {
    constexpr int kNone = -1;
    v = min(v, (uint32_t)__builtin_amdgcn_update_dpp(kNone, (int)v, 0xb1, 0xf, 0xf, false));      // quad_perm: lane ^ 1
    v = min(v, (uint32_t)__builtin_amdgcn_update_dpp(kNone, (int)v, 0x4e, 0xf, 0xf, false));      // quad_perm: lane ^ 2
    v = min(v, (uint32_t)__builtin_amdgcn_update_dpp(kNone, (int)v, 0x141, 0xf, 0xf, false));     // row_half_mirror: lane ^ 7
    if (kGroup == 16) v = min(v, (uint32_t)__builtin_amdgcn_update_dpp(kNone, (int)v, 0x140, 0xf, 0xf, false));  // row_mirror
    return v;
}

// The run of pairs [lo, hi) of one of the workgroups of a layer, in chunks of 64; wave w of it owns the chunks
// [first + w * per_wave, ...).  Every workgroup reads all ids (it needs the counts of the pairs before its run and of the
// whole layer) and numbers only its own: reading and counting takes a fraction of numbering, and no workgroup waits
// for another.
struct Run {
    int lo, hi, first, per_wave;                     // first: the wave's first chunk
    __device__ __forceinline__ Run(int n, int part, int split) {
        const int chunks = (n + kWave - 1) / kWave, each = (chunks + split - 1) / split;
        const int begin = min(part * each, chunks), end = min(begin + each, chunks);
        lo = begin * kWave;
        hi = min(end * kWave, n);
        per_wave = (end - begin + kWaves - 1) / kWaves;
        first = begin + wave_id() * per_wave;
    }
    __device__ __forceinline__ int item(int c) const { return (first + c) * kWave + lane_id(); }
};

// f(id) for the ids outside the run, four at a time where the layout allows; `before`: the id precedes the run.
template <typename F>
__device__ __forceinline__ void for_other_ids(const int32_t* __restrict__ ids, int n, bool vec4, const Run& run, F f) {
    if (run.lo == 0 && run.hi >= n) return;          // uniform
    const int tid = threadIdx.x;
    if (vec4) {
        const int4* v = reinterpret_cast<const int4*>(ids);
        constexpr int kBatch = 4;                    // independent loads in flight
        for (int i0 = 0; i0 < n / 4; i0 += kBatch * kThreads) {
            int4 q[kBatch];
#pragma unroll
            for (int u = 0; u < kBatch; ++u) {
                const int i = i0 + u * kThreads + tid, p = 4 * i;
                q[u] = make_int4(-1, -1, -1, -1);
                if (p < n && (p < run.lo || p >= run.hi)) q[u] = v[i];
            }
#pragma unroll
            for (int u = 0; u < kBatch; ++u) {
                if (i0 + u * kThreads >= n / 4) break;   // uniform
                const bool before = 4 * (i0 + u * kThreads + tid) < run.lo;
                f(q[u].x, before); f(q[u].y, before); f(q[u].z, before); f(q[u].w, before);
            }
        }
    } else {
        for (int p = tid; p < n; p += kThreads)
            if (p < run.lo || p >= run.hi) f(ids[p], p < run.lo);
    }
}

// Per-wave counts of the run -> what precedes each wave's chunks; returns the count over the whole layer.
__device__ __forceinline__ int run_bases(int* hist, int n_keys, int e, int before, int after) {
    int c[kWaves], running = before;
#pragma unroll
    for (int w = 0; w < kWaves; ++w) c[w] = hist[w * n_keys + e];      // all reads first: one LDS round trip, not one per wave
#pragma unroll
    for (int w = 0; w < kWaves; ++w) {
        hist[w * n_keys + e] = running;
        running += c[w];
    }
    return running + after;
}

// ------------------------------------------------------------------------------------------ METRO
constexpr int kIdCache = 8;      // int4 loads of ids a thread keeps in registers between the two passes
constexpr int kRunCache = 8;     // chunks of its run whose ids a wave keeps in registers

// Fewer steps than this in the chain (no more than spare slots or pairs, unless experts have no slot): no keys.  Preparing them costs two
// barriers' phases, 0.8 us; a call with lists, us, with keys / without: 16 experts, 4 spare slots 5.2 / 4.3 at 1 token, 128 experts, 16 spare
// slots 5.7 / 5.3 at 32 tokens, 256 experts, 32 spare slots 6.4 / 6.4, 512 experts, 64 spare slots 7.4 / 7.8.  Deciding by the steps
// themselves, counted in LDS, costs 0.1 us everywhere.  Fewer slots than experts say nothing: keys.  Without lists the keys are the
// faster everywhere.
constexpr uint32_t kFewSteps = 32;

// One workgroup per layer solves; with kLists, `split` workgroups solve the same layer and each emits its own run of
// pairs and the rows these get in the token lists of one rank ("route tokens", Sec. 4.3).  All pairs of an expert go to
// one replica, so the row of a pair is the slot's first row plus the number of earlier pairs of the expert: one stable
// numbering, by the keys of the run only.  Bound by latency (barriers, LDS round trips, the serial chain), by the instructions of the
// passes over the ids (16 waves on four issue ports: an instruction of all of them takes 16 cycles) and by fetching its code anew in
// every call (15 KB with lists, of which a call runs one form of the chain), so loops are not unrolled.  Kernel times in a layer with the
// rule below, us, against one workgroup that sorted its own pair_slot in three more passes: 64 pairs 9.9 -> 5.2, 2048 pairs 11.0 -> 6.2,
// 8192 pairs (256 experts) 19.2 -> 10.0; without lists, 58 layers of 8192 pairs 10.2 -> 5.7 a pass (7.9 with flags set behind a branch
// per id and the masks inside the chain).
template <bool kLists>
__global__ __launch_bounds__(kThreads) void metro_route_kernel(RouteArgs a) {
    __shared__ uint32_t s_active4[kMaxN / 4 + 1];  // a byte per expert: has pairs (kLists: of the run)
    __shared__ uint32_t s_host_lo[kMaxN], s_host_hi[kMaxN];
    __shared__ int s_rank[kMaxN];                  // chosen rank g* of every active expert
    __shared__ int s_slot[kMaxN + 1];              // chosen slot
    __shared__ uint32_t s_forced_lo[kWords][kMaxG], s_forced_hi[kWords][kMaxG];
    __shared__ uint32_t s_multi_lo[kWords], s_multi_hi[kWords];     // per word: active experts with several replicas
    __shared__ uint32_t s_bm_lo[kMaxG], s_bm_hi[kMaxG];
    __shared__ int s_err;
    __shared__ __attribute__((aligned(16))) uint32_t s_key[kMaxG][kChainRow];     // of a run of chain steps, by rank
    __shared__ __attribute__((aligned(16))) uint32_t s_best[kChain];
    __shared__ int s_list[kChain];                                  // their experts
    __shared__ __attribute__((aligned(16))) int s_hist[kLists ? kWaves * kMaxN : 1];             // pairs per expert: the run's, by wave
    __shared__ int s_before[kLists ? kMaxN : 1], s_after[kLists ? kMaxN : 1];
    __shared__ int s_off[kLists ? kMaxSpr : 1];                     // first row of every slot of list_rank

    const int layer = kLists ? 0 : blockIdx.x, part = kLists ? blockIdx.x : 0;
    const int N = a.N, G = a.G, spr = a.spr, S = G * spr;
    const int n_pairs = a.T * a.k;
    const int32_t* ids = a.ids + (size_t)layer * n_pairs;
    const int32_t* s2e = a.slot_to_expert + (size_t)layer * S;
    int32_t* pair_slot = a.pair_slot + (size_t)layer * n_pairs;
    const int tid = threadIdx.x;

    // The global loads go out first, so that their latency overlaps the LDS set-up; the ids stay in
    // registers for the emit pass (what does not fit is read again).
    const int4* v = reinterpret_cast<const int4*>(ids);
    const int n4 = a.vec4 ? n_pairs / 4 : 0;
    const Run run(n_pairs, part, kLists ? a.split : 1);
    int4 idc[kLists ? 1 : kIdCache];
    int key[kLists ? kRunCache : 1];
    uint8_t* s_active = reinterpret_cast<uint8_t*>(s_active4);
    if constexpr (kLists) {
#pragma unroll
        for (int c = 0; c < kRunCache; ++c) {
            const int p = run.item(c);
            key[c] = c < run.per_wave && p < run.hi ? ids[p] : -1;
        }
    } else {
#pragma unroll
        for (int c = 0; c < kIdCache; ++c) {
            idc[c] = make_int4(-1, -1, -1, -1);
            const int i = tid + c * kThreads;
            if (i < n4) idc[c] = v[i];
        }
    }
    int se[kMaxS / kThreads];
#pragma unroll
    for (int j = 0; j < kMaxS / kThreads; ++j) {
        const int sl = tid + j * kThreads;
        se[j] = sl < S ? s2e[sl] : -1;
    }

    for (int e = tid; e < N; e += kThreads) {
        s_host_lo[e] = 0;
        s_host_hi[e] = 0;
        s_rank[e] = -1;
        s_slot[e] = kNoSlot;
        if constexpr (kLists) s_before[e] = s_after[e] = 0;
    }
    if (tid <= kMaxN / 4) s_active4[tid] = 0;
    if constexpr (kLists)
        for (int i = tid; i < kWaves * N / 4; i += kThreads) reinterpret_cast<int4*>(s_hist)[i] = make_int4(0, 0, 0, 0);
    for (int i = tid; i < ((N + 63) >> 6) * kMaxG; i += kThreads) {
        (&s_forced_lo[0][0])[i] = 0;
        (&s_forced_hi[0][0])[i] = 0;
    }
    if (tid < kMaxG) { s_bm_lo[tid] = 0; s_bm_hi[tid] = 0; }
    if (tid == 0) {
        s_err = 0;
        s_slot[N] = -1;
    }
    __syncthreads();

    // Ranks hosting each expert (matrix A) and T[i] > 0 for every expert.
#pragma unroll
    for (int j = 0; j < kMaxS / kThreads; ++j) {
        const int sl = tid + j * kThreads;
        if (sl < S) {
            if (se[j] < -1 || se[j] >= N) { atomicOr(&s_err, METRO_FLAG_BAD_PLACEMENT); se[j] = -1; }
            else if (se[j] >= 0) set_bit64(s_host_lo, s_host_hi, se[j], sl / spr);
        }
    }
    // The 16 waves share four issue ports, so what counts in the passes over the ids is their instructions: flags are set
    // without a branch (every id outside [0, N) sets one past the experts'), ids out of range show in a maximum.
    uint32_t top = 0;                                    // of id + 1: more than N only if an id is out of range
    auto mark = [&](int id) {
        s_active[min((uint32_t)id, (uint32_t)N)] = 1;
        top = max(top, (uint32_t)id + 1u);
    };
    if constexpr (kLists) {
        int* mine = s_hist + wave_id() * N;
        auto count = [&](int id, int* counts) {
            if ((uint32_t)id < (uint32_t)N) atomicAdd(&counts[id], 1);
        };
#pragma unroll
        for (int c = 0; c < kRunCache; ++c)
            if (c < run.per_wave) {                      // uniform per wave
                mark(key[c]);
                count(key[c], mine);
            }
        for (int c = kRunCache; c < run.per_wave; ++c) {
            const int id = run.item(c) < run.hi ? ids[run.item(c)] : -1;
            mark(id);
            count(id, mine);
        }
        for_other_ids(ids, n_pairs, a.vec4, run, [&](int id, bool before) {
            top = max(top, (uint32_t)id + 1u);
            count(id, before ? s_before : s_after);
        });
    } else {
#pragma unroll
        for (int c = 0; c < kIdCache; ++c) {
            if (c * kThreads >= n4) break;               // uniform
            mark(idc[c].x); mark(idc[c].y); mark(idc[c].z); mark(idc[c].w);   // padding (-1) where not loaded
        }
        for (int i = tid + kIdCache * kThreads; i < n4; i += kThreads) {
            const int4 q = v[i];
            mark(q.x); mark(q.y); mark(q.z); mark(q.w);
        }
        if (!a.vec4)
            for (int i = tid; i < n_pairs; i += kThreads) mark(ids[i]);
    }
    if (top > (uint32_t)N) atomicOr(&s_err, METRO_FLAG_BAD_ID);
    __syncthreads();

    // Split the active experts: single replica (forced) or several (the serial chain).  Wave w has the experts of word w.
    const int word = wave_id(), n_words = (N + 63) >> 6;
    if (word < n_words) {
        uint64_t host = 0;
        const bool active = tid < N && (kLists ? s_active[tid] | s_before[tid] | s_after[tid] : s_active[tid]);
        if (active) host = join64(s_host_lo[tid], s_host_hi[tid]);
        const int r = __popcll(host);
        if (r == 1) {
            const int g = __ffsll((unsigned long long)host) - 1;
            s_rank[tid] = g;
            set_bit64(&s_forced_lo[word][0], &s_forced_hi[word][0], g, lane_id());
        } else if (r == 0 && active) {
            atomicOr(&s_err, METRO_FLAG_NO_REPLICA);
        }
        const uint64_t multi = __ballot(r > 1);
        if (lane_id() == 0) {
            s_multi_lo[word] = (uint32_t)multi;
            s_multi_hi[word] = (uint32_t)(multi >> 32);
        }
    }
    __syncthreads();

    // The chain: wave 0.  Load of rank g when expert e is served = forced experts below e (known beforehand) + chain picks so far.
    // With lists, few steps: the masks of a word's experts in registers, lane b those of expert 64 w + b, 150 to 230 cycles per expert.
    // Else the known part becomes a key per step and rank, (load, rank), beyond every load where the rank does not host the expert,
    // which all waves prepare for up to kChain steps; what remains in the chain is an add, a minimum over the ranks in registers
    // and a compare, about 55 cycles per expert up to 16 ranks, where every lane of a group of 8 or 16 learns the minimum.
    const bool few = kLists && min((uint32_t)(S - N), (uint32_t)n_pairs) < kFewSteps;    // uniform; any number of steps is right both ways
    if (__builtin_expect(few, 0)) {              // out of line: laid in between it costs the other way 0.1 us
        if (tid < kWave) {
            const int g = tid;                           // masks of ranks past G are zero
            int load = 0;
            for (int w = 0; w < n_words; ++w) {
                const uint64_t forced = join64(s_forced_lo[w][g], s_forced_hi[w][g]);
                const int mine = min((w << 6) + g, N - 1);
                const uint32_t host_lo = s_host_lo[mine], host_hi = s_host_hi[mine];
                uint64_t left = join64(__builtin_amdgcn_readfirstlane(s_multi_lo[w]), __builtin_amdgcn_readfirstlane(s_multi_hi[w]));
                int picked = 0;
                uint32_t best_of = 0xffffffffu;          // lane b: rank chosen for expert 64 w + b
                for (; left; left &= left - 1) {
                    const int b = __ffsll((unsigned long long)left) - 1;
                    const uint64_t hosts = join64(__builtin_amdgcn_readlane(host_lo, b), __builtin_amdgcn_readlane(host_hi, b));
                    const int now = load + __popcll(forced & ((1ull << b) - 1ull)) + picked;
                    const uint32_t best = wave_min(((hosts >> g) & 1ull) ? ((uint32_t)now << 6) | (uint32_t)g : 0xffffffffu) & 63u;
                    if ((uint32_t)g == best) ++picked;
                    if (g == b) best_of = best;
                }
                if (best_of != 0xffffffffu) s_rank[(w << 6) + g] = (int)best_of;
                load += __popcll(forced) + picked;
            }
        } else if constexpr (kLists) {                   // meanwhile: what precedes each wave's chunks, and T[i]
            for (int e = tid - kWave; e < N; e += kThreads - kWave) s_after[e] = run_bases(s_hist, N, e, s_before[e], s_after[e]);
        }
        __syncthreads();
    } else {
        const int group = G <= 8 ? 8 : G <= 16 ? 16 : kWave;
        // every word has `parts` waves: each prepares every parts-th of its steps
        const int parts = kWaves / n_words, of = wave_id() / parts, part_of = wave_id() - of * parts;
        const int lw = min(lane_id(), n_words - 1);
        const uint32_t my_lo = s_multi_lo[lw], my_hi = s_multi_hi[lw];
        const int upto = wave_inclusive_sum(lane_id() < n_words ? __popc(my_lo) + __popc(my_hi) : 0);      // lane w: up to word w
        const int steps = __builtin_amdgcn_readlane(upto, kWords - 1);
        uint32_t picked = 0;                                 // of this lane's rank, in units of the key
#pragma clang loop unroll(disable)
        for (int first = 0; first < max(steps, 1); first += kChain) {        // once, unless more than kChain experts have a choice
            if (of < n_words) {
                const int g = lane_id();                     // masks of ranks past G are zero
                uint64_t left = join64(__builtin_amdgcn_readlane(my_lo, of), __builtin_amdgcn_readlane(my_hi, of)), forced = 0;
                int load = 0;
#pragma clang loop unroll(disable)
                for (int w = 0; w <= of; ++w) {
                    load += __popcll(forced);
                    forced = join64(s_forced_lo[w][g], s_forced_hi[w][g]);
                }
                int i = (of > 0 ? __builtin_amdgcn_readlane(upto, of - 1) : 0) - first;
                for (int turn = part_of; left; left &= left - 1, ++i, turn = turn ? turn - 1 : parts - 1) {
                    if (turn || i < 0 || i >= kChain) continue;              // uniform
                    const int b = __ffsll((unsigned long long)left) - 1, e = (of << 6) + b;
                    const uint64_t hosts = join64(s_host_lo[e], s_host_hi[e]);
                    const uint32_t known = (uint32_t)(load + __popcll(forced & ((1ull << b) - 1ull)));
                    s_key[g][i] = (((hosts >> g) & 1ull) ? known << 6 : 0x40000000u) | (uint32_t)g;
                    if (g == 0) s_list[i] = e;
                }
            }
            __syncthreads();
            if (tid < kWave) {
                const int n = min(steps - first, kChain);
                const uint32_t* keys = s_key[tid & (group - 1)];
                auto chain = [&](auto least) {
                    uint4 ahead = *reinterpret_cast<const uint4*>(keys);
#pragma clang loop unroll(disable)                     // the code of a call is fetched anew, so what loops is cheaper
                    for (int i = 0; i < n; i += 4) {         // past the last step: keys of no step, whose picks nobody asks for
                        const uint32_t k[4] = {ahead.x, ahead.y, ahead.z, ahead.w};
                        ahead = *reinterpret_cast<const uint4*>(keys + min(i + 4, kChain - 4));
                        uint32_t m[4];
#pragma unroll
                        for (int u = 0; u < 4; ++u) {
                            const uint32_t v = k[u] + picked;
                            m[u] = least(v);
                            picked += v == m[u] ? 64u : 0u;
                        }
                        *reinterpret_cast<uint4*>(s_best + i) = make_uint4(m[0], m[1], m[2], m[3]);
                    }
                };
                if (group == 8) chain([](uint32_t v) { return group_min<8>(v); });
                else if (group == 16) chain([](uint32_t v) { return group_min<16>(v); });
                else chain([](uint32_t v) { return wave_min(v); });
                if (tid < n) s_rank[s_list[tid]] = (int)(s_best[tid] & 63u);     // a wave's LDS accesses are done in order
            } else if (kLists && first == 0) {               // meanwhile: what precedes each wave's chunks, and T[i]
                for (int e = tid - kWave; e < N; e += kThreads - kWave) s_after[e] = run_bases(s_hist, N, e, s_before[e], s_after[e]);
            }
            __syncthreads();
        }
    }

    // y[i][g*] = 1 -> the lowest slot of expert i on rank g*.
#pragma unroll
    for (int j = 0; j < kMaxS / kThreads; ++j) {
        const int sl = tid + j * kThreads;
        const int e = se[j];
        if (sl < S && e >= 0 && s_rank[e] == sl / spr) atomicMin(&s_slot[e], sl);         // rank -1: not active, or no replica
    }
    __syncthreads();
    const int lo = a.list_rank * spr;
    if constexpr (kLists) {                              // the last wave: rows per slot of the rank and their offsets
        if (wave_id() == kWaves - 1) {
            const int l = lane_id();
            const int e = l < spr ? s2e[lo + l] : -1;
            const int c = e >= 0 && e < N && s_slot[e] == lo + l ? s_after[e] : 0;
            const int incl = wave_inclusive_sum(c);
            s_off[l] = incl - c;
            if (part == 0) {
                if (l < spr) a.group_offsets[l] = incl - c;
                if (l == spr - 1) {
                    a.group_offsets[spr] = incl;
                    *a.n_pairs = incl;
                }
            }
        }
    }
    for (int e = tid; e < N; e += kThreads) {
        int slot = s_slot[e];
        if (slot == kNoSlot) s_slot[e] = slot = -1;
        if (part == 0) a.expert_slot[(size_t)layer * N + e] = slot;
        if (slot >= 0) set_bit64(s_bm_lo, s_bm_hi, slot / spr, slot % spr);
    }
    __syncthreads();
    if (part == 0) {
        if (tid < G) {
            const uint64_t bm = join64(s_bm_lo[tid], s_bm_hi[tid]);
            a.rank_bitmap[(size_t)layer * G + tid] = bm;
            a.rank_active[(size_t)layer * G + tid] = __popcll(bm);
        }
        if (tid == 0) a.err_flag[layer] = s_err;
    }

    // x from y: every pair of expert i goes to its activated replica.
    auto slot_of = [&](int id) { return s_slot[min((uint32_t)id, (uint32_t)N)]; };      // the one past the experts': -1
    if constexpr (!kLists) {
        int4* o = reinterpret_cast<int4*>(pair_slot);
#pragma unroll
        for (int c = 0; c < kIdCache; ++c) {
            const int i = tid + c * kThreads;
            if (i < n4) o[i] = make_int4(slot_of(idc[c].x), slot_of(idc[c].y), slot_of(idc[c].z), slot_of(idc[c].w));
        }
        for (int i = tid + kIdCache * kThreads; i < n4; i += kThreads) {
            const int4 q = v[i];
            o[i] = make_int4(slot_of(q.x), slot_of(q.y), slot_of(q.z), slot_of(q.w));
        }
        if (!a.vec4)
            for (int i = tid; i < n_pairs; i += kThreads) pair_slot[i] = slot_of(ids[i]);
    } else {
        int* mine = s_hist + wave_id() * N;
        const int bits = 32 - __clz(max(spr - 1, 1));
        auto emit = [&](int p, int id) {
            const int slot = slot_of(id), l = slot - lo;
            const bool here = l >= 0 && l < spr;         // slot -1 is on no rank
            int total;
            const int nth = wave_rank_by_key(l, here, bits, total);
            int row = -1;
            if (here) {
                const int base = mine[id];
                row = s_off[l] + base + nth;
                // the wave executes in lockstep: every read of mine[] above precedes the update below
                if (nth == total - 1) mine[id] = base + total;
                a.perm_pair[row] = p;
            }
            if (p < run.hi) {
                pair_slot[p] = slot;
                a.pair_row[p] = row;
            }
        };
#pragma unroll
        for (int c = 0; c < kRunCache; ++c)
            if (c < run.per_wave) emit(run.item(c), key[c]);             // uniform per wave
        for (int c = kRunCache; c < run.per_wave; ++c) emit(run.item(c), run.item(c) < run.hi ? ids[run.item(c)] : -1);
    }
}

// ------------------------------------------------------------------------------------------ token-balanced
// `split` workgroups per layer, each with its own run of pairs.  The occurrence number q of a pair (its place among the
// pairs of its expert) gives both results: replica q mod r, and -- since that replica gets every r-th pair of the
// expert -- place q / r among the replica's pairs, so the token lists need no sort of their own.  Issue-bound in the
// ballots of the numbering (about 80 instructions per 64 pairs), hence the runs; kernel time with lists 13.3 -> 6.7 us at 776
// pairs, 80.7 -> 11.8 us at 32768 (one workgroup, ids past the registers read one chunk at a time, the lists sorted again).
__global__ __launch_bounds__(kThreads) void token_balanced_kernel(RouteArgs a) {
    __shared__ int s_hist[kWaves * kMaxN];          // the run's pairs per expert, by wave; then their bases
    __shared__ int s_before[kMaxN], s_cnt[kMaxN];   // pairs before the run; after it, then T[i]
    __shared__ uint32_t s_host_lo[kMaxN], s_host_hi[kMaxN];
    __shared__ int s_base[kMaxN + 1];               // CSR of replicas per expert
    __shared__ int s_repl[kMaxS];                   // replica slots, ascending slot id within an expert
    __shared__ uint32_t s_bm_lo[kMaxG], s_bm_hi[kMaxG];
    __shared__ int s_wave_sum[kWaves];
    __shared__ int s_off[kMaxSpr];                  // first row of every slot of list_rank
    __shared__ int s_err;

    const int layer = blockIdx.x / a.split, part = blockIdx.x - layer * a.split;
    const int N = a.N, G = a.G, spr = a.spr, S = G * spr;
    const int n_pairs = a.T * a.k;
    const int32_t* ids = a.ids + (size_t)layer * n_pairs;
    const int32_t* s2e = a.slot_to_expert + (size_t)layer * S;
    int32_t* pair_slot = a.pair_slot + (size_t)layer * n_pairs;
    const int tid = threadIdx.x;

    const Run run(n_pairs, part, a.split);
    int key[kRunCache];
#pragma unroll
    for (int c = 0; c < kRunCache; ++c) {
        const int p = run.item(c);
        key[c] = c < run.per_wave && p < run.hi ? ids[p] : -1;
    }
    int se[kMaxS / kThreads];
#pragma unroll
    for (int j = 0; j < kMaxS / kThreads; ++j) {
        const int sl = tid + j * kThreads;
        se[j] = sl < S ? s2e[sl] : -1;
    }
    for (int e = tid; e < N; e += kThreads) { s_host_lo[e] = s_host_hi[e] = 0; s_before[e] = s_cnt[e] = 0; }
    for (int i = tid; i < kWaves * N; i += kThreads) s_hist[i] = 0;
    for (int i = tid; i < S; i += kThreads) s_repl[i] = kNoSlot;
    if (tid < kMaxG) { s_bm_lo[tid] = 0; s_bm_hi[tid] = 0; }
    if (tid == 0) s_err = 0;
    __syncthreads();

#pragma unroll
    for (int j = 0; j < kMaxS / kThreads; ++j) {
        const int sl = tid + j * kThreads;
        if (sl < S) {
            if (se[j] < -1 || se[j] >= N) { atomicOr(&s_err, METRO_FLAG_BAD_PLACEMENT); se[j] = -1; }
            else if (se[j] >= 0) set_bit64(s_host_lo, s_host_hi, se[j], sl / spr);
        }
    }
    bool bad = false;
    auto valid = [&](int id) {
        const bool ok = (uint32_t)id < (uint32_t)N;
        bad |= !ok && id != -1;
        return ok;
    };
    int* mine = s_hist + wave_id() * N;
#pragma unroll
    for (int c = 0; c < kRunCache; ++c)
        if (c < run.per_wave && valid(key[c])) atomicAdd(&mine[key[c]], 1);      // the first half is uniform
    for (int c = kRunCache; c < run.per_wave; ++c) {
        const int id = run.item(c) < run.hi ? ids[run.item(c)] : -1;
        if (valid(id)) atomicAdd(&mine[id], 1);
    }
    for_other_ids(ids, n_pairs, a.vec4, run, [&](int id, bool before) {
        if (valid(id)) atomicAdd(before ? &s_before[id] : &s_cnt[id], 1);
    });
    if (bad) atomicOr(&s_err, METRO_FLAG_BAD_ID);
    __syncthreads();

    // T[i], the bases of the run's chunks, and an exclusive scan of the replica counts r_e = popcount(host[e]) -> s_base
    {
        int r = 0;
        if (tid < N) {
            r = __popcll(join64(s_host_lo[tid], s_host_hi[tid]));
            s_cnt[tid] = run_bases(s_hist, N, tid, s_before[tid], s_cnt[tid]);
            if (s_cnt[tid] > 0 && r == 0) atomicOr(&s_err, METRO_FLAG_NO_REPLICA);
        }
        const int incl = wave_inclusive_sum(r);
        if (lane_id() == kWave - 1) s_wave_sum[wave_id()] = incl;
        __syncthreads();
        int before = 0;
        for (int w = 0; w < wave_id(); ++w) before += s_wave_sum[w];
        if (tid < N) s_base[tid] = before + incl - r;
        if (tid == N - 1) s_base[N] = before + incl;
    }
    __syncthreads();

    // Replica lists: the lowest slot of an expert on each hosting rank, ranks ascending (= ascending slot id).
    auto replica = [&](int e, int g) { return __popcll(join64(s_host_lo[e], s_host_hi[e]) & ((1ull << g) - 1ull)); };
#pragma unroll
    for (int j = 0; j < kMaxS / kThreads; ++j) {
        const int sl = tid + j * kThreads;
        if (sl < S && se[j] >= 0) atomicMin(&s_repl[s_base[se[j]] + replica(se[j], sl / spr)], sl);
    }
    __syncthreads();
    // Replica i of expert e gets pairs i, i + r, ...: it is activated iff i < T[e].
    const int lo = a.list_rank * spr;
    auto pairs_of = [&](int e, int sl) {                 // 0 for a copy that is no replica
        const int i = replica(e, sl / spr), r = s_base[e + 1] - s_base[e];
        return s_repl[s_base[e] + i] == sl && i < s_cnt[e] ? (s_cnt[e] - i + r - 1) / r : 0;
    };
#pragma unroll
    for (int j = 0; j < kMaxS / kThreads; ++j) {
        const int sl = tid + j * kThreads;
        if (sl < S && se[j] >= 0 && pairs_of(se[j], sl) > 0) set_bit64(s_bm_lo, s_bm_hi, sl / spr, sl % spr);
    }
    if (a.list_rank >= 0 && wave_id() == kWaves - 1) {   // rows per slot of the rank and their offsets
        const int l = lane_id();
        const int e = l < spr ? s2e[lo + l] : -1;
        const int c = e >= 0 && e < N ? pairs_of(e, lo + l) : 0;
        const int incl = wave_inclusive_sum(c);
        s_off[l] = incl - c;
        if (part == 0) {
            if (l < spr) a.group_offsets[l] = incl - c;
            if (l == spr - 1) {
                a.group_offsets[spr] = incl;
                *a.n_pairs = incl;
            }
        }
    }
    __syncthreads();
    if (part == 0) {
        if (tid < G) {
            const uint64_t bm = join64(s_bm_lo[tid], s_bm_hi[tid]);
            a.rank_bitmap[(size_t)layer * G + tid] = bm;
            a.rank_active[(size_t)layer * G + tid] = __popcll(bm);
        }
        if (tid == 0) a.err_flag[layer] = s_err;
    }

    const int bits = 32 - __clz(max(N - 1, 1));
    auto emit = [&](int p, int id) {
        const bool ok = id >= 0 && id < N;
        int total;
        const int nth = wave_rank_by_key(id, ok, bits, total);
        int slot = -1, row = -1;
        if (ok) {
            const int q = mine[id] + nth;
            // the wave executes in lockstep: every read of mine[] above precedes the update below
            if (nth == total - 1) mine[id] = q + 1;
            const int first = s_base[id], r = s_base[id + 1] - first;
            if (r > 0) {
                const int turn = q / r;
                slot = s_repl[first + q - turn * r];
                const int l = slot - lo;
                if (a.list_rank >= 0 && l >= 0 && l < spr) {
                    row = s_off[l] + turn;
                    a.perm_pair[row] = p;
                }
            }
        }
        if (p < run.hi) {
            pair_slot[p] = slot;
            if (a.list_rank >= 0) a.pair_row[p] = row;
        }
    };
#pragma unroll
    for (int c = 0; c < kRunCache; ++c)
        if (c < run.per_wave) emit(run.item(c), key[c]);                 // uniform per wave
    for (int c = kRunCache; c < run.per_wave; ++c) emit(run.item(c), run.item(c) < run.hi ? ids[run.item(c)] : -1);
}

// Workgroups per layer for the calls that number pairs: runs of at least 2048 pairs, no more workgroups than CUs, and no more
// than 64 readers of one layer's ids.  Counting the other runs' ids costs a workgroup up to 1 us whatever their number, numbering more
// of its own pairs costs it more.  Measured, 256 experts, a call with lists, us, runs of at least 1024 / 2048 / 4096 pairs, METRO and
// token-balanced: 2048 pairs 6.9 / 7.1 / 7.1 and 6.5 / 7.0 / 7.0, 4096 pairs 7.0 / 7.6 / 8.4 and 6.6 / 7.5 / 9.0, 8192 pairs 7.7 / 8.0 /
// 9.1 and 7.3 / 8.1 / 9.8, 32768 pairs 11.1 / 11.5 / 12.4 and 10.6 / 11.4 / 13.1; from 64 runs of 2048 on no difference.
inline int split_for(const RouteArgs& a, int L) {
    const int64_t n = (int64_t)a.T * a.k;
    const int64_t most = L >= 256 ? 1 : std::min(256 / L, 64);
    return (int)std::max<int64_t>(1, std::min((n + kRunPairs - 1) / kRunPairs, most));
}

// Whether an output shares memory with an input or with another output.  Workgroups of a layer read its inputs while others
// already write, and so do the waves of one workgroup with the ids that do not fit its registers (runs of more than 8192
// pairs), whose list rows go to any place.  Such a call gets one workgroup per layer, and its token lists come from a
// second launch, once the routing has consumed its inputs.
bool shares_memory(const RouteArgs& a, int L) {
    struct Range {
        uintptr_t begin, end;
        Range(const void* p, int64_t words) : begin((uintptr_t)p), end(p ? begin + 4 * (uintptr_t)words : begin) {}
    };
    const int64_t n = (int64_t)a.T * a.k, lists = a.list_rank >= 0;
    const bool own_count = lists && a.n_pairs != a.group_offsets + a.spr;       // else the last offset itself, the same value
    const Range all[] = {{a.ids, L * n}, {a.slot_to_expert, (int64_t)L * a.G * a.spr},        // the inputs
                         {a.pair_slot, L * n}, {a.expert_slot, (int64_t)L * a.N}, {a.rank_active, (int64_t)L * a.G},
                         {a.rank_bitmap, (int64_t)L * a.G * 2}, {a.err_flag, L}, {a.group_offsets, lists * (a.spr + 1)},
                         {a.perm_pair, lists * n}, {a.pair_row, lists * n}, {a.n_pairs, own_count}};
    for (int out = 2; out < (int)(sizeof(all) / sizeof(all[0])); ++out)
        for (int other = 0; other < out; ++other)
            if (all[out].begin < all[other].end && all[other].begin < all[out].end) return true;
    return false;
}

int check_route_args(const void* ids, const void* s2e, int L, int T, int k, int N, int G, int spr,
                     const void* pair_slot, const void* rank_active, const void* rank_bitmap,
                     const void* err_flag) {
    if (!s2e || !rank_active || !rank_bitmap || !err_flag) return METRO_ERR_INVALID_ARG;
    if (L < 1 || T < 0 || k < 1 || N < 1 || G < 1 || spr < 1 || k > N) return METRO_ERR_INVALID_ARG;
    if ((!ids || !pair_slot) && T > 0) return METRO_ERR_INVALID_ARG;   // an empty batch has no id tensor
    if (N > kMaxN || G > kMaxG || spr > kMaxSpr || G * spr > kMaxS || (int64_t)T * k >= (1 << 24))
        return METRO_ERR_UNSUPPORTED;
    return METRO_OK;
}

RouteArgs pack(const int32_t* ids, const int32_t* s2e, int T, int k, int N, int G, int spr, int32_t* pair_slot,
               int32_t* expert_slot, int32_t* rank_active, uint64_t* rank_bitmap, int32_t* err_flag) {
    RouteArgs a;
    a.ids = ids;
    a.slot_to_expert = s2e;
    a.T = T; a.k = k; a.N = N; a.G = G; a.spr = spr;
    const bool aligned = (((uintptr_t)ids | (uintptr_t)pair_slot) & 15) == 0 && ((int64_t)T * k) % 4 == 0;
    a.vec4 = aligned ? 1 : 0;
    a.pair_slot = pair_slot;
    a.expert_slot = expert_slot;
    a.rank_active = rank_active;
    a.rank_bitmap = rank_bitmap;
    a.err_flag = err_flag;
    a.list_rank = -1;
    a.split = 1;
    a.group_offsets = a.perm_pair = a.pair_row = a.n_pairs = nullptr;
    return a;
}

int add_lists(RouteArgs& a, int rank, int32_t* group_offsets, int32_t* perm_pair, int32_t* pair_row, int32_t* n_pairs) {
    if (!group_offsets || !n_pairs || rank < 0 || rank >= a.G) return METRO_ERR_INVALID_ARG;
    if ((!perm_pair || !pair_row) && a.T > 0) return METRO_ERR_INVALID_ARG;
    a.list_rank = rank;
    a.group_offsets = group_offsets;
    a.perm_pair = perm_pair;
    a.pair_row = pair_row;
    a.n_pairs = n_pairs;
    return METRO_OK;
}

}  // namespace
}  // namespace metro

extern "C" int metro_route(const int32_t* topk_ids, const int32_t* slot_to_expert, int L, int T, int k, int N,
                           int G, int spr, int32_t* pair_slot, int32_t* expert_slot, int32_t* rank_active,
                           uint64_t* rank_bitmap, int32_t* err_flag, void* stream) {
    using namespace metro;
    int rc = check_route_args(topk_ids, slot_to_expert, L, T, k, N, G, spr, pair_slot, rank_active, rank_bitmap,
                              err_flag);
    if (rc != METRO_OK) return rc;
    if (!expert_slot) return METRO_ERR_INVALID_ARG;
    RouteArgs a = pack(topk_ids, slot_to_expert, T, k, N, G, spr, pair_slot, expert_slot, rank_active,
                       rank_bitmap, err_flag);
    hipLaunchKernelGGL(metro_route_kernel<false>, dim3(L), dim3(kThreads), 0, (hipStream_t)stream, a);
    return hipGetLastError() == hipSuccess ? METRO_OK : METRO_ERR_HIP;
}

extern "C" int metro_route_token_balanced(const int32_t* topk_ids, const int32_t* slot_to_expert, int L, int T,
                                          int k, int N, int G, int spr, int32_t* pair_slot,
                                          int32_t* rank_active, uint64_t* rank_bitmap, int32_t* err_flag,
                                          void* stream) {
    using namespace metro;
    int rc = check_route_args(topk_ids, slot_to_expert, L, T, k, N, G, spr, pair_slot, rank_active, rank_bitmap,
                              err_flag);
    if (rc != METRO_OK) return rc;
    RouteArgs a = pack(topk_ids, slot_to_expert, T, k, N, G, spr, pair_slot, nullptr, rank_active, rank_bitmap,
                       err_flag);
    a.split = shares_memory(a, L) ? 1 : split_for(a, L);
    hipLaunchKernelGGL(token_balanced_kernel, dim3(L * a.split), dim3(kThreads), 0, (hipStream_t)stream, a);
    return hipGetLastError() == hipSuccess ? METRO_OK : METRO_ERR_HIP;
}

extern "C" int metro_route_permute(const int32_t* topk_ids, const int32_t* slot_to_expert, int T, int k, int N, int G,
                                   int spr, int rank, int32_t* pair_slot, int32_t* expert_slot, int32_t* rank_active,
                                   uint64_t* rank_bitmap, int32_t* err_flag, int32_t* group_offsets,
                                   int32_t* perm_pair, int32_t* pair_row, int32_t* n_pairs, void* stream) {
    using namespace metro;
    int rc = check_route_args(topk_ids, slot_to_expert, 1, T, k, N, G, spr, pair_slot, rank_active, rank_bitmap,
                              err_flag);
    if (rc != METRO_OK) return rc;
    if (!expert_slot) return METRO_ERR_INVALID_ARG;
    RouteArgs a = pack(topk_ids, slot_to_expert, T, k, N, G, spr, pair_slot, expert_slot, rank_active,
                       rank_bitmap, err_flag);
    rc = add_lists(a, rank, group_offsets, perm_pair, pair_row, n_pairs);
    if (rc != METRO_OK) return rc;
    if (shares_memory(a, 1)) {
        rc = metro_route(topk_ids, slot_to_expert, 1, T, k, N, G, spr, pair_slot, expert_slot, rank_active, rank_bitmap,
                         err_flag, stream);
        return rc != METRO_OK ? rc : moe_permute(pair_slot, T, k, rank, spr, group_offsets, perm_pair, pair_row, n_pairs, stream);
    }
    a.split = split_for(a, 1);
    hipLaunchKernelGGL(metro_route_kernel<true>, dim3(a.split), dim3(kThreads), 0, (hipStream_t)stream, a);
    return hipGetLastError() == hipSuccess ? METRO_OK : METRO_ERR_HIP;
}

extern "C" int metro_route_token_balanced_permute(const int32_t* topk_ids, const int32_t* slot_to_expert, int T, int k,
                                                  int N, int G, int spr, int rank, int32_t* pair_slot,
                                                  int32_t* rank_active, uint64_t* rank_bitmap, int32_t* err_flag,
                                                  int32_t* group_offsets, int32_t* perm_pair, int32_t* pair_row,
                                                  int32_t* n_pairs, void* stream) {
    using namespace metro;
    int rc = check_route_args(topk_ids, slot_to_expert, 1, T, k, N, G, spr, pair_slot, rank_active, rank_bitmap,
                              err_flag);
    if (rc != METRO_OK) return rc;
    RouteArgs a = pack(topk_ids, slot_to_expert, T, k, N, G, spr, pair_slot, nullptr, rank_active, rank_bitmap,
                       err_flag);
    rc = add_lists(a, rank, group_offsets, perm_pair, pair_row, n_pairs);
    if (rc != METRO_OK) return rc;
    if (shares_memory(a, 1)) {
        rc = metro_route_token_balanced(topk_ids, slot_to_expert, 1, T, k, N, G, spr, pair_slot, rank_active, rank_bitmap,
                                        err_flag, stream);
        return rc != METRO_OK ? rc : moe_permute(pair_slot, T, k, rank, spr, group_offsets, perm_pair, pair_row, n_pairs, stream);
    }
    a.split = split_for(a, 1);
    hipLaunchKernelGGL(token_balanced_kernel, dim3(a.split), dim3(kThreads), 0, (hipStream_t)stream, a);
    return hipGetLastError() == hipSuccess ? METRO_OK : METRO_ERR_HIP;
}
