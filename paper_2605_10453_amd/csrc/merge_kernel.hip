// Cross-workgroup merge for the streaming path and for rows_topk_kernel: one block per row combines the row's chunk
// partials (running max m_c, sum of exp s_c, top-k list per chunk) into the final ids and log-probabilities:
//     lse = M + ln sum_c s_c exp(m_c - M),   M = max_c m_c
// and the k first (logit desc, id asc) of all lists' entries.  The order of every reduction is fixed and the selection
// works on unique keys (order bits of the logit, then the inverted id), so the output does not depend on scheduling.
//
// What bounds it: the length of its chain of instructions.  There is hardly any work and one trip to memory (0.4 us; a second pass over the same lists
// took 3.6 us of the first one's 3.9), but a lone wavefront takes 8 to 28 cycles per dependent instruction (device_utils.hpp).
//
// Lists of up to 16 ids (10 in a launch of more than 24 rows of few lists) whose entries a block's threads can hold (SHORT, the usual call; plan.hpp:
// merge_short_lists): every thread keeps up to eight entries and one chunk's (m, s).
//   (1) T: the smallest of the maxima of k groups of entries (device_utils.hpp), so k entries reach it; two or three times as many do, where a sort
//       would leave hardly more than k, but they are ranked by all threads and the sort is a chain of 21 exchanges.  M = max m_c in the same steps.
//   (2) every wavefront puts its entries that reach T into a list of its own in shared memory (an addition to a common counter takes 174 cycles), and
//       the terms of the log-sum-exp are added, one per thread.
//   (3) the k first are found by counting.
// Two barriers.  Measured with one wavefront for all of this / now: one row, d = 4096, r = 512, V = 128256 33.9 / 32.7 us a call, with draws at V = 151936
// 45.7 / 45.4, 23 rows 42.4 / 41.2, the full head at d = 624, V = 23344, k = 1 12.7 / 11.3.  Rows with more entries at the bound than the lists hold, or with
// a logit that is no finite number, go on with what follows.
//
// Other calls (an instance of their own): one wavefront does everything that is a chain, without barriers, and the others only fetch lists:
//   (1) wavefront 0 reads the chunk maxima (the lists' heads), up to 8 per lane in flight.
//       T = the k-th largest of its 64 lanes' maxima: k heads reach it, so it bounds the answer from below.  (All-pairs
//       counting of 251 heads by 1024 threads took longer than the loads: 6.6 us a launch, 13.5 with 500 chunks and a draw.)
//       With fewer lists than k no head bounds anything: there T is the m-th largest of the lists' j-th entries, m j >= k.  (Every entry of 32 lists
//       of 64, as T = 0 admits them, is 40 us of (3): one row, r = 16, V = 2048, k = 64 55 us a call, 14 with this T.)
//       Wavefront 1 meanwhile finds the draw of a sampling call, wavefront 2 folds the log-sum-exp (by wavefront 0, before the bound / by wavefront 2:
//       4 rows, d = 1024, r = 128, V = 8192, k = 40 14.6 / 14.3 us a call, 16 rows, V = 128256, k = 32 22.5 / 22.1, one row, d = 2048, r = 256, k = 40 24.0 / 23.7).
//   (2) all threads: the lists' entries that reach T go to shared memory.  Where a row has few entries they were
//       requested at the start, before T is known (one trip instead of two); otherwise the first eight of the lists whose
//       heads reach T are read, and more of a list only where all eight are taken.
//   (3) the k first of them are found by counting, or, where they are many, by wavefront 0.
#include "gemv_parts.hpp"
#include "launch.hpp"

namespace slimspec {

namespace {

constexpr int kMergeHeads = 8;                                   // heads per lane in flight
constexpr int kMergeWaves = kRowMergeThreads / 64;
constexpr int kMergeMine = 64;                                   // entries of a wavefront's list at most
constexpr int kMergeLists = SLIMSPEC_KMAX_INTERNAL + kCandSlack; // lists that may hold winners, at most
constexpr int kMergeCand = kMergeLists * SLIMSPEC_KMAX_INTERNAL; // their entries, at most
constexpr int kMergeSel = 256;                                   // entries that are ranked all pairs, at most
static_assert(kMergeAhead * kRowMergeThreads <= kMergeCand, "entries taken ahead fit as well");
static_assert(kMergeShort <= kBoundMaxK, "lists that bound_of_groups serves");
static_assert(kMergeSel >= 2 * kMergeLists, "what a bound admits beyond this many are equal logits");

struct MergeLds {
    uint64_t cand[kMergeCand];
    uint64_t sel[kMergeSel];
    int list[kMergeLists];
    uint32_t n_list, n_cand, T, all_lists;
    float lse;
    uint64_t draw;
    float draw_z;
    // short lists
    uint64_t mine[kMergeWaves][kMergeMine + 8], wave_draw[kMergeWaves];
    uint32_t groups[128];
    int n_mine[kMergeWaves];
    float wave_s[kMergeWaves], wave_draw_z[kMergeWaves];
};

// The k largest of n keys in shared memory, by one wavefront: f(key, rank).
template <class F>
__device__ __forceinline__ void wave_rank_keys(const uint64_t *keys, int n, int k, int lane, F f) {
    for (int c0 = 0; c0 < n; c0 += 64) {
        const int c = c0 + lane;
        const uint64_t mine = (c < n) ? keys[c] : kNoKey;
        int rank = 0;
#pragma unroll 8
        for (int q = 0; q < n; ++q) rank += (keys[q] > mine) ? 1 : 0;
        if (c < n && rank < k) f(mine, rank);
    }
}

}  // namespace

// SHORT: lists that the code for short ones takes (the other code as well, for rows that it leaves); long lists have an instance without it, whose blocks
// would otherwise jump over it: the compiler's layout of one then moved calls of the other by up to 1.1 us (the router of four rows 50.8 / 51.9).
template <bool SHORT>
__global__ __launch_bounds__(kRowMergeThreads) void merge_kernel(
    const float2 *__restrict__ part_ms, const float *__restrict__ part_val, const int *__restrict__ part_id,
    int chunks, int k, int last_len, int j_th, int m_th, int32_t *__restrict__ out_ids, float *__restrict__ out_logprobs,
    const int32_t *__restrict__ id_map, SampleOut so, const float4 *__restrict__ part_smp)
{
    __shared__ MergeLds S;
    constexpr int NT = kRowMergeThreads, H = kMergeHeads;
    const int row = blockIdx.x, tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const float2 *ms = part_ms + (size_t)row * chunks;
    const float *pv = part_val + (size_t)row * chunks * k;
    const int *pi = part_id + (size_t)row * chunks * k;

    // Entries of the last chunk's list from last_len on are filler (it may have fewer than k columns; the others have k).
    const int n_entries = (chunks - 1) * k + last_len;
    constexpr int A = SHORT ? kMergeAhead : kMergeAheadLong;
    const bool ahead = SHORT || n_entries <= A * NT;
    float2 hm[H];
    if (SHORT) hm[0] = ms[min(tid, chunks - 1)];
    else if (wave == 0 || wave == 2) {
#pragma unroll
        for (int e = 0; e < H; ++e) hm[e] = ms[min(64 * e + lane, chunks - 1)];
    }
    float v_jth = 0.f;
    if (wave == 0 && j_th > 1) v_jth = pv[(size_t)min(lane, chunks - 1) * k + j_th - 1];
    float v_ahead[A];
    int id_ahead[A];
    if (ahead) {
#pragma unroll
        for (int u = 0; u < A; ++u) {
            if (u * NT >= n_entries) break;                      // (the same for all)
            const int e = min(tid + u * NT, n_entries - 1);
            v_ahead[u] = pv[e];
            id_ahead[u] = pi[e];
        }
    }

    float lse = 0.f;
    const auto emit = [&](uint64_t key, int rank) {
        const int id = (int)key_tiebreak(key);
        out_ids[(size_t)row * k + rank] = id_map ? id_map[id] : id;      // truncated vocabulary: column -> vocabulary id
        out_logprobs[(size_t)row * k + rank] = key_value(key) - lse;
    };
    const auto emit_draw = [&](uint64_t key, float z) {
        const int id = (int)key_tiebreak(key);
        so.lse[row] = lse;
        so.sample_ids[row] = id_map ? id_map[id] : id;
        so.sample_logprobs[row] = z - lse;
    };
    const auto rank_by_counting = [&](int n) {                   // the scan for every entry shared by as many lanes as there are
        const int p = lanes_per_item_log2(n, NT), P = 1 << p, c = tid >> p, part = tid & (P - 1);
        const uint64_t mine = c < n ? S.cand[c] : kNoKey;
        int rank = 0;
#pragma unroll 4
        for (int q = part; q < n; q += P) rank += S.cand[q] > mine ? 1 : 0;
        rank = lanes_sum(rank, P);
        if (c < n && part == 0 && rank < k) emit(mine, rank);
    };
    if constexpr (SHORT) {
        const bool have = tid < chunks;
        float4 draw = make_float4(0.f, 0.f, 0.f, 0.f);
        if (part_smp) draw = part_smp[(size_t)row * chunks + min(tid, chunks - 1)];
        const BoundPlan bound = make_bound_plan(min(n_entries, NT), k, 5);
        if (tid < kBoundGroups && tid >= bound.n_groups) S.groups[tid] = 0u;
        uint32_t bits[A], most = 0u;
#pragma unroll
        for (int u = 0; u < A; ++u) {
            bits[u] = 0u;
            if (u * NT >= n_entries) break;                      // (the same for all)
            if (tid + u * NT < n_entries) bits[u] = float_order_bits(v_ahead[u]);
            most = max(most, bits[u]);
        }
        if (bound.gl > 0) most = max(most, dpp_u32<0xB1>(most));
        if (bound.gl > 1) most = max(most, dpp_u32<0x4E>(most));
        if (bound.gl > 2) most = max(most, dpp_u32<0x141>(most));
        if (bound.gl > 3) most = max(most, dpp_u32<0x140>(most));
        if (bound.gl > 4) most = max(most, lane_xor16(most, lane));
        if ((tid & ((1 << bound.gl) - 1)) == 0 && (tid >> bound.gl) < bound.n_groups) S.groups[tid >> bound.gl] = most;
        __syncthreads();
        uint32_t top;
        const uint32_t T = bound_of_groups(S.groups, bound, k, lane, top);
        const float M = float_from_order_bits(top);              // the largest list's head; a row with a not-a-number ends up below
        uint32_t n_lane = 0u;
#pragma unroll
        for (int u = 0; u < A; ++u) {
            if (u * NT >= n_entries) break;
            n_lane += bits[u] >= T ? 1u : 0u;
        }
        const uint32_t upto = wave_prefix_sum(n_lane);
        const int n_mine = __builtin_amdgcn_readlane((int)upto, 63);      // entries of this wavefront
        int at = (int)(upto - n_lane);
#pragma unroll
        for (int u = 0; u < A; ++u) {
            if (u * NT >= n_entries) break;
            if (bits[u] >= T) S.mine[wave][min(at++, kMergeMine)] = u64_from(bits[u], ~(uint32_t)id_ahead[u]);      // (beyond: the list is not used)
        }
        if (lane < 8) S.mine[wave][min(n_mine, kMergeMine) + lane] = kNoKey;
        S.n_mine[wave] = n_mine;
        const float s = wave_sum(have ? hm[0].y * fast_exp(hm[0].x - M) : 0.f);
        S.wave_s[wave] = s;
        if (part_smp) {                                          // the largest z + g over the chunks (unique keys)
            const uint64_t key = have ? make_key(draw.x, (uint32_t)__float_as_int(draw.y)) : kNoKey, largest = wave_max_key(key);
            if (key == largest) { S.wave_draw[wave] = largest; S.wave_draw_z[wave] = draw.z; }
        }
        __syncthreads();
        // A wavefront ranks its own entries, eight at a time, the scan shared by eight lanes.
        int n_w[kMergeWaves], longest = 0;
        float sum = 0.f;
#pragma unroll
        for (int w = 0; w < kMergeWaves; ++w) {
            n_w[w] = __builtin_amdgcn_readfirstlane(S.n_mine[w]);
            longest = max(longest, n_w[w]);
            sum += S.wave_s[w];                                  // fixed order
        }
        lse = M + fast_log(sum);
        // (too many entries at the bound, or a logit that is no finite number, in whose chunk the sum is none either: the general code)
        if (__builtin_amdgcn_readfirstlane(sum < __builtin_huge_valf() ? 1 : 0) != 0 && longest <= kMergeMine) {
            for (int c0 = 0; c0 < n_mine; c0 += 8) {
                const uint64_t key = S.mine[wave][c0 + (lane >> 3)];       // (zeros behind the last)
                const int rank = rank_in_lists(S.mine, n_w, longest, key, lane);
                if (key != kNoKey && (lane & 7) == 0 && rank < k) emit(key, rank);
            }
            if (part_smp && tid == NT - 1) {
                int w = 0;
                for (int i = 1; i < kMergeWaves; ++i)
                    if (S.wave_draw[i] > S.wave_draw[w]) w = i;
                emit_draw(S.wave_draw[w], S.wave_draw_z[w]);
            }
            return;
        }
#pragma unroll
        for (int e = 0; e < H; ++e) hm[e] = ms[min(64 * e + lane, chunks - 1)];
    }

    if (wave == 0 || wave == 2) {
        // this lane's chunks in increasing order, H at a time
        // A chunk's maximum is its list's first entry, but not where the chunk holds a not-a-number: lists order those by their bits (a positive
        // one comes before +inf), while the maximum ignores them and is -inf, or has a sign and payload of its own, where there is nothing else.  With
        // such a head the list would not be taken, or T would admit no entry at all.  The chunk's sum is then no number either.
        const auto heads_in_lists = [&](int c0) {
            bool any = false;
#pragma unroll
            for (int e = 0; e < H; ++e) any |= !(hm[e].y < __builtin_huge_valf());
            if (__ballot(any) == 0ull) return;                   // as a rule (a branch per load: 300000 columns 0.9 us more)
#pragma unroll
            for (int e = 0; e < H; ++e)
                if (!(hm[e].y < __builtin_huge_valf())) hm[e].x = pv[(size_t)min(c0 + 64 * e + lane, chunks - 1) * k];
        };
        const auto load_heads = [&](int c0) {
            if (c0 == 0 && chunks <= 64 * H) return;             // still in registers
#pragma unroll
            for (int e = 0; e < H; ++e) hm[e] = ms[min(c0 + 64 * e + lane, chunks - 1)];
            heads_in_lists(c0);
        };
        heads_in_lists(0);
        // (at least 1 for a list, as list_bits)
        const auto bits_of = [&](int c0, int e) { return (c0 + 64 * e + lane < chunks) ? list_bits(hm[e].x) : 0u; };
        if (wave == 2) {
            float m_t = kNegInf, s_t = 0.f;
            for (int c0 = 0; c0 < chunks; c0 += 64 * H) {
                load_heads(c0);
                float m_new = m_t;
#pragma unroll
                for (int e = 0; e < H; ++e)
                    if (c0 + 64 * e + lane < chunks) m_new = fmaxf(m_new, hm[e].x);
                s_t = (m_t == kNegInf) ? 0.f : s_t * fast_exp(m_t - m_new);
#pragma unroll
                for (int e = 0; e < H; ++e)                      // a chunk with no logit above -inf adds nothing (its sum is not a number)
                    if (c0 + 64 * e + lane < chunks && hm[e].x != kNegInf) s_t += hm[e].y * fast_exp(hm[e].x - m_new);
                m_t = m_new;
            }
            const float M = wave_max(m_t);
            const float s = wave_sum(m_t == kNegInf ? 0.f : s_t * fast_exp(m_t - M));
            if (lane == 0) S.lse = M + fast_log(s);
        } else {
            uint32_t lane_bits = 0u;
            for (int c0 = 0; c0 < chunks; c0 += 64 * H) {
                load_heads(c0);
#pragma unroll
                for (int e = 0; e < H; ++e) lane_bits = max(lane_bits, bits_of(c0, e));
            }
            // (j-th entries: a lane has one list at most, the last one may not have as many; too few that have, or too few heads: everything)
            if (j_th > 1) lane_bits = lane < chunks - 1 || (lane == chunks - 1 && j_th <= last_len) ? list_bits(v_jth) : 0u;
            const uint32_t sorted = wave_sort_desc(lane_bits, lane);
            uint32_t T = max(1u, (uint32_t)__builtin_amdgcn_readlane((int)sorted, m_th - 1));
            const auto count = [&](uint32_t bound) {
                int n = 0;
                for (int c0 = 0; c0 < chunks; c0 += 64 * H) {
                    load_heads(c0);
#pragma unroll
                    for (int e = 0; e < H; ++e)
                        if (c0 + 64 * e < chunks) n += __popcll(__ballot(bits_of(c0, e) >= bound));
                }
                return n;
            };
            // many lists at the bound (k close to 64): raise it while k of them reach it
            int n = count(T), above = 0;
            if (n > k + kCandSlack) {
                uint32_t hi = (uint32_t)__builtin_amdgcn_readfirstlane((int)sorted) + 1u;        // no head reaches it
                while (n > k + kCandSlack && hi - T > 1u) {
                    const uint32_t mid = T + (hi - T) / 2;
                    const int c = count(mid);
                    if (c >= k) { T = mid; n = c; } else { hi = mid; above = c; }
                }
            }
            // Still more: lists with equal heads.  Of those, the first ones of the row suffice: their heads precede
            // every entry of the later ones.
            const bool ties = n > k + kCandSlack;
            int quota = ties ? k - above : n;                        // lists with a head equal to T that are taken (above: the heads beyond it)
            int at = 0;
            for (int c0 = 0; c0 < chunks; c0 += 64 * H) {
                load_heads(c0);
#pragma unroll
                for (int e = 0; e < H; ++e) {
                    if (c0 + 64 * e >= chunks) break;
                    const uint32_t b = bits_of(c0, e);
                    bool take = b >= T;
                    if (ties) {
                        const uint64_t equal = __ballot(b == T);
                        const int before = __builtin_amdgcn_mbcnt_hi((uint32_t)(equal >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)equal, 0u));
                        take = b > T || (b == T && before < quota);
                        quota = max(0, quota - (int)__popcll(equal));
                    }
                    const uint64_t mask = __ballot(take);
                    const int slot = at + __builtin_amdgcn_mbcnt_hi((uint32_t)(mask >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)mask, 0u));
                    if (take && slot < kMergeLists) S.list[slot] = c0 + 64 * e + lane;
                    at += __popcll(mask);
                }
            }
            if (lane == 0) { S.n_list = (uint32_t)min(at, kMergeLists); S.n_cand = 0u; S.T = T; S.all_lists = ties ? 0u : 1u; }
        }
    } else if (wave == 1 && part_smp) {
        // the Gumbel-max draw: the largest z + g over the chunks (unique keys)
        const float4 *smp = part_smp + (size_t)row * chunks;
        uint64_t best = kNoKey;
        float zb = 0.f;
        for (int c0 = 0; c0 < chunks; c0 += 64 * H) {
            float4 x[H];
#pragma unroll
            for (int e = 0; e < H; ++e) x[e] = smp[min(c0 + 64 * e + lane, chunks - 1)];
#pragma unroll
            for (int e = 0; e < H; ++e) {
                const uint64_t key = make_key(x[e].x, (uint32_t)__float_as_int(x[e].y));
                if (key > best) { best = key; zb = x[e].z; }
            }
        }
        const uint64_t top = wave_max_key(best);
        if (best == top) { S.draw = top; S.draw_z = zb; }        // (a clamped lane may hold the last chunk's as well: the same values)
    }
    __syncthreads();

    // ---- the entries that reach T
    const uint32_t T = S.T;
    const auto push = [&](bool in, float v, int id) {
        const uint32_t bits = float_order_bits(v);
        const bool take = in && bits >= T;
        const uint64_t mask = __ballot(take);
        if (mask == 0ull) return mask;
        const int before = __builtin_amdgcn_mbcnt_hi((uint32_t)(mask >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)mask, 0u));
        uint32_t base = 0u;
        if (take && before == 0) base = atomicAdd(&S.n_cand, (uint32_t)__popcll(mask));
        base = (uint32_t)__builtin_amdgcn_readlane((int)base, __ffsll((unsigned long long)mask) - 1);
        if (take) S.cand[base + before] = u64_from(bits, ~(uint32_t)id);
        return mask;
    };
    if (ahead && S.all_lists) {
#pragma unroll
        for (int u = 0; u < A; ++u) push(tid + u * NT < n_entries, v_ahead[u], id_ahead[u]);
    } else {
        // eight lanes per list, which is sorted: its next eight entries only where all of these were taken
        const int sub = lane & 7, n_list = (int)S.n_list;
        constexpr int GROUPS = NT / 8, PASSES = (kMergeLists + GROUPS - 1) / GROUPS;
        const auto entry = [&](int l, int p, bool &in) {
            const int e = S.list[min(l, n_list - 1)] * k + p;
            in = l < n_list && p < k && e < n_entries;
            return min(e, n_entries - 1);
        };
        float v[PASSES];
        int id[PASSES];
        bool in[PASSES];
#pragma unroll
        for (int u = 0; u < PASSES; ++u) {
            const int e = entry((tid >> 3) + u * GROUPS, sub, in[u]);
            v[u] = pv[e];
            id[u] = pi[e];
        }
#pragma unroll
        for (int u = 0; u < PASSES; ++u) {
            uint64_t taken = push(in[u], v[u], id[u]);
            for (int p = 8; p < k && ((taken >> (lane & 56)) & 0xffu) == 0xffu; p += 8) {
                bool more;
                const int e = entry((tid >> 3) + u * GROUPS, p + sub, more);
                taken = push(more, pv[e], pi[e]);
            }
        }
    }
    __syncthreads();

    // ---- the k first of them
    lse = S.lse;
    if (part_smp && tid == NT - 1) emit_draw(S.draw, S.draw_z);
    const int n = (int)S.n_cand;
    if (n <= kMergeSel) {
        rank_by_counting(n);                                     // (k = 64: one wavefront alone took 3 us)
    } else if (wave == 0) {
        // as with the lists: the k-th largest lane maximum, raised where it admits many
        uint32_t lane_bits = 0u;
        for (int c = lane; c < n; c += 64) lane_bits = max(lane_bits, (uint32_t)(S.cand[c] >> 32));
        const uint32_t sorted = wave_sort_desc(lane_bits, lane);
        uint32_t T2 = max(1u, (uint32_t)__builtin_amdgcn_readlane((int)sorted, k - 1));
        const auto count = [&](uint32_t bound) {
            int m = 0;
            for (int c0 = 0; c0 < n; c0 += 64) m += __popcll(__ballot(c0 + lane < n && (uint32_t)(S.cand[min(c0 + lane, n - 1)] >> 32) >= bound));
            return m;
        };
        int n2 = count(T2);
        uint32_t hi = (uint32_t)__builtin_amdgcn_readfirstlane((int)sorted) + 1u;
        while (n2 > k + 2 * kCandSlack && hi - T2 > 1u) {
            const uint32_t mid = T2 + (hi - T2) / 2;
            const int c = count(mid);
            if (c >= k) { T2 = mid; n2 = c; } else hi = mid;
        }
        if (n2 <= kMergeSel) {
            int at = 0;
            for (int c0 = 0; c0 < n; c0 += 64) {
                const uint64_t key = (c0 + lane < n) ? S.cand[c0 + lane] : kNoKey;
                const bool take = (uint32_t)(key >> 32) >= T2;
                const uint64_t mask = __ballot(take);
                if (take) S.sel[at + __builtin_amdgcn_mbcnt_hi((uint32_t)(mask >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)mask, 0u))] = key;
                at += __popcll(mask);
            }
            lds_wave_sync();
            wave_rank_keys(S.sel, n2, k, lane, emit);
        } else {                                                 // that many equal logits: the largest key, k times
            uint64_t last = ~0ull;
            for (int rank = 0; rank < k; ++rank) {
                uint64_t best = kNoKey;
                for (int c = lane; c < n; c += 64) { const uint64_t key = S.cand[c]; if (key < last) best = u64_max(best, key); }
                last = wave_max_key(best);
                if (lane == 0) emit(last, rank);
            }
        }
    }
}

hipError_t launch_merge(const float2 *part_ms, const float *part_val, const int *part_id,
                        int rows, int chunks, int chunk_cols, int V, int k, int32_t *out_ids, float *out_logprobs, const int32_t *id_map,
                        const SampleOut &so, const float4 *part_smp, hipStream_t st)
{
    const int last_len = merge_last_len(chunks, chunk_cols, V, k);
    // (j one more than it takes: m then leaves out the lists whose j-th entries are the smallest.  Not where (3) ranks all entries anyway.  Worked
    // out here: two divisions and a sort of its own in the kernel cost every call up to 0.5 us)
    int j_th = 1;
    if (chunks < k && (chunks - 1) * k + last_len > kMergeSel) j_th = (k + chunks - 1) / chunks + 1 < k ? (k + chunks - 1) / chunks + 1 : k;
    const auto launch = [&](auto kernel) {
        kernel<<<rows, kRowMergeThreads, 0, st>>>(part_ms, part_val, part_id, chunks, k, last_len, j_th, (k + j_th - 1) / j_th, out_ids, out_logprobs,
                                                  id_map, so, so.on ? part_smp : nullptr);
    };
    if (merge_short_lists(rows, chunks, last_len, k)) launch(merge_kernel<true>);
    else launch(merge_kernel<false>);
    return hipGetLastError();
}

}  // namespace slimspec
