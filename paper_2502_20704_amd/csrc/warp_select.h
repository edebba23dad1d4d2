// Temperature / top-k / top-p: the smallest kept scaled logit of the row a token is drawn from.
// Part of libfsd (gfx950); included by fsd_kernels.hip, which holds the host side and the C ABI.
#ifndef FSD_CSRC_WARP_SELECT_H_
#define FSD_CSRC_WARP_SELECT_H_

#include "accept_sample.h"
#include "device_common.h"
#include "pair_kernel.h"

namespace {

// ------------------------------------------------------------------------------------------
// sampling-method warpers (Sec. 4: the token is drawn with "whatever sampling method the user
// sets"): temperature, then top-k, then top-p, in that order, on the row the token is drawn from.
// One workgroup per sequence, or several (SPLIT), find the smallest kept scaled logit s = z inv_temp:
//   top-k   the k-th largest s: a select over the order-preserving 32-bit image of s;
//   top-p   the largest t with sum_{s >= t} e^(s - max) >= top_p sum_{kept} e^(s - max), by the same
//           select on weights; the weights are 2^40 fixed-point integers, so that the sums do not
//           depend on the order of the atomic additions (results are the same run to run).
// Ties at either threshold are kept.  accept_sample then drops every entry below the threshold; or (P.draw) this kernel, which
// has everything top-k kept in LDS by then, draws the token itself and writes the outputs.
// What bounds it: the passes over the row (range, sums or per-thread maxima, gathering) on few compute units, the
// selects in LDS, which are chains of barriers, and with SPLIT the round trips between the workgroups.

__device__ __forceinline__ unsigned ordered_key(float x) {
    const unsigned u = __float_as_uint(x);
    return (u & 0x80000000u) ? ~u : (u | 0x80000000u);
}
__device__ __forceinline__ float key_value(unsigned k) {
    return __uint_as_float((k & 0x80000000u) ? (k & 0x7FFFFFFFu) : ~k);
}

// The bound of a list of a row's largest entries, from the upper half of a key that enough of them reach.  A bound of +0 lets
// -0 in as well, whose key lies right below: the two are one number, and ties at a threshold are kept.
__device__ __forceinline__ unsigned list_bound(unsigned key) {
    return key == 0x80000000u ? 0x7FFFFFFFu : key;
}

// the bitwise or over the wavefront
__device__ __forceinline__ unsigned wave_or(unsigned v) {
    v |= static_cast<unsigned>(dpp_i<kDppSwap1>(static_cast<int>(v)));
    v |= static_cast<unsigned>(dpp_i<kDppSwap2>(static_cast<int>(v)));
    v |= static_cast<unsigned>(dpp_i<kDppHalfMirror>(static_cast<int>(v)));
    v |= static_cast<unsigned>(dpp_i<kDppMirror>(static_cast<int>(v)));
    unsigned all = 0u;
#pragma unroll
    for (int row = 0; row < 64; row += 16) all |= static_cast<unsigned>(__builtin_amdgcn_readlane(static_cast<int>(v), row));
    return all;
}

struct WarpParams {
    const char* target;
    const int32_t* parent;   // tree: [B,N]; NULL for a chain
    int rows;             // K or N
    long V;
    long nslots;
    float T;
    float inv_temp;
    int top_k;            // 0 = off
    float top_p;          // 1 = off
    float* thr;           // [B] out
    // SPLIT: memory of a sequence's workgroups, seq_bytes each (the exchange words of the reduction, which has ended)
    char* area;
    size_t seq_bytes;
    int list_keys;        // entries a workgroup's list has room for under top-k (see launch_warp_split)
    unsigned spin_limit;
    // 1 (SPLIT under top-k, at most 64 rows, lists with room for the places as well): this kernel draws the token and writes
    // the call's outputs, no accept_sample follows
    int draw;
    const int32_t* tokens;
    int max_depth;        // tree only
    unsigned seed_lo, seed_hi, off_lo, off_hi;
    int32_t* out_len;
    int32_t* out_tokens;
    int32_t* path_nodes;  // tree only
    int32_t* row_status;  // optional
    uint4* clear;         // see SampleParams
    long clear16;
    Ws ws;
};

constexpr int kWarpWG = 1024;

// An interval that holds every value of a bin of the value histogram: a cheap first question for the passes that
// gather one bin's entries (the bin itself is decided by the same operations as in the histogram).  The slack
// covers the rounding of those operations (1e-6 of a difference of at most 2048 bins) and of the bounds.
struct Interval { float lo, hi; };
__device__ __forceinline__ Interval bin_interval(float top, float scale, int bin) {
    const float slack = 0.01f / scale + fabsf(top) * 1e-6f, at = static_cast<float>(bin);
    return Interval{top - (at + 1.0f) / scale - slack, top - at / scale + slack};
}

// KEEP: the row fits 16 slots per thread (aligned bfloat16 rows up to 131072 entries), or a share of it
// split_keep (SPLIT), and is read once into registers; otherwise every pass streams it again, four loads in
// flight per thread.
constexpr int kWarpKeep = 16;
constexpr int kWarpList = 8192;   // entries the select can finish from LDS
constexpr int kWarpFastK = 512;   // largest top-k of the short way
constexpr int kWarpBins = 2048;   // bins of the value histogram (16 KB of LDS)
constexpr float kWarpRange = 28.0f;   // what lies further below the maximum weighs less than 2^-40: one bin

// SPLIT: gridDim.x workgroups share a sequence, each with at most split_keep slots of the row per thread, for the
// usual settings (top-k of at most kWarpFastK, or top-p alone).  One workgroup's time is a compute unit
// reading and passing over a whole row while most of the device is idle, so up to eight share a row and what is left
// for one of them is the select (rows of 128256 bfloat16 entries: 64 of them under temperature 0.7, top-k 50, top-p 0.9
// take 23 us with four workgroups each, 30 with one; 8 of them under top-p 0.95 25 us with eight, 49 with one):
//   top-k   every workgroup leaves the entries at or above the k-th largest of its own threads' maxima (the
//           row's k largest are among them) and counts itself; whoever counts last selects from all of them, a few
//           hundred for the usual k, and with their places in the row draws the token from what is kept: no
//           second kernel, whose start and passes over rows of which it drops nearly all cost more than the selection's end.
//           Up to 1024 of them stand in the registers of every wavefront, and the wavefronts look for the cut together, each
//           counting the entries above a candidate of its own: 4 bits a round with one barrier (count_select).  (A
//           select by 8-bit digits in LDS has seven barriers a digit and its additions queue at a few words.)
//   top-p   the workgroups agree on the row's range (one word each, zero until posted; the wait is bounded, and
//           all are resident, which the host checks), add their histograms of values in memory and count
//           themselves.  When all have (the same kind of wait) every one finds the bin of the crossing and leaves the entries its own
//           share has of it, and counts itself again; whoever counts last then selects from those.  (It used to gather the
//           bin from the row alone, a pass over the whole of it in one compute unit; that is left for bins with more
//           entries than the lists hold.  8 rows of 128256 bfloat16 entries under top-p 0.95: 30 -> 25 us.)
// Words and counts lie in the sequence's counter line, which every call clears.  What is left for others is stored
// with device-scope stores and performed (s_waitcnt) before the count.
constexpr int kWarpShare = 8;
constexpr int kSplitBins = kWarpWG;
constexpr size_t kSplitBytes = 16384;   // a sequence's memory, at least; under top-p 1024 bins and lists of 2048 keys
constexpr int kSplitKeys = 4096;        // keys and lengths of a sequence's lists under top-k, at most
constexpr int kCountKeys = 1024;        // keys count_select takes
constexpr int kRankKeys = 192;          // keys whose weights are summed up by rank, all pairs of them

// (two kernels, one under top-k and one under top-p alone: what they have in common is the row and the general selects, and with the
// one's registers and code in the other the top-p calls took 2 us longer)
enum { SPLIT_NONE = 0, SPLIT_TOP_K = 1, SPLIT_TOP_P = 2 };
// Slots of a share a thread keeps: 5, or 8 of binary32 rows, so that four workgroups, which is what 64 sequences have, hold rows of 131072 entries
// (64 of them, V=128256, top-k 50, top-p 0.9: whole call 135.3 us with 5, where one workgroup a row streams it, 116.0 with 8; bfloat16, whose
// rows fit either way, 78.8 and 79.2).  Rows of more than kSplitSlots slots are left to one workgroup.
constexpr int split_keep(bool bf16) { return bf16 ? 5 : 8; }
constexpr long kSplitSlots = 8L * 5 * kWarpWG;
template <bool BF16, int LD, bool KEEP, int SHARED = SPLIT_NONE>
__global__ __launch_bounds__(kWarpWG) void warp_select(WarpParams P) {
    constexpr bool SPLIT = SHARED != SPLIT_NONE, BY_K = SHARED == SPLIT_TOP_K;
    constexpr int VE = Slot<BF16>::VE;
    constexpr int ES = BF16 ? 2 : 4;
    __shared__ unsigned long long s_hist[256];
    __shared__ unsigned s_cnt[256];
    __shared__ unsigned long long s_wtot[4];
    __shared__ unsigned s_lkey[kWarpList];
    __shared__ unsigned long long s_bins[kWarpBins];
    __shared__ float s_red[kWarpWG / 64], s_red2[kWarpWG / 64];
    __shared__ int s_n, s_st, s_nlist, s_bin;
    __shared__ unsigned s_tmax[kWarpWG];
    __shared__ unsigned long long s_wsum[kWarpWG / 64], s_wtail[kWarpWG / 64];
    __shared__ unsigned s_prefix, s_mask, s_match;
    __shared__ unsigned long long s_need;
    __shared__ float s_max, s_min;
    __shared__ unsigned s_round[2][kWarpWG / 64], s_score;
    __shared__ unsigned long long s_above[kRankKeys + 1];
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int b = SPLIT ? blockIdx.y : blockIdx.x;

    // ---- the row the token will be drawn from: the first rejected position, or the row after the last
    // (chain); the row after the deepest node whose ancestors are all accepted, lowest index on ties (tree)
    int from = 0;
    // P.draw: what the outputs need
    [[maybe_unused]] int status = 0, n_acc = 0, winner = -1, my_par = -1, my_dep = 0, my_tok = 0;
    [[maybe_unused]] bool failed = false;
    if (tid == 0) { s_n = P.rows; s_st = 0; s_match = 0u; }
    __syncthreads();
    if (P.rows <= 64) {
        // a lane per position or node, every wavefront for itself, all words requested together (see accept_sample): the
        // pointer jumping by all sixteen wavefronts, two barriers a round, and the failure word behind it took 2.5 us of the
        // kernel on trees of 60 nodes (24.5 -> 22.0) and about 1 us of a whole call on chains of 8 (93.9 -> 92.7)
        const int pr = b * P.rows + (lane < P.rows ? lane : P.rows - 1);
        const int st = P.ws.pst[pr];
        const float div = P.ws.div[pr];
        if (P.parent) my_par = P.parent[pr];
        if (BY_K && P.draw) my_tok = P.tokens[pr];
        failed = failure_flagged(P.ws);
        const bool mine = lane < P.rows, ok = div <= P.T;
        if (__any(mine && st != 0)) {
            status = mine ? st : 0;
#pragma unroll
            for (int o = 32; o > 0; o >>= 1) status |= __shfl_xor(status, o);
        }
        if (P.parent == nullptr) {
            const unsigned long long no = __ballot(mine && !ok);
            from = n_acc = no ? static_cast<int>(__builtin_ctzll(no)) : P.rows;
        } else {
            // (a path that is too deep is for whoever writes the outputs to report: a malformed tree stops both)
            const TreePick pick = pick_path(lane, P.rows, BY_K && P.draw ? P.max_depth : kMaxRows, my_par, ok);
            status |= pick.status;
            if (status & FSD_ROW_BAD_PARENT) status &= ~FSD_ROW_TOO_DEEP;
            n_acc = pick.n;
            winner = pick.winner;
            my_dep = pick.my_dep;
            from = winner + 1;
        }
        if (failed) status |= FSD_ROW_INTERNAL;
        from = __builtin_amdgcn_readfirstlane(from);
        status = __builtin_amdgcn_readfirstlane(status);
        n_acc = __builtin_amdgcn_readfirstlane(n_acc);
        winner = __builtin_amdgcn_readfirstlane(winner);
        if (status && tid == 0) s_st = 1;
        __syncthreads();
    } else if (P.parent == nullptr) {
        for (int i = tid; i < P.rows; i += kWarpWG) {
            const int pr = b * P.rows + i;
            if (P.ws.pst[pr]) atomicOr(&s_st, 1);
            if (!(P.ws.div[pr] <= P.T)) atomicMin(&s_n, i);
        }
        __syncthreads();
    } else {
        // pointer jumping over the parents, as in accept_sample; the list's memory is free until the select
        const int rows = P.rows;
        int* par = reinterpret_cast<int*>(s_lkey);
        int* anc = par + rows;
        int* acc = anc + rows;
        int* dep = acc + rows;
        for (int j = tid; j < rows; j += kWarpWG) {
            const int pr = b * rows + j;
            int p = P.parent[pr];
            if (p < -1 || p >= j) { atomicOr(&s_st, 1); p = -1; }   // accept_sample reports it
            if (P.ws.pst[pr]) atomicOr(&s_st, 1);
            par[j] = p; anc[j] = p; dep[j] = 1;
            acc[j] = (P.ws.div[pr] <= P.T) ? 1 : 0;
        }
        __syncthreads();
        constexpr int PER = kMaxRows / kWarpWG;
        for (int span = 1; span < rows; span <<= 1) {
            int na[PER], nacc[PER], nd[PER];
#pragma unroll
            for (int q = 0; q < PER; ++q) {
                const int j = tid + q * kWarpWG;
                if (j < rows) {
                    const int a = anc[j];
                    na[q] = a; nacc[q] = acc[j]; nd[q] = dep[j];
                    if (a >= 0) { na[q] = anc[a]; nacc[q] = acc[j] & acc[a]; nd[q] = dep[j] + dep[a]; }
                }
            }
            __syncthreads();
#pragma unroll
            for (int q = 0; q < PER; ++q) {
                const int j = tid + q * kWarpWG;
                if (j < rows) { anc[j] = na[q]; acc[j] = nacc[q]; dep[j] = nd[q]; }
            }
            __syncthreads();
        }
        for (int j = tid; j < rows; j += kWarpWG) {
            if (acc[j]) atomicMax(&s_match, (static_cast<unsigned>(dep[j]) << 11) | static_cast<unsigned>(kMaxRows - 1 - j));
        }
        __syncthreads();
        const unsigned key = s_match;
        if (tid == 0) s_n = key ? (kMaxRows - 1 - static_cast<int>(key & (kMaxRows - 1))) + 1 : 0;
        __syncthreads();
    }
    if (P.rows > 64) {
        if (failure_flagged(P.ws) && tid == 0) s_st = 1;
        from = s_n;
        __syncthreads();
    }
    // P.draw: the outputs of the sequence, by one wavefront
    [[maybe_unused]] auto write_outputs = [&](int final_status, int token) __attribute__((always_inline)) {
        const int n = final_status ? 0 : n_acc;
        if (P.parent == nullptr) {
            write_chain(lane, P.rows, n, final_status != 0, my_tok, token, P.out_tokens + static_cast<size_t>(b) * (P.rows + 1));
        } else {
            write_path(lane, P.max_depth, final_status ? -1 : winner, n, my_par, my_dep, my_tok, final_status ? -1 : token,
                       P.path_nodes + static_cast<size_t>(b) * P.max_depth, P.out_tokens + static_cast<size_t>(b) * (P.max_depth + 1));
        }
        if (lane == 0) {
            P.out_len[b] = n;
            if (P.row_status) P.row_status[b] = final_status;
            if (failed) sequence_of_failed_call_done(P.ws);
        }
    };
    if constexpr (BY_K) {
        if (P.draw)
            clear_words(P.clear, P.clear16, (static_cast<long>(b) * gridDim.x + blockIdx.x) * kWarpWG + tid,
                        static_cast<long>(gridDim.x) * gridDim.y * kWarpWG);
    }
    if (s_st) {   // nothing will be drawn for this sequence
        if (tid == 0) P.thr[b] = neg_inf();
        if constexpr (BY_K) {
            if (P.draw && blockIdx.x == 0 && wave == 0) write_outputs(status, -1);
        }
        return;
    }
    const char* row = P.target + (static_cast<size_t>(b) * (P.rows + 1) + from) * static_cast<size_t>(P.V) * ES;

    constexpr int NK = SPLIT ? split_keep(BF16) : kWarpKeep;
    // this workgroup's share of the row
    const long share = SPLIT ? (P.nslots + gridDim.x - 1) / gridDim.x : P.nslots;
    const long sl_lo = SPLIT ? static_cast<long>(blockIdx.x) * share : 0;
    const long sl_hi = (sl_lo + share < P.nslots) ? sl_lo + share : P.nslots;
    bool whole = !SPLIT;   // SPLIT: the last workgroup passes over the whole row
    uint4 kept[KEEP ? NK : 1];
    if constexpr (KEEP) {
#pragma unroll
        for (int c = 0; c < NK; ++c) {
            const long sl = sl_lo + static_cast<long>(c) * kWarpWG + tid;
            kept[c] = load_slot<BF16, LD>(row, sl < sl_hi ? sl : P.nslots - 1, P.V);
        }
    }
    // one pass over the row: f(scaled logit, key, place in the row) for every entry
    auto for_slot = [&](const uint4& raw, long sl, auto&& f) __attribute__((always_inline)) {
        float z[VE];
        unpack<BF16>(raw, z);
#pragma unroll
        for (int e = 0; e < VE; ++e) {
            if (LD == LOAD_ALIGNED || sl * VE + e < P.V) {   // aligned rows have no ragged last slot
                const float sv = __fmul_rn(z[e], P.inv_temp);
                f(sv, ordered_key(sv), static_cast<int>(sl * VE + e));
            }
        }
    };
    auto for_each_at = [&](auto&& f) __attribute__((always_inline)) {
        if constexpr (KEEP) {
            if (!SPLIT || !whole) {
#pragma unroll
                for (int c = 0; c < NK; ++c) {
                    const long sl = sl_lo + static_cast<long>(c) * kWarpWG + tid;
                    // the copy is made opaque: what is derived from the kept words (scaled values, keys) would
                    // otherwise be hoisted out of the passes and kept as well, far beyond the register file
                    uint4 r = kept[c];
                    asm volatile("" : "+v"(r.x), "+v"(r.y), "+v"(r.z), "+v"(r.w));
                    if (sl < sl_hi) {
                        settle_slot<BF16, LD>(r, sl, P.V);
                        for_slot(r, sl, f);
                    }
                }
            }
        }
        if (!KEEP || (SPLIT && whole)) {
            constexpr int CH = 4;
            for (long base = 0; base < P.nslots; base += static_cast<long>(kWarpWG) * CH) {
                uint4 raw[CH];
#pragma unroll
                for (int c = 0; c < CH; ++c) {
                    const long sl = base + static_cast<long>(c) * kWarpWG + tid;
                    raw[c] = load_slot<BF16, LD>(row, sl < P.nslots ? sl : P.nslots - 1, P.V);
                }
#pragma unroll
                for (int c = 0; c < CH; ++c) {
                    const long sl = base + static_cast<long>(c) * kWarpWG + tid;
                    if (sl < P.nslots) {
                        settle_slot<BF16, LD>(raw[c], sl, P.V);
                        for_slot(raw[c], sl, f);
                    }
                }
            }
        }
    };
    auto for_each = [&](auto&& f) __attribute__((always_inline)) {
        for_each_at([&](float sv, unsigned key, int) __attribute__((always_inline)) { f(sv, key); });
    };
    // the row's maximum (s_max) and its smallest entry above -inf (s_min), from every thread's own
    auto block_range = [&](float m, float lo) __attribute__((always_inline)) {
        float neg = -lo;
        wave_max2(m, neg);
        __syncthreads();
        if (lane == 0) { s_red[wave] = m; s_red2[wave] = neg; }
        __syncthreads();
        if (wave == 0) {
            m = (lane < kWarpWG / 64) ? s_red[lane] : neg_inf();
            neg = (lane < kWarpWG / 64) ? s_red2[lane] : neg_inf();
            wave_max2(m, neg);
            if (lane == 0) { s_max = m; s_min = -neg; }
        }
        __syncthreads();
    };
    const bool want_k = BY_K || (!SPLIT && P.top_k > 0 && P.top_k < P.V), want_p = (SPLIT && !BY_K) || P.top_p < 1.0f;
    int bad = 0;   // P.draw: this thread has seen a NaN or +inf (or a logit that the temperature makes one)
    auto row_range = [&]() __attribute__((always_inline)) {
        float m = neg_inf(), lo = __builtin_inff();
        for_each([&](float sv, unsigned) {
            m = fmaxf(m, sv);
            lo = fminf(lo, (sv > neg_inf()) ? sv : __builtin_inff());
            if constexpr (BY_K) bad |= !(sv < __builtin_inff());
        });
        if (!BY_K || whole) block_range(m, lo);   // (under top-k nobody asks for the share's range)
        return m;   // this thread's maximum
    };
    // The need-th largest of n <= kCountKeys keys in LDS, or its digits down to bit `down_to` (the result is then the largest
    // multiple of 2^down_to with need keys at or above it): every wavefront holds all keys, 16 a lane, and in a round
    // tries the value that extends the digits found so far by its own number.
    auto count_select = [&](const unsigned* keys, int n, unsigned need, int down_to) __attribute__((always_inline)) -> unsigned {
        constexpr int PER = kCountKeys / 64;
        unsigned r[PER];
#pragma unroll
        for (int i = 0; i < PER; ++i) r[i] = (i * 64 + lane < n) ? keys[i * 64 + lane] : 0u;
        unsigned found = 0u;
        for (int shift = 28; shift >= down_to; shift -= 4) {
            const unsigned least = found | (static_cast<unsigned>(wave) << shift);
            unsigned count = 0u;
#pragma unroll
            for (int i = 0; i < PER; ++i) {
                if (i * 64 < n) count += static_cast<unsigned>(__popcll(__ballot(r[i] >= least)));
            }
            unsigned* const round = s_round[(shift >> 2) & 1];   // (the other one may still be read)
            if (lane == 0) round[wave] = count;
            __syncthreads();
            const unsigned long long enough = __ballot(round[lane & 15] >= need) & 0xFFFFull;   // (for all up to some number)
            found |= static_cast<unsigned>(enough ? 63 - __builtin_clzll(enough) : 0) << shift;
        }
        return found;
    };
    static_assert(kWarpWG / 64 == 16, "a digit of 4 bits a round");
    // Histogram additions of one thread, merged while consecutive entries fall in the same bin (the
    // leading digit of nearly every entry of a row is the same: adding them one by one would
    // serialise the whole workgroup on one LDS word).  s_hist takes the weights (1 per entry for
    // top-k), s_cnt the number of entries.
    struct Run { int bin; unsigned n; unsigned long long sum; };
    auto run_flush = [&](Run& r) __attribute__((always_inline)) {
        if (r.n) { atomicAdd(&s_hist[r.bin], r.sum); atomicAdd(&s_cnt[r.bin], r.n); }
        r.n = 0;
        r.sum = 0;
    };
    auto run_add = [&](Run& r, int bin, unsigned long long w) __attribute__((always_inline)) {
        if (bin != r.bin) { run_flush(r); r.bin = bin; }
        r.sum += w;
        r.n += 1;
    };
    // From the top: the digit at which the accumulated histogram reaches s_need; updates prefix and
    // need and leaves the number of entries that share the new prefix in s_match.  The 256 sums from
    // the top come from a parallel scan (a single thread walking the bins costs more than a pass
    // over the row); need_of(total), if given, first derives s_need from the histogram's total.  What is needed has been read by
    // all four wavefronts, and a barrier lies between, before the one that finds its bin writes the rest: a wavefront
    // that read the rest in its place could find a second bin, and the digits of both would end up in the prefix.
    struct AsNeeded {};   // (s_need as it stands)
    auto pick_from_top = [&](int shift, auto&& need_of) __attribute__((always_inline)) {
        constexpr bool DERIVED = !std::is_same_v<std::decay_t<decltype(need_of)>, AsNeeded>;
        __syncthreads();
        unsigned long long h = 0, v = 0;
        if (tid < 256) {
            h = s_hist[tid];
            v = h;
#pragma unroll
            for (int o = 1; o < 64; o <<= 1) {
                const unsigned long long x = __shfl_down(v, o);
                if (lane + o < 64) v += x;
            }
            if (lane == 0) s_wtot[wave] = v;
        }
        unsigned long long need = DERIVED ? 0ull : s_need;
        __syncthreads();
        if (tid < 256) {
            for (int w = wave + 1; w < 4; ++w) v += s_wtot[w];   // v = everything in bins >= tid
        }
        if constexpr (DERIVED) {
            if (tid == 0) need_of(v);
            __syncthreads();
            need = s_need;
            __syncthreads();
        }
        if (tid < 256) {
            const unsigned long long above = v - h;
            const bool here = (v >= need && above < need) || (tid == 0 && v < need);
            if (here) {
                s_prefix |= static_cast<unsigned>(tid) << shift;
                s_mask |= 255u << shift;
                s_need = need - above;
                s_match = s_cnt[tid];
            }
        }
        __syncthreads();
    };
    // Radix select from the top over an array of order-preserving keys in LDS, 8 bits a pass: the
    // smallest key whose entries, together with everything above them, weigh at least s_need.
    // wgt(sv, key) gives an entry's weight (0 = not taking part); first_total, called with the
    // total weight of the first histogram, may set s_need.  down_to: the last digit's shift (16: the upper half of
    // the key, a lower bound of it).
    // Digits in which all keys agree are theirs without a pass: a list's keys lie close together, and those of bfloat16 logits end in
    // zeros.  (A pass is six barriers.)
    auto lds_select = [&](const unsigned* keys, int n, auto&& wgt, auto&& first_total, int down_to = 0) __attribute__((always_inline)) {
        const unsigned first = keys[0];
        unsigned differ = 0u;
        for (int i = tid; i < n; i += kWarpWG) differ |= keys[i] ^ first;
        differ = wave_or(differ);
        if (tid == 0) s_match = 0u;
        __syncthreads();
        if (lane == 0 && differ) atomicOr(&s_match, differ);
        __syncthreads();
        differ = s_match;
        unsigned same = 0u;
#pragma unroll
        for (int shift = 0; shift < 32; shift += 8) same |= ((differ >> shift) & 255u) ? 0u : 255u << shift;
        if (tid == 0) { s_prefix = first & same & (~0u << down_to); s_mask = same & (~0u << down_to); }
        bool started = false;
        for (int shift = 24; shift >= down_to; shift -= 8) {
            if ((same >> shift) & 255u) continue;
            if (tid < 256) { s_hist[tid] = 0ull; s_cnt[tid] = 0u; }
            __syncthreads();
            const unsigned prefix = s_prefix, mask = s_mask;
            for (int i = tid; i < n; i += kWarpWG) {
                const unsigned key = keys[i];
                if ((key & mask) == prefix) {
                    const unsigned long long w = wgt(key_value(key), key);
                    if (w) {
                        const int bin = static_cast<int>((key >> shift) & 255u);
                        atomicAdd(&s_hist[bin], w);
                        atomicAdd(&s_cnt[bin], 1u);
                    }
                }
            }
            if (!started) pick_from_top(shift, first_total);
            else pick_from_top(shift, AsNeeded{});
            started = true;
        }
        __syncthreads();   // (no digit may have differed)
    };
    // The same select over the whole row (the general path): every digit is a pass over the row
    // until the entries that still share the prefix fit the list; then they are gathered there and
    // the remaining digits come from the list.
    auto row_select = [&](auto&& wgt, auto&& first_total) __attribute__((always_inline)) {
        if (tid == 0) { s_prefix = 0u; s_mask = 0u; }
        bool listed = false;
        for (int shift = 24; shift >= 0; shift -= 8) {
            if (tid < 256) { s_hist[tid] = 0ull; s_cnt[tid] = 0u; }
            __syncthreads();
            const unsigned prefix = s_prefix, mask = s_mask;
            if (listed) {
                const int nl = s_nlist;
                for (int i = tid; i < nl; i += kWarpWG) {
                    const unsigned key = s_lkey[i];
                    if ((key & mask) == prefix) {
                        const unsigned long long w = wgt(key_value(key), key);
                        if (w) {
                            const int bin = static_cast<int>((key >> shift) & 255u);
                            atomicAdd(&s_hist[bin], w);
                            atomicAdd(&s_cnt[bin], 1u);
                        }
                    }
                }
            } else {
                Run run{0, 0u, 0ull};
                for_each([&](float sv, unsigned key) {
                    if ((key & mask) == prefix) {
                        const unsigned long long w = wgt(sv, key);
                        if (w) run_add(run, static_cast<int>((key >> shift) & 255u), w);
                    }
                });
                run_flush(run);
            }
            if (shift == 24) pick_from_top(shift, first_total);
            else pick_from_top(shift, AsNeeded{});
            if (!listed && shift >= 16 && s_match <= static_cast<unsigned>(kWarpList)) {
                if (tid == 0) s_nlist = 0;
                __syncthreads();
                const unsigned prefix2 = s_prefix, mask2 = s_mask;
                for_each([&](float sv, unsigned key) {
                    if ((key & mask2) == prefix2 && wgt(sv, key)) {
                        const int at = atomicAdd(&s_nlist, 1);
                        if (at < kWarpList) s_lkey[at] = key;
                    }
                });
                __syncthreads();
                listed = true;
            }
        }
    };

    // The select over the whole row by value: every entry's weight goes to one of kWarpBins bins of equal
    // width below the row's maximum (the order of the bins is the order of the values, so the crossing lies in
    // the bin where the sum from the top crosses), the entries of that bin are gathered into the list,
    // and the list gives the exact key.  Three cheap passes over the row, where the select by digits
    // above needs one per digit with nearly all entries in a few bins (the leading digits are the
    // exponent).  The width follows the row's range, so that a row that temperature has flattened spreads as
    // well.  Nucleus 0.95 on 8 rows of 128256 bfloat16 entries: 164 -> 49 us for this kernel.  False if the crossing lies below the range (the last bin,
    // which keeps no sum of its own in LDS: masked entries would all queue there) or the list overflows
    // (a great many equal entries): the select by digits takes over.
    auto bin_select = [&](auto&& wgt, auto&& need_of) __attribute__((always_inline)) -> bool {
        static_assert(kWarpBins == 2 * kWarpWG, "two bins per thread in the scan");
        s_bins[tid] = 0ull;
        s_bins[tid + kWarpWG] = 0ull;
        if (tid == 0) { s_nlist = 0; s_bin = -1; }
        __syncthreads();
        const float top = s_max;
        const float scale = static_cast<float>(kWarpBins - 2) / fmaxf(fminf(top - s_min, kWarpRange), 1e-30f);
        auto bin_of = [&](float sv) __attribute__((always_inline)) -> int {
            return static_cast<int>(fminf(fmaxf((top - sv) * scale, 0.0f), static_cast<float>(kWarpBins - 1)));
        };
        unsigned long long tail = 0ull;
        for_each([&](float sv, unsigned key) {
            const unsigned long long w = wgt(sv, key);
            const int bin = bin_of(sv);
            if (bin == kWarpBins - 1) tail += w;
            else if (w) atomicAdd(&s_bins[bin], w);
        });
#pragma unroll
        for (int o = 32; o > 0; o >>= 1) tail += __shfl_xor(tail, o);
        __syncthreads();
        // running sums from the top, two bins per thread
        const unsigned long long h0 = s_bins[2 * tid], h1 = s_bins[2 * tid + 1];
        unsigned long long v = h0 + h1;
#pragma unroll
        for (int o = 1; o < 64; o <<= 1) {
            const unsigned long long x = __shfl_up(v, o);
            if (lane >= o) v += x;
        }
        if (lane == 63) { s_wsum[wave] = v; s_wtail[wave] = tail; }
        __syncthreads();
        unsigned long long above = v - h0 - h1, total = 0ull;
        for (int w = 0; w < kWarpWG / 64; ++w) {
            if (w < wave) above += s_wsum[w];
            total += s_wsum[w] + s_wtail[w];
        }
        const unsigned long long need = need_of(total);
        if (above < need && above + h0 >= need) { s_bin = 2 * tid; s_need = need - above; }
        if (above + h0 < need && above + h0 + h1 >= need) { s_bin = 2 * tid + 1; s_need = need - above - h0; }
        __syncthreads();
        const int chosen = s_bin;
        if (chosen < 0) return false;
        const Interval near = bin_interval(top, scale, chosen);
        for_each([&](float sv, unsigned key) {
            if (sv >= near.lo && sv <= near.hi && bin_of(sv) == chosen && wgt(sv, key)) {
                const int at = atomicAdd(&s_nlist, 1);
                if (at < kWarpList) s_lkey[at] = key;
            }
        });
        __syncthreads();
        const int nl = s_nlist;
        if (nl > kWarpList) return false;
        lds_select(s_lkey, nl, wgt, AsNeeded{});
        return true;
    };

    bool done_k = !want_k, done_p = !want_p;
    float t_k = neg_inf(), t_p = neg_inf();
    const float tmax = row_range();
    float cmax = s_max * kLog2e;
    auto one = [&](float, unsigned) __attribute__((always_inline)) -> unsigned long long { return 1ull; };
    // e^(s - max) in 2^-40 units; entries at -inf or below the top-k cut weigh nothing
    auto weight = [&](float sv, unsigned) __attribute__((always_inline)) -> unsigned long long {
        if (!(sv >= t_k)) return 0ull;
        // (two conversions to 32 bits, exact: a binary32 number has 24 significant ones)
        const float x = rintf(hw_exp2(fmaf(sv, kLog2e, -cmax)) * 0x1p40f);
        const unsigned hi = static_cast<unsigned>(x * 0x1p-32f);
        const unsigned lo = static_cast<unsigned>(fmaf(static_cast<float>(hi), -0x1p32f, x));
        return (static_cast<unsigned long long>(hi) << 32) | lo;
    };
    auto nucleus_need = [&](unsigned long long Z) __attribute__((always_inline)) -> unsigned long long {
        double need = static_cast<double>(P.top_p) * static_cast<double>(Z);
        unsigned long long n = static_cast<unsigned long long>(need);
        if (static_cast<double>(n) < need) ++n;
        return n ? n : 1ull;
    };
    auto first_k = [&](unsigned long long) __attribute__((always_inline)) -> unsigned long long { return static_cast<unsigned long long>(P.top_k); };

    // ---- any setting from the whole row: by value, or by digits where that does not settle it
    auto select_from_row = [&]() __attribute__((always_inline)) {
        if (!done_k) {
            if (!bin_select(one, first_k)) {
                __syncthreads();
                if (tid == 0) s_need = static_cast<unsigned long long>(P.top_k);
                __syncthreads();
                row_select(one, AsNeeded{});
            }
            t_k = key_value(s_prefix);
            __syncthreads();
        }
        if (!done_p) {
            if (!bin_select(weight, nucleus_need)) {
                __syncthreads();
                row_select(weight, [&](unsigned long long Z) { s_need = nucleus_need(Z); });
            }
            t_p = key_value(s_prefix);
        }
    };

    if constexpr (SPLIT) {
        unsigned* const line = P.ws.sdone + static_cast<size_t>(b) * kSdoneStride;
        unsigned* const count = line + 1;
        char* const area = P.area + static_cast<size_t>(b) * P.seq_bytes;
        const int g = static_cast<int>(blockIdx.x), W = static_cast<int>(gridDim.x);
        // everything this workgroup has stored is performed, then it counts itself: true for the last one
        auto count_self = [&](unsigned* at) __attribute__((always_inline)) -> bool {
            asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
            __syncthreads();
            if (tid == 0) s_bin = (__hip_atomic_fetch_add(at, 1u, __ATOMIC_RELAXED, AGENT) == static_cast<unsigned>(W) - 1u) ? 1 : 0;
            __syncthreads();
            const bool last = s_bin != 0;
            __syncthreads();   // (s_bin is used again)
            return last;
        };
        // this workgroup's keys (s_lkey, s_nlist) for whoever counts last: lists of cap keys, each behind its length
        auto leave_list = [&](unsigned* lists, int cap, unsigned* at) __attribute__((always_inline)) -> bool {
            const int left = s_nlist;
            for (int i = tid; i < left && i < cap; i += kWarpWG)
                __hip_atomic_store(lists + g * (cap + 1) + 1 + i, s_lkey[i], __ATOMIC_RELAXED, AGENT);
            if (tid == 0) __hip_atomic_store(lists + g * (cap + 1), static_cast<unsigned>(left), __ATOMIC_RELAXED, AGENT);
            return count_self(at);
        };
        // all lists into s_lkey: false if one was too long.  (A stretch of threads per list: all are read at once; at most
        // kSplitBytes / 4 <= kWarpList keys.)
        auto read_lists = [&](const unsigned* lists, int cap) __attribute__((always_inline)) -> bool {
            const int per = kWarpWG / W, w = tid / per, j0 = tid - w * per;
            const unsigned* const mine = lists + (w < W ? w : 0) * (cap + 1) + 1;
            unsigned key = __hip_atomic_load(mine + (j0 < cap ? j0 : 0), __ATOMIC_RELAXED, AGENT);
            int lens[kWarpShare], at0 = 0, my_n = 0, n = 0;
            bool fits = true;
#pragma unroll
            for (int q = 0; q < kWarpShare; ++q)
                lens[q] = static_cast<int>(__hip_atomic_load(lists + (q < W ? q : 0) * (cap + 1), __ATOMIC_RELAXED, AGENT));
#pragma unroll
            for (int q = 0; q < kWarpShare; ++q) {
                if (q >= W) break;
                fits &= lens[q] <= cap;
                if (q == w) { at0 = n; my_n = lens[q]; }
                n += lens[q];
            }
            if (!fits) return false;
            for (int j = j0; j < my_n; j += per) {
                if (j != j0) key = __hip_atomic_load(mine + j, __ATOMIC_RELAXED, AGENT);
                s_lkey[at0 + j] = key;
            }
            if (tid == 0) s_nlist = n;
            __syncthreads();
            return true;
        };
        if constexpr (BY_K) {
            // a list: its length, with the flag of an unusable logit, and the keys, or (P.draw) the length and pairs of key and
            // place in the row
            const int cap = P.list_keys;
            unsigned long long* const pairs = reinterpret_cast<unsigned long long*>(area);
            unsigned* const keys = reinterpret_cast<unsigned*>(area);
            unsigned* const s_place = reinterpret_cast<unsigned*>(s_bins);   // where in the row a key of s_lkey lies
            static_assert(sizeof(s_bins) >= kSplitKeys * 4 && kSplitKeys <= kWarpList, "the lists fit");
            const unsigned k = static_cast<unsigned>(P.top_k);
            s_tmax[tid] = ordered_key(tmax);
            if (tid == 0) s_nlist = 0;
            __syncthreads();
            const unsigned low = list_bound(count_select(s_tmax, kWarpWG, k, 16));   // (any bound with k entries at or above it)
            for_each_at([&](float, unsigned key, int place) {
                if (key >= low) {
                    const int at = atomicAdd(&s_nlist, 1);
                    if (at < cap) { s_lkey[at] = key; s_place[at] = static_cast<unsigned>(place); }
                }
            });
            const bool any_bad = __syncthreads_or(bad) != 0;
            const int left = s_nlist;
            const unsigned head_word = (any_bad ? 0x80000000u : 0u) | static_cast<unsigned>(left);
            if (P.draw) {
                unsigned long long* const at = pairs + g * (cap + 1);
                for (int i = tid; i < left && i < cap; i += kWarpWG) post64(at + 1 + i, (static_cast<unsigned long long>(s_lkey[i]) << 32) | s_place[i]);
                if (tid == 0) post64(at, head_word);
            } else {
                unsigned* const at = keys + g * (cap + 1);
                for (int i = tid; i < left && i < cap; i += kWarpWG) __hip_atomic_store(at + 1 + i, s_lkey[i], __ATOMIC_RELAXED, AGENT);
                if (tid == 0) __hip_atomic_store(at, head_word, __ATOMIC_RELAXED, AGENT);
            }
            if (!count_self(count)) return;
            // the lists one after the other into s_lkey and s_place, a stretch of threads each; an entry is asked for together
            // with the lengths, before it is known to be one
            const int per = kWarpWG / W, w = tid / per, j0 = tid - w * per;
            const int mine = (w < W ? w : 0) * (cap + 1) + 1;
            auto entry_at = [&](int j) __attribute__((always_inline)) -> unsigned long long {   // key, place
                if (P.draw) return read64(pairs + mine + j);
                return static_cast<unsigned long long>(__hip_atomic_load(keys + mine + j, __ATOMIC_RELAXED, AGENT)) << 32;
            };
            unsigned long long entry = entry_at(j0 < cap ? j0 : 0);
            int n = 0, at0 = 0, my_n = 0;
            bool fits = true, row_bad = false;
            unsigned head[kWarpShare];   // (all of them asked for in one go)
#pragma unroll
            for (int q = 0; q < kWarpShare; ++q) {
                const int from_list = (q < W ? q : 0) * (cap + 1);
                head[q] = P.draw ? static_cast<unsigned>(read64(pairs + from_list)) : __hip_atomic_load(keys + from_list, __ATOMIC_RELAXED, AGENT);
            }
#pragma unroll
            for (int q = 0; q < kWarpShare; ++q) {
                if (q >= W) break;
                const int len = static_cast<int>(head[q] & 0x7FFFFFFFu);
                fits &= len <= cap;
                row_bad |= (head[q] >> 31) != 0;
                if (q == w) { at0 = n; my_n = len; }
                n += len;
            }
            whole = true;
            float cut = 0.0f;
            if (fits) {
                for (int j = j0; j < my_n; j += per) {
                    if (j != j0) entry = entry_at(j);
                    s_lkey[at0 + j] = static_cast<unsigned>(entry >> 32);
                    s_place[at0 + j] = static_cast<unsigned>(entry);
                }
                __syncthreads();
                bool have_p = !want_p;
                if (n <= kCountKeys) {
                    if (tid == 0) { s_nlist = 0; s_match = 0u; s_prefix = ~0u; }
                    if (tid <= kRankKeys) s_above[tid] = 0ull;
                    t_k = key_value(count_select(s_lkey, n, k, 0));
                    if (want_p) {
                        // what top-k keeps, with its weights: an entry is kept if those above it weigh less than is needed
                        const unsigned key = tid < n ? s_lkey[tid] : 0u;
                        const float sv = key_value(key), m = wave_max(sv);   // (0: a NaN, which max() drops)
                        if (lane == 0 && m == m) atomicMax(&s_match, ordered_key(m));
                        __syncthreads();
                        cmax = key_value(s_match) * kLog2e;
                        if (sv >= t_k) {
                            const int at = atomicAdd(&s_nlist, 1);
                            if (at < kRankKeys) { s_tmax[at] = key; s_hist[at] = weight(sv, key); }
                        }
                        __syncthreads();
                        const int kept_k = s_nlist;
                        have_p = kept_k <= kRankKeys;
                        if (have_p) {
                            // (all pairs: 64 entries a wavefront, and a sixteenth of those they are compared with)
                            unsigned long long all = 0ull;
                            for (int i0 = 0; i0 < kept_k; i0 += 64) {
                                const int i = i0 + lane;
                                const unsigned own = s_tmax[i < kept_k ? i : 0];
                                unsigned long long above = 0ull;
                                for (int j = wave; j < kept_k; j += kWarpWG / 64) {
                                    const unsigned long long w = s_hist[j];
                                    if (i0 == 0) all += w;
                                    above += s_tmax[j] > own ? w : 0ull;
                                }
                                if (i < kept_k && above) atomicAdd(&s_above[i], above);
                            }
                            if (lane == 0) atomicAdd(&s_above[kRankKeys], all);
                            __syncthreads();
                            if (tid < kept_k && s_above[tid] < nucleus_need(s_above[kRankKeys])) atomicMin(&s_prefix, s_tmax[tid]);
                            __syncthreads();
                            t_p = key_value(s_prefix);
                        }
                    }
                } else {
                    if (tid == 0) s_need = static_cast<unsigned long long>(P.top_k);
                    unsigned top = 0u;
                    for (int i = tid; i < n; i += kWarpWG) top = s_lkey[i] > top ? s_lkey[i] : top;
                    block_range(key_value(top), 0.0f);   // (a thread without a key brings the NaN of key 0, which max() drops)
                    cmax = s_max * kLog2e;
                    lds_select(s_lkey, n, one, AsNeeded{});
                    t_k = key_value(s_prefix);
                }
                if (!have_p) {
                    __syncthreads();
                    lds_select(s_lkey, n, weight, [&](unsigned long long Z) { s_need = nucleus_need(Z); });
                    t_p = key_value(s_prefix);
                }
                cut = fmaxf(t_k, t_p);
            } else {
                // too long a list (a great many equal entries): the whole row, by this workgroup alone
                row_range();
                cmax = s_max * kLog2e;
                select_from_row();
                cut = fmaxf(t_k, t_p);
            }
            if (tid == 0) P.thr[b] = cut;
            if (!P.draw) return;
            Best best{neg_inf(), 0x7FFFFFFF};
            if (fits) {
                for (int i = tid; i < n; i += kWarpWG) {
                    const float sv = key_value(s_lkey[i]);
                    if (!(sv >= cut)) continue;
                    const unsigned place = s_place[i];
                    const U4 v = philox4x32_10(place >> 2, static_cast<unsigned>(b), P.off_lo, P.off_hi, P.seed_lo, P.seed_hi);
                    const unsigned word = (place & 3) == 0 ? v.x : (place & 3) == 1 ? v.y : (place & 3) == 2 ? v.z : v.w;
                    best = better(best, Best{__fadd_rn(sv, gumbel(word)), static_cast<int>(place)});
                }
            } else {
                if (tid == 0) s_score = score_key(-FLT_MAX);
                __syncthreads();
                const DrawArgs A{P.V, FSD_SAMPLE, P.seed_lo, P.seed_hi, P.off_lo, P.off_hi, true, cut, P.inv_temp};
                draw_share<BF16, LD, false, 8, kWarpWG>(A, b, row, false, nullptr, 0.0f, 0.0f, DrawChain{nullptr, 0, 0, nullptr}, 0, P.nslots, tid,
                                                        &s_score, best, bad);
                row_bad |= __syncthreads_or(bad) != 0;
            }
            best = wave_best(best);
            __syncthreads();
            if (lane == 0) { s_red[wave] = best.score; s_cnt[wave] = static_cast<unsigned>(best.idx); }
            __syncthreads();
            if (wave == 0) {
                const int from_wave = lane < kWarpWG / 64 ? lane : 0;
                best = wave_best(Best{s_red[from_wave], static_cast<int>(s_cnt[from_wave])});
                const bool none = best.idx == 0x7FFFFFFF || best.score == neg_inf();
                write_outputs((row_bad || none) ? FSD_ROW_NONFINITE : 0, best.idx);
            }
            return;
        } else {
            unsigned long long* const bins = reinterpret_cast<unsigned long long*>(area);
            unsigned long long* const words = reinterpret_cast<unsigned long long*>(line + 2);
            // this workgroup's part of the histogram is cleared before its word is posted
            for (int i = g * kSplitBins / W + tid; i < (g + 1) * kSplitBins / W; i += kWarpWG)
                __hip_atomic_store(bins + i, 0ull, __ATOMIC_RELAXED, AGENT);
            asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
            s_bins[tid] = 0ull;
            __syncthreads();
            if (tid == 0) post64(words + g, pack2(s_max, -s_min));
            if (wave == 0) {
                unsigned long long v = 1ull;
                for (unsigned polls = 0;; ++polls) {
                    v = read64(words + (lane < W ? lane : 0));
                    if (!__any(v == 0ull) || polls >= P.spin_limit) break;
                    __builtin_amdgcn_s_sleep(1);
                }
                const bool missing = __any(v == 0ull) != 0;
                float m = lo_f(v), neg = hi_f(v);
                wave_max2(m, neg);
                if (lane == 0) { s_max = m; s_min = -neg; s_bin = missing ? 1 : 0; }
            }
            __syncthreads();
            if (s_bin != 0) {   // a workgroup of this sequence never posted: the call reports it
                if (tid == 0) { flag_failure(P.ws); P.thr[b] = neg_inf(); }
                return;
            }
            cmax = s_max * kLog2e;
            const float top = s_max;
            const float scale = static_cast<float>(kSplitBins - 2) / fmaxf(fminf(top - s_min, kWarpRange), 1e-30f);
            auto bin_of = [&](float sv) __attribute__((always_inline)) -> int {
                return static_cast<int>(fminf(fmaxf((top - sv) * scale, 0.0f), static_cast<float>(kSplitBins - 1)));
            };
            unsigned long long tail = 0ull;   // (the last bin: see bin_select)
            for_each([&](float sv, unsigned key) {
                const unsigned long long w = weight(sv, key);
                const int bin = bin_of(sv);
                if (bin == kSplitBins - 1) tail += w;
                else if (w) atomicAdd(&s_bins[bin], w);
            });
#pragma unroll
            for (int o = 32; o > 0; o >>= 1) tail += __shfl_xor(tail, o);
            if (lane == 0 && tail) atomicAdd(&s_bins[kSplitBins - 1], tail);
            __syncthreads();
            const unsigned long long mine = s_bins[tid];
            if (mine) (void)__hip_atomic_fetch_add(bins + tid, mine, __ATOMIC_RELAXED, AGENT);
            if (!count_self(count)) {
                if (tid == 0) {
                    bool all = false;
                    for (unsigned polls = 0;; ++polls) {
                        all = __hip_atomic_load(count, __ATOMIC_RELAXED, AGENT) >= static_cast<unsigned>(W);
                        if (all || polls >= P.spin_limit) break;
                        __builtin_amdgcn_s_sleep(1);
                    }
                    s_bin = all ? 0 : 1;
                }
                __syncthreads();
                if (s_bin != 0) {
                    if (tid == 0) { flag_failure(P.ws); P.thr[b] = neg_inf(); }
                    return;
                }
                __syncthreads();   // (s_bin is used again)
            }
            // running sums from the top, one bin per thread
            const unsigned long long h = read64(bins + tid);
            unsigned long long v = h;
#pragma unroll
            for (int o = 1; o < 64; o <<= 1) {
                const unsigned long long x = __shfl_up(v, o);
                if (lane >= o) v += x;
            }
            if (lane == 63) s_wsum[wave] = v;
            if (tid == 0) { s_nlist = 0; s_bin = -1; }
            __syncthreads();
            unsigned long long above = v - h, total = 0ull;
            for (int w = 0; w < kWarpWG / 64; ++w) {
                if (w < wave) above += s_wsum[w];
                total += s_wsum[w];
            }
            const unsigned long long need = nucleus_need(total);
            if (tid < kSplitBins - 1 && above < need && above + h >= need) { s_bin = tid; s_need = need - above; }
            __syncthreads();
            const int chosen = s_bin;
            auto gather = [&]() __attribute__((always_inline)) {
                const Interval near = bin_interval(top, scale, chosen);
                for_each([&](float sv, unsigned key) {
                    if (sv >= near.lo && sv <= near.hi && bin_of(sv) == chosen && weight(sv, key)) {
                        const int at = atomicAdd(&s_nlist, 1);
                        if (at < kWarpList) s_lkey[at] = key;
                    }
                });
                __syncthreads();
            };
            // (behind the histogram: what is left of the sequence's memory)
            unsigned* const lists = reinterpret_cast<unsigned*>(bins + kSplitBins);
            const int cap = static_cast<int>((kSplitBytes - kSplitBins * 8) / 4) / W - 1;
            if (chosen >= 0) gather();
            if (!leave_list(lists, cap, line + 2 + 2 * kWarpShare)) return;
            if (chosen >= 0) {
                if (!read_lists(lists, cap)) {
                    whole = true;
                    if (tid == 0) s_nlist = 0;
                    __syncthreads();
                    gather();
                }
                const int nl = s_nlist;
                if (nl <= kWarpList) {
                    lds_select(s_lkey, nl, weight, AsNeeded{});
                    t_p = key_value(s_prefix);
                    done_p = true;
                }
            }
            if (done_p) {
                if (tid == 0) P.thr[b] = t_p;
                return;
            }
            whole = true;
            __syncthreads();
        }
    }

    // ---- the short way of a small top-k.  Every thread has noted the largest entry it saw; the k-th
    // largest of these 1024 maxima, L, has at least k entries of the row at or above it, so the k-th
    // largest entry is one of the entries >= L, and there are few of those (the entries are dealt to the
    // threads without regard to their values): they are gathered in one more pass and everything else
    // happens in LDS.  If the list overflows (many equal entries), the selects over the row take over.
    if (!SPLIT && want_k && P.top_k <= kWarpFastK) {
        s_tmax[tid] = ordered_key(tmax);
        if (tid == 0) { s_need = static_cast<unsigned long long>(P.top_k); s_nlist = 0; }
        __syncthreads();
        lds_select(s_tmax, kWarpWG, one, AsNeeded{}, 16);   // (any bound with k entries at or above it)
        const unsigned low = list_bound(s_prefix);   // at most the key of L
        for_each([&](float, unsigned key) {
            if (key >= low) {
                const int at = atomicAdd(&s_nlist, 1);
                if (at < kWarpList) s_lkey[at] = key;
            }
        });
        __syncthreads();
        const int nl = s_nlist;
        if (nl <= kWarpList) {
            if (tid == 0) s_need = static_cast<unsigned long long>(P.top_k);
            __syncthreads();
            lds_select(s_lkey, nl, one, AsNeeded{});
            t_k = key_value(s_prefix);
            done_k = true;
            __syncthreads();
            if (want_p) {   // everything top-k kept is in the list
                lds_select(s_lkey, nl, weight, [&](unsigned long long Z) { s_need = nucleus_need(Z); });
                t_p = key_value(s_prefix);
                done_p = true;
            }
        }
        __syncthreads();
    }

    select_from_row();
    if (tid == 0) P.thr[b] = fmaxf(t_k, t_p);
}

}  // namespace

#endif  // FSD_CSRC_WARP_SELECT_H_
