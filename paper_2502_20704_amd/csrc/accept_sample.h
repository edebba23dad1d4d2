// Acceptance (chain prefix, tree path, strict SD, reducible FSD) and the Gumbel-max draw.
// Part of libfsd (gfx950); included by fsd_kernels.hip, which holds the host side and the C ABI.
#ifndef FSD_CSRC_ACCEPT_SAMPLE_H_
#define FSD_CSRC_ACCEPT_SAMPLE_H_

#include "device_common.h"

namespace {

// ------------------------------------------------------------------------------------------
// kernel 2: acceptance + extra token

struct SampleParams {
    const char* target;
    const char* draft;        // strict SD only
    const int32_t* tokens;    // cand [B,K] or node_tokens [B,N]
    const int32_t* parent;    // tree only
    int rows;                 // K or N
    int max_depth;            // tree only
    long V;
    long nslots;
    int sps;                  // slots per sampler workgroup
    int GS;
    float T;
    int mode;
    unsigned seed_lo, seed_hi, off_lo, off_hi;
    int32_t* out_len;
    int32_t* out_tokens;
    int32_t* path_nodes;      // tree only
    int32_t* row_status;      // optional
    int cut;                  // warpers: the scale and the threshold below apply (FSD_SAMPLE only)
    const float* thr;         // optional [B]: warpers, smallest kept scaled logit of the sampled row (nullptr: all are kept)
    float inv_temp;           // warpers: binary32(1 / temperature), 1 otherwise
    uint4* clear;             // words of the reduction that count by the call's number (its arrival slots, see pair_kernel.h; the
    long clear16;             // words of a captured small_call), in 16-byte units: they go back to zero here
    Ws ws;
};

struct Best { float score; int idx; };

__device__ __forceinline__ Best better(Best a, Best b) {
    return (b.score > a.score || (b.score == a.score && b.idx < a.idx)) ? b : a;
}
// the best of the wavefront's 64: the maximum score, then the lowest index that has it (scores are never NaN)
__device__ __forceinline__ Best wave_best(Best v) {
    const float top = wave_max(v.score);
    return Best{top, wave_min(v.score == top ? v.idx : 0x7FFFFFFF)};
}

// what a draw needs beside the row: cut = the warpers' scale and threshold apply (FSD_SAMPLE only)
struct DrawArgs {
    long V;
    int mode;
    unsigned seed_lo, seed_hi, off_lo, off_hi;
    bool cut;
    float thr_b, inv_temp;
};
// strict SD on a tree: the rejected siblings' draft rows that shape the residual (their rows of the sequence's
// draft tensor, 1 / normalisers and log2-sum-exp2 values, one after the other in LDS)
struct DrawChain { const char* draft; int rows, n; const int* s; };

// The score a workgroup has seen so far, shared by its wavefronts through LDS as an order-preserving integer: the
// winner of the sequence reaches it.  (Read without any ordering: whatever value is seen is a score of this row.)
__device__ __forceinline__ unsigned score_key(float x) {
    const unsigned u = __float_as_uint(x);
    return (u & 0x80000000u) ? ~u : (u | 0x80000000u);
}
__device__ __forceinline__ float score_of_key(unsigned k) {
    return __uint_as_float((k & 0x80000000u) ? (k & 0x7FFFFFFFu) : ~k);
}
__device__ __forceinline__ float max3_nan(float a, float b, float c) {   // the maximum, or NaN if any of the three is
    float r;
    asm("v_maximum3_f32 %0, %1, %2, %3" : "=v"(r) : "v"(a), "v"(b), "v"(c));
    return r;
}

// The best score over slots [s0, s1) of the row, dealt to the workgroup's threads: of the row's entries or, with
// `residual`, of the positive part of p - q.  bad: a NaN or +inf logit was seen.  s_thr: the workgroup's shared score.
// STRIDE: the workgroup's threads.
//
// What bounds it: vector-ALU issue, most of it the random numbers (ten rounds of two 64-bit products per four entries);
// in small calls the chain from the row's first load to its last score.  Beside the random numbers an entry costs a
// bound of its score, one logarithm; only a wavefront with an entry that can still win does more.
// A lane takes NE = 8 entries a round (16 cost more registers than the loads
// in flight return: 64 rows of 128256 bfloat16 entries, before the bounds below: 14.8 us with either, 16 rows 8.2 with 8 and 9.4 with 16, 64 rows
// under top-k 10.6 and 12.2; 256 rows of 151936 binary32 entries 48.7 with 4 and 45.3 with 8) and requests the next
// round's rows, the draft's too, before it works on this one's.  (The residual's draw used to score the row's own
// entries along with it, for the case that no entry has any positive part; that case is now a second pass of the last
// workgroup.  With the earlier request of the draft row: strict SD on 64 rows of 128256 bfloat16 entries 23.1 -> 20.0 us.)
template <bool BF16, int LD, bool TREESD, int NE, int STRIDE = kWG>
__device__ __forceinline__ void draw_share(const DrawArgs& A, int b, const char* trow, bool residual, const char* drow,
                                           float lt, float ld, [[maybe_unused]] const DrawChain& C, long s0, long s1, int tid,
                                           unsigned* s_thr, Best& best, int& bad) {
    constexpr int VE = Slot<BF16>::VE;
    [[maybe_unused]] constexpr int ES = BF16 ? 2 : 4;
    constexpr int NS = NE / VE;
    // a score the winner is known to reach (see the bounds below), from the lowest finite one up: an entry
    // without mass, masked or cut off by the warpers, stays below
    float thr = -FLT_MAX;
    // a lane without a slot of its own re-reads the last one; its entries leave the draw
    auto request = [&](const char* row, long s, uint4 (&raw)[NS]) __attribute__((always_inline)) {
#pragma unroll
        for (int k = 0; k < NS; ++k) raw[k] = load_slot<BF16, LD>(row, (s + k * STRIDE < s1) ? s + k * STRIDE : s1 - 1, A.V);
    };
    auto entries = [&](uint4 (&raw)[NS], long s, float (&z)[NE]) __attribute__((always_inline)) {
#pragma unroll
        for (int k = 0; k < NS; ++k) {
            settle_slot<BF16, LD>(raw[k], (s + k * STRIDE < s1) ? s + k * STRIDE : s1 - 1, A.V);
            unpack<BF16>(raw[k], z + k * VE);
        }
    };
    // ln of the residual's entries (-inf where it has no mass) from the row's logits
    auto residual_of = [&](float (&z)[NE], [[maybe_unused]] uint4 (&rawd)[NS], long s) __attribute__((always_inline)) {
        float r[NE];
#pragma unroll
        for (int e = 0; e < NE; ++e) r[e] = hw_exp2(fmaf(z[e], kLog2e, -lt));
        if constexpr (TREESD) {
            // strict SD on a tree: p after the chain's rejections, minus the last draft row
            const int* ch = C.s;
            const float* iz = reinterpret_cast<const float*>(C.s + C.rows);
            const float* ldv = reinterpret_cast<const float*>(C.s + 2 * C.rows);
            for (int m = 0; m < C.n; ++m) {
                uint4 raw[NS];
                float zd[NE];
                request(C.draft + static_cast<size_t>(ch[m]) * static_cast<size_t>(A.V) * ES, s, raw);
                entries(raw, s, zd);
                const float ldm = ldv[m];
                if (m + 1 < C.n) {
                    const float izm = iz[m];
#pragma unroll
                    for (int e = 0; e < NE; ++e) r[e] = fmaxf(r[e] - hw_exp2(fmaf(zd[e], kLog2e, -ldm)), 0.0f) * izm;
                } else {
#pragma unroll
                    for (int e = 0; e < NE; ++e) r[e] = r[e] - hw_exp2(fmaf(zd[e], kLog2e, -ldm));
                }
            }
        } else {
            float zd[NE];
            entries(rawd, s, zd);
#pragma unroll
            for (int e = 0; e < NE; ++e) r[e] = r[e] - hw_exp2(fmaf(zd[e], kLog2e, -ld));
        }
#pragma unroll
        for (int e = 0; e < NE; ++e) z[e] = (r[e] > 0.0f) ? hw_log2(r[e]) * static_cast<float>(kLn2) : neg_inf();
    };
    // What a residual's score is bounded with before it is formed: its entry is at most p times the chain's factors, and
    // ln p is the exponential's own argument.  The constant covers the rounding of the exponential and the logarithm.
    float over = 2e-3f;
    if constexpr (TREESD) {
        if (residual) {
            const float* iz = reinterpret_cast<const float*>(C.s + C.rows);
            for (int m = 0; m + 1 < C.n; ++m) over = fmaf(hw_log2(iz[m]), static_cast<float>(kLn2), over);
        }
    }
    uint4 next[NS], nextd[NS];
    request(trow, s0 + tid, next);
    const bool pair = !TREESD && residual;
    if (pair) request(drow, s0 + tid, nextd);
    // The trip count is the same for every lane (the thresholds are wavefront reductions), but not for every
    // wavefront: one without a slot of its own in the last round leaves, where the random numbers of lanes that have
    // nothing to draw would cost the others' issue slots (128 rows of 35456 bfloat16 entries, whole call: 33.4 us with them, 32.2 without).
    const long before = static_cast<long>(__builtin_amdgcn_readfirstlane(tid >> 6)) * 64;   // this wavefront's first slot of a round
    for (long sb = s0; sb + before < s1; sb += NS * STRIDE) {
        const long s = sb + tid;
        float z[NE];   // what is scored: the logits, or ln of the residual's entries
        uint4 raw[NS], rawd[NS];
#pragma unroll
        for (int k = 0; k < NS; ++k) { raw[k] = next[k]; rawd[k] = nextd[k]; }
        if (sb + NS * STRIDE < s1) {
            request(trow, s + NS * STRIDE, next);
            if (pair) request(drow, s + NS * STRIDE, nextd);
        }
        entries(raw, s, z);
        if (A.cut) {
            // temperature, then the kept set of top-k / top-p: everything else leaves the draw
            bool any_kept = false;
#pragma unroll
            for (int e = 0; e < NE; ++e) {
                bad |= !(z[e] < __builtin_inff());
                const float sv = __fmul_rn(z[e], A.inv_temp);
                const bool keep = sv >= A.thr_b;
                z[e] = keep ? sv : neg_inf();
                any_kept |= keep;
            }
            // A wavefront without a kept entry has nothing to draw: no random numbers are formed for it.
            // (Top-k keeps a handful of a row's entries: nearly every wavefront leaves here.  Before, such
            // a wavefront had no score to reach and evaluated all its variates.  C2's shape with
            // temperature 0.7, top-k 50, top-p 0.9: 33.0 -> 10.6 us for this kernel.)
            if (!__any(any_kept)) continue;
        }
        if (sb + before + 63 + (NS - 1) * STRIDE >= s1) {   // some lane lacks a slot
            asm volatile("");   // stays a branch
#pragma unroll
            for (int k = 0; k < NS; ++k) {
                if (s + k * STRIDE >= s1) {
#pragma unroll
                    for (int e = 0; e < VE; ++e) z[k * VE + e] = neg_inf();
                }
            }
        }
        auto index_of = [&](int e) __attribute__((always_inline)) { return static_cast<int>((s + (e / VE) * STRIDE) * VE + e % VE); };
        if (A.mode == FSD_SAMPLE) {
            // Bounds of a variate G = -ln(-ln u) from x = 1 - u, which is exact in binary32: -ln u lies above x, so
            //     G <= -ln x,    and    G >= -ln x - 2.82 x
            // (-ln x - G is convex in x, 0 at 0 and at most 2.8116 at the largest x).  1e-3 covers the rounding of
            // the hardware logarithm and of the variate's own routine by a wide margin.  An entry whose upper bound
            // stays below a score the winner must reach cannot be the argmax: its variate, two exact-operation
            // logarithms, is never evaluated.  The largest lower bound of a score in the wavefront is such a score, and so
            // is the best one any wavefront of the workgroup has seen.  (The bounds used to be a binade wide, from the
            // position of the leading one of x: nearly every round then had entries to evaluate, which cost two thirds of
            // a round; and a residual's entries were formed, three transcendental instructions each, before any bound.
            // This kernel: 64 rows of 128256 bfloat16 entries 15.0 -> 13.5 us, strict SD on them 20.2 -> 18.3, 256 rows
            // of 151936 binary32 entries 44.2 -> 35.0.)
            float gub[NE], ub[NE];
            unsigned w[NE];
#pragma unroll
            for (int q = 0; q < NE / 4; ++q) {
                // (a last round whose second slots this wavefront does not have, in binary32: no numbers)
                if (q * 4 / VE > 0 && sb + before + (q * 4 / VE) * STRIDE >= s1) {
                    w[q * 4 + 0] = w[q * 4 + 1] = w[q * 4 + 2] = w[q * 4 + 3] = 0u;
                    continue;
                }
                const U4 r = philox4x32_10(static_cast<unsigned>(index_of(4 * q)) >> 2, static_cast<unsigned>(b), A.off_lo,
                                           A.off_hi, A.seed_lo, A.seed_hi);
                w[q * 4 + 0] = r.x; w[q * 4 + 1] = r.y; w[q * 4 + 2] = r.z; w[q * 4 + 3] = r.w;
            }
            // (1 - u) = (2^24 - 1 - 2 (w >> 9)) 2^-24: both operations are exact
            auto x_of = [&](unsigned word) __attribute__((always_inline)) {
                return fmaf(static_cast<float>(word >> 9), -0x1p-23f, 1.0f - 0x1p-24f);
            };
#pragma unroll
            for (int e = 0; e < NE; ++e) {
                gub[e] = fmaf(hw_log2(x_of(w[e])), -0x1.62e43p-1f, 1e-3f);
                ub[e] = (residual ? fmaf(fmaf(z[e], kLog2e, -lt), static_cast<float>(kLn2), over) : z[e]) + gub[e];
            }
            float top = ub[0];   // (NaN if any is: a NaN logit goes on to be found)
#pragma unroll
            for (int e = 1; e + 1 < NE; e += 2) top = max3_nan(top, ub[e], ub[e + 1]);
            top = max3_nan(top, ub[NE - 1], ub[NE - 1]);
            thr = fmaxf(thr, score_of_key(__hip_atomic_load(s_thr, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP)));
            if (!__any(!(top < thr))) continue;
            if (residual) {
                residual_of(z, rawd, s);
#pragma unroll
                for (int e = 0; e < NE; ++e) ub[e] = __fadd_rn(z[e], gub[e]);
            }
            float lo = neg_inf();
#pragma unroll
            for (int e = 0; e < NE; ++e)   // (max() drops the NaN of a NaN logit)
                lo = fmaxf(lo, __fadd_rn(z[e], gub[e] + fmaf(x_of(w[e]), -2.82f, -2e-3f)));
            thr = fmaxf(thr, wave_max(lo));
            // The entries that are left, at most a few per wavefront: every lane works through its own,
            // lowest index first (one pass of the loop serves one entry of every lane that has any).
            unsigned todo = 0;
#pragma unroll
            for (int e = 0; e < NE; ++e) todo |= !(ub[e] < thr) ? (1u << e) : 0u;
            while (__any(todo != 0)) {
                if (todo != 0) {
                    const int e = __builtin_ctz(todo);
                    todo &= todo - 1;
                    float zz = z[0];
                    unsigned ww = w[0];
#pragma unroll
                    for (int i = 1; i < NE; ++i) {
                        zz = (e == i) ? z[i] : zz;
                        ww = (e == i) ? w[i] : ww;
                    }
                    bad |= !(zz < __builtin_inff());   // (a NaN or +inf logit is never below a threshold)
                    const float score = __fadd_rn(zz, gumbel(ww));
                    if (score > best.score) best = Best{score, index_of(e)};
                }
            }
            const float seen = wave_max(best.score);
            thr = fmaxf(thr, seen);
            if ((tid & 63) == 0) (void)__hip_atomic_fetch_max(s_thr, score_key(thr), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
        } else {
            if (residual) {
                residual_of(z, rawd, s);
            } else {
#pragma unroll
                for (int e = 0; e < NE; ++e) bad |= !(z[e] < __builtin_inff());
            }
#pragma unroll
            for (int e = 0; e < NE; ++e) {
                if (z[e] > best.score) best = Best{z[e], index_of(e)};
            }
        }
    }
}

// The tree rule over at most 64 nodes, one per lane (the same in every lane but my_dep): depth and node of the deepest
// accepted path, status bits of a malformed tree.  my_par: an invalid parent becomes -1.
struct TreePick { int n, winner, my_dep, status; };
__device__ __forceinline__ TreePick pick_path(int lane, int rows, int max_depth, int& my_par, bool accepted) {
    TreePick r{0, -1, 0, 0};
    const bool mine = lane < rows;
    const bool bad_parent = my_par < -1 || my_par >= lane;
    if (__any(mine && bad_parent)) r.status |= FSD_ROW_BAD_PARENT;
    if (bad_parent) my_par = -1;
    // pointer jumping: after r rounds `at` names the 2^r-th ancestor, the rest covers that stretch:
    // ancestor + 1 (8 bits), depth (8 bits), accepted
    int at = (my_par + 1) | (1 << 8) | (accepted ? 1 << 16 : 0);
    for (int span = 1; span < rows; span <<= 1) {
        const int up = at & 0xFF, far = __shfl(at, up ? up - 1 : 0);
        if (up) at = (far & 0xFF) | ((at & 0xFF00) + (far & 0xFF00)) | (at & far & (1 << 16));
    }
    r.my_dep = (at >> 8) & 0xFF;
    const bool good = mine && (at >> 16);
    if (__any(mine && r.my_dep > max_depth)) r.status |= FSD_ROW_TOO_DEEP;
    const float deepest = wave_max(good ? static_cast<float>(r.my_dep) : 0.0f);   // deepest, then lowest index
    if (deepest > 0.0f) {
        r.n = static_cast<int>(deepest);
        r.winner = static_cast<int>(__builtin_ctzll(__ballot(good && r.my_dep == r.n)));
    }
    return r;
}
// a path of n nodes that ends at `winner` (-1: none) and the token behind it, a node per lane
__device__ __forceinline__ void write_path(int lane, int max_depth, int winner, int n, int my_par, int my_dep, int my_tok, int token,
                                           int32_t* pn, int32_t* out) {
    // the nodes of the path are the winner and its ancestors; a node's place is its depth
    unsigned long long path = 0;
    for (int j = winner; j >= 0; j = __builtin_amdgcn_readlane(my_par, j)) path |= 1ull << j;
    for (int i = n + lane; i < max_depth; i += 64) pn[i] = -1;
    for (int i = n + lane; i <= max_depth; i += 64) out[i] = i == n ? token : -1;
    if ((path >> lane) & 1) { pn[my_dep - 1] = lane; out[my_dep - 1] = my_tok; }
}

// the tokens of a chain of at most 64 positions, one a lane: n accepted ones, the drawn token, padding (all of it padding
// if the sequence has failed)
__device__ __forceinline__ void write_chain(int lane, int rows, int n, bool failed, int my_tok, int token, int32_t* out) {
    for (int i = lane; i <= rows; i += 64) out[i] = (failed || i > n) ? -1 : (i == n) ? token : my_tok;
}

// A workgroup's share of a sequence's draw in one word that says by itself whether it has arrived: score, then the flag
// of an unusable logit and the index plus one (all ones: no entry).  Never zero.
__device__ __forceinline__ unsigned long long share_word(Best m, int bad) {
    const unsigned at = m.idx == 0x7FFFFFFF ? 0x7FFFFFFFu : static_cast<unsigned>(m.idx) + 1u;
    return (static_cast<unsigned long long>(__float_as_uint(m.score)) << 32) | (bad ? 0x80000000u : 0u) | at;
}
__device__ __forceinline__ Best share_best(unsigned long long w) {
    const unsigned at = static_cast<unsigned>(w) & 0x7FFFFFFFu;
    return Best{__uint_as_float(static_cast<unsigned>(w >> 32)), at == 0x7FFFFFFFu ? 0x7FFFFFFF : static_cast<int>(at) - 1};
}
// A call that has failed, by the one workgroup of a sequence that writes its outputs, once it has: the last sequence to come here puts the
// failure word, which nothing looks at after this kernel, back to zero, so that the same call replayed from a captured
// graph, with the same number, does not find a failure of the last time.  Every workgroup that writes outputs has looked at
// the word by then.  Another one of a sequence may still look, find no failure and work on what the reduction left: it is in bounds whatever
// that is, and for nothing, since it writes no outputs.  (warp_select: outputs of a call without failure are written by whoever is the last to
// count itself, and where the writing workgroup has come here it never counts itself, so nobody is the last.)  (gridDim.y: the sequences.)
__device__ __forceinline__ void sequence_of_failed_call_done(const Ws& w) {
    const unsigned done = atomicAdd(w.counters + 4, 1u);
    if (done == gridDim.y - 1) __hip_atomic_store(reinterpret_cast<unsigned long long*>(w.counters + 2), 0ull, __ATOMIC_RELAXED, AGENT);
}
// The reduction kernel has ended: its words go back to zero, so that the same call replayed from a captured graph, with the
// same number, does not find them set.
__device__ __forceinline__ void clear_words(uint4* words, long n16, long thread, long nthreads) {
    for (long i = thread; i < n16; i += nthreads) words[i] = make_uint4(0u, 0u, 0u, 0u);
}

// How often the sequence's last workgroup looks for a share.  The workgroups it waits for come before it in the grid
// and wait for nobody, so they have started before it and end whatever else the device does.
constexpr unsigned kShareLooks = 1u << 22;

// What bounds it in calls of a few sequences is a chain of latencies: arguments, results of the reduction, row, variates,
// share, merge, outputs.  So the arguments' cache lines are requested together, all words the acceptance needs in one
// go, up to 64 positions or nodes are decided by every wavefront for itself (no barrier), the last workgroup of a sequence looks for
// the others' shares (it used to be whoever counted itself last, one round trip more), and nothing is waited for that
// the outputs do not need.  1 sequence of 4 positions, V=32000, binary32: 5.5 -> 4.0 us; of 8, V=128256, bfloat16: 5.8 -> 4.1;
// 32 trees of 60 nodes 16.8 -> 9.7 (their path used to be written node by node, a load behind every store);
// 64 sequences of 8 13.5 -> 12.0.
template <bool BF16, int LD, int KIND>
__global__ __launch_bounds__(kWG) void accept_sample(SampleParams P) {
    constexpr int ES = BF16 ? 2 : 4;
    constexpr bool TREE = KIND == KIND_TREE, TREESD = KIND == KIND_TREESD, CHAIN = !TREE && !TREESD;
    constexpr bool BY_RATIO = KIND == KIND_SD || KIND == KIND_RFSD;
    extern __shared__ int s_dyn[];   // tree: par[N], anc[N], acc[N], dep[N]
    __shared__ int s_n, s_st, s_key;
    __shared__ unsigned s_thr;
    __shared__ Best s_best[4];
    __shared__ int s_bad[4];

    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int gs = blockIdx.x, b = blockIdx.y;
    const int rows = P.rows;
    // one argument from every cache line they lie in: loaded where they are used, each line would be a miss of its own
    asm volatile("" ::"s"(P.rows), "s"(P.seed_lo), "s"(P.inv_temp), "s"(P.ws.div), "s"(P.ws.nonce));

    // ---- which positions are accepted
    const bool few = rows <= 64;      // a lane per position or node, every wavefront for itself
    const int pr = b * rows + (lane < rows ? lane : rows - 1);
    const unsigned long long fail_word = __hip_atomic_load(reinterpret_cast<const unsigned long long*>(P.ws.counters + 2), __ATOMIC_RELAXED, AGENT);
    int n = 0;         // accepted prefix length / path depth
    int sample_row = 0;
    int winner = -1;
    int nchain = 0;    // strict SD on a tree: rejected siblings whose draft rows shape the residual
    int status = 0;
    int my_par = -1, my_dep = 0, my_tok = 0;   // few: this lane's node (or position)
    // Sec. 4 eq. 4 (NaN compares false); Sec. 3 eq. 1-2 in the log domain: min(1, p/q) > u  <=>  min(0, ln p - ln q) - ln u > 0;
    // reducible FSD (Sec. 4.3): either rule accepts
    auto accepted = [&](int i, float div, double ratio) __attribute__((always_inline)) -> bool {
        bool ok = false;
        if constexpr (KIND != KIND_SD) ok = div <= P.T;
        if constexpr (BY_RATIO) {
            const U4 r = philox4x32_10((static_cast<unsigned>(i) >> 2) | (1u << 30), static_cast<unsigned>(b),
                                       P.off_lo, P.off_hi, P.seed_lo, P.seed_hi);
            const unsigned wsel = (i & 3) == 0 ? r.x : (i & 3) == 1 ? r.y : (i & 3) == 2 ? r.z : r.w;
            const double u = static_cast<double>(word_to_uniform(wsel));
            const double thr = ratio < 0.0 ? ratio : 0.0;
            ok = ok || (thr - log(u) > 0.0);
        }
        return ok;
    };
    if (tid == 0) { s_n = rows; s_st = 0; s_key = 0; s_thr = score_key(-FLT_MAX); }
    if (!TREESD && few) {
        const int st = P.ws.pst[pr];
        float div = 0.0f;
        double ratio = 0.0;
        if constexpr (KIND != KIND_SD) div = P.ws.div[pr];
        if constexpr (BY_RATIO) ratio = P.ws.lr[pr];
        if constexpr (TREE) my_par = P.parent[pr];
        my_tok = P.tokens[pr];   // (for the outputs)
        __syncthreads();
        const bool mine = lane < rows;
        if (__any(mine && st != 0)) {
            int bits = mine ? st : 0;
#pragma unroll
            for (int o = 32; o > 0; o >>= 1) bits |= __shfl_xor(bits, o);
            status = bits;
        }
        if constexpr (CHAIN) {
            const unsigned long long no = __ballot(mine && !accepted(lane, div, ratio));
            n = no ? static_cast<int>(__builtin_ctzll(no)) : rows;
            sample_row = n;
        } else {
            const TreePick pick = pick_path(lane, rows, P.max_depth, my_par, accepted(lane, div, ratio));
            n = pick.n;
            winner = pick.winner;
            my_dep = pick.my_dep;
            status |= pick.status;
            sample_row = winner + 1;
        }
    } else if constexpr (CHAIN) {
        __syncthreads();
        for (int i = tid; i < rows; i += kWG) {
            const size_t at = static_cast<size_t>(b) * rows + i;
            const int st = P.ws.pst[at];
            const bool ok = accepted(i, KIND != KIND_SD ? P.ws.div[at] : 0.0f, BY_RATIO ? P.ws.lr[at] : 0.0);
            if (st) atomicOr(&s_st, st);
            if (!ok) atomicMin(&s_n, i);
        }
        __syncthreads();
        n = s_n;
        sample_row = n;
        status = s_st;
    } else if constexpr (TREESD) {
        // the walk kernel has decided: depth, last node, and the residual chain the token comes from
        // (if the walk gave up on a bounded wait it may have written nothing: the header is then
        // whatever an earlier call left, so nothing in it is trusted)
        const int* hdr = P.ws.tsd + static_cast<size_t>(b) * (4 + rows);
        const int h0 = hdr[0], h1 = hdr[1], h2 = hdr[2], h3 = hdr[3];
        const bool gave_up = fail_word == P.ws.nonce;
        status = gave_up ? FSD_ROW_INTERNAL : h0;
        n = gave_up ? 0 : h1;
        sample_row = gave_up ? 0 : h2 + 1;
        nchain = __builtin_amdgcn_readfirstlane(gave_up ? 0 : h3);
        if (n < 0 || n > P.max_depth || sample_row < 0 || sample_row > rows || nchain < 0 || nchain > rows) {
            n = 0; sample_row = 0; nchain = 0;
            status = FSD_ROW_INTERNAL;
        }
        int* ch = s_dyn;
        float* iz = reinterpret_cast<float*>(s_dyn + rows);
        float* ldv = reinterpret_cast<float*>(s_dyn + 2 * rows);
        for (int m = tid; m < nchain; m += kWG) {
            const int c = hdr[4 + m];
            ch[m] = c;
            iz[m] = P.ws.tsd_invz[static_cast<size_t>(b) * rows + m];
            ldv[m] = static_cast<float>(P.ws.lse2[2 * (static_cast<size_t>(b) * rows + c) + 1]);
        }
        __syncthreads();
    } else {
        int* par = s_dyn;
        int* anc = s_dyn + rows;
        int* acc = s_dyn + 2 * rows;
        int* dep = s_dyn + 3 * rows;
        __syncthreads();
        for (int j = tid; j < rows; j += kWG) {
            const size_t at = static_cast<size_t>(b) * rows + j;
            int p = P.parent[at];
            if (p < -1 || p >= j) { atomicOr(&s_st, FSD_ROW_BAD_PARENT); p = -1; }
            const int st = P.ws.pst[at];
            if (st) atomicOr(&s_st, st);
            par[j] = p; anc[j] = p; dep[j] = 1;
            acc[j] = accepted(j, P.ws.div[at], 0.0) ? 1 : 0;
        }
        __syncthreads();
        // pointer jumping: after r rounds anc[j] is the 2^r-th ancestor, acc/dep cover that stretch
        for (int span = 1; span < rows; span <<= 1) {
            int na[kMaxRows / kWG], nacc[kMaxRows / kWG], nd[kMaxRows / kWG];
#pragma unroll
            for (int q = 0; q < kMaxRows / kWG; ++q) {
                const int j = tid + q * kWG;
                if (j < rows) {
                    const int a = anc[j];
                    na[q] = a; nacc[q] = acc[j]; nd[q] = dep[j];
                    if (a >= 0) { na[q] = anc[a]; nacc[q] = acc[j] & acc[a]; nd[q] = dep[j] + dep[a]; }
                }
            }
            __syncthreads();
#pragma unroll
            for (int q = 0; q < kMaxRows / kWG; ++q) {
                const int j = tid + q * kWG;
                if (j < rows) { anc[j] = na[q]; acc[j] = nacc[q]; dep[j] = nd[q]; }
            }
            __syncthreads();
        }
        for (int j = tid; j < rows; j += kWG) {
            if (dep[j] > P.max_depth) atomicOr(&s_st, FSD_ROW_TOO_DEEP);
            if (acc[j]) atomicMax(&s_key, (dep[j] << 11) | (kMaxRows - 1 - j));   // deepest, then lowest index
        }
        __syncthreads();
        const int key = s_key;
        if (key) { n = key >> 11; winner = kMaxRows - 1 - (key & (kMaxRows - 1)); }
        sample_row = winner + 1;
        status = s_st;
    }
    if (status & FSD_ROW_BAD_PARENT) status &= ~FSD_ROW_TOO_DEEP;   // depths mean nothing in a malformed tree
    const bool failed = __any(fail_word == P.ws.nonce) != 0;
    if (failed) status |= FSD_ROW_INTERNAL;   // a bounded wait of an earlier kernel expired

    // (the same in every lane: scalars from here on)
    status = __builtin_amdgcn_readfirstlane(status);
    n = __builtin_amdgcn_readfirstlane(n);
    sample_row = __builtin_amdgcn_readfirstlane(sample_row);
    winner = __builtin_amdgcn_readfirstlane(winner);

    // ---- Gumbel-max over this workgroup's share of the sampled target row
    const char* trow = P.target + (static_cast<size_t>(b) * (rows + 1) + sample_row) * static_cast<size_t>(P.V) * ES;
    bool residual = false;
    const char* drow = nullptr;
    float lt = 0.0f, ld = 0.0f;
    if constexpr (TREESD) {
        if (nchain > 0 && !status) {
            residual = true;
            lt = static_cast<float>(P.ws.lse2[2 * (static_cast<size_t>(b) * rows + s_dyn[nchain - 1])]);
        }
    }
    if constexpr (BY_RATIO) {
        if (n < rows) {   // rejected at n: the residual of Sec. 3 eq. 3 needs the draft row as well
            residual = true;
            drow = P.draft + (static_cast<size_t>(b) * rows + n) * static_cast<size_t>(P.V) * ES;
            lt = static_cast<float>(P.ws.lse2[2 * (b * rows + n)]);
            ld = static_cast<float>(P.ws.lse2[2 * (b * rows + n) + 1]);
        }
    }
    const bool merges = gs == P.GS - 1;   // the sequence's last workgroup merges the shares and writes the outputs
    long s0 = static_cast<long>(gs) * P.sps;
    long s1 = (s0 + P.sps < P.nslots) ? s0 + P.sps : P.nslots;
    Best all{neg_inf(), 0x7FFFFFFF};   // the sequence's winner
    int final_status = status;
    auto share_of = [&](int& bd) __attribute__((always_inline)) -> Best {
        Best best{neg_inf(), 0x7FFFFFFF};
        int bad = 0;
        if (!status) {
            const bool cut = P.cut && P.mode == FSD_SAMPLE;
            const DrawArgs A{P.V, P.mode, P.seed_lo, P.seed_hi, P.off_lo, P.off_hi, cut, (cut && P.thr) ? P.thr[b] : neg_inf(), P.inv_temp};
            const DrawChain C{P.draft + static_cast<size_t>(b) * rows * static_cast<size_t>(P.V) * ES, rows, nchain, s_dyn};
            // binary32: a share of one slot a lane takes 4 entries a round, any longer one 8 (a second slot that no
            // lane has still costs its instructions; whole calls on 16 sequences of 2, V=64000: 18.5 us with 8 entries,
            // 17.9 with 4; on 40 of 2, V=50048, shares of two slots a lane: 23.5 and 24.1)
            if (!BF16 && s1 - s0 <= kWG)
                draw_share<BF16, LD, TREESD, 4 + 4 * BF16>(A, b, trow, residual, drow, lt, ld, C, s0, s1, tid, &s_thr, best, bad);
            else
                draw_share<BF16, LD, TREESD, 8>(A, b, trow, residual, drow, lt, ld, C, s0, s1, tid, &s_thr, best, bad);
        }
        best = wave_best(best);
        bad = __any(bad);
        if (lane == 0) { s_best[wave] = best; s_bad[wave] = bad; }
        __syncthreads();
        Best m = s_best[0];
        bd = s_bad[0];
#pragma unroll
        for (int k = 1; k < 4; ++k) { m = better(m, s_best[k]); bd |= s_bad[k]; }
        return m;
    };
    for (;;) {
        int bd = 0;
        const Best mine = share_of(bd);
        if (!merges) {
            // The sampler's shares are cleared with the exchange words at the start of the call, so nothing has to
            // order this store: whoever merges looks until the word is there.
            if (tid == 0)
                __hip_atomic_store(P.ws.spart + static_cast<size_t>(b) * P.GS + gs, share_word(mine, bd), __ATOMIC_RELAXED, AGENT);
        } else if (wave == 0) {
            // one share per lane, this workgroup's own in the last (alone: nobody else's)
            const unsigned long long* const slot = P.ws.spart + static_cast<size_t>(b) * P.GS;
            unsigned long long w = share_word(mine, bd);
            bool late = false;
            if (s1 - s0 < P.nslots) {
                const bool other = lane < gs;
                for (unsigned looks = 0;; ++looks) {
                    const unsigned long long v = __hip_atomic_load(slot + (other ? lane : 0), __ATOMIC_RELAXED, AGENT);
                    late = __any(other && v == 0) != 0;
                    if (!late || looks >= kShareLooks) { w = other ? v : w; break; }
                    __builtin_amdgcn_s_sleep(1);
                }
            }
            all = wave_best(share_best(w));
            bd = __any((w & 0x80000000u) != 0);
            if (late) final_status |= FSD_ROW_INTERNAL;   // a share never arrived (never expected)
            if (!final_status && (bd || (all.idx == 0x7FFFFFFF && !residual))) final_status |= FSD_ROW_NONFINITE;
        }
        if constexpr (BY_RATIO || TREESD) {
            if (!merges || !residual) break;
            if (tid == 0) { s_st = final_status; s_key = all.idx; }
            __syncthreads();
            if (s_st || s_key != 0x7FFFFFFF) break;
            // No entry has a positive part (p = q to rounding, which a genuine rejection all but excludes): the
            // token is drawn from the row itself, by this workgroup alone.  (A rejected row is one the reduction
            // has found usable: it has an entry above -inf.)
            residual = false;
            s0 = 0;
            s1 = P.nslots;
        } else {
            break;
        }
    }
    if (merges && wave == 0) {
        const int token = all.idx;
        if (final_status) n = 0;
        const int width = CHAIN ? rows + 1 : P.max_depth + 1;
        int32_t* const out = P.out_tokens + static_cast<size_t>(b) * width;
        if constexpr (TREESD) {
            // the walk has written the path and its tokens; add the drawn token, or take it all back
            if (final_status) {
                int32_t* pn = P.path_nodes + static_cast<size_t>(b) * P.max_depth;
                for (int i = lane; i < P.max_depth; i += 64) pn[i] = -1;
                for (int i = lane; i < width; i += 64) out[i] = -1;
            } else if (lane == 0) {
                out[n] = token;
            }
        } else if constexpr (TREE) {
            int32_t* const pn = P.path_nodes + static_cast<size_t>(b) * P.max_depth;
            if (few) {
                write_path(lane, P.max_depth, final_status ? -1 : winner, n, my_par, my_dep, my_tok, final_status ? -1 : token, pn, out);
            } else {
                for (int i = n + lane; i < P.max_depth; i += 64) pn[i] = -1;
                for (int i = n + lane; i < width; i += 64) out[i] = (i == n && !final_status) ? token : -1;
                if (lane == 0 && !final_status) {
                    const int* par = s_dyn;
                    int jn = winner;
                    for (int i = n - 1; i >= 0 && jn >= 0; --i) {
                        pn[i] = jn;
                        out[i] = P.tokens[static_cast<size_t>(b) * rows + jn];
                        jn = par[jn];
                    }
                }
            }
        } else if (few) {
            write_chain(lane, rows, n, final_status != 0, my_tok, token, out);
        } else {
            for (int i = lane; i < width; i += 64) {
                int v = -1;
                if (!final_status) {
                    if (i < n) v = P.tokens[static_cast<size_t>(b) * rows + i];
                    else if (i == n) v = token;
                }
                out[i] = v;
            }
        }
        if (lane == 0) {
            P.out_len[b] = n;
            if (P.row_status) P.row_status[b] = final_status;
            if (P.cut && P.thr == nullptr) P.ws.thr[b] = neg_inf();   // (nothing was selected: nothing is cut)
            if (failed) sequence_of_failed_call_done(P.ws);
        }
    }
    clear_words(P.clear, P.clear16, (static_cast<long>(b) * gridDim.x + gs) * kWG + tid, static_cast<long>(gridDim.x) * gridDim.y * kWG);
}

}  // namespace

#endif  // FSD_CSRC_ACCEPT_SAMPLE_H_
