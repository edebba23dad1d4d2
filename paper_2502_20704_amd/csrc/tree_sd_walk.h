// The walk of strict SD over a token tree.
// Part of libfsd (gfx950); included by fsd_kernels.hip, which holds the host side and the C ABI.
#ifndef FSD_CSRC_TREE_SD_WALK_H_
#define FSD_CSRC_TREE_SD_WALK_H_

#include "device_common.h"
#include "accept_sample.h"

namespace {

// ------------------------------------------------------------------------------------------
// strict SD over a token tree: the walk
//
// The tree analogue of strict SD's acceptance (Sec. 3, eq. 1-3, applied child by child as in the
// tree-verification methods Sec. 2 cites).  At the current context with target distribution p the
// children are tried in index order: child j is accepted iff min(1, p(x_j)/q_j(x_j)) > y_j; after a
// rejection p becomes the normalised positive part of p - q_j.  The first child of a context is tested
// against the log-ratio the reduction kernel has stored; a later child needs p after the rejections
// so far at its token, which is kept for every child and brought up to date with each rejection, and
// every rejection that is followed by another sibling costs one pass over the vocabulary for its
// normaliser.  The token itself is drawn by accept_sample from what this kernel leaves in the workspace.
//
// gridDim.x workgroups share a sequence (all of them resident at once, which the host checks):
// every one walks the same tree and takes the same decisions, a pass is split between them, and
// the partial sums meet through 64-bit words in the workspace that are zero until posted, one
// round of words per pass.  Every workgroup adds the partials in the same order, so all see the
// same normaliser.  Waiting is bounded: a workgroup that gives up sets the call's internal-error
// flag and leaves.  Workgroup 0 of a sequence writes the outputs.
struct WalkParams {
    const char* target;
    const char* draft;
    const int32_t* tokens;    // [B,N]
    const int32_t* parent;    // [B,N]
    int rows;                 // N
    int max_depth;
    long V;
    long nslots;
    unsigned seed_lo, seed_hi, off_lo, off_hi;
    int32_t* path_nodes;      // [B,max_depth]
    int32_t* out_tokens;      // [B,max_depth+1]
    float* user_ratio;        // optional [B,N]
    unsigned spin_limit;
    Ws ws;
};

constexpr int kWalkWG = 1024;
// Slots of a row a thread keeps of the distribution in force (KEEP): 24 bfloat16 entries, 16 binary32 ones.  A
// 1024-thread workgroup has 128 registers, which the kept entries share with a draft row in flight (twice the
// registers an entry for binary32) and the positive parts formed from both: with 24 binary32 entries 77 registers were
// spilled and the walk took twice as long as one that reads everything again (one tree of 24 nodes,
// V=128256: 46 us against 23); with 16 it is 8, 10 on unaligned rows (bfloat16, 24 entries: 16 and 20).
template <bool BF16> struct WalkKeep { static constexpr int CH = BF16 ? 3 : 4; };

// What bounds the walk is its chain of dependent steps (a context's tries, and a pass after every rejection
// but the last), each of which costs round trips to memory.  So nothing is read or formed twice and
// little is waited for:
//   - a context's children sit on the lanes of the first wavefront (64 at a time): their tokens' entries,
//     log-ratios and uniform numbers are fetched together, and each child's own value of the distribution in
//     force is brought up to date after every rejection, instead of being formed along the whole chain at its
//     try.  (In float64: done by all sixteen wavefronts alike it would take each step a microsecond or two of
//     every SIMD.)  The decision goes to the others through LDS;
//   - with KEEP (a workgroup's share of a row is at most WalkKeep's slots a thread) the distribution in force stays
//     with the thread from pass to pass, so a pass reads one draft row instead of the target row and all rejected
//     ones, and that row is requested before the try whose rejection needs it.  (Where the share is longer, which
//     more trees bring about as well, a pass reads the rejected rows again: V=128256 from 43 trees on, binary32 from 33.)
// 32 trees of 60 nodes, V=128256 bfloat16: 72-83 -> 50-54 us.  Whole calls on trees of 24 nodes, binary32, before
// any of this -> now: V=32000, 1 tree 46.1 -> 34.6; V=128256, 4 trees 76.8 -> 57.0, 32 trees 194.7 -> 167.8.
template <bool BF16, int LD, bool KEEP>
__global__ __launch_bounds__(kWalkWG) void tree_sd_walk(WalkParams P) {
    constexpr int VE = Slot<BF16>::VE;
    constexpr int ES = BF16 ? 2 : 4;
    extern __shared__ int s_walk[];   // par[N], tok[N], chain[N], 1/Z[N], then Z[N] (float64)
    __shared__ double s_red[kWalkWG / 64];
    __shared__ int s_st, s_accept[2];
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int b = blockIdx.y, N = P.rows;
    const int g = blockIdx.x, GSW = gridDim.x;
    const bool writer = (g == 0);
    int* par = s_walk;
    int* tok = s_walk + N;
    int* chain = s_walk + 2 * N;
    float* s_invz = reinterpret_cast<float*>(s_walk + 3 * N);
    double* Zs = reinterpret_cast<double*>(s_walk + 4 * N);
    const double* lr_of = P.ws.lr + static_cast<size_t>(b) * N;
    const double* lse_of = P.ws.lse2 + 2 * static_cast<size_t>(b) * N;
    int* hdr = P.ws.tsd + static_cast<size_t>(b) * (4 + N);
    float* invz = P.ws.tsd_invz + static_cast<size_t>(b) * N;
    int32_t* pn = P.path_nodes + static_cast<size_t>(b) * P.max_depth;
    int32_t* out = P.out_tokens + static_cast<size_t>(b) * (P.max_depth + 1);

    if (tid == 0) s_st = 0;
    __syncthreads();
    for (int j = tid; j < N; j += kWalkWG) {
        const size_t pr = static_cast<size_t>(b) * N + j;
        int p = P.parent[pr];
        if (p < -1 || p >= j) { atomicOr(&s_st, FSD_ROW_BAD_PARENT); p = -1; }
        const int st = P.ws.pst[pr];
        if (st) atomicOr(&s_st, st);
        par[j] = p;
        tok[j] = P.tokens[pr];
        if (writer && P.user_ratio) P.user_ratio[pr] = __builtin_nanf("");
    }
    if (writer) {
        for (int i = tid; i < P.max_depth; i += kWalkWG) pn[i] = -1;
        for (int i = tid; i <= P.max_depth; i += kWalkWG) out[i] = -1;
    }
    __syncthreads();
    for (int j = tid; j < N; j += kWalkWG) {   // a node deeper than the outputs can hold?
        int depth = 1;
        for (int a = par[j]; a >= 0 && depth <= P.max_depth; a = par[a]) ++depth;
        if (depth > P.max_depth) atomicOr(&s_st, FSD_ROW_TOO_DEEP);
    }
    __syncthreads();
    int status = s_st;
    if (status & FSD_ROW_BAD_PARENT) status &= ~FSD_ROW_TOO_DEEP;
    if (failure_flagged(P.ws)) status |= FSD_ROW_INTERNAL;
    if (status) {
        if (writer && tid == 0) { hdr[0] = status; hdr[1] = 0; hdr[2] = -1; hdr[3] = 0; }
        return;
    }
    // this workgroup's share of a pass
    const long share = (P.nslots + GSW - 1) / GSW;
    const long sl_lo = static_cast<long>(g) * share;
    const long sl_hi = (sl_lo + share < P.nslots) ? sl_lo + share : P.nslots;
    int round = 0;   // passes so far in this sequence
    int tries = 0;

    // p and q of an entry: 2^(z log2e - lse2) with the argument formed in float64 and split into a
    // binary32 part for the hardware exponential and a remainder applied as 1 + ln2 * rest.  A
    // binary32 argument would carry the rounding of lse2 (about 1e-6 at |lse2| = 20) into every
    // entry of the row alike, and a later sibling's log-ratio multiplies such a common error by
    // p/(p - q); this way only the exponential's own rounding is left, which averages out in the sums.
    auto prob = [&](float z, double lse2) __attribute__((always_inline)) -> float {
        const double x = fma(static_cast<double>(z), kLog2eD, -lse2);
        const float xh = static_cast<float>(x);
        // (a masked entry, -inf or far below the row: xh is -inf and the difference no number; both bounds hold
        // for any entry that has a probability, and max() drops the NaN)
        const float xl = fminf(fmaxf(static_cast<float>(x - static_cast<double>(xh)), -1.0f), 1.0f);
        return hw_exp2(xh) * fmaf(xl, static_cast<float>(kLn2), 1.0f);
    };
    // (the value of a row's entry in float64, for the tests against single tokens)
    auto prob64 = [&](const char* row, int x, double lse2) __attribute__((always_inline)) -> double {
        return exp2(static_cast<double>(load_elem<BF16>(row, x)) * kLog2eD - lse2);
    };
    // CH slots per thread at a time, row by row: the CH loads of a row are in flight together
    constexpr int CH = KEEP ? WalkKeep<BF16>::CH : BF16 ? 4 : 8;
    auto slot_of = [&](long base, int c) __attribute__((always_inline)) -> long {
        const long sl = base + static_cast<long>(c) * kWalkWG + tid;
        return sl < sl_hi ? sl : P.nslots - 1;
    };
    auto request = [&](const char* row, long base, uint4 (&raw)[CH]) __attribute__((always_inline)) {
#pragma unroll
        for (int c = 0; c < CH; ++c) raw[c] = load_slot<BF16, LD>(row, slot_of(base, c), P.V);
    };

    const size_t rowb = static_cast<size_t>(P.V) * ES;
    const char* const drafts = P.draft + static_cast<size_t>(b) * N * rowb;
    int cur = -1, n = 0, nrej = 0, last_j = -1, before_last = 0;
    for (;;) {   // every value below that steers the walk is the same in all threads
        const char* trow = P.target + (static_cast<size_t>(b) * (N + 1) + (cur + 1)) * rowb;
        nrej = 0; last_j = -1; before_last = 0;
        int next = -1;
        // KEEP: this thread's entries of the distribution in force
        float dist[KEEP ? CH : 1][VE];
        bool formed = false, leave = false;
        for (int from = cur + 1; from < N && !leave;) {
            // the next children of the context, one per lane
            int child = -1, count = 0, last_seen = from - 1;
            bool more_after = false;   // children beyond these 64
            for (int base = from; base < N && !more_after; base += 64) {
                unsigned long long found = __ballot(base + lane < N && par[(base + lane < N) ? base + lane : 0] == cur);
                while (found) {
                    if (count == 64) { more_after = true; break; }
                    const int j = base + __builtin_ctzll(found);
                    found &= found - 1;
                    if (lane == count) child = j;
                    ++count;
                    last_seen = j;
                }
            }
            if (count == 0) break;
            from = more_after ? last_seen + 1 : N;
            // (idle lanes repeat the first child, which is read while all lanes are active: in an arm of the selection
            // it would be the first idle lane's)
            const int first = __builtin_amdgcn_readlane(child, 0);
            const int mine = child >= 0 ? child : first;
            uint4 raw[CH];
            if constexpr (KEEP) {
                if (!formed) request(trow, sl_lo, raw);
            }
            int x = 0;
            double first_ratio = 0.0, r = 0.0, lq = 0.0, log_u = 0.0;   // first wavefront only
            if (wave == 0) {
                x = tok[mine];
                const double lt2 = lse_of[2 * mine], ld2 = lse_of[2 * mine + 1];
                first_ratio = lr_of[mine];
                r = prob64(trow, x, lt2);
                lq = (static_cast<double>(load_elem<BF16>(drafts + mine * rowb, x)) * kLog2eD - ld2) * kLn2;
                for (int m = 0; m < nrej; ++m)   // (only beyond a context's first 64 children)
                    r = fmax(r - prob64(drafts + chain[m] * rowb, x, lse_of[2 * chain[m] + 1]), 0.0) / Zs[m];
                // Sec. 3 eq. 1-2 in the log domain, with the uniform number of the child's index
                const U4 rw = philox4x32_10((static_cast<unsigned>(mine) >> 2) | (1u << 30), static_cast<unsigned>(b), P.off_lo,
                                            P.off_hi, P.seed_lo, P.seed_hi);
                const unsigned wsel = (mine & 3) == 0 ? rw.x : (mine & 3) == 1 ? rw.y : (mine & 3) == 2 ? rw.z : rw.w;
                log_u = log(static_cast<double>(word_to_uniform(wsel)));
            }
            if constexpr (KEEP) {
                if (!formed) {
                    const double lt2c = lse_of[2 * first];
#pragma unroll
                    for (int c = 0; c < CH; ++c) {
                        float z[VE];
#pragma unroll
                        for (int e = 0; e < VE; ++e) dist[c][e] = 0.0f;
                        if (sl_lo + static_cast<long>(c) * kWalkWG + wave * 64 >= sl_hi) continue;   // (nobody's here)
                        settle_slot<BF16, LD>(raw[c], slot_of(sl_lo, c), P.V);
                        unpack<BF16>(raw[c], z);
                        const bool in = sl_lo + static_cast<long>(c) * kWalkWG + tid < sl_hi;
#pragma unroll
                        for (int e = 0; e < VE; ++e) dist[c][e] = in ? prob(z[e], lt2c) : 0.0f;
                        __builtin_amdgcn_sched_barrier(0);   // (one slot at a time: all at once would not fit the registers)
                    }
                    formed = true;
                }
            }

            for (int k = 0; k < count; ++k) {
                const int j = __builtin_amdgcn_readlane(child, k);
                const char* drow = drafts + j * rowb;
                const bool more = k + 1 < count || more_after;
                float at_x = 0.0f;
                if (more) {   // what the pass after a rejection reads
                    if (wave == 0) at_x = load_elem<BF16>(drow, x);
                    if constexpr (KEEP) request(drow, sl_lo, raw);
                }
                if (wave == 0) {
                    const double ratio = (nrej == 0) ? first_ratio : (r > 0.0) ? log(r) - lq : -__builtin_inf();
                    const double thr = ratio < 0.0 ? ratio : 0.0;
                    if (writer && lane == k && P.user_ratio) P.user_ratio[static_cast<size_t>(b) * N + j] = static_cast<float>(ratio);
                    if (lane == k) s_accept[tries & 1] = (thr - log_u > 0.0) ? 1 : 0;
                }
                __syncthreads();
                // (two slots in turn: nobody writes the one that is read here before the next try's barrier)
                const bool accepted = s_accept[tries & 1] != 0;
                ++tries;
                if (accepted) { next = j; leave = true; break; }
                last_j = j;
                before_last = nrej;
                if (!more) { leave = true; break; }
                // ---- the normaliser of the positive part of p - q_j, p being the distribution in force
                [[maybe_unused]] const double lt2j = lse_of[2 * j];
                const double ld2j = lse_of[2 * j + 1];
                double acc = 0.0;
                float left[KEEP ? CH : 1][VE];
                if constexpr (KEEP) {
#pragma unroll
                    for (int c = 0; c < CH; ++c) {
                        float zd[VE];
#pragma unroll
                        for (int e = 0; e < VE; ++e) left[c][e] = 0.0f;
                        if (sl_lo + static_cast<long>(c) * kWalkWG + wave * 64 >= sl_hi) continue;
                        settle_slot<BF16, LD>(raw[c], slot_of(sl_lo, c), P.V);
                        unpack<BF16>(raw[c], zd);
                        float part = 0.0f;
#pragma unroll
                        for (int e = 0; e < VE; ++e) {
                            left[c][e] = fmaxf(dist[c][e] - prob(zd[e], ld2j), 0.0f);
                            part += left[c][e];
                        }
                        acc += static_cast<double>(part);
                        __builtin_amdgcn_sched_barrier(0);
                    }
                } else {
                    for (long base = sl_lo; base < sl_hi; base += static_cast<long>(kWalkWG) * CH) {
                        float pv[CH][VE];
                        request(trow, base, raw);
#pragma unroll
                        for (int c = 0; c < CH; ++c) {
                            float z[VE];
                            settle_slot<BF16, LD>(raw[c], slot_of(base, c), P.V);
                            unpack<BF16>(raw[c], z);
                            const bool in = base + static_cast<long>(c) * kWalkWG + tid < sl_hi;
#pragma unroll
                            for (int e = 0; e < VE; ++e) pv[c][e] = in ? prob(z[e], lt2j) : 0.0f;
                        }
                        for (int m = 0; m < nrej; ++m) {
                            request(drafts + chain[m] * rowb, base, raw);
                            const double ldm = lse_of[2 * chain[m] + 1];
                            const float izm = s_invz[m];
#pragma unroll
                            for (int c = 0; c < CH; ++c) {
                                float zd[VE];
                                settle_slot<BF16, LD>(raw[c], slot_of(base, c), P.V);
                                unpack<BF16>(raw[c], zd);
#pragma unroll
                                for (int e = 0; e < VE; ++e)
                                    pv[c][e] = fmaxf(pv[c][e] - prob(zd[e], ldm), 0.0f) * izm;
                            }
                        }
                        request(drow, base, raw);
#pragma unroll
                        for (int c = 0; c < CH; ++c) {
                            float zd[VE];
                            settle_slot<BF16, LD>(raw[c], slot_of(base, c), P.V);
                            unpack<BF16>(raw[c], zd);
                            float part = 0.0f;
#pragma unroll
                            for (int e = 0; e < VE; ++e) part += fmaxf(pv[c][e] - prob(zd[e], ld2j), 0.0f);
                            acc += static_cast<double>(part);
                        }
                    }
                }
                acc = wave_sum(acc);
                __syncthreads();   // the previous round's readers are done with s_red
                if (lane == 0) s_red[wave] = acc;
                __syncthreads();
                double Z = 0.0;
                for (int w = 0; w < kWalkWG / 64; ++w) Z += s_red[w];   // same order in every thread
                if (GSW > 1) {
                    // ---- meet the other workgroups of the sequence: post this share, read all of them
                    unsigned long long* const words = P.ws.wz + (static_cast<size_t>(b) * N + round) * kWalkShare;
                    if (tid == 0) post64(words + g, dbits(Z));
                    __syncthreads();   // everyone has read s_red
                    if (tid < GSW) {
                        unsigned long long v = 0;
                        unsigned polls = 0;
                        for (;;) {
                            v = read64(words + tid);
                            if (v != 0 || polls++ >= P.spin_limit) break;
                            __builtin_amdgcn_s_sleep(2);
                        }
                        s_red[tid] = (v != 0) ? bitsd(v) : __builtin_nan("");
                    }
                    __syncthreads();
                    Z = 0.0;
                    for (int w = 0; w < GSW; ++w) Z += s_red[w];
                    if (Z != Z) {   // a workgroup of this sequence never posted: give up, the call reports it
                        if (tid == 0) flag_failure(P.ws);
                        return;
                    }
                }
                ++round;
                if (Z > 0.0) {
                    const float iz = static_cast<float>(1.0 / Z);
                    if (tid == 0) {
                        chain[nrej] = j; Zs[nrej] = Z; s_invz[nrej] = iz;
                        if (writer) invz[nrej] = iz;
                    }
                    if constexpr (KEEP) {
#pragma unroll
                        for (int c = 0; c < CH; ++c) {
#pragma unroll
                            for (int e = 0; e < VE; ++e) dist[c][e] = left[c][e] * iz;
                        }
                    }
                    if (wave == 0) r = fmax(r - exp2(static_cast<double>(at_x) * kLog2eD - ld2j), 0.0) / Z;
                    __syncthreads();
                    ++nrej;
                }
            }
        }
        if (next < 0) break;
        if (writer && tid == 0) { pn[n] = next; out[n] = tok[next]; }
        ++n;
        cur = next;
    }
    // ---- what the sampler needs: the residual chain ends with the last rejected child, whose
    // normaliser nobody needs
    if (writer && tid == 0) {
        hdr[0] = 0;
        hdr[1] = n;
        hdr[2] = cur;
        const int nchain = (last_j >= 0) ? before_last + 1 : 0;
        hdr[3] = nchain;
        for (int m = 0; m < before_last && m < nchain; ++m) hdr[4 + m] = chain[m];
        if (nchain > 0) hdr[4 + nchain - 1] = last_j;
    }
}

}  // namespace

#endif  // FSD_CSRC_TREE_SD_WALK_H_
