// FSD on a few sequences in one launch.
// Part of libfsd (gfx950); included by fsd_kernels.hip, which holds the host side and the C ABI.
#ifndef FSD_CSRC_SMALL_CALL_H_
#define FSD_CSRC_SMALL_CALL_H_

#include "accept_sample.h"
#include "device_common.h"
#include "pair_kernel.h"

namespace {

// ------------------------------------------------------------------------------------------
// a small call: reduction, draw and acceptance in one kernel
//
// What bounds a call of a few sequences is not work but a chain: a kernel's start, the logits from memory, and a round
// trip through the memory's side (1-1.5 us) wherever wavefronts meet.  In the two kernels of a large call it has six
// such trips: the members' arrival, their sums, the divergence's shares, the rows' results from one kernel to the next, the sampled row, the
// draw's shares.  Here it has two, the sums and the divergence's shares:
//   - Every word says by itself whether it is this call's: half of it is half of the call's number.  So nothing is
//     cleared and nobody's arrival is waited for.  (A replay of a captured call has the number of the replay before: there
//     the words are cleared, by a kernel before this one or by the sampler behind it.)
//   - The draw needs the target row and the random numbers, which are the same for every row, but not the
//     divergences.  While the teams work, workgroups that wait for nobody draw from all target rows; acceptance
//     then only picks one.  (The chip is mostly idle in such a call.)
//   - One workgroup a sequence (16 pairs, if there are no draws), the last of the grid, reads the draws' and the members' words itself.
// Where the draws of all rows would be too much, or need what this kernel does not have (reducible FSD, the warpers), it leaves
// the results to the kernels that follow, as pair_kernel does.
// The teams' wavefronts hold NV slots of each row a lane, for one pair each: there is no second step and nothing to
// overlap.  All divergences are evaluated pointwise, for bfloat16 too: half as much a lane as in the large shape.
// NV is 2 where that makes few wavefronts (kSmallWaves), else 4, and the next larger one where a team would have more than 64
// members (one word of each a lane), the words would not fit the workspace or the teams the device.
struct SmallParams {
    const char* target;
    const char* draft;
    const int32_t* tokens;
    const int32_t* parent;  // tree only
    int rows;               // K or N
    int npairs;             // B * rows
    int max_depth;          // tree only
    long V;
    long nslots;
    int G;                  // wavefronts per pair
    int np;                 // words of a member's share of the divergence
    int team_wgs;           // the grid: the teams' workgroups, the draws' (GS for every target row), one per sequence
    int draw_wgs;           // 0: the draw follows in kernels of its own, the results go to the workspace (ws)
    int GS;
    int sps;                // slots per draw
    int finish;             // without draws: pairs of a finishing workgroup
    float T;
    int mode;
    unsigned seed_lo, seed_hi, off_lo, off_hi;
    unsigned spin_limit;
    int32_t* out_len;
    int32_t* out_tokens;
    int32_t* path_nodes;    // tree only
    int32_t* row_status;    // optional
    float* user_div;        // optional
    long words16;                // the words below in 16-byte units, rounded up
    unsigned long long* words;   // sums [pair][member][4], shares of the divergence [pair][member][np], draws [b][row][GS][2]
    unsigned long long nonce;
    // without draws: where the results go, what the kernels that follow need cleared (16-byte units)
    Ws ws;
    float* user_ratio;      // optional, reducible FSD only
    int want_ratio;         // reducible FSD: ln p(x) - ln q(x) at the candidate token as well
    uint4* clear_a;
    long clear_a16;
    uint4* clear_b;
    long clear_b16;
};

constexpr int kSmallTeam = 64;
// Pairs of a finishing workgroup where the reduction alone is asked for: four a wavefront, or one where reducible FSD asks for the
// candidate's log-ratio too, a chain of its own (two merges and logarithms in float64) for every pair.  Whole calls of reducible FSD, the
// persistent teams, four pairs and one (us): JS, bfloat16 B=4 K=8 V=32000 17.5, 20.1 and 14.0, V=128256 20.7, 25.5 and 18.3; binary32 B=4
// K=8 V=32000 15.3, 19.9 and 13.5, B=8 17.3, 23.6 and 16.4.
constexpr int small_finish_pairs(bool want_ratio) { return want_ratio ? 4 : 16; }
// words of a divergence's share: JS a sum and a status; TV three sums, KL two and a mark, and a status; bfloat16 KL two sums
// in float64, the mark and the status in the last bits of the first
constexpr int small_share_words(int mode) { return mode == MODE_JS ? 2 : 4; }
// Bfloat16 KL is made of float64 sums in large calls (pair_kernel's single pass): for results of order one its error is the
// rounding of the result, and it grows in proportion as they get smaller.  The pointwise terms have no such error; so that they are
// not behind for large results either, the rows' normalisers, the sums over a wavefront and the shares are float64 here,
// and a share is corrected for the rounding of its factor, which all entries have in common.
template <bool BF16, int MODE> constexpr bool kWideKl = BF16 && MODE == MODE_KLP;
constexpr unsigned kSaturated = 1u, kLate = 2u;

__device__ __forceinline__ unsigned long long tagged(unsigned payload, unsigned long long nonce, int i) {
    return ((i & 1) ? (nonce << 32) : (nonce & 0xFFFFFFFF00000000ull)) | payload;
}
__device__ __forceinline__ bool is_tagged(unsigned long long w, unsigned long long nonce, int i) {
    return static_cast<unsigned>(w >> 32) == static_cast<unsigned>((i & 1) ? nonce : nonce >> 32);
}
// every lane reads the N words at each of its R places (lanes without an entry of their own repeat another's): false if one of the
// wavefront's words has not come within `limit` looks
template <int N, int R>
__device__ __forceinline__ bool await_tagged(const unsigned long long* (&at)[R], unsigned long long nonce, unsigned limit,
                                             unsigned long long (&w)[R][N]) {
    for (unsigned polls = 0;; ++polls) {
        bool missing = false;
#pragma unroll
        for (int r = 0; r < R; ++r) {
#pragma unroll
            for (int i = 0; i < N; ++i) w[r][i] = read64(at[r] + i);
        }
#pragma unroll
        for (int r = 0; r < R; ++r) {
#pragma unroll
            for (int i = 0; i < N; ++i) missing |= !is_tagged(w[r][i], nonce, i);
        }
        if (!__any(missing)) return true;
        if (polls >= limit) return false;
        __builtin_amdgcn_s_sleep(1);
    }
}

template <bool BF16, int NV, int MODE, int LD>
__device__ __forceinline__ void small_team(const SmallParams& P, int gwave) {
    constexpr int VE = Slot<BF16>::VE, ES = BF16 ? 2 : 4, NE = NV * VE, NP = small_share_words(MODE);
    constexpr float kTiny = 2e-38f;
    constexpr bool WIDE = kWideKl<BF16, MODE>;
    const int lane = threadIdx.x & 63;
    const int pair = gwave / P.G, member = gwave - pair * P.G;
    if (pair >= P.npairs) return;
    const int b = pair / P.rows, j = pair - b * P.rows;
    int ctx = j;
    if (P.parent) {
        const int par = P.parent[pair];
        ctx = (par >= -1 && par < j) ? par + 1 : 0;   // (small_finish reports an invalid one)
    }
    const char* const trow = P.target + (static_cast<size_t>(b) * (P.rows + 1) + ctx) * static_cast<size_t>(P.V) * ES;
    const char* const drow = P.draft + static_cast<size_t>(pair) * static_cast<size_t>(P.V) * ES;
    unsigned long long* const sums = P.words + static_cast<size_t>(pair) * P.G * 4;
    unsigned long long* const shares = P.words + static_cast<size_t>(P.npairs) * P.G * 4 + static_cast<size_t>(pair) * P.G * NP;

    const long s0 = static_cast<long>(member) * (64 * NV) + lane;
    uint4 ra[NV], rb[NV];
#pragma unroll
    for (int k = 0; k < NV; ++k) {
        const long s = s0 + 64 * k, at = s < P.nslots ? s : P.nslots - 1;
        ra[k] = load_slot<BF16, LD>(trow, at, P.V);
        rb[k] = load_slot<BF16, LD, true>(drow, at, P.V);
    }
    // ---- maximum, then sums of 2^(z log2e - k) with k = ceil(max log2e)
    float mt = neg_inf(), md = neg_inf();
#pragma unroll
    for (int k = 0; k < NV; ++k) {
        const long s = s0 + 64 * k, at = s < P.nslots ? s : P.nslots - 1;
        settle_slot<BF16, LD>(ra[k], at, P.V);
        settle_slot<BF16, LD>(rb[k], at, P.V);
        if (s >= P.nslots) { ra[k] = slot_neg_inf<BF16>(); rb[k] = slot_neg_inf<BF16>(); }
        float a[VE], c[VE];
        unpack<BF16>(ra[k], a);
        unpack<BF16>(rb[k], c);
#pragma unroll
        for (int e = 0; e < VE; e += 2) {
            mt = fmaxf(fmaxf(mt, a[e]), a[e + 1]);
            md = fmaxf(fmaxf(md, c[e]), c[e + 1]);
        }
    }
    wave_max2(mt, md);
    const float kt = reference_exponent(mt), kd = reference_exponent(md);
    float et[NE], ed[NE], st = 0.0f, sd = 0.0f, wsum = 0.0f, dmax = neg_inf();
    [[maybe_unused]] double st64 = 0.0, sd64 = 0.0, wsum64 = 0.0;   // WIDE: binary32 sums of 16 entries, added up in float64
#pragma unroll
    for (int k = 0; k < NV; ++k) {
        float a[VE], c[VE];
        unpack<BF16>(ra[k], a);
        unpack<BF16>(rb[k], c);
#pragma unroll
        for (int e = 0; e < VE; ++e) {
            const float xa = hw_exp2(fmaf(a[e], kLog2e, -kt)), xb = hw_exp2(fmaf(c[e], kLog2e, -kd));
            et[k * VE + e] = xa;
            ed[k * VE + e] = xb;
            st += xa;
            sd += xb;
            if constexpr (MODE == MODE_KLP) {   // sum p (a - b) beside the pointwise terms (see pair_kernel)
                const float diff = a[e] - c[e];
                dmax = fmaxf(dmax, diff);       // +inf iff the draft masks an entry the target does not
                wsum = fmaf(xa, __builtin_amdgcn_fmed3f(diff, -FLT_MAX, FLT_MAX), wsum);
            }
        }
        if constexpr (WIDE) {
            if (k & 1) {
                st64 += static_cast<double>(st);
                sd64 += static_cast<double>(sd);
                wsum64 += static_cast<double>(wsum);
                st = sd = wsum = 0.0f;
            }
        }
    }
    if constexpr (WIDE) {
        st64 = wave_sum(st64);
        sd64 = wave_sum(sd64);
        st = static_cast<float>(st64);
        sd = static_cast<float>(sd64);
    } else {
        wave_sumf2(st, sd);
    }
    if (lane < 4) {
        const float mine = lane == 0 ? kt : lane == 1 ? kd : lane == 2 ? st : sd;
        post64(sums + member * 4 + lane, tagged(__float_as_uint(mine), P.nonce, lane));
    }
    if constexpr (WIDE) wsum64 = wave_sum(wsum64);
    else if constexpr (MODE == MODE_KLP) wsum = wave_sumf(wsum);
    if constexpr (MODE == MODE_KLP) dmax = wave_max(dmax);

    // ---- the rows' normalisers relative to this wavefront's own references
    const unsigned long long* at[1] = {sums + (lane < P.G ? lane : P.G - 1) * 4};
    unsigned long long w[1][4];
    const bool ok = await_tagged<4, 1>(at, P.nonce, P.spin_limit, w);
    TeamNorm n{kt, kd, 0.0f, 0.0f, ok};
    [[maybe_unused]] double zt64 = 0.0;
    if constexpr (WIDE) {
        // (this wavefront's own sums as they were before they were rounded for the others)
        const double mt64 = lane == member ? st64 : static_cast<double>(lo_f(w[0][2])), md64 = lane == member ? sd64 : static_cast<double>(lo_f(w[0][3]));
        zt64 = wave_sum(lane < P.G ? ldexp(mt64, kdiff(lo_f(w[0][0]), kt)) : 0.0);
        n.zt = static_cast<float>(zt64);
        n.zd = static_cast<float>(wave_sum(lane < P.G ? ldexp(md64, kdiff(lo_f(w[0][1]), kd)) : 0.0));
    } else {
        const unsigned long long packed[2] = {(w[0][1] << 32) | static_cast<unsigned>(w[0][0]), (w[0][3] << 32) | static_cast<unsigned>(w[0][2])};
        merge_round(packed, lane < P.G, n);
    }
    const float rzt = __builtin_amdgcn_rcpf(n.zt), rzd = __builtin_amdgcn_rcpf(n.zd);
    const float ft = ((st > 0.0f) || (st != st)) ? rzt : rzt * 0.0f, fd = ((sd > 0.0f) || (sd != sd)) ? rzd : rzd * 0.0f;

    // ---- the divergence's terms (as in pair_kernel's phase 2)
    const float ftc = fmaxf(ft, 0x1p-80f), fdc = fmaxf(fd, 0x1p-80f);   // max() drops NaN: see below
    const float cq = (ftc == fdc) ? 1.0f : fdc * __builtin_amdgcn_rcpf(ftc);
    const bool unusable = ft != ft || fd != fd;
    float part[3] = {0.0f, 0.0f, 0.0f};
    [[maybe_unused]] double share64 = 0.0;
    if constexpr (MODE == MODE_TV) {
#pragma unroll
        for (int i = 0; i < NE; ++i) tv_terms(et[i], ed[i] * cq, part[0], part[1], part[2]);
        wave_sumf2(part[0], part[1]);
        part[2] = wave_sumf(part[2]);
#pragma unroll
        for (int i = 0; i < 3; ++i) part[i] = unusable ? ft + fd : part[i] * ftc;
    } else {
        float acc = 0.0f;
        [[maybe_unused]] double acc64 = 0.0;
#pragma unroll
        for (int i = 0; i < NE; ++i) {
            const float p = (MODE == MODE_KLP) ? fmaf(et[i], ft, kTiny) : et[i];
            const float q = (MODE == MODE_KLP) ? fmaf(ed[i], fd, kTiny) : ed[i] * cq;
            pointwise_term<MODE>(p, q, acc);
            if constexpr (WIDE) {
                if (i % 16 == 15) { acc64 += static_cast<double>(acc); acc = 0.0f; }
            }
        }
        if constexpr (WIDE) {
            // in proportion to 1 / zt64 instead of its binary32 rounding ft (2^-22 apart at most, where ft is not 0)
            double exact = 2.0 - zt64 * static_cast<double>(ft);
            if (!(fabs(exact - 1.0) < 0x1p-20)) exact = 1.0;
            share64 = unusable ? static_cast<double>(ft + fd) : wave_sum(acc64) * exact;
            if (dmax == __builtin_inff()) share64 += __builtin_inf();   // NaN stays NaN
            wsum64 = ft > 0.0f ? wsum64 * (static_cast<double>(ft) * exact) : 0.0;
        } else {
            acc = wave_sumf(acc);
            if constexpr (MODE != MODE_KLP) acc *= ftc;
            if (unusable) acc = ft + fd;
            if constexpr (MODE == MODE_KLP) {
                if (dmax == __builtin_inff()) acc += __builtin_inff();   // NaN stays NaN
                part[1] = wsum * ft;
            }
            part[0] = acc;
        }
        if constexpr (MODE == MODE_KLP) {
            const float dl = ((kt - hw_log2(ft)) - (kd - hw_log2(fd))) * static_cast<float>(kLn2);
            const bool sat = (ft > 0.0f) && dmax > neg_inf() && (fd == 0.0f || dmax - dl > 80.0f);
            part[2] = sat ? 1.0f : 0.0f;
        }
    }
    if (lane < NP) {
        unsigned mine;
        if constexpr (WIDE) {
            const unsigned long long bits = static_cast<unsigned long long>(__double_as_longlong(lane < 2 ? share64 : wsum64));
            mine = static_cast<unsigned>((lane & 1) ? bits >> 32 : bits);
            if (lane == 0) mine = (mine & ~(kSaturated | kLate)) | (part[2] > 0.0f ? kSaturated : 0u) | (ok ? 0u : kLate);
        } else {
            const float val = (lane == 0 || NP == 2) ? part[0] : lane == 1 ? part[1] : part[2];
            mine = lane == NP - 1 ? (ok ? 0u : static_cast<unsigned>(FSD_ROW_INTERNAL)) : __float_as_uint(val);
        }
        post64(shares + member * NP + lane, tagged(mine, P.nonce, lane));
    }
}

struct SmallShared {
    unsigned thr;
    Best best[4];
    int bad[4];
    float div[64];
    int status[64];
    Best drawn[65];
    int drawn_status[65];
};

// the best score of a share of one target row, whichever row the token will come from
template <bool BF16, int LD>
__device__ __forceinline__ void small_draw(const SmallParams& P, int row_of_all, int g, SmallShared& s) {
    constexpr int ES = BF16 ? 2 : 4;
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int b = row_of_all / (P.rows + 1);
    if (tid == 0) s.thr = score_key(-FLT_MAX);
    __syncthreads();
    const char* const trow = P.target + static_cast<size_t>(row_of_all) * static_cast<size_t>(P.V) * ES;
    const long s0 = static_cast<long>(g) * P.sps, s1 = (s0 + P.sps < P.nslots) ? s0 + P.sps : P.nslots;
    const DrawArgs A{P.V, P.mode, P.seed_lo, P.seed_hi, P.off_lo, P.off_hi, false, neg_inf(), 1.0f};
    const DrawChain C{nullptr, 0, 0, nullptr};
    Best best{neg_inf(), 0x7FFFFFFF};
    int bad = 0;
    draw_share<BF16, LD, false, 8>(A, b, trow, false, nullptr, 0.0f, 0.0f, C, s0, s1, tid, &s.thr, best, bad);
    best = wave_best(best);
    bad = __any(bad);
    if (lane == 0) { s.best[wave] = best; s.bad[wave] = bad; }
    __syncthreads();
    if (tid < 2) {
        Best m = s.best[0];
        int bd = s.bad[0];
#pragma unroll
        for (int k = 1; k < 4; ++k) { m = better(m, s.best[k]); bd |= s.bad[k]; }
        const unsigned long long share = share_word(m, bd);
        unsigned long long* const at = P.words + static_cast<size_t>(P.npairs) * P.G * (4 + P.np) +
                                       (static_cast<size_t>(row_of_all) * P.GS + g) * 2;
        post64(at + tid, tagged(tid ? static_cast<unsigned>(share) : static_cast<unsigned>(share >> 32), P.nonce, tid));
    }
}

// a sequence's divergences, its accepted prefix or path and its token
template <bool BF16, int MODE>
__device__ __forceinline__ void small_finish(const SmallParams& P, int wg, SmallShared& s) {
    constexpr int NP = small_share_words(MODE);
    constexpr bool WIDE = kWideKl<BF16, MODE>;
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int rows = P.rows;
    // this workgroup's pairs: a sequence's, or, where only the reduction is asked for, a fixed number
    const int b = wg;
    const int pair0 = P.draw_wgs ? b * rows : wg * P.finish, pair1 = P.draw_wgs ? pair0 + rows : min(pair0 + P.finish, P.npairs);
    const size_t mine_at = static_cast<size_t>(P.draw_wgs ? b : 0) * rows + (lane < rows ? lane : rows - 1);
    const int token_in = P.tokens[mine_at];
    int my_par = P.parent ? P.parent[mine_at] : -1;
    if (P.draw_wgs == 0) {
        const uint4 zero = make_uint4(0u, 0u, 0u, 0u);
        const long step = static_cast<long>((P.npairs + P.finish - 1) / P.finish) * kWG;
        for (long i = static_cast<long>(wg) * kWG + tid; i < P.clear_a16; i += step) P.clear_a[i] = zero;
        for (long i = static_cast<long>(wg) * kWG + tid; i < P.clear_b16; i += step) P.clear_b[i] = zero;
    }
    // the draws first: they are there long before the divergences.  (Four rows a wavefront at a time: each on its own, the
    // round trips of a tree's rows were the longest part of its call.)
    const unsigned long long* const draws = P.words + static_cast<size_t>(P.npairs) * P.G * (4 + NP);
    for (int base = wave; base <= rows && P.draw_wgs; base += 16) {
        const unsigned long long* at[4];
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            const int r = base + 4 * k <= rows ? base + 4 * k : base;
            at[k] = draws + ((static_cast<size_t>(b) * (rows + 1) + r) * P.GS + (lane < P.GS ? lane : P.GS - 1)) * 2;
        }
        unsigned long long w[4][2];
        const bool there = await_tagged<2, 4>(at, P.nonce, kShareLooks, w);
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            const int r = base + 4 * k;
            if (r > rows) break;
            const unsigned long long share = (w[k][0] << 32) | static_cast<unsigned>(w[k][1]);
            const Best m = wave_best(share_best(share));
            const int st = !there ? FSD_ROW_INTERNAL : (__any((share & 0x80000000u) != 0) || m.idx == 0x7FFFFFFF) ? FSD_ROW_NONFINITE : 0;
            if (lane == 0) { s.drawn[r] = m; s.drawn_status[r] = st; }
        }
    }
    // four pairs a wavefront at a time
    const unsigned long long* const sums = P.words;
    const unsigned long long* const shares = P.words + static_cast<size_t>(P.npairs) * P.G * 4;
    const bool in = lane < P.G;
    // log2-sum-exp2 of a pair's rows from the team's sums, in float64
    auto row_logs = [&](int pair, double& lse2_t, double& lse2_d) __attribute__((always_inline)) -> bool {
        const unsigned long long* p1[1] = {sums + (static_cast<size_t>(pair) * P.G + (in ? lane : P.G - 1)) * 4};
        unsigned long long u[1][4];
        const bool there = await_tagged<4, 1>(p1, P.nonce, P.spin_limit, u);
        const float kt = lo_f(u[0][0]), kd = lo_f(u[0][1]);
        const double St = in ? static_cast<double>(lo_f(u[0][2])) : 0.0, Sd = in ? static_cast<double>(lo_f(u[0][3])) : 0.0;
        const float Kt = wave_max((St > 0.0) ? kt : neg_inf()), Kd = wave_max((Sd > 0.0) ? kd : neg_inf());
        const double Zt = wave_sum((St > 0.0) ? ldexp(St, kdiff(kt, Kt)) : 0.0), Zd = wave_sum((Sd > 0.0) ? ldexp(Sd, kdiff(kd, Kd)) : 0.0);
        lse2_t = static_cast<double>(Kt) + log2(Zt);
        lse2_d = static_cast<double>(Kd) + log2(Zd);
        return there;
    };
    // a share's first sum, or KL's second (WIDE: float64 in two words, whose last bits in the first are marks)
    auto number = [](const unsigned long long (&v)[NP], int i) __attribute__((always_inline)) -> double {
        if constexpr (WIDE)
            return __longlong_as_double(static_cast<long long>((v[2 * i + 1] << 32) | (static_cast<unsigned>(v[2 * i]) & ~(i ? 0u : kSaturated | kLate))));
        else
            return static_cast<double>(lo_f(v[i]));
    };
    for (int base = pair0 + wave; base < pair1; base += 16) {
        const unsigned long long* at[4];
        [[maybe_unused]] unsigned again = 0;   // pairs whose KL has terms that leave binary32's range
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            const int pair = base + 4 * k < pair1 ? base + 4 * k : base;
            at[k] = shares + (static_cast<size_t>(pair) * P.G + (in ? lane : P.G - 1)) * NP;
        }
        // what reducible FSD's log-ratio takes is there before the shares are
        double log_p = 0.0, log_q = 0.0, first_t = 0.0, first_d = 0.0;
        bool first_ok = true;
        int x = 0;
        if (P.want_ratio) {   // (one pair a wavefront)
            constexpr int ES = BF16 ? 2 : 4;
            x = P.tokens[base];
            const long at_x = (x < 0 || x >= P.V) ? 0 : x;
            log_p = static_cast<double>(load_elem<BF16>(P.target + (static_cast<size_t>(base) + base / rows) * P.V * ES, at_x));
            log_q = static_cast<double>(load_elem<BF16>(P.draft + static_cast<size_t>(base) * P.V * ES, at_x));
            first_ok = row_logs(base, first_t, first_d);
        }
        unsigned long long w[4][NP];
        const bool there = await_tagged<NP, 4>(at, P.nonce, P.spin_limit, w);
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            const int pair = base + 4 * k;
            if (pair >= pair1) break;
            const bool late = WIDE ? (w[k][0] & kLate) != 0 : static_cast<unsigned>(w[k][NP - 1]) != 0;
            int status = (!there || __any(late)) ? FSD_ROW_INTERNAL : 0;
            const double first = wave_sum(in ? number(w[k], 0) : 0.0);
            double value;
            if constexpr (MODE == MODE_TV) {   // the lighter side (see pair_kernel)
                const double other = wave_sum(in ? static_cast<double>(lo_f(w[k][1])) : 0.0);
                const double mass = wave_sum(in ? static_cast<double>(lo_f(w[k][2])) : 0.0);
                value = (mass != mass) ? __builtin_nan("") : (mass <= 1.0 ? first : other);
            } else {
                value = 0.5 * kLn2 * first;
            }
            if (value != value) status |= FSD_ROW_NONFINITE;   // NaN / +inf logits, or a row without mass
            if (value < 0.0) value = 0.0;
            if (P.want_ratio && !first_ok) status |= FSD_ROW_INTERNAL;
            if constexpr (MODE == MODE_KLP) {
                const bool saturated = __any(in && (WIDE ? (w[k][0] & kSaturated) != 0 : lo_f(w[k][2]) > 0.0f));
                if (!status && value < __builtin_inf() && saturated) again |= 1u << k;
            }
            if (status) value = __builtin_nan("");
            if (P.draw_wgs == 0 && lane == 0) {
                if (P.want_ratio) {
                    double ratio = __builtin_nan("");
                    if (x < 0 || x >= P.V) {
                        status |= FSD_ROW_BAD_TOKEN;
                    } else if (!(status & FSD_ROW_NONFINITE)) {
                        const double lp = log_p - first_t * kLn2, lq = log_q - first_d * kLn2;
                        ratio = (lp == -__builtin_inf()) ? -__builtin_inf() : lp - lq;
                    }
                    P.ws.lr[pair] = ratio;
                    if (P.user_ratio) P.user_ratio[pair] = static_cast<float>(ratio);
                }
                P.ws.div[pair] = static_cast<float>(value);
                P.ws.lse2[2 * pair] = first_t;
                P.ws.lse2[2 * pair + 1] = first_d;
                P.ws.pst[pair] = status;
                if (status & FSD_ROW_INTERNAL) flag_failure(P.ws);
            }
            if (lane == 0) {
                if (P.draw_wgs) {
                    s.div[pair - pair0] = static_cast<float>(value);
                    s.status[pair - pair0] = status;
                }
                if (P.user_div) P.user_div[pair] = static_cast<float>(value);
            }
        }
        if constexpr (MODE == MODE_KLP) {
            // The log-domain value where it is larger by more than its own rounding can explain.  (One pair after the other, behind the
            // others' code, which its logarithms in float64 made half as long again: bfloat16 KL, 5 sequences of 1, V=64896 8.0 -> 7.6 us a call, one of 9,
            // V=130176 10.7 -> 10.4; binary32 KL 1 %.)
            for (again = __builtin_amdgcn_readfirstlane(again); again != 0; again &= again - 1) {
                const int pair = base + 4 * __builtin_ctz(again);
                const unsigned long long* p[1] = {shares + (static_cast<size_t>(pair) * P.G + (in ? lane : P.G - 1)) * NP};
                unsigned long long v[1][NP];
                double lse2_t = first_t, lse2_d = first_d;
                bool ok = await_tagged<NP, 1>(p, P.nonce, P.spin_limit, v);
                if (!P.want_ratio) ok = row_logs(pair, lse2_t, lse2_d) && ok;
                const double first = wave_sum(in ? number(v[0], 0) : 0.0), logs = wave_sum(in ? number(v[0], 1) : 0.0);
                const double dl = (lse2_t - lse2_d) * kLn2, log_value = logs - dl;
                double value = fmax(0.5 * kLn2 * first, 0.0);
                if (log_value - value > 4e-7 * (fabs(logs) + fabs(dl))) value = log_value;
                if (!ok) value = __builtin_nan("");
                if (lane == 0) {
                    if (P.draw_wgs) {
                        s.div[pair - pair0] = static_cast<float>(value);
                        if (!ok) s.status[pair - pair0] = FSD_ROW_INTERNAL;
                    } else {
                        P.ws.div[pair] = static_cast<float>(value);
                        if (!ok) { P.ws.pst[pair] = FSD_ROW_INTERNAL; flag_failure(P.ws); }
                    }
                    if (P.user_div) P.user_div[pair] = static_cast<float>(value);
                }
            }
        }
    }
    if (P.draw_wgs == 0) return;
    __syncthreads();
    if (wave != 0) return;
    const bool mine = lane < rows;
    const float div = mine ? s.div[lane] : 0.0f;
    int status = mine ? s.status[lane] : 0;
    if (__any(status != 0)) {
#pragma unroll
        for (int o = 32; o > 0; o >>= 1) status |= __shfl_xor(status, o);
    }
    const bool accepted = div <= P.T;   // Sec. 4 eq. 4 (NaN compares false)
    int n, row, winner = -1, my_dep = 0;
    if (P.parent) {
        const TreePick pick = pick_path(lane, rows, P.max_depth, my_par, accepted);
        status |= pick.status;
        if (status & FSD_ROW_BAD_PARENT) status &= ~FSD_ROW_TOO_DEEP;   // depths mean nothing in a malformed tree
        n = pick.n;
        winner = pick.winner;
        my_dep = pick.my_dep;
        row = winner + 1;
    } else {
        const unsigned long long no = __ballot(mine && !accepted);
        n = no ? static_cast<int>(__builtin_ctzll(no)) : rows;
        row = n;
    }
    const int token = s.drawn[row].idx;
    if (!status) status = s.drawn_status[row];
    if (status) n = 0;
    if (P.parent) {
        write_path(lane, P.max_depth, status ? -1 : winner, n, my_par, my_dep, token_in, status ? -1 : token,
                   P.path_nodes + static_cast<size_t>(b) * P.max_depth, P.out_tokens + static_cast<size_t>(b) * (P.max_depth + 1));
    } else {
        int32_t* const out = P.out_tokens + static_cast<size_t>(b) * (rows + 1);
        for (int i = lane; i <= rows; i += 64) {
            int v = -1;
            if (!status) v = i < n ? token_in : i == n ? token : -1;
            out[i] = v;
        }
    }
    if (lane == 0) {
        P.out_len[b] = n;
        if (P.row_status) P.row_status[b] = status;
    }
}

template <bool BF16, int NV, int MODE, int LD>
__global__ __launch_bounds__(kWG) void small_call(SmallParams P) {
    __shared__ SmallShared s;
    const int wg = static_cast<int>(blockIdx.x);
    if (wg < P.team_wgs) {
        small_team<BF16, NV, MODE, LD>(P, wg * (kWG / 64) + __builtin_amdgcn_readfirstlane(static_cast<int>(threadIdx.x >> 6)));
    } else if (wg < P.team_wgs + P.draw_wgs) {
        const int d = wg - P.team_wgs, row = d / P.GS;
        small_draw<BF16, LD>(P, row, d - row * P.GS, s);
    } else {
        small_finish<BF16, MODE>(P, wg - P.team_wgs - P.draw_wgs, s);
    }
}

}  // namespace

#endif  // FSD_CSRC_SMALL_CALL_H_
