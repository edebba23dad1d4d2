// Host side and C ABI of libfsd, the FSD candidate-verification step for gfx950 (MI355X).
//
// A verify call launches
//   zero_counters   (device_common.h) clears the counters and exchange words of the call (only where there
//                   are more than 4 MB of them: otherwise the reduction kernel does it itself)
//   pair_kernel     (pair_kernel.h) the vocabulary reduction: one (target row, draft row) pair is
//                   split over a team of G wavefronts; every wavefront loads its slice of both rows
//                   ONCE into registers with 128-bit loads, the team exchanges the softmax
//                   normalisers through 64-bit words in the workspace, and the divergence (paper
//                   App. C.1-C.3) is accumulated from the registers.  One member per pair (they take
//                   turns) adds the team's partial sums in a fixed order: run-to-run identical results.
//   tree_sd_walk    (tree_sd_walk.h) strict SD on a token tree only: the walk over the children
//   warp_select     (warp_select.h) warped calls only: the cut of temperature / top-k / top-p
//   accept_sample   (accept_sample.h) per sequence: the accepted prefix (Sec. 4, eq. 4) or accepted
//                   tree path (Sec. 6.4) or the strict-SD acceptance (Sec. 3, eq. 1-2), then the extra
//                   token by Gumbel-max over the vocabulary of one target row, split over GS workgroups.
// The plain FSD calls on a few sequences launch small_call (small_call.h) alone, and fsd_calibrate_threshold the
// kernels of calibrate.h.
//
// Nothing here is shared with the CPU oracle: Philox4x32-10 and the exact-operation logarithm
// are implemented a second time from their published / stated definitions.

#include <hip/hip_runtime.h>
#include <hip/hip_ext.h>
#include <stdint.h>
#include <float.h>
#include <limits.h>
#include <math.h>

#include <atomic>
#include <chrono>

#include "fsd.h"

#include "device_common.h"
#include "pair_kernel.h"
#include "accept_sample.h"
#include "small_call.h"
#include "tree_sd_walk.h"
#include "warp_select.h"
#include "calibrate.h"

// Workspace of fsd_verify_chain_static, the entry point for callers that cannot allocate: device
// memory that exists from the moment the library is loaded until the process ends, one copy per
// GPU.  Host code never uses this name as an address (on the host it is only a stand-in for the
// symbol): static_scratch() asks the runtime for the array's device address once per device.
static __device__ __align__(256) unsigned char scratch[FSD_STATIC_SCRATCH_BYTES];

namespace {

// ------------------------------------------------------------------------------------------
// host side: planning, workspace, launches

struct Plan {
    int VE, NV, G, spm, GS, sps;   // G = wavefronts per pair
    long nslots;
    size_t off_counters, n_counters, off_state, off_wz, off_part1, off_arrive, zero_bytes, off_div, off_pst, off_lse2, off_lr, off_spart,
        off_thr, off_tsd, off_tsdz, bytes;
};

inline size_t align_up(size_t x, size_t a) { return (x + a - 1) / a * a; }

constexpr int kMaxTeam = 256;     // wavefronts per pair (merged in rounds of 64)
int g_shape_nv = 0;               // 0 = chosen by make_plan (see fsd_debug_set_shape)

// wavefronts per pair when every lane holds nv slots of each row.  A team is a run of consecutive
// wavefronts of the grid, not of whole workgroups: at V = 128256 (bfloat16, 5 slots per lane) 51
// members do, 40 teams fit the device instead of the 39 of 52, and 512 pairs take 13 rounds, not 14.
long team_size(long nslots, int nv) {
    const long per_wave = 64L * nv;
    return (nslots + per_wave - 1) / per_wave;
}

bool make_plan(int B, int rows, long V, int dtype, Plan& p) {
    if (B < 1 || B > 65535 || rows < 1 || rows > kMaxRows || V < 1) return false;
    if (dtype != FSD_F32 && dtype != FSD_BF16) return false;
    if (static_cast<long>(B) * rows >= (1L << 24)) return false;
    if (V > fsd_max_vocab(dtype)) return false;
    p.VE = (dtype == FSD_BF16) ? 8 : 4;
    p.nslots = (V + p.VE - 1) / p.VE;
    // 32 vocabulary entries of each row per lane: 4 slots of bfloat16, 8 of binary32
    p.NV = (dtype == FSD_BF16) ? 4 : 8;
    if (g_shape_nv && !(dtype == FSD_BF16 && g_shape_nv > 5) && team_size(p.nslots, g_shape_nv) <= kMaxTeam) p.NV = g_shape_nv;
    const long G = team_size(p.nslots, p.NV);
    if (G > kMaxTeam) return false;
    p.G = static_cast<int>(G);
    p.spm = static_cast<int>((p.nslots + G - 1) / G);
    long GS = (kSampleWGs + B - 1) / B;
    const long maxgs = (p.nslots + kWG - 1) / kWG;
    if (GS > maxgs) GS = maxgs;
    if (GS > 64) GS = 64;
    if (GS < 1) GS = 1;
    p.GS = static_cast<int>(GS);
    p.sps = static_cast<int>((p.nslots + GS - 1) / GS);
    const size_t R = static_cast<size_t>(B) * rows;
    size_t o = 0;
    p.off_counters = o; p.n_counters = 64 + static_cast<size_t>(B) * kSdoneStride; o = align_up(o + p.n_counters * 4, 256);
    p.off_state = o; o = align_up(o + R * 8, 256);
    p.off_wz = o; o = align_up(o + R * kWalkShare * 8, 256);
    // (a share is one word of 8 bytes; it used to be 32 bytes, and the size that callers are told stays what it was)
    p.off_spart = o; o = align_up(o + static_cast<size_t>(B) * p.GS * 32, 256);
    // the two exchange arrays: 8 words of 8 bytes for every member of the plan's team, twice what the mode that posts
    // most (4 words a member) needs of it, so that a shape may have twice the members (small binary32 calls do).  A call
    // lays them out densely for its own mode and shape (see carve) and clears only that much
    p.off_part1 = o; o = align_up(o + R * p.G * 32, 256) + align_up(R * p.G * 32, 256);
    p.zero_bytes = o;
    p.off_div = o; o = align_up(o + R * 4, 256);
    p.off_pst = o; o = align_up(o + R * 4, 256);
    p.off_lse2 = o; o = align_up(o + R * 16, 256);
    p.off_lr = o; o = align_up(o + R * 8, 256);
    p.off_thr = o; o = align_up(o + static_cast<size_t>(B) * 4, 256);
    p.off_tsd = o; o = align_up(o + static_cast<size_t>(B) * (4 + rows) * 4, 256);
    p.off_tsdz = o; o = align_up(o + static_cast<size_t>(B) * rows * 4, 256);
    p.off_arrive = o; o = align_up(o + static_cast<size_t>(kMaxArrive) * 8, 256);
    p.bytes = o;
    return true;
}

// upper bound of the wavefronts a grid of this device can hold at once (32 per compute unit)
long max_resident_wavefronts() {
    static long cached[16] = {};
    int dev = 0;
    (void)hipGetDevice(&dev);
    if (dev < 0 || dev >= 16) dev = 0;
    if (cached[dev] == 0) {
        int cus = 0;
        if (hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess || cus < 1) cus = 1024;
        cached[dev] = static_cast<long>(cus) * 32;
    }
    return cached[dev];
}

// a number for every call: never 0, never the same twice in a process, and unlikely to be what
// another process left in memory (the failure word and the arrival slots compare against it)
unsigned long long next_nonce() {
    static std::atomic<unsigned long long> counter{
        static_cast<unsigned long long>(std::chrono::steady_clock::now().time_since_epoch().count()) * 0x9E3779B97F4A7C15ull};
    unsigned long long n = 0;
    while (n == 0) n = counter.fetch_add(0x9E3779B97F4A7C15ull, std::memory_order_relaxed);
    return n;
}

// G, n1, n2: wavefronts per pair and exchange words per member of this call's reduction kernel (G (n1 + n2) is at most
// 8 times the plan's G: the caller checks); zero_bytes: how much of the workspace's head the call has to clear
Ws carve(void* workspace, const Plan& p, int B, int rows, int G, int n1, int n2, size_t& zero_bytes) {
    char* base = static_cast<char*>(workspace);
    const size_t R = static_cast<size_t>(B) * rows;
    Ws w;
    w.counters = reinterpret_cast<unsigned*>(base + p.off_counters);
    w.sdone = w.counters + 64;
    w.state = reinterpret_cast<unsigned long long*>(base + p.off_state);
    w.part1 = reinterpret_cast<unsigned long long*>(base + p.off_part1);
    const size_t off_part2 = align_up(p.off_part1 + R * G * n1 * 8, 256);
    w.part2 = reinterpret_cast<double*>(base + off_part2);
    zero_bytes = align_up(off_part2 + R * G * n2 * 8, 256);
    w.div = reinterpret_cast<float*>(base + p.off_div);
    w.pst = reinterpret_cast<int*>(base + p.off_pst);
    w.lse2 = reinterpret_cast<double*>(base + p.off_lse2);
    w.lr = reinterpret_cast<double*>(base + p.off_lr);
    w.spart = reinterpret_cast<unsigned long long*>(base + p.off_spart);
    w.thr = reinterpret_cast<float*>(base + p.off_thr);
    w.tsd = reinterpret_cast<int*>(base + p.off_tsd);
    w.tsd_invz = reinterpret_cast<float*>(base + p.off_tsdz);
    w.wz = reinterpret_cast<unsigned long long*>(base + p.off_wz);
    w.arrive = reinterpret_cast<unsigned long long*>(base + p.off_arrive);
    w.nonce = next_nonce();
    return w;
}

unsigned g_spin_limit = 1u << 22;
unsigned g_selection_spin_limit = UINT_MAX;   // test hook: a smaller limit for the selection's wait alone
// The entropy form of JS (bfloat16 logits) carries an absolute error of a few 1e-7 whatever the
// result: below this floor (nats) a pair is evaluated again in the pointwise form, so that what the
// caller sees is within 2e-3 relative everywhere (with a margin of five to ten).
constexpr float kJsFloor = 1e-3f;
float g_js_floor = kJsFloor;
bool g_exact_js = false;   // test hook: bfloat16 JS in the pointwise form only
bool g_self_clear = true;  // test hook: 0 = every call launches the clearing kernel
bool g_small_calls = true; // test hook: 0 = no call takes small_call
#ifdef FSD_PHASE_TIMING
unsigned long long* g_dbg = nullptr;
#endif

// ---- optional event timing of pair_kernel
constexpr int kMaxProf = 4096;
bool g_prof_on = false;
int g_prof_n = 0;
hipEvent_t g_prof_ev[2 * kMaxProf];
bool g_prof_made = false;
hipEvent_t* g_prof_pair = nullptr;   // the two events of the reduction launch being timed, if any

// How many workgroups of a kernel are resident at once on the current device, and how much unused
// dynamic LDS to ask for so that the hardware cannot place more than that number on any one CU.
// Without the padding a grid that does not fill every slot may be spread unevenly (some CUs full,
// others half empty), and the team members that share a pair then all run at the pace of the most
// crowded CU.  The padding leaves 8 KB of slack so that it can only lower the count it is checked
// against, never the number of workgroups that really fit.
struct Residency { int total; unsigned pad_lds; };

int g_last_grid = 0, g_last_total = 0;

template <typename Kernel>
Residency residency_of(Kernel kernel, int threads, Residency (&cache)[16], int most = 0) {
    int dev = 0;
    (void)hipGetDevice(&dev);
    if (dev < 0 || dev >= 16) dev = 0;
    if (cache[dev].total == 0) {
        int per_cu = 0, cus = 0, lds_cu = 0;
        if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, kernel, threads, 0) != hipSuccess) per_cu = 1;
        if (hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess) cus = 64;
        if (hipDeviceGetAttribute(&lds_cu, hipDeviceAttributeMaxSharedMemoryPerMultiprocessor, dev) != hipSuccess) lds_cu = 0;
        if (most > 0 && per_cu > most) per_cu = most;   // (the padding below keeps them apart)
        if (per_cu < 1) per_cu = 1;
        if (cus < 1) cus = 1;
        unsigned pad = 0;
        hipFuncAttributes attr;
        if (lds_cu > 16384 && hipFuncGetAttributes(&attr, reinterpret_cast<const void*>(kernel)) == hipSuccess) {
            const long stat = static_cast<long>(attr.sharedSizeBytes);
            const long want = ((static_cast<long>(lds_cu) - 8192) / per_cu - stat) / 1024 * 1024;
            if (want > 0 && (stat + want) * (per_cu + 1) > lds_cu) {
                bool ok = true;
                if (stat + want > 65536)
                    ok = hipFuncSetAttribute(reinterpret_cast<const void*>(kernel), hipFuncAttributeMaxDynamicSharedMemorySize,
                                             static_cast<int>(want)) == hipSuccess;
                int check = 0;
                if (ok && hipOccupancyMaxActiveBlocksPerMultiprocessor(&check, kernel, threads, static_cast<size_t>(want)) == hipSuccess &&
                    check == per_cu)
                    pad = static_cast<unsigned>(want);
            }
        }
        (void)hipGetLastError();
        cache[dev] = Residency{per_cu * cus, pad};
    }
    g_last_total = cache[dev].total;
    return cache[dev];
}

template <bool BF16, int NV, int MODE, int LD, bool TSHARED = false, bool EVEN = false>
void launch_pair_k(hipStream_t st, const PairParams& P0) {
    // persistent grid: as many whole teams as fit on the device at once (at least one, whose workgroups
    // fit by the limit on the team size), in whole workgroups; the wavefronts left over leave at once
    static Residency cache[16] = {};
    const Residency res = residency_of(pair_kernel<BF16, NV, MODE, LD, TSHARED, EVEN>, kWG, cache, pair_kernel_most(BF16, NV, MODE));
    const long waves_per_wg = kWG / 64;
    long nteams = res.total * waves_per_wg / P0.G;
    if (nteams > P0.npairs) nteams = P0.npairs;
    if (nteams < 1) nteams = 1;
    const long grid = (nteams * P0.G + waves_per_wg - 1) / waves_per_wg;
    PairParams P = P0;
    P.nteams = static_cast<int>(nteams);
    g_last_grid = static_cast<int>(grid);
    if (g_prof_pair) {
        // timed launch: the events take the start and the end of this dispatch itself (what a
        // kernel trace shows), not the time between two markers around it in the stream
        hipExtLaunchKernelGGL((pair_kernel<BF16, NV, MODE, LD, TSHARED, EVEN>), dim3(static_cast<unsigned>(grid)), dim3(kWG), res.pad_lds, st,
                              g_prof_pair[0], g_prof_pair[1], 0, P);
    } else {
        hipLaunchKernelGGL((pair_kernel<BF16, NV, MODE, LD, TSHARED, EVEN>), dim3(static_cast<unsigned>(grid)), dim3(kWG), res.pad_lds, st, P);
    }
}
template <bool BF16, int NV, int MODE>
void launch_pair_a(int load, hipStream_t st, const PairParams& P) {
    // a tree (shared target rows) has variants of its own, for 16-byte aligned rows and, on others, for the
    // library's own shapes of large calls.  (A small binary32 call, 4 slots, is one step per wavefront and has no sibling
    // to share with: 1 tree of 16 nodes, V=32001, with and without 16.4 us JS, 31.7 strict SD; of 8, V=128001 34.6 and 33.7.)
    constexpr bool kOwn = BF16 ? (NV == 4 || NV == 6) : (NV >= 8);
    const bool shared = P.parent != nullptr;
    if (load == LOAD_ALIGNED) {
        if (shared) launch_pair_k<BF16, NV, MODE, LOAD_ALIGNED, true>(st, P);
        else launch_pair_k<BF16, NV, MODE, LOAD_ALIGNED>(st, P);
    } else {
        if constexpr (kOwn) {
            if (shared) { launch_pair_k<BF16, NV, MODE, LOAD_WIDE, true>(st, P); return; }
        }
        // Chains of bfloat16 rows some of which begin in the middle of a 32-bit word: see pair_kernel's EVEN.  (Other rows would only pay for it, V=128258
        // 71.7 -> 74.9 us; trees of odd rows 208 -> 211, the entropy form's kernel has no registers left there.)
        if constexpr (BF16 && (NV == 6 || (NV == 4 && (MODE == MODE_LSE || MODE == MODE_KL)))) {
            if (P.V % 2 != 0 || ((reinterpret_cast<uintptr_t>(P.target) | reinterpret_cast<uintptr_t>(P.draft)) & 2) != 0) {
                launch_pair_k<BF16, NV, MODE, LOAD_WIDE, false, true>(st, P);
                return;
            }
        }
        launch_pair_k<BF16, NV, MODE, LOAD_WIDE>(st, P);
    }
}
template <bool BF16, int NV>
void launch_pair_m(int mode, int load, hipStream_t st, const PairParams& P) {
    switch (mode) {
        case MODE_KL: launch_pair_a<BF16, NV, MODE_KL>(load, st, P); break;
        case MODE_JS: launch_pair_a<BF16, NV, MODE_JS>(load, st, P); break;
        case MODE_TV: launch_pair_a<BF16, NV, MODE_TV>(load, st, P); break;
        case MODE_KLP: launch_pair_a<BF16, NV, MODE_KLP>(load, st, P); break;
        case MODE_JSE: launch_pair_a<BF16, NV, MODE_JS>(load, st, P); break;   // (its own shape is launched by launch_pair)
        default: launch_pair_a<BF16, NV, MODE_LSE>(load, st, P); break;
    }
}
// the large shape of the bfloat16 single-pass kernels: see where it is chosen
template <int MODE>
void launch_pair_single(int load, hipStream_t st, const PairParams& P) {
    if (load != LOAD_ALIGNED) launch_pair_k<true, 8, MODE, LOAD_WIDE, true>(st, P);
    else if (P.parent != nullptr) launch_pair_k<true, 8, MODE, LOAD_ALIGNED, true>(st, P);
    else launch_pair_k<true, 8, MODE, LOAD_ALIGNED>(st, P);
}
// rows shorter than a slot: one shape
template <bool BF16>
void launch_pair_elem(int mode, hipStream_t st, const PairParams& P) {
    switch (mode) {
        case MODE_KL: launch_pair_k<BF16, 2, MODE_KL, LOAD_ELEM>(st, P); break;
        case MODE_JS: launch_pair_k<BF16, 2, MODE_JS, LOAD_ELEM>(st, P); break;
        case MODE_TV: launch_pair_k<BF16, 2, MODE_TV, LOAD_ELEM>(st, P); break;
        case MODE_KLP: launch_pair_k<BF16, 2, MODE_KLP, LOAD_ELEM>(st, P); break;
        default: launch_pair_k<BF16, 2, MODE_LSE, LOAD_ELEM>(st, P); break;
    }
}
void launch_pair(int dtype, int NV, int mode, int load, hipStream_t st, const PairParams& P) {
    const bool prof = g_prof_on && g_prof_n < kMaxProf;
    if (prof) {
        if (!g_prof_made) {
            for (int i = 0; i < 2 * kMaxProf; ++i) (void)hipEventCreate(&g_prof_ev[i]);
            g_prof_made = true;
        }
        g_prof_pair = &g_prof_ev[2 * g_prof_n];
    }
    if (load == LOAD_ELEM) {
        if (dtype == FSD_BF16) launch_pair_elem<true>(mode, st, P);
        else launch_pair_elem<false>(mode, st, P);
    } else if (dtype == FSD_BF16) {
        if (NV == 2) launch_pair_m<true, 2>(mode, load, st, P);
        else if (NV == 6) {   // the library's own shape of the two-phase kernels
            if (mode == MODE_JSE) launch_pair_a<true, 6, MODE_JSE>(load, st, P);
            else if (mode == MODE_TV) launch_pair_a<true, 6, MODE_TV>(load, st, P);
            else launch_pair_a<true, 6, MODE_JS>(load, st, P);
        }
        else if (NV == 5) launch_pair_m<true, 5>(mode, load, st, P);
        else if (NV == 8) {   // the library's own shape of the single-pass kernels
            if (mode == MODE_KL) launch_pair_single<MODE_KL>(load, st, P);
            else launch_pair_single<MODE_LSE>(load, st, P);
        }
        else launch_pair_m<true, 4>(mode, load, st, P);
    } else {
        if (NV == 2) launch_pair_m<false, 2>(mode, load, st, P);
        else if (NV == 4) launch_pair_m<false, 4>(mode, load, st, P);
        else if (NV == 10) {   // the library's own shape of the two-phase kernels
            if (mode == MODE_KLP) launch_pair_a<false, 10, MODE_KLP>(load, st, P);
            else if (mode == MODE_TV) launch_pair_a<false, 10, MODE_TV>(load, st, P);
            else launch_pair_a<false, 10, MODE_JS>(load, st, P);
        }
        else launch_pair_m<false, 8>(mode, load, st, P);
    }
    if (prof) {
        g_prof_pair = nullptr;
        ++g_prof_n;
    }
}

template <bool BF16, int LD>
void launch_sample_k(int kind, dim3 grid, size_t lds, hipStream_t st, const SampleParams& P) {
    switch (kind) {
        case KIND_CHAIN: hipLaunchKernelGGL((accept_sample<BF16, LD, KIND_CHAIN>), grid, dim3(kWG), lds, st, P); break;
        case KIND_TREE: hipLaunchKernelGGL((accept_sample<BF16, LD, KIND_TREE>), grid, dim3(kWG), lds, st, P); break;
        case KIND_RFSD: hipLaunchKernelGGL((accept_sample<BF16, LD, KIND_RFSD>), grid, dim3(kWG), lds, st, P); break;
        case KIND_TREESD: hipLaunchKernelGGL((accept_sample<BF16, LD, KIND_TREESD>), grid, dim3(kWG), lds, st, P); break;
        default: hipLaunchKernelGGL((accept_sample<BF16, LD, KIND_SD>), grid, dim3(kWG), lds, st, P); break;
    }
}
void launch_sample(int dtype, int load, int kind, dim3 grid, size_t lds, hipStream_t st, const SampleParams& P) {
    if (dtype == FSD_BF16) {
        if (load == LOAD_ALIGNED) launch_sample_k<true, LOAD_ALIGNED>(kind, grid, lds, st, P);
        else if (load == LOAD_WIDE) launch_sample_k<true, LOAD_WIDE>(kind, grid, lds, st, P);
        else launch_sample_k<true, LOAD_ELEM>(kind, grid, lds, st, P);
    } else {
        if (load == LOAD_ALIGNED) launch_sample_k<false, LOAD_ALIGNED>(kind, grid, lds, st, P);
        else if (load == LOAD_WIDE) launch_sample_k<false, LOAD_WIDE>(kind, grid, lds, st, P);
        else launch_sample_k<false, LOAD_ELEM>(kind, grid, lds, st, P);
    }
}

// ---- small calls (small_call.h): every pair's wavefronts at once, one step each
// Which of its forms a call may take, each where it is the fastest.  Whole calls (us) by the persistent teams, by the reduction in one
// step with the sampler behind it, and in one launch; (n) is n sequences of 8 unless said otherwise, [n] one tree of n nodes.
//   reduction  one step of the whole device, until the members' words cost more than the teams' second step.
//     JS   bfloat16 V=32000 [60] 16.7 14.6, 3 of 60 19.9 19.2; V=64000 (8) 18.6 16.6, (12) 19.6 19.6; V=128256 [30] 18.4 17.1, [36] 19.0 19.5, (4)
//          18.9 17.3, (5) 19.7 19.1, (6) 20.1 20.9, 7 of 5 18.8 18.5, 8 of 5 19.1 19.7; V=256000, 5 of 4 21.3 20.7; V=210901, 2 of 14 23.6 21.7
//          binary32 V=32000 [30] 13.8 13.8, 22 of 5 17.6 17.6, 28 of 5 19.7 21.1, 7 of 16 nodes 17.8 17.9, 10 of 16 nodes 22.7 21.5; V=50257, 14 of 5 18.1
//          17.8, 18 of 5 20.2 21.3; V=64000, 11 of 5 18.1 18.0, 16 of 5 20.8 22.6, 6 of 16 nodes 23.0 22.0; V=100000, 7 of 5 17.9 18.7; V=128256, 6 of 5 18.0
//          19.3.  (From 1 million entries on, where the teams need one step, about 2 million, that is the faster one.  The binary32 lines
//          come from teams of one wavefront a SIMD, as `step` below does; with today's the break-even of chains lies at 3.5 million entries, of long rows and
//          under TV at 3.25, and what lies between the two is up to 11 % slower in one step of the device than it would be with the teams.)
//     TV   bfloat16 V=32000 [60] 15.7 14.9; V=64000 (4) 14.9 14.6, (6) 15.2 16.2; V=128256 (2) 15.1 15.2, (3) 15.6 16.4; V=200000, 4 of 4 18.1 17.6,
//          6 of 4 19.6 20.1; rows that are not 16-byte aligned V=40265, 21 of 4 19.7 17.6, V=235817, 2 of 9 22.3 19.1
//          binary32 V=32000 [30] 13.6 14.5, [60] 15.1 16.1, 28 of 5 19.5 21.5; V=50257, 14 of 5 18.3 18.4, 18 of 5 19.9 21.4; V=64000 (4) 15.2 17.2, 14 of 5
//          19.8 21.6; V=98752 [41], three steps of the teams, 21.5 20.6
//     KL   binary32 V=32000, 22 of 5 19.8 18.8, 37 of 5 25.6 24.7, 10 of 16 nodes 26.3 22.7; V=64000, 11 of 5 20.3 19.3, 19 of 5 25.8 25.2; V=100000, 7 of 5 20.3
//          20.4, 10 of 5 23.0 25.5; V=128256, 6 of 5 20.1 21.0, 8 of 5 22.6 25.1; bfloat16 has a single pass in large calls: V=32000 [30] 13.3 14.9
//     Reducible FSD: JS bfloat16 V=64000 (12) 20.5 19.3, V=128256 (4) 19.6 17.1, (6) 20.9 21.0; TV V=64000 (8) 19.5 17.2, V=128256 (5) 20.3 20.9.
//   one launch draws from all rows, and one workgroup a sequence reads all its words: worth less the more of both there is.
//     JS   bfloat16 V=128256 (2) 16.4 14.4 11.3, (3) 16.8 15.9 14.8, (4) 18.9 17.3 17.7; [16] 16.7 14.8 12.2, [30] 18.4 17.1 18.6; V=32000 [30] 16.3 14.4
//          11.9, [60] 16.7 14.6 17.0; V=64000 [30] 16.7 14.7 12.8
//          binary32 V=32000 [30] 13.8 13.8 11.8, [60] 15.1 15.5 18.9; V=64000 [30] 15.0 15.9 16.1; V=128256 [16] 15.6 15.5 14.8, (3) 18.8 18.0 17.4
//     KL   bfloat16 V=32000, 8 of 5 12.9 14.4 10.3, 12 of 5 13.0 14.6 14.2, [16] 13.2 14.1 10.4, [30] 13.3 14.9 14.5
//   replays    of one launch have a kernel before it that clears its words, 2 us: the larger ones take the reduction instead, in the same
//          shape, so that a replay gives what the eager call gives.  JS, V=32000 8 of 5 bfloat16 15.3 13.0 11.6, binary32 13.4 13.8
//          11.9, 12 of 5 binary32 14.2 15.3 15.1; V=64000 [30] bfloat16 16.3 14.2 15.0; V=128256 (3) 16.4 16.0 16.5; KL binary32 V=64000 (6) 20.9 19.1
//          20.5; but TV binary32 V=64000 (4) 14.6 17.5 15.3.
struct SmallForms { bool reduction, whole, whole_replayed; };
SmallForms small_forms(int kind, int dtype, int div, int B, int rows, long V, bool aligned) {
    constexpr long M = 1L << 20;
    const bool bf16 = dtype == FSD_BF16, tv = div == FSD_DIV_TV, js = div == FSD_DIV_JS, single_pass = bf16 && div == FSD_DIV_KL, long_rows = V > 3L << 15;
    const long entries = static_cast<long>(B) * rows * V, drawn = static_cast<long>(B) * (rows + 1) * V, bytes = drawn * (bf16 ? 2 : 4);
    const bool ratio = kind == KIND_RFSD;
    SmallForms f{false, false, false};
    if (single_pass) f.reduction = false;   // (reducible FSD: its normalisers' sums are float64 there)
    else if (ratio) f.reduction = entries <= (tv ? 9 * M / 2 : 6 * M);
    else if (bf16 && js) f.reduction = entries <= (!long_rows || V > 1L << 17 || !aligned ? 6 * M : kind == KIND_CHAIN ? 5 * M : 4 * M);   // (4 slots a lane, many members)
    else if (bf16) f.reduction = entries <= (!aligned ? 9 * M / 2 : V > 1L << 17 ? 15 * M / 4 : 2 * M);
    else if (div == FSD_DIV_KL) f.reduction = entries <= 6 * M;
    else {
        // pairs that teams of 8 slots a lane and a wavefront a SIMD take in a step (see the table above)
        const long step = max_resident_wavefronts() / 8 / team_size((V + 3) / 4, 8), pairs = static_cast<long>(B) * rows;
        if (js) f.reduction = entries <= (long_rows ? 4 * M : 6 * M) && (entries <= M || pairs > step);
        else f.reduction = entries <= (long_rows ? 4 * M : 9 * M / 2) && pairs > (long_rows ? 2 * step : step);
    }
    const long most = single_pass ? 40 * M : js && !bf16 ? 144 * M : 120 * M;   // rows times bytes drawn from
    f.whole = !ratio && rows <= 32 && entries <= (single_pass ? 9 * M / 8 : 6 * M) && drawn <= 4 * M && rows * bytes <= most;
    f.whole_replayed = (tv && !bf16) || (bytes <= 6 * M && rows * bytes <= 60 * M);
    return f;
}
// Draws of all target rows in the same launch: workgroups aimed at, at most, and rounds one
// of them may take (half the workgroups, with twice the rounds: 1 sequence of 8, V=128256 8.5 -> 9.2; twice as many: 4 of 8 15.2 -> 16.1).
constexpr long kSmallDraws = 1024, kSmallRounds = 4;
// Two slots a lane while that leaves a wavefront a SIMD or less of its own, else four: half the words to read for
// twice the work of a step.  Whole calls with two and four (us): V=32000, bfloat16, 512 wavefronts 7.41 and 7.58, 1024 9.15 and
// 8.49; binary32, 504 6.90 and 6.80, 1008 7.67 and 7.06, 2016 10.7 and 8.3; V=32001 504 7.57 and 8.09, 1008 8.92 and 8.62.
constexpr long kSmallWaves = 640;

template <bool BF16, int NV, int MODE, int LD>
bool launch_small_k(hipStream_t st, SmallParams& P, int B, bool captured) {
    static Residency cache[16] = {};
    const Residency res = residency_of(small_call<BF16, NV, MODE, LD>, kWG, cache);
    if (P.team_wgs > res.total) return false;   // (the members of a team wait for each other; they come first in the grid)
    g_last_grid = P.team_wgs;
    const int finish = P.draw_wgs ? B : (P.npairs + P.finish - 1) / P.finish;
    P.words16 = (static_cast<long>(P.npairs) * P.G * (4 + P.np) + static_cast<long>(P.draw_wgs) * 2 + 1) / 2;
    if (captured && P.draw_wgs) {
        // A replay has the number of the call that was recorded: what the replay before it left would count as its own.  (Where
        // the sampler follows it clears the words, see run: whatever this kernel's wavefronts had to post is there by then.)
        hipLaunchKernelGGL(zero_counters, dim3(static_cast<unsigned>((P.words16 + 255) / 256)), dim3(256), 0, st,
                           reinterpret_cast<uint4*>(P.words), P.words16);
    }
    hipLaunchKernelGGL((small_call<BF16, NV, MODE, LD>), dim3(static_cast<unsigned>(P.team_wgs + P.draw_wgs + finish)), dim3(kWG), 0, st, P);
    return true;
}
template <bool BF16, int NV, int LD>
bool launch_small_m(int div, hipStream_t st, SmallParams& P, int B, bool captured) {
    return div == FSD_DIV_JS ? launch_small_k<BF16, NV, MODE_JS, LD>(st, P, B, captured)
         : div == FSD_DIV_TV ? launch_small_k<BF16, NV, MODE_TV, LD>(st, P, B, captured) : launch_small_k<BF16, NV, MODE_KLP, LD>(st, P, B, captured);
}
enum { SMALL_NONE = 0, SMALL_REDUCED = 1, SMALL_DONE = 2 };   // launched: nothing, the reduction alone, the whole call
std::atomic<int> g_last_route{SMALL_NONE};   // of the last verify call (see fsd_debug_last_route)
template <bool BF16, int LD>
int launch_small(int div, hipStream_t st, SmallParams& P, int B, int plan_G, SmallForms may, bool captured) {
    constexpr int VE = Slot<BF16>::VE;
    P.np = small_share_words(div == FSD_DIV_JS ? MODE_JS : MODE_TV);
    const long all = static_cast<long>(B) * (P.rows + 1), round = 8 / VE * kWG;
    long GS = may.whole ? kSmallDraws / all : 0;
    if (GS > (P.nslots + round - 1) / round) GS = (P.nslots + round - 1) / round;
    if (GS > 64) GS = 64;
    if (P.nslots > GS * round * kSmallRounds) GS = 0;
    bool no_room = false;   // (one launch in a larger shape than its teams need is slower than the teams: 7 sequences of 11, V=47744 TV 18.6 and 16.6)
    const auto launch = [&](int NV) {
        P.G = static_cast<int>(team_size(P.nslots, NV));
        const long words = static_cast<long>(P.npairs) * P.G * (4 + P.np);
        P.team_wgs = (P.npairs * P.G + kWG / 64 - 1) / (kWG / 64);
        if (P.G > kSmallTeam) return false;
        // the words lie in the place of the arrival slots, or, more of them, in that of the exchange words
        const bool few = words + all * GS * 2 <= kMaxArrive;
        if (!few && P.G * (4 + P.np) > plan_G * 8) return false;
        P.words = few ? P.ws.arrive : P.ws.part1;
        P.GS = few ? static_cast<int>(GS) : 0;
        P.draw_wgs = static_cast<int>(all) * P.GS;
        P.sps = P.GS ? static_cast<int>((P.nslots + P.GS - 1) / P.GS) : 0;
        if (!P.GS && !may.reduction) { no_room = true; return false; }
        if (captured && !may.whole_replayed) P.draw_wgs = P.GS = 0;
        return NV == 2 ? launch_small_m<BF16, 2, LD>(div, st, P, B, captured)
             : NV == 4 ? launch_small_m<BF16, 4, LD>(div, st, P, B, captured) : launch_small_m<BF16, 8, LD>(div, st, P, B, captured);
    };
    const bool two = P.npairs * team_size(P.nslots, 2) <= kSmallWaves;
    if ((two && launch(2)) || launch(4) || (!no_room && launch(8))) return P.draw_wgs ? SMALL_DONE : SMALL_REDUCED;
    return SMALL_NONE;
}

// The workgroups that share a sequence wait for each other, so the whole grid has to be resident:
// as many per sequence as fit (at most kWalkShare, and no more than there are passes' worth of
// slots), a single one otherwise.
template <bool BF16, int LD>
void launch_walk(int B, long nslots, size_t lds, hipStream_t st, const WalkParams& P) {
    int dev = 0, cus = 0;
    (void)hipGetDevice(&dev);
    if (hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess) cus = 0;
    const auto shares = [&](auto kernel) -> long {
        int per_cu = 0;
        if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, kernel, kWalkWG, lds) != hipSuccess) per_cu = 0;
        (void)hipGetLastError();
        long gsw = (static_cast<long>(per_cu) * cus) / B;
        if (gsw > kWalkShare) gsw = kWalkShare;
        const long by_work = (nslots + kWalkWG - 1) / kWalkWG;
        if (gsw > by_work) gsw = by_work;
        return gsw < 1 ? 1 : gsw;
    };
    if constexpr (LD != LOAD_ELEM) {
        // the distribution in force in registers where a workgroup's share of a row allows it
        const long gsw = shares(tree_sd_walk<BF16, LD, true>);
        if ((nslots + gsw - 1) / gsw <= static_cast<long>(WalkKeep<BF16>::CH) * kWalkWG) {
            hipLaunchKernelGGL((tree_sd_walk<BF16, LD, true>), dim3(static_cast<unsigned>(gsw), static_cast<unsigned>(B)), dim3(kWalkWG), lds, st, P);
            return;
        }
    }
    const long gsw = shares(tree_sd_walk<BF16, LD, false>);
    hipLaunchKernelGGL((tree_sd_walk<BF16, LD, false>), dim3(static_cast<unsigned>(gsw), static_cast<unsigned>(B)), dim3(kWalkWG), lds, st, P);
}

std::atomic<int> g_last_selection{0};   // workgroups a sequence of the last warped call's selection (see fsd_debug_last_selection)

// Keys a workgroup's list has to hold under top-k.  A share's entries are dealt to T threads (1024, or as many as have
// any); the k-th largest of their maxima has about T ln(T / (T - k)) entries at or above it, with the variance of
// the number of draws that reach k of T places.  Four of its standard deviations are added, and a
// sixteenth for the bound's missing lower half (entries that agree with it in the upper 16 bits).
long list_keys(long k, long T) {
    if (k >= T) return LONG_MAX;
    const double x = -log1p(-static_cast<double>(k) / static_cast<double>(T)), n = static_cast<double>(T) * x;
    return static_cast<long>(n * 1.0625 + 4.0 * sqrt(static_cast<double>(T) * (expm1(x) - x))) + 1;
}

// Rows of fewer entries are left to one workgroup.  Whole calls, one workgroup a row and several (us):
//   top-p 0.95, 8 sequences   bfloat16   V=8200 40.3 and 39.7;              V=12001 42.8 and 43.4, 16001 47.8 and 47.4
//                             binary32   V=16000 44.4 and 44.9, 20000 51.7 and 50.9; V=12001 44.6 and 44.6, 16001 (1 sequence) 33.4 and 32.4
//   top-k 50, top-p 0.9, 8 sequences of 32   bfloat16   V=16000 32.0 and 28.8, 24000 34.9 and 31.4; V=16001 34.2 and 32.2, 24001 38.6 and 35.3
//                             binary32   V=16000 35.1 and 30.9, 32000 43.9 and 39.1, 40000 49.2 and 42.9; V=16001 36.8 and 32.5, 20001 41.3 and 35.8
// Under top-k the lines are those of a selection with a draw kernel behind it on either side, where both took the same time (of 8 sequences,
// bfloat16 V=24000 39.5 and 39.3, binary32 40000 48.3 and 47.5, 20001 43.5 and 43.3).  That is what a recorded call, a long chain or a large top-k still has;
// where several workgroups draw the token as well they are the faster ones below the lines too, by the second row's 2 to 7 us.
// (Binary32 rows are streamed by the one workgroup, unaligned ones of either type with moves for their last slot.)
constexpr long split_least(bool bf16, bool aligned, bool top_k) {
    return top_k ? (bf16 ? 24000 : aligned ? 40000 : 20000) : (!aligned ? 16000 : bf16 ? 0 : 20000);
}

// warp_select with several workgroups per sequence: false (nothing launched) if the row is short, if fewer than two
// per sequence are resident (under top-p alone they wait for each other), if a share does not fit their registers, or
// if it takes fewer workgroups than that for their lists to hold a large top-k.  (A list that overflows costs the last
// workgroup the whole row again: 8 rows of 128256 bfloat16 entries, top-k 512: 69 us a call with eight workgroups a
// row, 55 with one, 49 with four.)
template <bool BF16, int LD, int SHARED>
bool launch_warp_split_k(int B, hipStream_t st, WarpParams& P) {
    constexpr bool want_k = SHARED == SPLIT_TOP_K;
    if (P.V < split_least(BF16, LD == LOAD_ALIGNED, want_k)) return false;
    static std::atomic<long> resident[16] = {};
    int dev = 0;
    (void)hipGetDevice(&dev);
    if (dev < 0 || dev >= 16) dev = 0;
    long total = resident[dev].load(std::memory_order_relaxed);
    if (total == 0) {
        int per_cu = 0, cus = 0;
        if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, warp_select<BF16, LD, true, SHARED>, kWarpWG, 0) != hipSuccess) per_cu = 0;
        if (hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess) cus = 0;
        (void)hipGetLastError();
        total = static_cast<long>(per_cu) * cus;
        if (total < 1) total = 1;
        resident[dev].store(total, std::memory_order_relaxed);
    }
    long W = total / B;
    if (W > kWarpShare) W = kWarpShare;
    const long by_work = (P.nslots + kWarpWG - 1) / kWarpWG;
    if (W > by_work) W = by_work;
    if (want_k) {
        const auto needed = [&](long w) {
            const long share = (P.nslots + w - 1) / w;
            return list_keys(P.top_k, share < kWarpWG ? share : kWarpWG);
        };
        while (W >= 2 && needed(W) > kSplitKeys / W - 1) --W;
        // the draw in the same launch needs the places of the keys as well, twice the memory; where a sequence has that (fewer
        // than 8 rows of the usual vocabularies under a top-k of hundreds do not), a list has as many entries as one of keys alone
        if (P.draw && W >= 2) {
            const long words = static_cast<long>(P.seq_bytes / 8);
            P.list_keys = static_cast<int>((words < kSplitKeys ? words : kSplitKeys) / W - 1);
            if (needed(W) > P.list_keys) P.draw = 0;
        }
        if (!P.draw && W >= 2) P.list_keys = static_cast<int>(kSplitKeys / W - 1);
    }
    if (W < 2 || P.nslots > kSplitSlots || (P.nslots + W - 1) / W > static_cast<long>(split_keep(BF16)) * kWarpWG) return false;
    g_last_selection.store(static_cast<int>(W), std::memory_order_relaxed);
    hipLaunchKernelGGL((warp_select<BF16, LD, true, SHARED>), dim3(static_cast<unsigned>(W), static_cast<unsigned>(B)), dim3(kWarpWG), 0, st, P);
    return true;
}

template <bool BF16, int LD>
bool launch_warp_split(int B, hipStream_t st, WarpParams& P) {
    return P.top_k > 0 && P.top_k < P.V ? launch_warp_split_k<BF16, LD, SPLIT_TOP_K>(B, st, P) : launch_warp_split_k<BF16, LD, SPLIT_TOP_P>(B, st, P);
}

// how the kernels fetch a slot of these rows (see load_slot)
int load_of(const void* a, const void* b, long V, int VE) {
    if (V < VE) return LOAD_ELEM;
    return (V % VE == 0 && reinterpret_cast<uintptr_t>(a) % 16 == 0 && reinterpret_cast<uintptr_t>(b) % 16 == 0) ? LOAD_ALIGNED : LOAD_WIDE;
}

// Device address of the static scratch array on the current device (nullptr if the runtime will not
// give it).  Every GPU holds its own copy of the array at its own address, so the address is looked
// up once per device, with that device current, and kept.
void* static_scratch() {
    static std::atomic<void*> ptr[64] = {};
    int dev = 0;
    if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= 64) return nullptr;
    void* p = ptr[dev].load(std::memory_order_acquire);
    if (!p) {
        if (hipGetSymbolAddress(&p, HIP_SYMBOL(scratch)) != hipSuccess || !p) {
            (void)hipGetLastError();
            return nullptr;
        }
        ptr[dev].store(p, std::memory_order_release);
    }
    return p;
}

// the common body of the entry points
int run(int kind, const void* target, const void* draft, const int32_t* tokens, const int32_t* parent, int B,
        int rows, int max_depth, int V, int dtype, int div, float T, int mode, uint64_t seed, uint64_t offset,
        int32_t* out_len, int32_t* path_nodes, int32_t* out_tokens, float* user_vals, float* user_ratio,
        int32_t* row_status, void* workspace, size_t workspace_bytes, void* hip_stream,
        float temperature = 1.0f, int top_k = 0, float top_p = 1.0f, bool static_ws = false) {
    if (!target || !draft || !tokens || !out_len || !out_tokens) return FSD_ERR_NULL;
    const bool tree = (kind == KIND_TREE || kind == KIND_TREESD);
    if (tree && (!parent || !path_nodes)) return FSD_ERR_NULL;
    if (dtype != FSD_F32 && dtype != FSD_BF16) return FSD_ERR_DTYPE;
    if (kind != KIND_SD && kind != KIND_TREESD && (div < FSD_DIV_KL || div > FSD_DIV_TV)) return FSD_ERR_DIV;
    if (mode != FSD_SAMPLE && mode != FSD_GREEDY) return FSD_ERR_MODE;
    if (T != T) return FSD_ERR_SHAPE;
    if (tree && (max_depth < 1 || max_depth > kMaxRows)) return FSD_ERR_SHAPE;
    if (!(temperature >= 1e-3f && temperature <= 1e3f) || top_k < 0 || !(top_p > 0.0f && top_p <= 1.0f)) return FSD_ERR_SHAPE;
    Plan p;
    if (!make_plan(B, rows, V, dtype, p)) return FSD_ERR_SHAPE;
    if (static_ws) {
        // the library's own buffer instead of the caller's
        if (p.bytes > static_cast<size_t>(FSD_STATIC_SCRATCH_BYTES)) return FSD_ERR_TOO_LARGE;
        workspace = static_scratch();
        if (!workspace) return FSD_ERR_LAUNCH;
    } else if (!workspace || reinterpret_cast<uintptr_t>(workspace) % 256 != 0 || workspace_bytes < p.bytes) {
        return FSD_ERR_WORKSPACE;
    }

    hipStream_t st = static_cast<hipStream_t>(hip_stream);
    const int load = load_of(target, draft, V, p.VE);
    const int R = B * rows;

    const int plan_G = p.G;   // what the workspace is laid out for
    // which reduction kernel, and its shape
    int k1mode = (kind == KIND_SD || kind == KIND_TREESD) ? MODE_LSE : div;
    if (k1mode == MODE_KL && dtype == FSD_F32) k1mode = MODE_KLP;
    // bfloat16 JS: the entropy form (reducible FSD, whose finisher also forms the candidates' log-ratios,
    // and the shapes of the tuning hook stay with the pointwise form)
    if (load == LOAD_ELEM) {
        // a row shorter than a slot: one lane of one wavefront, in the smallest shape (the only one with
        // element-wise loads)
        p.NV = 2;
        p.G = 1;
        p.spm = static_cast<int>(p.nslots);
    } else if (k1mode == MODE_JS && dtype == FSD_BF16 && kind != KIND_RFSD && !g_exact_js && !g_shape_nv) {
        k1mode = MODE_JSE;
    }
    if (load != LOAD_ELEM && dtype == FSD_BF16 && !g_shape_nv && (k1mode == MODE_JS || k1mode == MODE_TV || k1mode == MODE_JSE)) {
        // The bfloat16 two-phase kernels are bound by instruction issue, a third of it per step and not
        // per entry: they hold 6 slots of each row per lane (96 logits a step), which fits two wavefronts
        // per SIMD (256 registers) because 5 of the 12 chunks of each set of kept exponentials live in
        // LDS.  The workspace is laid out for the larger team of the 4-slot shape.
        p.NV = 6;
        p.G = static_cast<int>(team_size(p.nslots, p.NV));
        p.spm = static_cast<int>((p.nslots + p.G - 1) / p.G);
        // entropy form: whole chunks of 64 NV slots per member, so that only the last one with any
        // slots has lanes without one (those lanes cost it selections the others do not pay for)
        if (k1mode == MODE_JSE) p.spm = 64 * p.NV;
    }
    if (load != LOAD_ELEM && dtype == FSD_BF16 && !g_shape_nv && (k1mode == MODE_LSE || k1mode == MODE_KL)) {
        // The bfloat16 single-pass kernels hold 8 slots of each row per lane once the rows are enough for several rounds of their teams
        // (a step's reductions and exchange, a fifth of its instructions with 4 slots, are then shared by twice the logits); with
        // fewer the last round is too empty.  A tree's siblings read their target row once.  Whole calls, us, 4 and 8 slots:
        //   strict SD, from nearly four rounds   V=128256, 24 sequences of 8 35.7 and 36.3, 40 49.0 and 47.7, 64 66.7 and 64.3, 256 218 and 203; trees of 60, 5
        //     sequences 73.5 and 75.0, 6 79.3 and 76.1, 15 117.3 and 114.4, 32 195.7 and 183.8; V=32000, 24 trees 74.2 and 70.7; V=200000, 4 92.0 and 88.9.  (In
        //     between a last round that is nearly empty goes either way: V=56128, 20 trees 86.1 and 85.2, 22 84.5 and 86.0.)
        //   KL, whose 4-slot kernel waits for memory more than it computes   trees of 60, from 24 rounds: V=128256, 8.3 rounds 70.6 and 76.0, 11 93.5 and 96.2, 18
        //     140.9 and 146.0, 24 184.9 and 180.5, 48 366 and 355; V=32000, 18 143.8 and 142.2, 24 189.4 and 183.3.  Chains, from 32: V=128256, 10 60.8 and
        //     61.5, 20 107.1 and 107.1, 40 193.3 and 189.2; V=32000, 20 105.2 and 105.7, 28 145.3 and 141.5, 40 195.7 and 188.8; V=200000, 10 60.9 and
        //     63.2, 28 144.2 and 145.9, 40 192.2 and 192.7.
        //   rows that are not 16-byte aligned   strict SD on trees, from seven: V=106053, 4.1 rounds 91.7 and 94.8, 6.2 103.2 and 105.4, 7.2 106.7 and 106.5,
        //     9.3 118.7 and 117.2; V=128259 230 and 220.  KL on trees, 4.1 51.2 and 55.9, 14 133.1 and 134.6, 24 215.3 and 212.1.  But chains, V=128259, strict SD
        //     74.9 and 85.8, KL 72.0 and 83.0: never.
        const long G8 = team_size(p.nslots, 8);
        const long round = max_resident_wavefronts() / 8 * pair_kernel_most(true, 8, k1mode) / G8, rows_read = parent ? R + B : 2L * R;
        const long quarters = k1mode == MODE_KL ? (parent ? 4 * 24 : 4 * 32) : load == LOAD_ALIGNED ? 15 : 4 * 7;   // of a round
        if ((parent || load == LOAD_ALIGNED) && 4 * rows_read >= quarters * round) {
            p.NV = 8;
            p.G = static_cast<int>(G8);
            p.spm = static_cast<int>((p.nslots + G8 - 1) / G8);
        }
    }
    if (dtype == FSD_F32 && load != LOAD_ELEM && !g_shape_nv) {
        // (Of what small_call does not take: strict SD above all, and the calls its rule leaves to the teams.)
        // A call whose pairs all fit the device at once is one step per wavefront, and its time the chain of that
        // step: half the slots per lane (twice the members, who post at most twice what the workspace is laid
        // out for) shorten it.  Strict SD: one sequence of 4 positions, V=32000: 13.8 -> 12.8 us a call; 8 of 4 14.1 -> 12.9; one of 8, V=128256
        // 14.6 -> 14.4; 4 of 5, V=64000 14.3 -> 13.6.  The line is drawn at the most wavefronts it was
        // measured to help with (1280; TV and JS at 2384, more than one step, 21.9 -> 22.6).
        const long G4 = team_size(p.nslots, 4);
        if (G4 <= kMaxTeam && static_cast<long>(R) * G4 * 32 <= 5 * max_resident_wavefronts()) {
            p.NV = 4;
            p.G = static_cast<int>(G4);
            p.spm = static_cast<int>((p.nslots + G4 - 1) / G4);
        } else if (k1mode != MODE_LSE) {
            // The two-phase kernels hold 10 slots a lane, or 8 where the call is of few steps and 8 slots make
            // less of them (whole calls, us, 8 and 10 slots: 16 sequences of 8, V=64000, 2 and 2 steps 25.9 and 27.6; 8 of 16, V=128256, 4 and 4
            // steps 37.0 and 38.7; 64 of 16, V=32000, 8 and 7 57.0 and 59.3; 128 of 16, V=128256, 64 and 52 381 and 359; 256 of 16, V=151936, 152 and
            // 121 917 and 831, where one wavefront a SIMD, with 8 slots and a third set of exponentials, took 936).  Not where 8 slots make a team
            // one of more rounds of 64 members, whose words every merge then reads in more rounds: 12 of 6, V=151936, 3 and 3 steps, 75 and 60 members 33.5
            // and 33.2; 5 of 8, V=400000, 4 and 4, 196 and 157 48.5 and 46.5; but 5 of 8, V=200000, 2 and 2, 98 and 79 JS 29.2 and 30.7, KL 32.6 and
            // 35.2; 8 of 8, V=256000, 4 and 4, 125 and 100 40.0 and 41.3, KL 45.3 and 47.6.  Such teams up to four steps: 14 of 8, V=200000, 6 and 5 52.5 and 51.5.
            const long G8 = team_size(p.nslots, 8), G10 = team_size(p.nslots, 10), waves = max_resident_wavefronts() / 4;
            const auto steps = [&](long G) { const long teams = waves / G > 0 ? waves / G : 1; return (R + teams - 1) / teams; };
            const bool eight = (G8 + 63) / 64 == (G10 + 63) / 64 && steps(G8) <= (G8 <= 64 ? 8 : 4) && steps(G8) * 8 < steps(G10) * 10;
            p.NV = eight ? 8 : 10;
            p.G = static_cast<int>(eight ? G8 : G10);
            p.spm = static_cast<int>((p.nslots + p.G - 1) / p.G);
        }
    }
    // exchange words a member posts in this mode: only those are laid out and cleared
    const bool two_phase = (k1mode == MODE_JS || k1mode == MODE_TV || k1mode == MODE_KLP || k1mode == MODE_JSE);
    const int n1 = two_phase ? 2 : 4;
    const int n2 = (k1mode == MODE_TV || k1mode == MODE_KLP) ? 2 : two_phase ? 1 : 0;
    size_t zero_bytes = 0;
    const Ws ws = carve(workspace, p, B, rows, p.G, n1, n2, zero_bytes);
    if (zero_bytes > p.zero_bytes) return FSD_ERR_WORKSPACE;   // the exchange words would run into what follows them (no shape here does)

    const bool warped = (temperature != 1.0f) || (top_k > 0 && top_k < V) || (top_p < 1.0f);
    // Small calls: the reduction in one step, or the whole of a plain FSD call on a few sequences in one launch, unless a test or the
    // profiler has asked for the kernels of a large call
    int launched = SMALL_NONE;
    uint4* clear_last = nullptr;   // what the sampler clears once the reduction has ended (see SampleParams)
    long clear_last16 = 0;
    bool captured = false;
    SmallForms may{false, false, false};
    if ((kind == KIND_CHAIN || kind == KIND_TREE || kind == KIND_RFSD) && load != LOAD_ELEM && g_small_calls && !g_shape_nv && !g_prof_on && g_self_clear &&
        static_cast<long>(R) * V <= 6L << 20 && !(k1mode == MODE_JSE && g_js_floor != kJsFloor)) {
        hipStreamCaptureStatus capture = hipStreamCaptureStatusNone;
        captured = hipStreamIsCapturing(st, &capture) != hipSuccess || capture != hipStreamCaptureStatusNone;
        if (captured) (void)hipGetLastError();
        may = small_forms(kind, dtype, div, B, rows, V, load == LOAD_ALIGNED);
        if (warped && mode == FSD_SAMPLE) may.whole = false;
    }
    if (may.whole || may.reduction) {
        SmallParams P;
        P.target = static_cast<const char*>(target);
        P.draft = static_cast<const char*>(draft);
        P.tokens = tokens;
        P.parent = tree ? parent : nullptr;
        P.rows = rows;
        P.npairs = R;
        P.max_depth = max_depth;
        P.V = V;
        P.nslots = p.nslots;
        P.T = T;
        P.mode = mode;
        P.seed_lo = static_cast<unsigned>(seed);
        P.seed_hi = static_cast<unsigned>(seed >> 32);
        P.off_lo = static_cast<unsigned>(offset);
        P.off_hi = static_cast<unsigned>(offset >> 32);
        P.spin_limit = g_spin_limit;
        P.out_len = out_len;
        P.out_tokens = out_tokens;
        P.path_nodes = path_nodes;
        P.row_status = row_status;
        P.user_div = user_vals;
        P.nonce = ws.nonce;
        P.ws = ws;
        P.user_ratio = user_ratio;
        P.want_ratio = (kind == KIND_RFSD) ? 1 : 0;
        P.finish = small_finish_pairs(kind == KIND_RFSD);
        P.clear_a = reinterpret_cast<uint4*>(ws.counters + 4);
        P.clear_a16 = static_cast<long>((p.n_counters - 4) * 4 / 16);
        P.clear_b = reinterpret_cast<uint4*>(ws.spart);
        P.clear_b16 = (static_cast<long>(B) * p.GS + 1) / 2;
        launched =
            dtype == FSD_BF16 ? (load == LOAD_ALIGNED ? launch_small<true, LOAD_ALIGNED>(div, st, P, B, plan_G, may, captured)
                                                      : launch_small<true, LOAD_WIDE>(div, st, P, B, plan_G, may, captured))
                              : (load == LOAD_ALIGNED ? launch_small<false, LOAD_ALIGNED>(div, st, P, B, plan_G, may, captured)
                                                      : launch_small<false, LOAD_WIDE>(div, st, P, B, plan_G, may, captured));
        if (launched == SMALL_REDUCED && captured) {
            clear_last = reinterpret_cast<uint4*>(P.words);
            clear_last16 = P.words16;
        }
    }
    g_last_route.store(launched, std::memory_order_relaxed);
    if (launched == SMALL_DONE) return (hipGetLastError() == hipSuccess) ? FSD_OK : FSD_ERR_LAUNCH;
    const bool reduced = launched == SMALL_REDUCED;

    // The calls have no clearing kernel: the reduction clears what it and the kernels after it need (see
    // clear_own_words in pair_kernel.h; C2: -3 us a call, C4: -2 us), unless there are more than 4 MB to
    // clear (inside the reduction kernel that costs what the kernel of its own costs, C3: 7.5 MB) or
    // the grid is too large for the arrival slots.
    const bool self_clear = g_self_clear && zero_bytes <= (4u << 20) && max_resident_wavefronts() <= kMaxArrive;
    if (self_clear && !reduced) {
        clear_last = reinterpret_cast<uint4*>(ws.arrive);
        clear_last16 = kMaxArrive / 2;
    }
    if (!self_clear && !reduced) {
        const long n16 = static_cast<long>(zero_bytes / 16);
        hipLaunchKernelGGL(zero_counters, dim3(static_cast<unsigned>((n16 + 255) / 256)), dim3(256), 0, st,
                           reinterpret_cast<uint4*>(ws.counters), n16);
    }

    PairParams pp;
    pp.self_clear = self_clear ? 1 : 0;
    // what no team owns: the sampler's counters (all but the first four words: the failure word, words 2-3,
    // is never cleared here, so that a flag raised early cannot be lost) and its shares
    pp.clear_a = reinterpret_cast<uint4*>(ws.counters + 4);
    pp.clear_a16 = static_cast<long>((p.n_counters - 4) * 4 / 16);
    // (the walk's shares lie right before the sampler's: strict SD over a tree has both cleared)
    pp.clear_b = reinterpret_cast<uint4*>(kind == KIND_TREESD ? reinterpret_cast<char*>(ws.wz) : reinterpret_cast<char*>(ws.spart));
    pp.clear_b16 = static_cast<long>((p.off_spart - (kind == KIND_TREESD ? p.off_wz : p.off_spart)) / 16) + (static_cast<long>(B) * p.GS + 1) / 2;
    pp.target = static_cast<const char*>(target);
    pp.draft = static_cast<const char*>(draft);
    pp.parent = tree ? parent : nullptr;
    pp.cand = tokens;
    pp.rows = rows;
    pp.npairs = R;
    pp.V = V;
    pp.nslots = p.nslots;
    pp.spm = p.spm;
    pp.G = p.G;
    pp.spin_limit = g_spin_limit;
#ifdef FSD_PHASE_TIMING
    pp.dbg = g_dbg;
#endif
    pp.user_div = user_vals;
    pp.user_ratio = user_ratio;
    pp.want_ratio = (kind == KIND_RFSD) ? 1 : 0;
    pp.js_floor = g_js_floor;
    pp.ws = ws;
    if (!reduced) launch_pair(dtype, p.NV, k1mode, load, st, pp);

    SampleParams sp;
    sp.target = static_cast<const char*>(target);
    sp.draft = static_cast<const char*>(draft);
    sp.tokens = tokens;
    sp.parent = parent;
    sp.rows = rows;
    sp.max_depth = max_depth;
    sp.V = V;
    sp.nslots = p.nslots;
    sp.sps = p.sps;
    sp.GS = p.GS;
    sp.T = T;
    sp.mode = mode;
    sp.seed_lo = static_cast<unsigned>(seed);
    sp.seed_hi = static_cast<unsigned>(seed >> 32);
    sp.off_lo = static_cast<unsigned>(offset);
    sp.off_hi = static_cast<unsigned>(offset >> 32);
    sp.out_len = out_len;
    sp.out_tokens = out_tokens;
    sp.path_nodes = path_nodes;
    sp.row_status = row_status;
    sp.ws = ws;
    sp.cut = 0;
    sp.thr = nullptr;
    sp.inv_temp = 1.0f;
    sp.clear = clear_last;
    sp.clear16 = clear_last16;
    if (warped && mode == FSD_SAMPLE) {
        // warpers: one more kernel finds, per sequence, the smallest kept scaled logit
        WarpParams wp;
        wp.target = static_cast<const char*>(target);
        wp.parent = (kind == KIND_TREE) ? parent : nullptr;
        wp.rows = rows;
        wp.V = V;
        wp.nslots = p.nslots;
        wp.T = T;
        wp.inv_temp = static_cast<float>(1.0 / static_cast<double>(temperature));
        wp.top_k = top_k;
        wp.top_p = top_p;
        wp.thr = ws.thr;
        wp.ws = ws;
        // one workgroup a row keeps an aligned bfloat16 row in registers.  (Unaligned rows are streamed: with the
        // moves of their last slot the kept form spills 107 registers.  Calls on 4 sequences under top-k 50, kept and streamed:
        // V=8197 58.1 and 34.7 us, V=32001 59.1 and 38.9, V=128259 66.6 and 53.6.)
        const bool keep = dtype == FSD_BF16 && load == LOAD_ALIGNED && p.nslots <= static_cast<long>(kWarpKeep) * kWarpWG;
        wp.area = reinterpret_cast<char*>(ws.part1);
        wp.seq_bytes = static_cast<size_t>(rows) * plan_G * 64;
        wp.spin_limit = g_spin_limit < g_selection_spin_limit ? g_spin_limit : g_selection_spin_limit;
        wp.list_keys = 0;
        wp.tokens = tokens;
        wp.max_depth = max_depth;
        wp.seed_lo = sp.seed_lo; wp.seed_hi = sp.seed_hi; wp.off_lo = sp.off_lo; wp.off_hi = sp.off_hi;
        wp.out_len = out_len;
        wp.out_tokens = out_tokens;
        wp.path_nodes = path_nodes;
        wp.row_status = row_status;
        wp.clear = clear_last;
        wp.clear16 = clear_last16;
        const bool want_k = top_k > 0 && top_k < V, want_p = top_p < 1.0f;
        // the draw with the selection (by several workgroups a row), but for a recorded call whose reduction has words to be cleared
        // where the lists go
        wp.draw = (want_k && rows <= 64 && (clear_last == nullptr || clear_last == reinterpret_cast<uint4*>(ws.arrive))) ? 1 : 0;
        const auto warp = [&](auto kernel) {
            g_last_selection.store(1, std::memory_order_relaxed);
            hipLaunchKernelGGL(kernel, dim3(B), dim3(kWarpWG), 0, st, wp);
        };
        // several workgroups a sequence, where a setting allows it, the workspace has room for what they leave each
        // other and all of them are resident
        const bool split = load != LOAD_ELEM && (want_k ? top_k <= kWarpFastK : want_p) && wp.seq_bytes >= kSplitBytes &&
                           (dtype == FSD_BF16 ? (load == LOAD_ALIGNED ? launch_warp_split<true, LOAD_ALIGNED>(B, st, wp)
                                                                      : launch_warp_split<true, LOAD_WIDE>(B, st, wp))
                                              : (load == LOAD_ALIGNED ? launch_warp_split<false, LOAD_ALIGNED>(B, st, wp)
                                                                      : launch_warp_split<false, LOAD_WIDE>(B, st, wp)));
        if (split && wp.draw) return (hipGetLastError() == hipSuccess) ? FSD_OK : FSD_ERR_LAUNCH;   // (it has drawn the token as well)
        if (split) {
            // (launched)
        } else if (!want_k && !want_p) {
            // nothing to select: temperature alone keeps everything, and the sampler leaves the cut that says so
            g_last_selection.store(1, std::memory_order_relaxed);
        } else if (dtype == FSD_BF16) {
            if (keep) warp(warp_select<true, LOAD_ALIGNED, true>);
            else if (load == LOAD_ALIGNED) warp(warp_select<true, LOAD_ALIGNED, false>);
            else if (load == LOAD_WIDE) warp(warp_select<true, LOAD_WIDE, false>);
            else warp(warp_select<true, LOAD_ELEM, false>);
        } else {
            if (load == LOAD_ALIGNED) warp(warp_select<false, LOAD_ALIGNED, false>);
            else if (load == LOAD_WIDE) warp(warp_select<false, LOAD_WIDE, false>);
            else warp(warp_select<false, LOAD_ELEM, false>);
        }
        if (want_k || want_p) sp.thr = ws.thr;
        sp.cut = 1;
        sp.inv_temp = wp.inv_temp;
    }
    if (kind == KIND_TREESD) {
        // strict SD on a tree: up to kWalkShare workgroups per sequence walk the tree before the token is drawn
        WalkParams wk;
        wk.target = sp.target;
        wk.draft = sp.draft;
        wk.tokens = tokens;
        wk.parent = parent;
        wk.rows = rows;
        wk.max_depth = max_depth;
        wk.V = V;
        wk.nslots = p.nslots;
        wk.seed_lo = sp.seed_lo; wk.seed_hi = sp.seed_hi; wk.off_lo = sp.off_lo; wk.off_hi = sp.off_hi;
        wk.path_nodes = path_nodes;
        wk.out_tokens = out_tokens;
        wk.user_ratio = user_ratio;
        wk.ws = ws;
        wk.spin_limit = g_spin_limit;
        const size_t wlds = static_cast<size_t>(rows) * 24 + 16;
        if (dtype == FSD_BF16) {
            if (load == LOAD_ALIGNED) launch_walk<true, LOAD_ALIGNED>(B, p.nslots, wlds, st, wk);
            else if (load == LOAD_WIDE) launch_walk<true, LOAD_WIDE>(B, p.nslots, wlds, st, wk);
            else launch_walk<true, LOAD_ELEM>(B, p.nslots, wlds, st, wk);
        } else {
            if (load == LOAD_ALIGNED) launch_walk<false, LOAD_ALIGNED>(B, p.nslots, wlds, st, wk);
            else if (load == LOAD_WIDE) launch_walk<false, LOAD_WIDE>(B, p.nslots, wlds, st, wk);
            else launch_walk<false, LOAD_ELEM>(B, p.nslots, wlds, st, wk);
        }
    }
    const size_t lds = (kind == KIND_TREE) ? static_cast<size_t>(rows) * 16
                     : (kind == KIND_TREESD) ? static_cast<size_t>(rows) * 12 : 0;
    launch_sample(dtype, load, kind, dim3(p.GS, B), lds, st, sp);

    return (hipGetLastError() == hipSuccess) ? FSD_OK : FSD_ERR_LAUNCH;
}

}  // namespace

// ------------------------------------------------------------------------------------------
// C ABI

extern "C" {

int64_t fsd_max_vocab(int dtype) {
    // 256 wavefronts per pair, 64 lanes, 32 entries of each row per lane
    if (dtype == FSD_BF16 || dtype == FSD_F32) return static_cast<int64_t>(kMaxTeam) * 64 * 32;
    return 0;
}

size_t fsd_workspace_bytes(int B, int rows_per_seq, int V, int dtype) {
    Plan p;
    if (!make_plan(B, rows_per_seq, V, dtype, p)) return 0;
    return p.bytes;
}

size_t fsd_calibrate_workspace_bytes(int B, int K) {
    if (B < 1 || K < 1 || K > kMaxRows || static_cast<long>(B) * K >= (1L << 24)) return 0;
    return align_up(sizeof(CalibState), 256) + align_up(static_cast<size_t>(B) * K * 4, 256);
}

int fsd_calibrate_threshold(const float* divergences, int B, int K, float target_fraction, float* T_out,
                            float* fraction_out, void* workspace, size_t workspace_bytes, void* hip_stream) {
    if (!divergences || !T_out) return FSD_ERR_NULL;
    const size_t need = fsd_calibrate_workspace_bytes(B, K);
    if (need == 0 || !(target_fraction > 0.0f) || !(target_fraction <= 1.0f)) return FSD_ERR_SHAPE;
    if (!workspace || reinterpret_cast<uintptr_t>(workspace) % 256 != 0 || workspace_bytes < need) return FSD_ERR_WORKSPACE;
    hipStream_t st = static_cast<hipStream_t>(hip_stream);
    CalibState* state = static_cast<CalibState*>(workspace);
    unsigned* keys = reinterpret_cast<unsigned*>(static_cast<char*>(workspace) + align_up(sizeof(CalibState), 256));
    const long n = static_cast<long>(B) * K;
    // rank = ceil(fraction n), in exact arithmetic on the binary32 fraction
    const double want = static_cast<double>(target_fraction) * static_cast<double>(n);
    long rank = static_cast<long>(want);
    if (static_cast<double>(rank) < want) ++rank;
    if (rank < 1) rank = 1;
    if (rank > n) rank = n;
    const unsigned blocks = static_cast<unsigned>(n / 4096 + 1 > 1024 ? 1024 : n / 4096 + 1);
    hipLaunchKernelGGL(calib_keys, dim3((B + 255) / 256), dim3(256), 0, st, divergences, B, K, keys);
    hipLaunchKernelGGL(calib_init, dim3(1), dim3(256), 0, st, state, static_cast<unsigned>(rank));
    for (int shift = 24; shift >= 0; shift -= 8) {
        hipLaunchKernelGGL(calib_hist, dim3(blocks), dim3(256), 0, st, keys, n, shift, state);
        hipLaunchKernelGGL(calib_pick, dim3(1), dim3(256), 0, st, state, shift);
    }
    hipLaunchKernelGGL(calib_count, dim3(blocks), dim3(256), 0, st, keys, n, state);
    hipLaunchKernelGGL(calib_result, dim3(1), dim3(1), 0, st, state, n, T_out, fraction_out);
    return (hipGetLastError() == hipSuccess) ? FSD_OK : FSD_ERR_LAUNCH;
}

const char* fsd_status_string(int status) {
    switch (status) {
        case FSD_OK: return "ok";
        case FSD_ERR_NULL: return "a required pointer is NULL";
        case FSD_ERR_SHAPE: return "size out of range or T is NaN";
        case FSD_ERR_DTYPE: return "unknown dtype";
        case FSD_ERR_DIV: return "unknown divergence";
        case FSD_ERR_WORKSPACE: return "workspace missing, misaligned or too small";
        case FSD_ERR_MODE: return "unknown sampling mode";
        case FSD_ERR_LAUNCH: return "kernel launch failed";
        case FSD_ERR_TOO_LARGE: return "sizes need more scratch memory than the static buffer holds (FSD_STATIC_SCRATCH_BYTES)";
        default: return "unknown status";
    }
}

int fsd_verify_chain(const void* target_logits, const void* draft_logits, const int32_t* cand_tokens, int B, int K,
                     int V, int dtype, int div, float T, int mode, uint64_t seed, uint64_t offset,
                     int32_t* accept_len, int32_t* out_tokens, float* divergences, int32_t* row_status,
                     void* workspace, size_t workspace_bytes, void* hip_stream) {
    return run(KIND_CHAIN, target_logits, draft_logits, cand_tokens, nullptr, B, K, 0, V, dtype, div, T, mode, seed,
               offset, accept_len, nullptr, out_tokens, divergences, nullptr, row_status, workspace, workspace_bytes,
               hip_stream);
}

int fsd_verify_tree(const void* target_logits, const void* draft_logits, const int32_t* node_tokens,
                    const int32_t* parent, int B, int N, int max_depth, int V, int dtype, int div, float T,
                    int mode, uint64_t seed, uint64_t offset, int32_t* path_len, int32_t* path_nodes,
                    int32_t* out_tokens, float* divergences, int32_t* row_status, void* workspace,
                    size_t workspace_bytes, void* hip_stream) {
    return run(KIND_TREE, target_logits, draft_logits, node_tokens, parent, B, N, max_depth, V, dtype, div, T, mode,
               seed, offset, path_len, path_nodes, out_tokens, divergences, nullptr, row_status, workspace,
               workspace_bytes, hip_stream);
}

int sd_verify_chain(const void* target_logits, const void* draft_logits, const int32_t* cand_tokens, int B, int K,
                    int V, int dtype, int mode, uint64_t seed, uint64_t offset, int32_t* accept_len,
                    int32_t* out_tokens, float* log_ratio, int32_t* row_status, void* workspace,
                    size_t workspace_bytes, void* hip_stream) {
    return run(KIND_SD, target_logits, draft_logits, cand_tokens, nullptr, B, K, 0, V, dtype, FSD_DIV_KL, 0.0f, mode,
               seed, offset, accept_len, nullptr, out_tokens, log_ratio, nullptr, row_status, workspace, workspace_bytes,
               hip_stream);
}

int fsd_verify_tree_warped(const void* target_logits, const void* draft_logits, const int32_t* node_tokens,
                           const int32_t* parent, int B, int N, int max_depth, int V, int dtype, int div, float T,
                           int mode, uint64_t seed, uint64_t offset, float temperature, int top_k, float top_p,
                           int32_t* path_len, int32_t* path_nodes, int32_t* out_tokens, float* divergences,
                           int32_t* row_status, void* workspace, size_t workspace_bytes, void* hip_stream) {
    return run(KIND_TREE, target_logits, draft_logits, node_tokens, parent, B, N, max_depth, V, dtype, div, T, mode,
               seed, offset, path_len, path_nodes, out_tokens, divergences, nullptr, row_status, workspace,
               workspace_bytes, hip_stream, temperature, top_k, top_p);
}

int fsd_verify_chain_warped(const void* target_logits, const void* draft_logits, const int32_t* cand_tokens, int B,
                            int K, int V, int dtype, int div, float T, int mode, uint64_t seed, uint64_t offset,
                            float temperature, int top_k, float top_p, int32_t* accept_len, int32_t* out_tokens,
                            float* divergences, int32_t* row_status, void* workspace, size_t workspace_bytes,
                            void* hip_stream) {
    return run(KIND_CHAIN, target_logits, draft_logits, cand_tokens, nullptr, B, K, 0, V, dtype, div, T, mode, seed,
               offset, accept_len, nullptr, out_tokens, divergences, nullptr, row_status, workspace, workspace_bytes,
               hip_stream, temperature, top_k, top_p);
}

int sd_verify_tree(const void* target_logits, const void* draft_logits, const int32_t* node_tokens,
                   const int32_t* parent, int B, int N, int max_depth, int V, int dtype, int mode, uint64_t seed,
                   uint64_t offset, int32_t* path_len, int32_t* path_nodes, int32_t* out_tokens, float* log_ratio,
                   int32_t* row_status, void* workspace, size_t workspace_bytes, void* hip_stream) {
    return run(KIND_TREESD, target_logits, draft_logits, node_tokens, parent, B, N, max_depth, V, dtype, FSD_DIV_KL,
               0.0f, mode, seed, offset, path_len, path_nodes, out_tokens, nullptr, log_ratio, row_status, workspace,
               workspace_bytes, hip_stream);
}

int rfsd_verify_chain(const void* target_logits, const void* draft_logits, const int32_t* cand_tokens, int B, int K,
                      int V, int dtype, int div, float T, int mode, uint64_t seed, uint64_t offset,
                      int32_t* accept_len, int32_t* out_tokens, float* divergences, float* log_ratio,
                      int32_t* row_status, void* workspace, size_t workspace_bytes, void* hip_stream) {
    return run(KIND_RFSD, target_logits, draft_logits, cand_tokens, nullptr, B, K, 0, V, dtype, div, T, mode, seed,
               offset, accept_len, nullptr, out_tokens, divergences, log_ratio, row_status, workspace,
               workspace_bytes, hip_stream);
}

int fsd_verify_chain_static(const void* target_logits, const void* draft_logits, const int32_t* cand_tokens, int B,
                            int K, int V, int dtype, int div, float T, int mode, uint64_t seed, uint64_t offset,
                            int32_t* accept_len, int32_t* out_tokens, float* divergences, int32_t* row_status,
                            void* hip_stream) {
    return run(KIND_CHAIN, target_logits, draft_logits, cand_tokens, nullptr, B, K, 0, V, dtype, div, T, mode, seed,
               offset, accept_len, nullptr, out_tokens, divergences, nullptr, row_status, nullptr, 0, hip_stream,
               1.0f, 0, 1.0f, true);
}

int fsd_profile_enable(int on) {
    g_prof_on = (on != 0);
    return FSD_OK;
}

int fsd_profile_collect(float* mean_ms, float* min_ms) {
    const int n = g_prof_n;
    double sum = 0.0;
    float mn = 0.0f;
    for (int i = 0; i < n; ++i) {
        (void)hipEventSynchronize(g_prof_ev[2 * i + 1]);
        float ms = 0.0f;
        (void)hipEventElapsedTime(&ms, g_prof_ev[2 * i], g_prof_ev[2 * i + 1]);
        sum += ms;
        if (i == 0 || ms < mn) mn = ms;
    }
    if (mean_ms) *mean_ms = n ? static_cast<float>(sum / n) : 0.0f;
    if (min_ms) *min_ms = mn;
    g_prof_n = 0;
    return n;
}

int fsd_debug_set_shape(int wavefronts, int slots_per_thread) {
    const bool ok = (wavefronts == 0 || wavefronts == 4) &&
                    (slots_per_thread == 0 || slots_per_thread == 2 || slots_per_thread == 4 || slots_per_thread == 5 ||
                     slots_per_thread == 8);
    if (!ok) return FSD_ERR_SHAPE;
    g_shape_nv = slots_per_thread;
    return FSD_OK;
}

size_t fsd_debug_warp_threshold_offset(int B, int rows_per_seq, int V, int dtype) {
    Plan p;
    if (!make_plan(B, rows_per_seq, V, dtype, p)) return 0;
    return p.off_thr;
}

void fsd_debug_last_launch(int* grid, int* resident) {
    if (grid) *grid = g_last_grid;
    if (resident) *resident = g_last_total;
}

int fsd_debug_last_route(void) { return g_last_route.load(std::memory_order_relaxed); }

int fsd_debug_set_small_calls(int on) {
    const int prev = g_small_calls ? 1 : 0;
    g_small_calls = (on != 0);
    return prev;
}

int fsd_debug_last_selection(void) { return g_last_selection.load(std::memory_order_relaxed); }

float fsd_debug_set_js_floor(float floor_nats) {
    const float prev = g_js_floor;
    g_js_floor = floor_nats;
    return prev;
}

int fsd_debug_set_exact_js(int on) {
    const int prev = g_exact_js ? 1 : 0;
    g_exact_js = (on != 0);
    return prev;
}

int fsd_debug_set_self_clear(int on) {
    const int prev = g_self_clear ? 1 : 0;
    g_self_clear = (on != 0);
    return prev;
}

unsigned fsd_debug_set_spin_limit(unsigned polls) {
    const unsigned prev = g_spin_limit;
    g_spin_limit = polls;
    return prev;
}

unsigned fsd_debug_set_selection_spin_limit(unsigned polls) {
    const unsigned prev = g_selection_spin_limit;
    g_selection_spin_limit = polls;
    return prev;
}

#ifdef FSD_PHASE_TIMING
void fsd_debug_set_dbg(void* p) { g_dbg = static_cast<unsigned long long*>(p); }
#endif

}  // extern "C"
