// Many independent assignment instances in one launch (the same phase loop
// as solve.hip, arXiv:2203.03732 Section 2.2, with the same proposal rounds
// and tie-break, so every instance's result is identical to a
// single-instance solve on its rounded costs).
//
// Each workgroup pops instances from a queue (largest n first) and solves an
// instance alone: the column keys, the duals, the free and taken lists and
// the active rows of a round all live in LDS, the round barrier is
// __syncthreads, and only the rounded-cost matrix (built beforehand by the
// batched cost kernels) and short lists derived from it are read from memory.
// The kernel does not need co-resident workgroups, so it can be captured in
// a HIP graph and replayed.
//
// The same loop solves a single instance of few columns, or its last phases
// (solo_kernel).
//
// Candidate lists. A free row looks for the first column with
// v = k + t(a) = y(b) - 1 =: need. Its v never fall (t only grows) and need
// never falls (y(b) only grows), so a list of all columns with v < V, taken
// at any time, holds every column the row can find while need < V. Each row
// keeps such a list of at most CAP entries (column, k) with its V, and
// minv, a bound below which it can find nothing: most rows of a phase are
// settled by minv alone (LDS) or by one 128-byte list, read by 8 lanes,
// instead of their 2n bytes of the matrix. A row whose need has passed V
// reads its whole row once (one wave, every chunk in flight), which finds its
// column and writes the next list, with V as high as CAP allows. A row
// with more than CAP columns at v = need gets no list and is read whole
// whenever it is scanned.
//
// Bound: at first instruction issue (every row is read whole once and its list
// made: ~2.8 us a row of 2,048 and wave with 16 waves a CU), later latency: a
// phase of list rows alone takes ~2 us (filter, scan and check, each ended by
// a workgroup barrier), one with whole rows ~3 us more. Whole batched calls,
// against keys compared per column and every scan reading the matrix: 512
// instances of n in [64, 1024], d = 16, eps = 0.05 1.63 -> 1.12 ms (0.91 with
// the present cost build); loss and gradient of 64 x 2048, d = 64, eps = 0.01
// 10.8 -> 5.6 ms (there against teams of 4 workgroups an instance; 5.0 with the
// present build and first lists).
#include "cost_common.h"
#include "device_common.h"
#include "internal.h"
#include "round_slots.h"

#include <cmath>
#include <type_traits>

namespace prot {
namespace {

constexpr uint32_t kListFill = 0x7FFF0000u;  // column 0 with a k that never matches
constexpr uint16_t kNone16 = 0xFFFF;
// Largest y(b) and -y(a): Lemma 3.2 keeps them within K + 2 <= 0x7FFF, so only
// a cost matrix with entries outside [0, 1] (which its rounding reports) gets
// one past it; the point builds place every cost in [0, K]. Up to here need
// stays below the padding's 0x7FFF.
constexpr uint32_t kDualTop = 0x7FFF;
// Rows of a wave from which they are looked at together (kPeek), and instances
// whose 16 waves can have as many. Whole solves, from 8 rows and n > 128 / from 4
// and n > 63, us: 1 x 128, d = 2, eps = 0.2 52.1 / 48.1, 64 x 250, eps = 0.1 71.5 / 67.2;
// from 2 rows 64 x 50, eps = 0.05 5% slower.
constexpr int kPeekMin = 4;
constexpr int32_t kPeekMinN = 63;
constexpr int32_t kBatchWideMax = 256;
constexpr int32_t kBatchNarrowMaxN = 256, kBatchNarrowMin = 1024;
// A column's key: the round above the proposing row in reverse order, so that
// the larger key wins and within a round the smaller row. A key of an earlier
// round never wins, so keys are not cleared between rounds; before the round
// field runs out they are (at a phase start).
constexpr int kKeyRowBits = 11;
constexpr uint32_t kKeyRowMask = (1u << kKeyRowBits) - 1u;
constexpr uint32_t kKeyRounds = 1u << (32 - kKeyRowBits);

__device__ inline uint32_t batch_key(uint32_t r, int b)
{
    return (r << kKeyRowBits) | (kKeyRowMask - (uint32_t)b);
}

// CAP: entries of a row's candidate list, read by CAP / 4 lanes (16 bytes each).
template <int NMAX, int NT, int CAP>
struct BatchShared {
    alignas(16) uint32_t key[NMAX];
    alignas(16) uint16_t t[NMAX];  // -y(a)
    uint16_t mate[NMAX];       // row matched to the column (kNone16: none)
    uint16_t y[NMAX];          // y(b)
    uint16_t minv[NMAX];       // no column of row b has k + t below this
    uint16_t V[NMAX];          // row b's list holds every column with k + t < V (0: no list)
    uint16_t F[2][NMAX];       // free rows: this phase / next phase
    // active rows of this round / the next: rows with a list from the front,
    // rows without one from the back; their scan positions
    uint16_t ab[2][NMAX];
    uint16_t ap[2][NMAX];
    // what a row found this round: a column, or nothing (kNone16) and the
    // smallest k + t it has
    uint16_t pa[NMAX];
    uint16_t pm[NMAX];
    alignas(16) uint32_t stage[NT / 64][CAP];  // a wave's list on its way to memory
    uint32_t wcnt[16];
    long long red_k[16];
    double red_c[16];
    unsigned long long red_s[16];
    uint32_t nF[2];
    // rows with a list, rows without, whether any row proposed: by round_slots.h
    uint32_t nl[kRoundSlots], nd[kRoundSlots], prop[kRoundSlots];
    uint32_t tr_scan[2], tr_none[2];  // per-phase record: entries examined, rows that found none
    uint32_t over;  // a dual passed kDualTop
    int32_t job;
};

// Workgroup barrier for LDS only: stores to global memory may still be in
// flight (__syncthreads waits for them).
__device__ inline void barrier_lds()
{
    asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
}

// x, opaque to the compiler: what is made of it where this stands is not kept
// in registers through the loops around.
__device__ inline int not_hoisted(int x)
{
    asm volatile("" : "+v"(x));
    return x;
}

// Index for this lane's entry of a list with the given counter (every lane
// of the wave calls; one atomic per wave).
__device__ inline uint32_t wave_push(uint32_t *counter, bool want)
{
    const unsigned long long bal = __ballot(want);
    uint32_t at = 0;
    if (bal != 0ull && (threadIdx.x & 63) == 0) at = atomicAdd(counter, (uint32_t)__popcll(bal));
    return __builtin_amdgcn_readfirstlane(at) + lanes_below(bal);
}

// Two 16-bit values at a time.
typedef uint16_t u16x2 __attribute__((ext_vector_type(2)));
__device__ inline u16x2 as_pair(uint32_t w) { return __builtin_bit_cast(u16x2, w); }
__device__ inline uint32_t as_word(u16x2 v) { return __builtin_bit_cast(uint32_t, v); }

// In each half: 1 if its value exceeds D's, else 0 (a saturating subtraction
// and a minimum; written out because the compiler takes the pair apart into
// two compares and two selects). one: 1 in both halves.
__device__ inline uint32_t pairs_above(uint32_t v, uint32_t D, uint32_t one)
{
    uint32_t r;
    asm("v_pk_sub_u16 %0, %1, %2 clamp" : "=v"(r) : "v"(v), "v"(D));
    asm("v_pk_min_u16 %0, %1, %2" : "=v"(r) : "v"(r), "v"(one));
    return r;
}
// Bit e set iff element e of four pairs is at most D, from the OR of
// pairs_above(word w) << 2w.
__device__ inline uint32_t low_bits(uint32_t x) { return ~(x | (x >> 15)) & 0xFFu; }

// Bit i set iff any of bits 4 i .. 4 i + 3 is.
__device__ inline uint32_t rows_of(unsigned long long x)
{
    x |= x >> 2;
    x = (x | x >> 1) & 0x1111111111111111ull;
    x = (x | x >> 3) & 0x0303030303030303ull;
    x = (x | x >> 6) & 0x000F000F000F000Full;
    x = (x | x >> 12) & 0x000000FF000000FFull;
    return (uint32_t)(x | x >> 24) & 0xFFFFu;
}

// The rounded costs of columns col0 .. col0 + 7 of a row. A matrix of bytes
// (kBytes) holds padding as 0xFF, which becomes the 0x7FFF of a 16-bit one.
template <bool kBytes>
__device__ inline uint4 load_8(const int16_t *__restrict__ k, int64_t at)
{
    if constexpr (!kBytes) return *reinterpret_cast<const uint4 *>(k + at);
    const uint2 v = *reinterpret_cast<const uint2 *>(reinterpret_cast<const uint8_t *>(k) + at);
    auto widen = [](uint32_t w, uint32_t sel) {
        const u16x2 p = as_pair(__builtin_amdgcn_perm(0u, w, sel));
        return as_word(p | (((p + (u16x2)(uint16_t)1) >> (u16x2)(uint16_t)8) *
                            (u16x2)(uint16_t)0x7F00));
    };
    return make_uint4(widen(v.x, 0x0C010C00u), widen(v.x, 0x0C030C02u), widen(v.y, 0x0C010C00u),
                      widen(v.y, 0x0C030C02u));
}

// A whole row held by one wave: chunk c is columns 512 c + 8 lane .. + 7.
template <int NC>
struct RowRegs {
    uint4 c[NC];
};
template <int NC, bool kBytes>
__device__ RowRegs<NC> load_row(const int16_t *__restrict__ k, int64_t row, int n, int lane)
{
    RowRegs<NC> r;
#pragma unroll
    for (int c = 0; c < NC; ++c) {
        const int col0 = c * 512 + lane * 8;
        r.c[c] = make_uint4(0x7FFF7FFFu, 0x7FFF7FFFu, 0x7FFF7FFFu, 0x7FFF7FFFu);
        if (col0 < n) r.c[c] = load_8<kBytes>(k, row + col0);
    }
    return r;
}

// d[i] for a lane's own index i: a tree of bitwise selects (registers cannot
// be indexed by a lane's value, and a select written with ?: is turned back
// into an array in memory).
template <int N>
struct SelectWord {
    static __device__ inline uint32_t get(const uint32_t (&d)[N], uint32_t i)
    {
        const uint32_t m = 0u - (i & 1u);
        uint32_t h[N / 2];
#pragma unroll
        for (int e = 0; e < N / 2; ++e) h[e] = (d[2 * e] & ~m) | (d[2 * e + 1] & m);
        return SelectWord<N / 2>::get(h, i >> 1);
    }
};
template <>
struct SelectWord<1> {
    static __device__ inline uint32_t get(const uint32_t (&d)[1], uint32_t) { return d[0]; }
};

// First admissible column of a row in scan order from column `origin`, by one
// wave; every column is compared. The row's bounds and list are renewed:
// *minv = the smallest k + t if nothing is admissible (a column taken this
// phase counts with its raised t), and the columns with v < *V go to `stage`
// (kListCap entries of LDS; *V = 0 if more than that have v = need, then there
// is no list). V - 1 starts *window above the smallest v and is halved towards it
// until the list fits, or widened while it holds fewer than kListCap / 4.
// k: the row; S_t: the duals in LDS.
// Bound: instruction issue (about 3 instructions per 2 columns and pass over
// the row: the sums and their minimum, then one or two list masks).
template <int NC, int kListCap>
__device__ Hit direct_row(const RowRegs<NC> &k, const uint16_t *S_t, int n,
                          int origin, int need, int lane, uint32_t *stage, uint16_t *minv,
                          uint16_t *V, int *window)
{
    const uint32_t one = 0x10001u;
    const u16x2 need2 = (u16x2)(uint16_t)need;
    uint32_t d[4 * NC];  // k + t - need
    u16x2 mn2 = (u16x2)(uint16_t)0xFFFF;
#pragma unroll
    for (int c = 0; c < NC; ++c) {
        const uint32_t kw[4] = {k.c[c].x, k.c[c].y, k.c[c].z, k.c[c].w};
        const int col0 = c * 512 + lane * 8;
        const uint4 t = *reinterpret_cast<const uint4 *>(S_t + (col0 < n ? col0 : 0));
        const uint32_t tw[4] = {t.x, t.y, t.z, t.w};
#pragma unroll
        for (int w = 0; w < 4; ++w) {
            const u16x2 v = as_pair(kw[w]) + as_pair(tw[w]) - need2;
            d[4 * c + w] = as_word(v);
            mn2 = __builtin_elementwise_min(mn2, v);
        }
    }
    const int mn = (int)wave_min_u32(min(as_word(mn2) & 0xFFFFu, as_word(mn2) >> 16));
    // bit 8c + e: column 512 c + 8 lane + e has v <= need + D
    auto mask_of = [&](int D) {
        const uint32_t D2 = (uint32_t)D * 0x10001u;
        uint32_t W = 0;
#pragma unroll
        for (int c = 0; c < NC; ++c) {
            uint32_t x = 0;
#pragma unroll
            for (int w = 0; w < 4; ++w)
                x |= pairs_above(d[4 * c + w], D2, one) << (2 * w);
            W |= low_bits(x) << (8 * c);
        }
        return W;
    };
    Hit h{-1, -1};
    *minv = (uint16_t)min(0xFFFF, need + mn);
    if (mn == 0) {
        const uint32_t M = mask_of(0);
        uint32_t G = 0;  // columns from the origin on
#pragma unroll
        for (int c = 0; c < NC; ++c) {
            const int s = origin - (c * 512 + lane * 8);
            G |= (s <= 0 ? 0xFFu : s >= 8 ? 0u : (0xFFu << s) & 0xFFu) << (8 * c);
        }
        uint32_t j = 0x7FFFFFFFu;
        if (M != 0u) {
            const uint32_t A = M & G;
            const int i = __builtin_ctz(A ? A : M);
            const int col = (i >> 3) * 512 + lane * 8 + (i & 7);
            j = (uint32_t)(A ? col - origin : col - origin + n);
        }
        h.j = (int)wave_min_u32(j);
        h.a = origin + h.j < n ? origin + h.j : origin + h.j - n;
    }
    // padding has v - need = 0x7FFF - need, above dcap
    const int dcap = 0x7FFE - need;
    if (mn > dcap) {  // (nothing within 15 bits: every v is at least minv)
        *V = 0;
        return h;
    }
    int D = min(mn + *window, dcap);
    uint32_t W, incl;
    int cnt;
    for (bool grown = false;;) {
        W = mask_of(D);
        incl = wave_inclusive_sum_u32((uint32_t)__builtin_popcount(W));
        cnt = __builtin_amdgcn_readlane((int)incl, 63);
        if (cnt > kListCap) {
            if (D == mn) break;
            D = mn + ((D - mn) >> 1);
            grown = true;  // do not widen again
        } else if (!grown && cnt < kListCap / 4 && D < dcap) {
            const int next = min(D + 1 + ((D - mn) >> 1), dcap);
            if (D - mn > 64) grown = true;
            D = next;
        } else {
            break;
        }
    }
    *window = D - mn;
    if (cnt > kListCap) {
        // too many at the smallest v: an empty list up to it, or none
        if (mn == 0) {
            *V = 0;
            return h;
        }
        D = mn - 1;
        W = 0u;
        cnt = 0;
        incl = 0u;
    }
    *V = (uint16_t)(need + D + 1);
    uint32_t at = incl - (uint32_t)__builtin_popcount(W);
    while (W) {
        const int i = __builtin_ctz(W);
        W &= W - 1u;
        const int col = (i >> 3) * 512 + lane * 8 + (i & 7);
        const uint32_t pair = SelectWord<4 * NC>::get(d, (uint32_t)i >> 1);
        const uint32_t v = ((i & 1) ? pair >> 16 : pair & 0xFFFFu) + (uint32_t)need;
        stage[at++] = (uint32_t)col | ((v - S_t[col]) << 16);
    }
#pragma unroll
    for (int i = 0; i < kListCap; i += 64)
        if (i + lane >= cnt && i + lane < kListCap) stage[i + lane] = kListFill;
    return h;
}

// An instance: nb rows, na >= nb columns.
struct LdsJob {
    int nb, na;
    const int16_t *k;  // or bytes (kBytes)
    int64_t ldk;
    uint32_t *lists;
    int64_t T, max_phases, bound;
    int origin;
    int64_t *trace, *rtime;  // may be null
    const uint32_t *first;   // bounds of lists made beforehand (first_lists_kernel), or null
};
// Its totals, and where its free rows are (S.F[cur]).
struct LdsRun {
    int64_t phases, sum_free, rounds, max_rounds;
    unsigned long long scanned;  // this thread's share
    int status;                  // 0, 1 stopped at max_phases, 2 by the bound, 4 by kDualTop
    int cur;
};

// Initial state (Section 2.2): y(b) = 1, y(a) = 0, M empty.
template <int NMAX, int NT, int CAP>
__device__ void lds_cold(const LdsJob &J, BatchShared<NMAX, NT, CAP> &S)
{
    for (int i = threadIdx.x; i < ((J.na + 7) & ~7); i += NT) S.t[i] = 0;
    for (int i = threadIdx.x; i < J.na; i += NT) S.mate[i] = kNone16;
    for (int i = threadIdx.x; i < J.nb; i += NT) {
        S.y[i] = 1;
        S.F[0][i] = (uint16_t)i;
    }
    if (threadIdx.x == 0) S.nF[0] = (uint32_t)J.nb;
}

// The phases from the state in S (t, mate, y, F[0] and nF[0], set by any
// thread) until at most T rows are free. kSingle: a single instance, whose
// phases are recorded and whose duals are watched (kDualTop). kPeek: rows are
// likely to find their column at once (rows_content).
template <int NMAX, int NT, int CAP, bool kSingle, bool kBytes, bool kPeek>
__device__ void lds_phases(const LdsJob &J, LdsRun &R, BatchShared<NMAX, NT, CAP> &S)
{
    constexpr int NC = NMAX / 512;
    constexpr int kWaves = NT / 64;
    constexpr int kListCap = CAP, kListLanes = CAP / 4;
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int n = J.na;
    const int16_t *k = J.k;
    const int64_t ldk = J.ldk;
    uint32_t *lists = J.lists;
    const bool timed = J.rtime != nullptr;
    // no lists (V = 0) and nothing known (minv = 0 makes every row look), or
    // the lists made beforehand
    for (int i = tid; i < n; i += NT) {
        const uint32_t f = J.first && i < J.nb ? J.first[i] : 0u;
        S.key[i] = 0u;
        S.minv[i] = (uint16_t)f;
        S.V[i] = (uint16_t)(f >> 16);
    }
    if (tid == 0) {
        S.nF[1] = 0;
        S.over = 0;
        for (int i = 0; i < kRoundSlots; ++i) S.nl[i] = S.nd[i] = S.prop[i] = 0;
        S.tr_scan[0] = S.tr_scan[1] = S.tr_none[0] = S.tr_none[1] = 0;
    }
    int64_t phases = R.phases, sum_free = 0, rounds = 0, max_rounds = R.max_rounds;
    unsigned long long scanned = 0;  // this thread's share
    // the last finished phase's record, written by thread 0 once every wave
    // has passed a barrier after adding to it
    int64_t traced = -1;
    uint32_t tr_free = 0;
    int64_t tr_rounds = 0;
    auto write_trace = [&]() {
        if (traced < 0 || tid != 0) return;
        const int e = (int)(traced & 1);
        if (J.trace && traced < kTraceCap) {
            int64_t *t = J.trace + 4 * traced;
            t[0] = tr_free;
            t[1] = tr_rounds;
            t[2] = S.tr_scan[e];
            t[3] = (int64_t)tr_free - S.tr_none[e];
        }
        S.tr_scan[e] = S.tr_none[e] = 0;
        traced = -1;
    };
    uint32_t r = 0;
    int cur = 0, q = 0;
    int s = 0;           // slot of the round's counters (round_slots.h)
    int status = R.status;
    int window = 4;      // of this wave's last list (direct_row)
    bool quick = true;   // this wave looks at 512 columns before a whole row
    bool peek = true;    // and at 32 before those (kPeek)
    uint32_t block = 8;
    // A dual rises by at most one a phase, so it can be past kDualTop only after
    // that many of them; from then on each phase of a single instance looks
    // before it scans. (A batch's costs are in range; its solves took 1% longer
    // with the test.)
    auto look_past_top = [&]() {
        for (int i = tid; i < n; i += NT)
            if (S.t[i] > kDualTop || (i < J.nb && S.y[i] > kDualTop)) S.over = 1;
    };
    __syncthreads();
    for (;;) {
        const uint32_t nF = S.nF[cur];
        if ((int64_t)nF <= J.T || status != 0) break;
        if (J.max_phases > 0 && phases >= J.max_phases) {
            status = 1;
            break;
        }
        if (J.bound > 0 && phases >= J.bound) {
            status = 2;
            break;
        }
        const unsigned long long scanned_before = scanned;
        uint32_t none = 0;  // rows of this wave that found no column
        phases += 1;
        sum_free += nF;
        const int nx = cur ^ 1;
        if (r + (uint32_t)n + 2u >= kKeyRounds) {
            for (int i = tid; i < n; i += NT) S.key[i] = 0u;
            r = 0;
        }
        // The rows of B' sorted by what they need: nothing (no column can be
        // admissible: exhausted as a scan would be), their list, or their row.
        for (uint32_t i0 = wave * 64; i0 < nF; i0 += NT) {
            const bool in = i0 + lane < nF;
            int b = 0, need = 0;
            bool skip = false, listed = false;
            if (in) {
                b = S.F[cur][i0 + lane];
                need = (int)S.y[b] - 1;
                skip = need < (int)S.minv[b];
                listed = !skip && need < (int)S.V[b];
            }
            const uint32_t f = wave_push(&S.nF[nx], skip);
            if (kSingle) none += (uint32_t)__popcll(__ballot(skip));
            const uint32_t l = wave_push(&S.nl[s], listed);
            const uint32_t dd = wave_push(&S.nd[s], in && !skip && !listed);
            if (skip) {
                S.y[b] = (uint16_t)(need + 2);
                S.F[nx][f] = (uint16_t)b;
                scanned += (unsigned long long)n;
            } else if (in) {
                const uint32_t at = listed ? l : (uint32_t)(NMAX - 1) - dd;
                S.ab[q][at] = (uint16_t)b;
                S.ap[q][at] = 0;
            }
        }
        if (kSingle && phases >= (int64_t)kDualTop) look_past_top();
        __syncthreads();
        // (written between the last barrier and this one only)
        if (kSingle && phases >= (int64_t)kDualTop && S.over) {
            status = 4;
            break;
        }
        if (kSingle) write_trace();
        int64_t phase_rounds = 0;
        for (;;) {
            r += 1;
            const uint32_t nl = S.nl[s], nd = S.nd[s];
            const int64_t t_start = timed ? (int64_t)wall_clock64() : 0;
            if (tid == 0) {
                // (nF[cur]: read by everyone before the barrier that began
                // the phase, next used after the phase)
                for (int i = 0; i < kRoundSlots; ++i)
                    if (cleared_by(s, i)) S.nl[i] = S.nd[i] = S.prop[i] = 0;
                S.nF[cur] = 0;
            }
            // Rows without a list: one wave each, up to 64 of the wave's rows at
            // a time (8 at first, to find out which way suits them). Where admissible columns are many (rows that overflow
            // their lists) the 512 columns from the row's position usually
            // hold one: `quick` looks there first and leaves the misses to
            // the whole-row pass. It is on while at least half its rows hit,
            // and comes back when half the rows of a whole-row pass overflow.
            int rows;
            for (uint32_t i0 = wave; i0 < nd; i0 += kWaves * rows) {
                rows = (int)min(block, (nd - i0 + kWaves - 1) / kWaves);
                block = 64u;
                unsigned long long left = rows == 64 ? ~0ull : (1ull << rows) - 1ull;
                auto slot = [&](int e) { return NMAX - 1 - (int)i0 - e * kWaves; };
                if (quick) {
                    auto start_of = [&](int b, int pos) {
                        int c = (J.origin == 0 ? b : 0) + pos;
                        return c >= n ? c - n : c;
                    };
                    // Many rows: first the 32 columns from each row's position,
                    // 16 rows at a time, 4 lanes a row. On while at least half
                    // the rows hit.
                    if (kPeek && peek && rows >= kPeekMin) {
                        const int ln = not_hoisted(lane);
                        auto peek_at = [&](int e, int *b, int *c) {
                            *b = -1;
                            uint4 kv = make_uint4(~0u, ~0u, ~0u, ~0u);
                            if (e < rows) {
                                *b = S.ab[q][slot(e)];
                                *c = start_of(*b, S.ap[q][slot(e)]);
                                const int col0 = (*c & ~7) + (ln & 3) * 8;
                                if (col0 < n) kv = load_8<kBytes>(k, (int64_t)*b * ldk + col0);
                            }
                            return kv;
                        };
                        int bn, cn = 0;
                        uint4 kn = peek_at(ln >> 2, &bn, &cn);
                        for (int e0 = 0; e0 < rows; e0 += 16) {
                            const int b = bn, c = cn, e = e0 + (ln >> 2);
                            const uint4 kv = kn;
                            if (e0 + 16 < rows) kn = peek_at(e + 16, &bn, &cn);
                            const int origin = J.origin == 0 ? b : 0;
                            const int end = c < origin ? origin : n;
                            const int col0 = (c & ~7) + (ln & 3) * 8;
                            uint32_t m = 0;
                            if (b >= 0 && col0 < end)
                                m = match_mask(kv, *reinterpret_cast<const uint4 *>(&S.t[col0]),
                                               (int)S.y[b] - 1) &
                                    range_mask(col0, c, end);
                            // the first of a row's lanes with a hit proposes
                            const uint32_t lower = (1u << (ln & 3)) - 1u;
                            const bool mine =
                                m != 0u && ((uint32_t)(__ballot(m != 0u) >> (ln & 60)) & lower) == 0u;
                            if (mine) {
                                const int a = col0 + __builtin_ctz(m), at = slot(e);
                                const int j = a >= origin ? a - origin : a - origin + n;
                                scanned += (unsigned long long)(j - (int)S.ap[q][at] + 1);
                                S.pa[at] = (uint16_t)a;
                                S.ap[q][at] = (uint16_t)j;
                                S.prop[s] = 1;
                                atomicMax(&S.key[a], batch_key(r, b));
                            }
                            left &= ~((unsigned long long)rows_of(__ballot(mine)) << e0);
                        }
                        peek = 2 * __builtin_popcountll(left) <= rows;
                    }
                    auto load_window = [&](int e, int *b, int *c) {
                        *b = __builtin_amdgcn_readfirstlane((int)S.ab[q][slot(e)]);
                        *c = start_of(*b, __builtin_amdgcn_readfirstlane((int)S.ap[q][slot(e)]));
                        const int col0 = (*c & ~7) + lane * 8;
                        return col0 < n ? load_8<kBytes>(k, (int64_t)*b * ldk + col0)
                                        : make_uint4(~0u, ~0u, ~0u, ~0u);
                    };
                    int bn, cn;
                    uint4 kn;
                    unsigned long long todo = left;
                    if (todo) kn = load_window(__builtin_ctzll(todo), &bn, &cn);
                    while (todo) {
                        const int e = __builtin_ctzll(todo);
                        const int b = bn, c = cn, at = slot(e);
                        const uint4 kv = kn;
                        todo &= todo - 1ull;
                        if (todo) kn = load_window(__builtin_ctzll(todo), &bn, &cn);
                        const int need = __builtin_amdgcn_readfirstlane((int)S.y[b] - 1);
                        const int col0 = (c & ~7) + lane * 8;
                        // a scan that started at origin + pos wraps at n and ends
                        // before its origin
                        const int origin = J.origin == 0 ? b : 0;
                        const int end = c < origin ? origin : n;
                        uint32_t m = 0;
                        if (col0 < end)
                            m = match_mask(kv, *reinterpret_cast<const uint4 *>(&S.t[col0]), need) &
                                range_mask(col0, c, end);
                        const unsigned long long bal = __ballot(m != 0u);
                        if (bal == 0ull) continue;
                        left &= ~(1ull << e);
                        const int L = __builtin_ctzll(bal);
                        const int a = (c & ~7) + L * 8 +
                                      __builtin_ctz((uint32_t)__builtin_amdgcn_readlane((int)m, L));
                        if (lane != 0) continue;
                        const int j = a >= origin ? a - origin : a - origin + n;
                        scanned += (unsigned long long)(j - (int)S.ap[q][at] + 1);
                        S.pa[at] = (uint16_t)a;
                        S.ap[q][at] = (uint16_t)j;
                        S.prop[s] = 1;
                        atomicMax(&S.key[a], batch_key(r, b));
                    }
                    quick = 2 * __builtin_popcountll(left) <= rows;
                }
                // whole rows; the next row's loads in flight while one is compared
                if (left == 0ull) continue;
                int en = __builtin_ctzll(left), overflowed = 0;
                const int full = __builtin_popcountll(left);
                int bn = __builtin_amdgcn_readfirstlane((int)S.ab[q][slot(en)]);
                RowRegs<NC> kn = load_row<NC, kBytes>(k, (int64_t)bn * ldk, n, lane);
                // A row's list is stored while the next row is looked at,
                // before the loads of the row after that: the wait for those
                // loads then does not wait for a store just issued.
                int stored = -1;
                auto store_list = [&]() {
                    if (stored >= 0 && lane < kListLanes)
                        *reinterpret_cast<uint4 *>(lists + (int64_t)stored * kListCap + lane * 4) =
                            *reinterpret_cast<const uint4 *>(&S.stage[wave][lane * 4]);
                };
                while (left) {
                    const int b = bn, at = slot(en);
                    const RowRegs<NC> kr = kn;
                    left &= left - 1ull;
                    store_list();
                    if (left) {
                        en = __builtin_ctzll(left);
                        bn = __builtin_amdgcn_readfirstlane((int)S.ab[q][slot(en)]);
                        kn = load_row<NC, kBytes>(k, (int64_t)bn * ldk, n, lane);
                    }
                    const int need = __builtin_amdgcn_readfirstlane((int)S.y[b] - 1);
                    const int pos = S.ap[q][at];
                    const int origin = J.origin == 0 ? b : 0;
                    uint16_t minv, V;
                    const Hit h = direct_row<NC, CAP>(kr, S.t, n, origin, need, lane, S.stage[wave],
                                                 &minv, &V, &window);
                    stored = V ? b : -1;
                    overflowed += V == 0;
                    if (lane != 0) continue;
                    S.V[b] = V;
                    S.pa[at] = (uint16_t)h.a;
                    if (h.j >= 0) {
                        scanned += (unsigned long long)(h.j - pos + 1);
                        S.ap[q][at] = (uint16_t)h.j;
                        S.prop[s] = 1;
                        atomicMax(&S.key[h.a], batch_key(r, b));
                    } else {
                        scanned += (unsigned long long)(n - pos);
                        S.pm[at] = minv;
                    }
                }
                store_list();
                if (2 * overflowed >= full) quick = peek = true;
            }
            // rows with a list: kListLanes lanes each
            for (uint32_t i0 = wave * (64 / kListLanes); i0 < nl; i0 += NT / kListLanes) {
                const uint32_t i = i0 + (uint32_t)(lane / kListLanes);
                const bool in = i < nl;
                int b = 0, need = 0, pos = 0, origin = 0;
                uint32_t j = 0x7FFFFFFFu, lo = 0x7FFFFFFFu;
                if (in) {
                    b = S.ab[q][i];
                    const uint4 e = *reinterpret_cast<const uint4 *>(
                        lists + (int64_t)b * kListCap + (lane % kListLanes) * 4);
                    need = (int)S.y[b] - 1;
                    pos = S.ap[q][i];
                    origin = J.origin == 0 ? b : 0;
                    const uint32_t ew[4] = {e.x, e.y, e.z, e.w};
#pragma unroll
                    for (int u = 0; u < 4; ++u) {
                        const int a = (int)(ew[u] & 0xFFFFu);
                        const uint32_t v = (ew[u] >> 16) + S.t[a];
                        const uint32_t ja = (uint32_t)(a >= origin ? a - origin : a - origin + n);
                        if (v == (uint32_t)need) j = min(j, ja);
                        lo = min(lo, v);
                    }
                }
                j = group_min_u32<kListLanes>(j);
                lo = group_min_u32<kListLanes>(lo);
                if (!in || lane % kListLanes != 0) continue;
                if (j != 0x7FFFFFFFu) {
                    const int a = origin + (int)j < n ? origin + (int)j : origin + (int)j - n;
                    scanned += (unsigned long long)((int)j - pos + 1);
                    S.pa[i] = (uint16_t)a;
                    S.ap[q][i] = (uint16_t)j;
                    S.prop[s] = 1;
                    atomicMax(&S.key[a], batch_key(r, b));
                } else {
                    scanned += (unsigned long long)(n - pos);
                    S.pa[i] = kNone16;
                    S.pm[i] = (uint16_t)min(lo, (uint32_t)S.V[b]);  // v >= V off the list
                }
            }
            // (the lists written are read after the next barrier at the earliest)
            barrier_lds();
            if (timed && tid == 0 && 4u * r <= 3u * (uint32_t)kRoundTimeCap) {
                J.rtime[4 * (r - 1)] = t_start;
                J.rtime[4 * (r - 1) + 1] = (int64_t)wall_clock64();
                J.rtime[4 * (r - 1) + 2] = nl + nd;
                J.rtime[4 * (r - 1) + 3] = phases;
            }
            if (S.prop[s]) phase_rounds += 1;
            // Winners: step (II), the column's old mate is free in the next
            // phase, and (III a) for the column, y(a) -= 1, at once: every
            // slack v - need is >= 0, so raising t also takes the column out of
            // every row's sight for the rest of the phase. Losers look on from
            // one position after the column they lost. A row that found nothing
            // stays free in M', (III b).
            const uint32_t top = nl + nd;
            for (uint32_t i0 = wave * 64; i0 < top; i0 += NT) {
                const uint32_t i = i0 + lane;
                const uint32_t at = i < nl ? i : (uint32_t)(NMAX - 1) - (i - nl);
                int a = kNone16, b = 0;
                int freed = kNone16;
                bool won = false, lost = false, listed = false;
                if (i < top) {
                    a = S.pa[at];
                    b = S.ab[q][at];
                    if (a != kNone16) {
                        won = S.key[a] == batch_key(r, b);
                        lost = !won;
                        if (won) {
                            freed = S.mate[a];
                            S.mate[a] = (uint16_t)b;
                            S.t[a] = (uint16_t)(S.t[a] + 1u);
                        } else {
                            // (this round may just have given the row a list)
                            listed = (int)S.y[b] - 1 < (int)S.V[b];
                        }
                    } else {
                        freed = b;
                        S.y[b] = (uint16_t)(S.y[b] + 1u);
                        S.minv[b] = S.pm[at];
                    }
                }
                if (kSingle) none += (uint32_t)__popcll(__ballot(i < top && a == kNone16));
                const uint32_t f = wave_push(&S.nF[nx], freed != kNone16);
                const uint32_t l = wave_push(&S.nl[losers_slot(s)], listed);
                const uint32_t dd = wave_push(&S.nd[losers_slot(s)], lost && !listed);
                if (freed != kNone16) S.F[nx][f] = (uint16_t)freed;
                if (lost) {
                    const uint32_t to = listed ? l : (uint32_t)(NMAX - 1) - dd;
                    S.ab[q ^ 1][to] = (uint16_t)b;
                    S.ap[q ^ 1][to] = (uint16_t)(S.ap[q][at] + 1);
                }
            }
            __syncthreads();
            q ^= 1;
            const int lost_s = losers_slot(s);
            if (S.nl[lost_s] + S.nd[lost_s] == 0u) {  // nobody lost: M' is maximal
                s = phase_slot(s);
                break;
            }
            s = lost_s;
        }
        rounds += phase_rounds;
        if (phase_rounds > max_rounds) max_rounds = phase_rounds;
        cur = nx;
        if (kSingle) {
            const uint32_t sc = wave_sum_u32((uint32_t)(scanned - scanned_before));
            if (lane == 0) {
                if (sc) atomicAdd(&S.tr_scan[(phases - 1) & 1], sc);
                if (none) atomicAdd(&S.tr_none[(phases - 1) & 1], none);
            }
            traced = phases - 1;
            tr_free = nF;
            tr_rounds = phase_rounds;
        }
    }
    if (kSingle && phases >= (int64_t)kDualTop) {
        look_past_top();
        __syncthreads();
        if (S.over) status = 4;
    }
    if (kSingle) {
        __syncthreads();
        write_trace();
    }
    R.phases = phases;
    R.sum_free += sum_free;
    R.rounds += rounds;
    R.max_rounds = max_rounds;
    R.scanned += scanned;
    R.status = status;
    R.cur = cur;
}

// The matching from the mates: mb = S.ap[0], ma = S.ap[1] (kNone16: free; the
// free rows are F[cur], the free columns the never-taken ones). complete
// (Section 2.1): i-th free b (ascending) with the i-th free a (ascending).
template <int NMAX, int NT, int CAP>
__device__ void lds_matching(const LdsJob &J, int cur, bool complete, BatchShared<NMAX, NT, CAP> &S)
{
    constexpr int kWaves = NT / 64;
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const uint32_t nfree = S.nF[cur];
    uint16_t *mb = S.ap[0], *ma = S.ap[1];
    for (int i = tid; i < J.nb; i += NT) {
        mb[i] = kNone16;
        S.pa[i] = 0;
    }
    __syncthreads();
    for (int i = tid; i < J.na; i += NT) {
        const uint16_t b = S.mate[i];
        ma[i] = b;
        if (b != kNone16) mb[b] = (uint16_t)i;
    }
    for (uint32_t i = tid; i < nfree; i += NT) S.pa[S.F[cur][i]] = 1;
    __syncthreads();
    // ascending list of the i < n with flag(i), by all threads
    auto ordered_list = [&](int n, auto flag, uint16_t *out) {
        int base = 0;
        for (int i0 = 0; i0 < n; i0 += NT) {
            const bool f = i0 + tid < n && flag(i0 + tid);
            const unsigned long long bal = __ballot(f);
            if (lane == 0) S.wcnt[wave] = (uint32_t)__popcll(bal);
            __syncthreads();
            int before = base, total = base;
            for (int w = 0; w < kWaves; ++w) {
                if (w < wave) before += (int)S.wcnt[w];
                total += (int)S.wcnt[w];
            }
            if (f) out[before + (int)lanes_below(bal)] = (uint16_t)(i0 + tid);
            base = total;
            __syncthreads();
        }
        return base;
    };
    if (!complete) return;
    const int nb = ordered_list(J.nb, [&](int i) { return S.pa[i] != 0; }, S.ab[0]);
    const int na = ordered_list(J.na, [&](int i) { return S.mate[i] == kNone16; }, S.ab[1]);
    const int m = min(nb, na);
    for (int i = tid; i < m; i += NT) {
        mb[S.ab[0][i]] = S.ab[1][i];
        ma[S.ab[1][i]] = S.ab[0][i];
    }
    __syncthreads();
}

template <int NMAX, int NT, int CAP, bool kPeek>
__device__ void solve_instance(const BatchArgs &A, int inst, BatchShared<NMAX, NT, CAP> &S, bool timed)
{
    constexpr int kWaves = NT / 64;
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int n = A.n_arr[inst];
    const int64_t off = A.pt_off[inst];
    const int16_t *k = A.k + A.k_off[inst];
    const int64_t ldk = A.ldk_arr[inst];
    const int64_t T = (int64_t)floor(A.eps * (double)n + 1e-9);
    // the watchdog: a cold start needs at most (2n(K + 2) - n) / (T + 1)
    // phases (Lemma 3.2 with eq. (4)); more means a fault
    const int64_t bound =
        A.phase_bound ? A.phase_bound
                      : (2 * (int64_t)n * ((int64_t)floor(1.0 / A.eps) + 2) - n) / (T + 1);
    const LdsJob J{n, n, k, ldk, A.lists + off * CAP, T, A.max_phases, bound, A.origin,
                   nullptr, timed ? A.rtime : nullptr, A.first ? A.first + off : nullptr};
    LdsRun R{};
    lds_cold(J, S);
    lds_phases<NMAX, NT, CAP, false, false, kPeek>(J, R, S);
    unsigned long long scanned = R.scanned;
    const int status = R.status == 2 ? -4 : R.status;
    if (R.status == 2 && tid == 0)
        __hip_atomic_fetch_or(A.err, 256, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    const uint32_t nfree = S.nF[R.cur];
    lds_matching(J, R.cur, A.complete && status >= 0, S);
    const uint16_t *mb = S.ap[0], *ma = S.ap[1];

    // Outputs and per-instance statistics (fixed-order reductions).
    const float *X = A.X + off * A.d, *Y = A.Y + off * A.d;
    long long ks = 0;
    double cs = 0.0;
    for (int i = tid; i < n; i += NT) {
        const int a = mb[i] == kNone16 ? -1 : (int)mb[i];
        A.mate_a[off + i] = ma[i] == kNone16 ? -1 : (int)ma[i];
        A.mate_b[off + i] = a;
        A.y_a[off + i] = -(int32_t)S.t[i];
        A.y_b[off + i] = S.y[i];
        if (a >= 0) {
            ks += k[(int64_t)i * ldk + a];
            double s = 0.0;
            for (int e = 0; e < A.d; ++e) {
                const double dq = __dsub_rn((double)X[(int64_t)i * A.d + e], (double)Y[(int64_t)a * A.d + e]);
                s = __dadd_rn(s, __dmul_rn(dq, dq));
            }
            cs = __dadd_rn(cs, s);
        }
    }
    for (int o = 32; o > 0; o >>= 1) {
        ks += __shfl_xor(ks, o);
        cs = __dadd_rn(cs, __shfl_xor(cs, o));
        scanned += __shfl_xor(scanned, o);
    }
    if (lane == 0) {
        S.red_k[wave] = ks;
        S.red_c[wave] = cs;
        S.red_s[wave] = scanned;
    }
    __syncthreads();
    if (tid == 0) {
        for (int w = 1; w < kWaves; ++w) {
            ks += S.red_k[w];
            cs = __dadd_rn(cs, S.red_c[w]);
            scanned += S.red_s[w];
        }
        InstanceStats &st = A.stats[inst];
        const float m = A.m[inst];
        st.phases = R.phases;
        st.sum_free = R.sum_free;
        st.rounds = R.rounds;
        st.max_rounds = R.max_rounds;
        st.scanned = (int64_t)scanned;
        st.matched_in_phases = n - (int64_t)nfree;
        st.completed_pairs = A.complete ? (int64_t)nfree : 0;
        st.sum_k = ks;
        st.threshold = T;
        st.status = status;
        st.kmax = m > 0.0f ? (int32_t)floor(1.0 / A.eps) : 0;
        st.cost_scale = (double)m;
        st.cost = m > 0.0f ? cs / (double)m : 0.0;
    }
    __syncthreads();
}

template <int NMAX, int NT, bool kPeek>
// (4 waves per SIMD: two workgroups of 512 threads or one of 1,024 a CU)
__global__ void __launch_bounds__(NT, 4) batch_solve_kernel(BatchArgs A)
{
    __shared__ BatchShared<NMAX, NT, kBatchListCap> S;
    for (;;) {
        if (threadIdx.x == 0)
            S.job = (int32_t)__hip_atomic_fetch_add(A.queue, 1u, __ATOMIC_RELAXED,
                                                    __HIP_MEMORY_SCOPE_AGENT);
        __syncthreads();
        const int job = S.job;
        __syncthreads();
        if (job >= A.batch) break;
        solve_instance<NMAX, NT, kBatchListCap, kPeek>(A, A.order[job], S, A.rtime != nullptr && job == 0);
    }
}

// One instance, from the start (cold) or from the state that a phase loop of
// many workgroups left in the outputs once few rows were free. The outputs,
// the completion and the control block are those of the kernels that follow
// the loop.
// Bound: latency, three workgroup barriers and two dependent LDS or list
// reads a phase, ~2.5 us more where a row is read whole. Euclidean cost,
// d = 2, eps = 0.01, whole solves: n = 300 (1,259 phases) 8.4 -> 3.4 ms, 1,024
// (1,416) 9.4 -> 5.2, 2,048 (1,528) 10.7 -> 7.6; with lists of 32 entries 3.8,
// 5.4 and 8.0, of 128 3.2, 5.0 and 7.7 but squared costs 3 to 5 % slower.
template <int NMAX, int NT, int CAP, bool kBytes>
__global__ void __launch_bounds__(NT, 4) solo_kernel(SoloArgs A)
{
    __shared__ BatchShared<NMAX, NT, CAP> S;
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    Ctl *c = A.ctl;
    const LdsJob J{A.n_b, A.n_a, A.k, A.ldk, A.lists, A.T, A.max_phases, A.phase_bound, A.origin,
                   A.trace, nullptr, A.cold ? A.first : nullptr};
    const int32_t err = c->err;
    // the loop failed: the outputs are marked invalid (every vertex free); the
    // host reports the error
    auto no_matching = [&]() {
        for (int i = tid; i < A.n_b; i += NT) A.mate_b[i] = -1;
        for (int i = tid; i < A.n_a; i += NT) A.mate_a[i] = -1;
    };
    LdsRun R{};
    if (A.cold) {
        lds_cold(J, S);
        if (A.trace && tid < 4) A.trace[tid] = 0;
    } else {
        if (err & kErrLoop) {
            no_matching();
            return;
        }
        if (err & 16) return;  // (nothing ran)
        R.phases = c->phases;
        R.sum_free = c->sum_free;
        R.rounds = c->rounds;
        R.max_rounds = c->max_rounds;
        R.scanned = tid == 0 ? c->scanned : 0ull;
        R.status = c->status;
        if (tid == 0) S.nF[0] = 0;
        __syncthreads();
        for (int i = tid; i < ((A.n_a + 7) & ~7); i += NT)
            S.t[i] = i < A.n_a ? (uint16_t)-A.y_a[i] : 0;
        for (int i = tid; i < A.n_a; i += NT) {
            const int32_t m = A.mate_a[i];
            S.mate[i] = m >= 0 ? (uint16_t)m : kNone16;
        }
        for (int i0 = wave * 64; i0 < A.n_b; i0 += NT) {
            const int i = i0 + lane;
            const bool is_free = i < A.n_b && A.mate_b[i] < 0;
            if (i < A.n_b) S.y[i] = (uint16_t)A.y_b[i];
            const uint32_t f = wave_push(&S.nF[0], is_free);
            if (is_free) S.F[0][f] = (uint16_t)i;
        }
    }
    lds_phases<NMAX, NT, CAP, true, kBytes, false>(J, R, S);
    if (R.status == 4) {
        if (tid == 0) __hip_atomic_fetch_or(&c->err, 64, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        no_matching();
        return;
    }
    // (a solve stopped early keeps its state, without the completion)
    lds_matching(J, R.cur, A.complete && R.status == 0 && err == 0, S);
    const uint32_t nfree = S.nF[R.cur];
    for (int i = tid; i < A.n_a; i += NT) {
        const uint16_t m = S.ap[1][i];
        A.mate_a[i] = m == kNone16 ? -1 : (int)m;
        A.y_a[i] = -(int32_t)S.t[i];
    }
    for (int i = tid; i < A.n_b; i += NT) {
        const uint16_t m = S.ap[0][i];
        A.mate_b[i] = m == kNone16 ? -1 : (int)m;
        A.y_b[i] = S.y[i];
    }
    unsigned long long scanned = R.scanned;
    for (int o = 32; o > 0; o >>= 1) scanned += __shfl_xor(scanned, o);
    if (lane == 0) S.red_s[wave] = scanned;
    __syncthreads();
    if (tid == 0) {
        scanned = 0;
        for (int w = 0; w < NT / 64; ++w) scanned += S.red_s[w];
        c->scanned = scanned;
        c->status = R.status;
        c->phases = R.phases;
        c->sum_free = R.sum_free;
        c->rounds = R.rounds;
        c->max_rounds = R.max_rounds;
        c->free_after = nfree;
    }
}

// The first list of every row of a new instance (t = 0, need = 0), before a
// solve whose few workgroups would otherwise make them alone: grid (kFirstRows
// rows a block, instances), a wave its rows one after the other. first[row] =
// V << 16 | minv. Bound: instruction issue (direct_row), ~2.8 us a row of 2,048
// and wave; 131,072 such rows take ~0.1 ms, 0.36 on the 64 workgroups of their
// solve.
constexpr int kFirstRows = 8;
template <int NMAX, int CAP, bool kBytes>
__global__ void __launch_bounds__(256, 4)
first_lists_kernel(const int32_t *n_arr, const int32_t *ldk_arr, const int64_t *pt_off,
                   const int64_t *k_off, const int16_t *k_all, int n_b, int n_a, int64_t ldk_one,
                   uint32_t *lists, uint32_t *first)
{
    __shared__ alignas(16) uint16_t zero[NMAX];
    __shared__ alignas(16) uint32_t stage[4][CAP];
    const int inst = blockIdx.y;
    const int nb = n_arr ? n_arr[inst] : n_b, na = n_arr ? nb : n_a;
    const int64_t ldk = ldk_arr ? ldk_arr[inst] : ldk_one, off = pt_off ? pt_off[inst] : 0;
    const int16_t *k = k_all + (k_off ? k_off[inst] : 0);
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    if ((int)blockIdx.x * kFirstRows >= nb) return;
    for (int i = threadIdx.x; i < NMAX; i += 256) zero[i] = 0;
    __syncthreads();
    int window = 4;
    for (int e = wave; e < kFirstRows; e += 4) {
        const int b = (int)blockIdx.x * kFirstRows + e;
        if (b >= nb) return;
        const RowRegs<NMAX / 512> kr = load_row<NMAX / 512, kBytes>(k, (int64_t)b * ldk, na, lane);
        uint16_t minv, V;
        direct_row<NMAX / 512, CAP>(kr, zero, na, 0, 0, lane, stage[wave], &minv, &V, &window);
        if (V && lane < CAP / 4)
            *reinterpret_cast<uint4 *>(lists + (off + b) * CAP + lane * 4) =
                *reinterpret_cast<const uint4 *>(&stage[wave][lane * 4]);
        if (lane == 0) first[off + b] = ((uint32_t)V << 16) | minv;
    }
}

__global__ void batch_reset_kernel(unsigned int *queue) { *queue = 0u; }

// The variant for a batch: n_max picks the LDS layout and the registers a row
// takes, the batch the waves an instance gets: 16 while every instance has a
// compute unit to itself, 8 beyond, 4 for many small ones. Whole calls in us
// with layouts of 1,024 -> 512 columns: 10 x 500 407 -> 374, 8 x 256 235 -> 218
// (16 waves); 512 x [300, 500] 554 -> 508 (8 waves; 16: 593, 4: 608);
// 2,000 x [100, 256], 8 -> 4 waves 649 -> 585, but 306 x [39, 247] 174 -> 215.
template <bool kPeek, class F>
auto pick_batch_kernel(int32_t n_max, int32_t batch, F f)
{
    if (n_max > 1024) return f(batch_solve_kernel<2048, 1024, kPeek>, 1024);
    if (n_max > 512)
        return batch > kBatchWideMax ? f(batch_solve_kernel<1024, 512, kPeek>, 512)
                                     : f(batch_solve_kernel<1024, 1024, kPeek>, 1024);
    if (batch <= kBatchWideMax) return f(batch_solve_kernel<512, 1024, kPeek>, 1024);
    return n_max <= kBatchNarrowMaxN && batch >= kBatchNarrowMin
               ? f(batch_solve_kernel<512, 256, kPeek>, 256)
               : f(batch_solve_kernel<512, 512, kPeek>, 512);
}

// Whether most rows have so many columns at their smallest cost that they find
// one among the first they look at and are done in a few phases: large eps in
// few dimensions. Then lists made beforehand are wasted: whole solves of 16 x 700
// without / with them, us: d = 4 eps = 0.1 87 / 96, 0.05 246 / 245; d = 8 0.14 99 / 106,
// 0.07 262 / 223; d = 16 0.3 96 / 106, 0.14 184 / 132; d = 32 0.3 170 / 152. The line is
// a fit to where the two meet at d = 4, 5, 8, 16 and 32. And a wave looks at 32
// columns of 16 rows at once before it takes rows singly (kPeek): without / with,
// d = 2 1 x 1,000, eps = 0.2 98 / 61, 64 x 1,024, eps = 0.1 167 / 120; but 512 x [64, 1024],
// d = 16, eps = 0.05, beyond the line, 915 / 925 (its registers), and 64 x 250, d = 2,
// eps = 0.01 2,346 / 2,420.
bool rows_content(int32_t d, double eps) { return eps > 0.0167 * std::pow((double)d, 0.86); }

template <class F>
auto with_batch_kernel(int32_t n_max, int32_t batch, int32_t d, double eps, F f)
{
    return n_max > kPeekMinN && rows_content(d, eps) ? pick_batch_kernel<true>(n_max, batch, f)
                                                     : pick_batch_kernel<false>(n_max, batch, f);
}

}  // namespace

int32_t batch_max_n() { return 2048; }

// The first lists are made beforehand, on every compute unit, where the
// solve's workgroups leave some idle and rows need lists: in two or three
// dimensions the first scans mostly find a column among the 512 they look at
// first. Whole calls in us, without / with: 64 x 2,048, d = 64 5,112 / 4,857;
// 4 x 2,048, d = 8 1,027 / 608; 8 x 256, d = 32 206 / 194; 256 x 900, d = 16
// 1,316 / 1,287; but 100 x 2,048, d = 2 1,202 / 1,362 and 50 x 400, d = 3 143 /
// 155. One instance: a cost matrix of 300 x 517 93 / 82, 300 x 300, d = 16 139 /
// 114, but 100 x 1,000, d = 8 (nearly every row content at once) 55 / 58.
bool many_dims(int32_t d) { return d > 3; }
bool batch_first_lists(int32_t batch, int32_t d, double eps)
{
    return batch <= kBatchWideMax && many_dims(d) && !rows_content(d, eps);
}

hipError_t launch_solo(const SoloArgs &a, hipStream_t s, hipEvent_t ev_start, hipEvent_t ev_stop)
{
    SoloArgs copy = a;
    void *args[] = {&copy};
    auto pick = [&](auto bytes) -> const void * {
        constexpr bool kBytes = decltype(bytes)::value;
        return a.n_a > 1024  ? (const void *)solo_kernel<2048, 1024, kSoloListCap, kBytes>
               : a.n_a > 512 ? (const void *)solo_kernel<1024, 1024, kSoloListCap, kBytes>
                             : (const void *)solo_kernel<512, 1024, kSoloListCap, kBytes>;
    };
    const void *fn = a.k8 ? pick(std::true_type{}) : pick(std::false_type{});
    if (a.cold && a.first) {
        auto lists = [&](auto nmax, auto bytes) {
            hipLaunchKernelGGL((first_lists_kernel<decltype(nmax)::value, kSoloListCap,
                                                   decltype(bytes)::value>),
                               dim3((a.n_b + kFirstRows - 1) / kFirstRows), dim3(256), 0, s,
                               nullptr, nullptr, nullptr, nullptr, a.k, a.n_b, a.n_a, a.ldk,
                               a.lists, a.first);
        };
        // (kSoloColdCells entries and n_a <= 2 n_b: at most 565 columns)
        static_assert(2 * kSoloColdCells <= 1024 * 1024, "columns of a solve from the start");
        auto by_size = [&](auto bytes) {
            if (a.n_a > 512) lists(std::integral_constant<int, 1024>{}, bytes);
            else lists(std::integral_constant<int, 512>{}, bytes);
        };
        if (a.k8) by_size(std::true_type{});
        else by_size(std::false_type{});
    }
    return hipExtLaunchKernel(fn, dim3(1), dim3(1024), args, 0, s, ev_start, ev_stop, 0);
}

hipError_t batch_grid(int32_t n_max, int32_t batch, int32_t d, double eps, int *grid)
{
    int per_cu = 0, dev = 0, cus = 0;
    hipError_t e = with_batch_kernel(n_max, batch, d, eps, [&](auto fn, int threads) {
        return hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, fn, threads, 0);
    });
    if (e != hipSuccess) return e;
    if ((e = hipGetDevice(&dev)) != hipSuccess) return e;
    if ((e = hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev)) != hipSuccess)
        return e;
    int g = per_cu * cus;
    if (g > batch) g = batch;
    *grid = g < 1 ? 1 : g;
    return hipSuccess;
}

hipError_t launch_batch_solve(const BatchArgs &a, int32_t n_max, int grid, hipStream_t s)
{
    hipLaunchKernelGGL(batch_reset_kernel, dim3(1), dim3(1), 0, s, a.queue);
    if (a.batch == 0) return hipGetLastError();
    if (a.first) {
        auto lists = [&](auto nmax) {
            hipLaunchKernelGGL((first_lists_kernel<decltype(nmax)::value, kBatchListCap, false>),
                               dim3((n_max + kFirstRows - 1) / kFirstRows, a.batch), dim3(256), 0,
                               s, a.n_arr, a.ldk_arr, a.pt_off, a.k_off, a.k, 0, 0, (int64_t)0,
                               a.lists, a.first);
        };
        if (n_max > 1024) lists(std::integral_constant<int, 2048>{});
        else if (n_max > 512) lists(std::integral_constant<int, 1024>{});
        else lists(std::integral_constant<int, 512>{});
    }
    with_batch_kernel(n_max, a.batch, a.d, a.eps, [&](auto fn, int threads) {
        hipLaunchKernelGGL(fn, dim3(grid), dim3(threads), 0, s, a);
        return 0;
    });
    return hipGetLastError();
}

}  // namespace prot
