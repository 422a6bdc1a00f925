// HIP kernels (gfx950) that score repetend candidates: one candidate per lane.
//
// Per candidate (Tessel, arXiv 2311.15269; Alg. 1, body of the loop over repetends):
//   decode   index -> lead vector (n_i of Eq. 3) + per-device block orders
//   build    walk the orders in an executable (topological) sequence, detect orders that
//            can never run, repair them in the REPAIR space, track the per-device memory
//            prefix (Eq. 1 [2]) and leave a compact "program" of the window
//   period   the repetend time t_R of Eq. 4 (with compaction of neighbouring repetends):
//            the least period of the rigidly repeated window.  The window is a max-plus
//            linear map on (device free times, end times of the micro-batches that are in
//            flight at the window boundary); its growth rate is the maximum cycle ratio
//   argmin   (period, index) lexicographic, lane -> wave -> block record -> grid merge
//
// Three kernels compute the same thing, the third in tessel_graph.hip (what the fast kernel does not take, within its
// tables):
//   eval_kernel       general: multi-device blocks, cyclic device scan, 16-bit program in LDS,
//                     Karp's formula over V+1 sweeps
//   eval_fast_kernel  single-device blocks: bit-mask build, program words in VGPRs, eigenvector
//                     test after every sweep; what it cannot finish goes to the general kernel
//
// State that is indexed per lane at run time (device records, micro-batch tokens) lives in
// LDS laid out [slot][lane], which is bank-conflict free for any per-lane slot.
#include <hip/hip_runtime.h>
#include <stdint.h>
#include <limits.h>
#include <stdlib.h>
#include <algorithm>

#include "tessel_device.h"
#include "tessel_common.h"

namespace tessel {

// ------------------------------------------------------------------ 4-bit counters per type
// next micro-batch index of every block type: lead + occurrences placed, 4 bits each
struct Mu {
    uint64_t lo, hi;
    static constexpr int kTypeBits = 5;          // of a program entry of the path for graphs
    __device__ __forceinline__ void clear() { lo = 0; hi = 0; }
    __device__ __forceinline__ uint32_t get(uint32_t g) const
    {
        uint64_t w = g < 16 ? lo : hi;
        return (uint32_t)(w >> ((g & 15u) * 4u)) & 15u;
    }
    __device__ __forceinline__ void set(uint32_t g, uint32_t v)
    {
        uint64_t m = 15ull << ((g & 15u) * 4u), x = (uint64_t)v << ((g & 15u) * 4u);
        if (g < 16) lo = (lo & ~m) | x; else hi = (hi & ~m) | x;
    }
    __device__ __forceinline__ void inc(uint32_t g)
    {
        uint64_t x = 1ull << ((g & 15u) * 4u);
        if (g < 16) lo += x; else hi += x;
    }
};

// the same for up to 64 block types and windows of up to 16 micro-batches, 8 bits each (problems that only the general
// kernel's path for graphs takes)
struct MuWide {
    uint64_t w[8];
    __device__ __forceinline__ void clear()
    {
#pragma unroll
        for (int k = 0; k < 8; k++) w[k] = 0;
    }
    __device__ __forceinline__ uint64_t word(uint32_t g) const
    {
        const uint64_t a = g & 8u ? w[1] : w[0], b = g & 8u ? w[3] : w[2], c = g & 8u ? w[5] : w[4], d = g & 8u ? w[7] : w[6];
        const uint64_t lo = g & 16u ? b : a, hi = g & 16u ? d : c;
        return g & 32u ? hi : lo;
    }
    __device__ __forceinline__ uint32_t get(uint32_t g) const { return (uint32_t)(word(g) >> ((g & 7u) * 8u)) & 255u; }
    __device__ __forceinline__ void add(uint32_t g, uint64_t x)
    {
#pragma unroll
        for (int k = 0; k < 8; k++) w[k] += (g >> 3) == (uint32_t)k ? x : 0ull;
    }
    __device__ __forceinline__ void set(uint32_t g, uint32_t v)
    {
        const uint32_t sh = (g & 7u) * 8u;
        add(g, ((uint64_t)v << sh) - (word(g) & (255ull << sh)));
    }
    __device__ __forceinline__ void inc(uint32_t g) { add(g, 1ull << ((g & 7u) * 8u)); }
    static constexpr int kTypeBits = 6;          // of a program entry
};

// entry y of eight: a select tree, so that the table comes through scalar loads
template <class T>
__device__ __forceinline__ T sel8(const T (&v)[kMaxLTW], uint32_t y)
{
    const T a = y & 1u ? v[1] : v[0], b = y & 1u ? v[3] : v[2], c = y & 1u ? v[5] : v[4], d = y & 1u ? v[7] : v[6];
    const T lo = y & 2u ? b : a, hi = y & 2u ? d : c;
    return y & 4u ? hi : lo;
}
__device__ __forceinline__ uint32_t sel4u(const uint32_t (&v)[kMaxLT], uint32_t y)
{
    uint32_t a = y & 1u ? v[1] : v[0];
    uint32_t b = y & 1u ? v[3] : v[2];
    return y & 2u ? b : a;
}

__device__ __forceinline__ int sel4(const int32_t (&v)[kMaxLTW], uint32_t y)
{
    int a = y & 1u ? v[1] : v[0];
    int b = y & 1u ? v[3] : v[2];
    return y & 2u ? b : a;
}

// remove the 2-bit entry at position pos (entries above move down)
__device__ __forceinline__ uint64_t remove_at(uint64_t x, uint32_t pos)
{
    uint64_t low = x & ((1ull << (2u * pos)) - 1ull);
    uint64_t high = ((x >> (2u * pos)) >> 2) << (2u * pos);
    return low | high;
}

// position of the first entry equal to y among the first len entries, or 64 if none
__device__ __forceinline__ uint32_t find_first(uint64_t x, uint32_t len, uint32_t y)
{
    uint64_t z = x ^ (0x5555555555555555ull * y);
    uint64_t hit = ~(z | (z >> 1)) & 0x5555555555555555ull;
    if (len < 32) hit &= (1ull << (2u * len)) - 1ull;
    return hit ? (uint32_t)__builtin_ctzll(hit) >> 1 : 64u;
}

// ------------------------------------------------------------------ one window sweep (general kernel)
// Program entry: bits 0-4 home code of the block type (device*4 + symbol), bits 5-10 token
// slot.  s = max(free time of its device(s), end of the micro-batch's previous block);
// both become s + t.  A chain's first block reads a token slot nobody has written: 0.
template <bool TP>
__device__ __forceinline__ void sweep_window(const KParams &P, const uint16_t *prog, uint32_t *state,
                                             const int32_t *t_tab, const uint32_t *mask_tab)
{
    const int total = P.total;
    for (int k = 0; k < total; k++) {
        uint32_t e = prog[k * kWave];
        uint32_t loc = e & 31u, ts = e >> 5;
        uint32_t tok = state[ts * kWave];
        uint32_t t = (uint32_t)t_tab[loc];
        if (!TP) {
            uint32_t ds = loc >> 2;
            uint32_t en = max(state[ds * kWave], tok) + t;
            state[ds * kWave] = en;
            state[ts * kWave] = en;
        } else {
            uint32_t mask = mask_tab[loc], s = tok;
            for (int d = 0; d < P.D; d++)
                if (mask >> d & 1u) s = max(s, state[d * kWave]);
            uint32_t en = s + t;
            for (int d = 0; d < P.D; d++)
                if (mask >> d & 1u) state[d * kWave] = en;
            state[ts * kWave] = en;
        }
    }
    // window boundary: micro-batches mu >= N_R are mu - N_R of the next window
    for (int p = 0; p < P.npaths; p++)
        for (int mu = 0; mu < P.NR; mu++) {
            int base = P.D + p * 2 * P.NR + mu;
            state[base * kWave] = state[(base + P.NR) * kWave];
            state[(base + P.NR) * kWave] = 0;
        }
}

__device__ __forceinline__ int reduced_slot(const KParams &P, int v)
{
    if (v < P.D) return v;
    int p = (v - P.D) / P.NR, mu = (v - P.D) % P.NR;
    return P.D + p * 2 * P.NR + mu;
}

// Least period of the repeated window = ceil(maximum cycle ratio) of the max-plus map x -> F(x)
// that one sweep applies to the V = D + npaths*N_R boundary values (plus the constant 0 that
// keeps start times non-negative).  Karp: with x(j) the vector after j+1 sweeps from 0 and
// n = V+1 sweeps in total, lambda = max_v min_{j<n-1} (x_v(n-1) - x_v(j)) / (n-1-j).
// Two passes over the same sweeps so that no history has to be stored.  (General kernel.)
// Before that, the shortcut the fast kernel lives on: iterate x <- F(x) from 0; as soon as every boundary value that
// means anything (`live`: devices with blocks, micro-batches that are in flight at the boundary) has grown by the
// same delta over one sweep, x is an eigenvector and delta the maximum cycle ratio, exactly.
constexpr int kGeneralTries = 6;
template <int VM, bool TP>
__device__ __forceinline__ int least_period(const KParams &P, const uint16_t *prog, uint32_t *state, const int32_t *t_tab,
                            const uint32_t *mask_tab, uint32_t live)
{
    const int V = P.nsweeps - 1, n = P.nsweeps;
    uint32_t xn[VM], bn[VM], bd[VM];
    for (int s = 0; s < P.nslots; s++) state[s * kWave] = 0;
    {
        uint32_t *prev = xn;
#pragma unroll
        for (int v = 0; v < VM; v++) prev[v] = 0;
        bool done = false;
        uint32_t T = 0;
        for (int j = 0; j < kGeneralTries; j++) {
            if (__ballot(!done) == 0) break;
            sweep_window<TP>(P, prog, state, t_tab, mask_tab);
            bool same = true, have = false;
            uint32_t delta = 0;
#pragma unroll
            for (int v = 0; v < VM; v++) {
                if (v < V) {
                    const uint32_t x = state[reduced_slot(P, v) * kWave];
                    const uint32_t dv = x - prev[v];
                    prev[v] = x;
                    if (live >> v & 1u) {
                        if (!have) { delta = dv; have = true; }
                        else if (dv != delta) same = false;
                    }
                }
            }
            if (!done && same && have) { T = delta; done = true; }
        }
        // every lane of the wave is here for a candidate that needs a period (the caller's lanes diverged before)
        if (done) return (int)T;
    }
    for (int s = 0; s < P.nslots; s++) state[s * kWave] = 0;
    for (int j = 0; j < n; j++) sweep_window<TP>(P, prog, state, t_tab, mask_tab);
#pragma unroll
    for (int v = 0; v < VM; v++) {
        xn[v] = v < V ? state[reduced_slot(P, v) * kWave] : 0u;
        bn[v] = 0xFFFFFFFFu; bd[v] = 1u;
    }
    for (int s = 0; s < P.nslots; s++) state[s * kWave] = 0;
    for (int j = 0; j < n - 1; j++) {
        sweep_window<TP>(P, prog, state, t_tab, mask_tab);
        uint32_t den = (uint32_t)(n - 1 - j);
#pragma unroll
        for (int v = 0; v < VM; v++) {
            if (v < V) {
                uint32_t a = xn[v] - state[reduced_slot(P, v) * kWave];
                // a/den < bn/bd  <=>  a*bd < bn*den   (all below 2^31, checked at problem creation)
                bool better = bn[v] == 0xFFFFFFFFu || (uint64_t)a * bd[v] < (uint64_t)bn[v] * den;
                if (better) { bn[v] = a; bd[v] = den; }
            }
        }
    }
    uint32_t T = 0;
#pragma unroll
    for (int v = 0; v < VM; v++) {
        if (v < V) {
            uint32_t c = (bn[v] + bd[v] - 1u) / bd[v];
            T = max(T, c);
        }
    }
    return (int)T;
}

// ------------------------------------------------------------------ candidate decoding
// index -> leads (4-bit counters by block type id) and, per device, the order of its blocks as
// 2-bit local symbols (first block in the lowest bits).  Returns kOk or the structural reject
// reason of the FACTORIAL space.
// (Problems with more than four block types on a device, sampled spaces only: the third bit of the symbol at position p
// is bit p of rem2[d].)
template <int DM, class CNT = Mu>
__device__ __forceinline__ int decode_candidate(const KParams &P, uint64_t idx, uint64_t (&rem)[DM], int (&remlen)[DM], CNT &mu,
                                                uint32_t (&rem2)[DM])
{
    const uint32_t NR = (uint32_t)P.NR;
    mu.clear();
#pragma unroll
    for (int d = 0; d < DM; d++) rem2[d] = 0;
#pragma unroll
    for (int d = 0; d < DM; d++) { rem[d] = 0; remlen[d] = 0; }
    if (P.space == kFactorial) {
        uint64_t rest = idx;
        bool dup = false, tpm = false;
        uint64_t seen_types = 0;
#pragma unroll
        for (int d = 0; d < DM; d++) {
            if (d >= P.D) continue;
            const uint32_t n = (uint32_t)P.ntd[d] * NR;
            uint32_t r = (uint32_t)(rest % P.cdev[d]);
            rest /= P.cdev[d];
            uint64_t list = P.init_list[d], o = 0;
            uint32_t firstlab = 0xFFFFFFFFu, seencnt = 0;
            for (uint32_t pos = 0; pos < n; pos++) {
                uint32_t f = P.fact[n - 1 - pos];
                uint32_t digit = r / f;
                r -= digit * f;
                uint32_t code = (uint32_t)(list >> (5u * digit)) & 31u;
                uint64_t low = list & ((1ull << (5u * digit)) - 1ull);
                list = low | (((list >> (5u * digit)) >> 5) << (5u * digit));
                uint32_t y = code >> 3, lab = code & 7u;
                o |= (uint64_t)y << (2u * pos);
                uint32_t fl = byte_of(firstlab, y), sc = byte_of(seencnt, y);
                if (fl == 0xFFu) firstlab = (firstlab & ~(0xFFu << (8u * y))) | (lab << (8u * y));
                else {
                    uint32_t want = fl + sc;                 // labels continue cyclically (Property 1)
                    if (want >= NR) want -= NR;
                    if (lab != want) dup = true;
                }
                seencnt += 1u << (8u * y);
            }
            rem[d] = o; remlen[d] = (int)n;
            for (int y = 0; y < P.ntd[d]; y++) {
                uint32_t g = byte_of(P.type_of[d], (uint32_t)y), fl = byte_of(firstlab, (uint32_t)y);
                if (seen_types >> g & 1u) { if (mu.get(g) != fl) tpm = true; }
                else { mu.set(g, fl); seen_types |= 1ull << g; }
            }
        }
        if (dup) return kDup;
        if (tpm) return kTpMismatch;
        if (P.dag) {
            for (int e = 0; e < P.ndeps; e++)
                if (mu.get(P.dsrc[e]) < mu.get(P.ddst[e])) return kProp2;
        } else
        for (int g = 0; g < P.K; g++) {
            int p = P.pred[g];
            if (p >= 0 && mu.get((uint32_t)p) < mu.get((uint32_t)g)) return kProp2;
        }
    } else if (P.space == kCanonical) {
        uint64_t rest = idx;
        const uint32_t B = NR + 1;
#pragma unroll
        for (int d = 0; d < DM; d++) {
            if (d >= P.D) continue;
            const uint32_t n = (uint32_t)P.ntd[d] * NR;
            uint64_t r = rest % P.cdev[d];
            rest /= P.cdev[d];
            uint32_t c[kMaxLT];
#pragma unroll
            for (int y = 0; y < kMaxLT; y++) c[y] = y < P.ntd[d] ? NR : 0u;
            uint64_t o = 0;
            for (uint32_t pos = 0; pos < n; pos++) {
                bool chosen = false;
#pragma unroll
                for (int y = 0; y < kMaxLT; y++) {
                    if (!chosen && c[y] > 0) {
                        c[y]--;
                        uint64_t w = P.wtab[((c[0] * B + c[1]) * B + c[2]) * B + c[3]];
                        if (r < w) { o |= (uint64_t)y << (2u * pos); chosen = true; }
                        else { r -= w; c[y]++; }
                    }
                }
            }
            rem[d] = o; remlen[d] = (int)n;
        }
        const int8_t *row = P.leadtab + rest * (uint64_t)P.K;
        for (int g = 0; g < P.K; g++) mu.set((uint32_t)g, (uint32_t)row[g]);
    } else {
        uint64_t z = mix64(P.seed + 0x9E3779B97F4A7C15ULL * (idx + 1));
        const uint32_t a = (uint32_t)z, b = (uint32_t)(z >> 32);
        if (P.has_fixed) {
            for (int g = 0; g < P.K; g++) mu.set((uint32_t)g, P.fixed[g]);
        } else if (P.dag) {
            // consumers before producers: a type's lead is the largest (consumer's lead + step) over its dependencies
            for (int k = 0; k < P.K; k++) {
                const uint32_t i = P.rtopo[k];
                uint32_t lead = 0;
                for (int e = 0; e < P.ndeps; e++) {
                    if (P.dsrc[e] != i) continue;
                    const uint32_t u = (stream_word(a, b, (kDrawLeadBase + (uint32_t)e) >> 1) >> (16u * ((uint32_t)e & 1u))) & 0xFFFFu;
                    const uint32_t step = (P.dcross[e] && u < P.step_q16) ? 1u : 0u;
                    lead = max(lead, mu.get(P.ddst[e]) + step);
                }
                mu.set(i, min(NR - 1u, lead));
            }
        } else {
            for (int k = 0; k < P.K; k++) {
                uint32_t i = P.rtopo[k];
                int j = P.succ[i];
                uint32_t lead = 0;
                if (j >= 0) {
                    uint32_t e = kDrawLeadBase + P.edge_out[i];
                    uint32_t u = (stream_word(a, b, e >> 1) >> (16u * (e & 1u))) & 0xFFFFu;
                    uint32_t step = (P.cross_out[i] && u < P.step_q16) ? 1u : 0u;
                    lead = min(NR - 1u, mu.get((uint32_t)j) + step);
                }
                mu.set(i, lead);
            }
        }
#pragma unroll
        for (int d = 0; d < DM; d++) {
            if (d >= P.D) continue;
            const uint32_t n = (uint32_t)P.ntd[d] * NR;
            uint32_t c0 = P.ntd[d] > 0 ? NR : 0u, c1 = P.ntd[d] > 1 ? NR : 0u, c2 = P.ntd[d] > 2 ? NR : 0u;
            uint32_t cw = 0;                              // up to eight types: the blocks left of every type, four bits each
            for (int y = 0; y < P.ntd[d]; y++) cw |= NR << (4 * y);
            uint64_t o = 0;
            uint32_t o2 = 0;
            uint32_t word = 0;
            for (uint32_t pos = 0; pos < n; pos++) {
                uint32_t j = kDrawOrdBase + 32u * (uint32_t)d + pos;
                if ((pos & 1u) == 0) word = stream_word(a, b, j >> 1);
                uint32_t u = (word >> (16u * (pos & 1u))) & 0xFFFFu;
                uint32_t digit = (u * (n - pos)) >> 16;
                uint32_t y;
                if (P.many) {
                    // symbol = number of cumulative counts at or below the digit
                    uint32_t acc = 0;
                    y = 0;
#pragma unroll
                    for (int k = 0; k < kMaxLTW - 1; k++) { acc += (cw >> (4 * k)) & 15u; y += digit >= acc ? 1u : 0u; }
                    cw -= 1u << (4u * y);
                    o2 |= (y >> 2) << pos;
                } else {
                    y = (digit >= c0) + (digit >= c0 + c1) + (digit >= c0 + c1 + c2);
                    c0 -= y == 0; c1 -= y == 1; c2 -= y == 2;
                }
                o |= (uint64_t)(y & 3u) << (2u * pos);
            }
            rem[d] = o; remlen[d] = (int)n; rem2[d] = o2;
        }
    }

    return kOk;
}

template <int DM, class CNT = Mu>
__device__ __forceinline__ int decode_candidate(const KParams &P, uint64_t idx, uint64_t (&rem)[DM], int (&remlen)[DM], CNT &mu)
{
    uint32_t rem2[DM];
    return decode_candidate<DM, CNT>(P, idx, rem, remlen, mu, rem2);
}

// ------------------------------------------------------------------ one candidate (general path)
template <int DM, int VM>
__device__ __forceinline__ int evaluate(const KParams &P, uint64_t idx, uint16_t *prog, uint32_t *state, const int32_t *t_tab,
                        const uint32_t *mask_tab, int &period, int (&peak)[DM])
{
    uint64_t rem[DM];
    int remlen[DM];
    Mu mu;
    period = 0;
#pragma unroll
    for (int d = 0; d < DM; d++) peak[d] = 0;
    {
        int st = decode_candidate<DM>(P, idx, rem, remlen, mu);
        if (st != kOk) return st;
    }

    // ---------------- memory at the window entry: blocks that ran before it (type i has
    // handled micro-batches 0 .. lead_i - 1)
    int memcur[DM];
#pragma unroll
    for (int d = 0; d < DM; d++) {
        memcur[d] = 0;
        if (d < P.D)
            for (int y = 0; y < P.ntd[d]; y++)
                memcur[d] += P.m_of[d][y] * (int)mu.get(byte_of(P.type_of[d], (uint32_t)y));
        peak[d] = INT_MIN;
    }

    // ---------------- build: place blocks in an executable sequence
    const bool repair = P.space == kSampledRepair;
    int placed = 0;
    const int total = P.total;
    bool deadlock = false;

    // places block type g (its next occurrence) taking entry pos[dd] of every device dd it occupies
    auto place = [&](uint32_t g, uint32_t mask, uint32_t home, uint32_t tokbase, int m, uint32_t pos_d, int d_static) {
        uint32_t mug = mu.get(g);
        prog[placed * kWave] = (uint16_t)(home | ((tokbase + mug) << 5));
        mu.inc(g);
        placed++;
#pragma unroll
        for (int dd = 0; dd < DM; dd++) {
            if (dd >= P.D) continue;
            bool here = (mask >> dd) & 1u;
            if (!here) continue;
            uint32_t pos = 0;
            if (dd == d_static) pos = pos_d;
            else if (pos_d != 0xFFFFFFFFu && repair) {
                // multi-device block placed out of line: its earliest entry on the other devices
                uint32_t ysym = 0;
                for (int y = 0; y < P.ntd[dd]; y++) if (byte_of(P.type_of[dd], (uint32_t)y) == g) ysym = (uint32_t)y;
                pos = find_first(rem[dd], (uint32_t)remlen[dd], ysym);
            }
            rem[dd] = remove_at(rem[dd], pos);
            remlen[dd]--;
            memcur[dd] += m;
            peak[dd] = max(peak[dd], memcur[dd]);
        }
    };

    while (placed < total && !deadlock) {
        bool progress = false;
#pragma unroll
        for (int d = 0; d < DM; d++) {
            if (d >= P.D || remlen[d] == 0) continue;
            uint32_t y = (uint32_t)rem[d] & 3u;
            uint32_t g = byte_of(P.type_of[d], y), pr = byte_of(P.pred_of[d], y);
            uint32_t mask = byte_of(P.mask_of[d], y);
            bool ok = pr == 0xFFu || mu.get(pr) > mu.get(g);
            if (P.tp && mask != (1u << d)) {
                // a multi-device block runs when it heads the list of all its devices; it is
                // placed from its lowest device
                if ((mask & ((1u << d) - 1u)) != 0) ok = false;
#pragma unroll
                for (int dd = 0; dd < DM; dd++) {
                    if (dd >= P.D || dd == d || !((mask >> dd) & 1u)) continue;
                    bool head = remlen[dd] > 0 && byte_of(P.type_of[dd], (uint32_t)rem[dd] & 3u) == g;
                    if (!head) ok = false;
                }
            }
            if (ok) {
                place(g, mask, byte_of(P.home_of[d], y), byte_of(P.tok_of[d], y), sel4(P.m_of[d], y), 0u, d);
                progress = true;
            }
        }
        if (progress) continue;
        if (!repair) { deadlock = true; break; }
        // Nothing at the head of any list can run.  Ascending over devices, then over the
        // device's remaining entries in list order: the first block whose producers are
        // placed goes next (only the first entry of each type can be that block).
        bool done = false;
#pragma unroll
        for (int d = 0; d < DM; d++) {
            if (done || d >= P.D || remlen[d] == 0) continue;
            uint32_t best_pos = 64u, best_y = 0;
#pragma unroll
            for (int y = 0; y < kMaxLT; y++) {
                if (y >= P.ntd[d]) continue;
                uint32_t g = byte_of(P.type_of[d], (uint32_t)y), pr = byte_of(P.pred_of[d], (uint32_t)y);
                bool ready = pr == 0xFFu || mu.get(pr) > mu.get(g);
                uint32_t pos = ready ? find_first(rem[d], (uint32_t)remlen[d], (uint32_t)y) : 64u;
                if (pos < best_pos) { best_pos = pos; best_y = (uint32_t)y; }
            }
            if (best_pos < 64u) {
                uint32_t y = best_y;
                place(byte_of(P.type_of[d], y), byte_of(P.mask_of[d], y), byte_of(P.home_of[d], y),
                      byte_of(P.tok_of[d], y), sel4(P.m_of[d], y), best_pos, d);
                done = true;
            }
        }
        if (!done) { deadlock = true; }     // cannot happen: unplaced blocks form a DAG
    }
    if (deadlock) {
#pragma unroll
        for (int d = 0; d < DM; d++) peak[d] = 0;
        return kDeadlock;
    }
    int peak_max = INT_MIN;
#pragma unroll
    for (int d = 0; d < DM; d++) {
        if (d >= P.D || peak[d] == INT_MIN) peak[d] = 0;      // a device without blocks
        if (d < P.D) peak_max = max(peak_max, peak[d]);
    }
    if (peak_max > P.M) return kMem;

    // ---------------- period
    // boundary values that mean anything: devices with blocks; micro-batch j of a chain is in flight at the
    // boundary when the chain's first block is j or more ahead (its counter now reads lead + N_R)
    uint32_t live = 0;
    for (int d = 0; d < P.D; d++) live |= (P.ntd[d] > 0 ? 1u : 0u) << d;
    for (int g = 0, path = 0; g < P.K; g++)
        if (P.pred[g] < 0) {
            const int lead = (int)mu.get((uint32_t)g) - P.NR;
            for (int j = 0; j < P.NR; j++)
                if (lead > j && P.D + path * P.NR + j < 32) live |= 1u << (P.D + path * P.NR + j);
            path++;
        }
    period = P.tp ? least_period<VM, true>(P, prog, state, t_tab, mask_tab, live)
                  : least_period<VM, false>(P, prog, state, t_tab, mask_tab, live);
    return kOk;
}

// ------------------------------------------------------------------ dependency graphs that are not chains
// A block type may have several producers and several consumers (Sec. III-A, Eq. 1 [3]).  State of a sweep, in LDS
// [slot][lane]: the D device times, then for every unbranched stretch of the graph with a type somebody consumes a
// ring of 2 N_R end times by micro-batch (micro-batches N_R and up belong to the next window and move down at the
// window boundary) and N_R more slots for the boundary's comparison.  Program entry: type id
// in bits 0-4 (0-5 for problems with more than 32 types), micro-batch above.  Tables by type id in LDS: t, device mask,
// producer mask (two words where there are more than 32 types), first ring slot.
struct DagTables {
    const int32_t *t; const uint32_t *mask, *pred, *pred_hi, *tok;
    __device__ __forceinline__ uint64_t producers(uint32_t g) const { return pred[g] | (pred_hi ? (uint64_t)pred_hi[g] << 32 : 0ull); }
};

template <int TB>
__device__ __forceinline__ void sweep_window_dag(const KParams &P, const DagTables &Tb, const uint16_t *prog, uint32_t *state)
{
    const int total = P.total;
    for (int k = 0; k < total; k++) {
        const uint32_t e = prog[k * kWave];
        const uint32_t g = e & ((1u << TB) - 1u), m = e >> TB;
        uint32_t s = 0;
        for (uint32_t rest = Tb.mask[g]; rest; rest &= rest - 1u) s = max(s, state[__builtin_ctz(rest) * kWave]);
        for (uint64_t rest = Tb.producers(g); rest; rest &= rest - 1ull) s = max(s, state[(Tb.tok[__builtin_ctzll(rest)] + m) * kWave]);
        const uint32_t en = s + (uint32_t)Tb.t[g];
        for (uint32_t rest = Tb.mask[g]; rest; rest &= rest - 1u) state[__builtin_ctz(rest) * kWave] = en;
        if (Tb.tok[g] != kNoRing) state[(Tb.tok[g] + m) * kWave] = en;
    }
}

// The window boundary: every ring moves down by N_R micro-batches and the device times stay, all less `shift` (0, or
// the period under test: times are then taken from the start of the next window, not below 0).  Returns whether every
// value that crosses the boundary and means anything grew by `want` over the window (`first`: by any one amount,
// which is handed back in `want`): ring entries below the lead of the ring's first type (micro-batches it handled
// before the window), compared with the copy the last boundary kept of them behind the ring (later types of the
// ring's stretch overwrite the entries themselves); device times against `prevfree`.
template <int DM, class CNT>
__device__ __forceinline__ bool boundary_dag(const KParams &P, const DagTables &Tb, uint32_t *state, const CNT &lead, uint32_t (&prevfree)[DM],
                                             uint32_t shift, bool first, uint32_t &want, uint32_t &top, uint32_t &most)
{
    bool same = true, have = !first;
    top = 0;
    most = 0;                                    // the largest growth (of a first kind of call)
#pragma unroll
    for (int d = 0; d < DM; d++) {
        if (d >= P.D) continue;
        const uint32_t x = state[d * kWave], y = x > shift ? x - shift : 0u;
        if (P.ntd[d] > 0) {
            const uint32_t dv = y - prevfree[d];
            most = max(most, dv);
            if (!have) { want = dv; have = true; } else if (dv != want) same = false;
        }
        prevfree[d] = y; state[d * kWave] = y;
        top = max(top, y);
    }
    for (int r = 0; r < P.ntok; r++) {
        const uint32_t base = P.ring_base[r], kept = P.ring_kept[r];
        const uint32_t lg = lead.get((uint32_t)P.ring_head[r]);
        for (int m = 0; m < P.NR; m++) {
            const uint32_t old = state[(kept + m) * kWave], x = state[(base + m + P.NR) * kWave];
            const uint32_t y = x > shift ? x - shift : 0u;
            if ((uint32_t)m < lg) {
                const uint32_t dv = y - old;
                most = max(most, dv);
                if (!have) { want = dv; have = true; } else if (dv != want) same = false;
                top = max(top, y);
            }
            const uint32_t keep = (uint32_t)m < lg ? y : 0u;
            state[(base + m) * kWave] = keep;
            state[(kept + m) * kWave] = keep;
            state[(base + m + P.NR) * kWave] = 0;
        }
    }
    return same && have;
}

// Least period of the repeated window.  First the eigenvector search of the other kernels (sweeps from 0 until every
// boundary value grows by the same amount, which is then the period); if that does not settle, the definition: the
// least T in [LB, UB] for which start times exist, by bisection; start times exist for T iff the sweeps from 0, with
// every boundary value taken T later each time, come to rest (Kleene iteration of the longest-path equations; it
// rests after at most as many windows as values cross the boundary, or passes UB).
template <int DM, class CNT>
__device__ __forceinline__ int least_period_dag(const KParams &P, const DagTables &Tb, const uint16_t *prog, uint32_t *state, const CNT &lead)
{
    uint32_t prevfree[DM];
    auto reset = [&]() {
        for (int s = 0; s < P.nslots; s++) state[s * kWave] = 0;
#pragma unroll
        for (int d = 0; d < DM; d++) prevfree[d] = 0;
    };
    reset();
    bool done = false;
    uint32_t T = 0, bound = (uint32_t)P.UB;
    for (int j = 0; j < P.dag_tries; j++) {
        if (__ballot(!done) == 0) break;
        sweep_window_dag<CNT::kTypeBits>(P, Tb, prog, state);
        uint32_t delta = 0, top, most;
        const bool eig = boundary_dag<DM>(P, Tb, state, lead, prevfree, 0u, true, delta, top, most);
        // no cycle ratio exceeds the largest growth of one sweep, whatever the values before it
        bound = min(bound, most);
        if (!done && eig) { T = delta; done = true; }
    }
    if (__ballot(!done) == 0) return (int)T;
    // bisection between the lower bound and the least growth seen (a growth of the last sweeps is within a unit or two of
    // the ratio, so one to three steps instead of the seven or eight from the serial time), until every lane has its period
    int crossing = P.D;
    for (int r = 0; r < P.ntok; r++) crossing += (int)lead.get((uint32_t)P.ring_head[r]);
    uint32_t lo = done ? T : (uint32_t)P.LB, hi = done ? T : max(bound, (uint32_t)P.LB);
    while (__ballot(lo < hi) != 0) {
        const uint32_t mid = lo + (hi - lo) / 2u;
        const bool open = lo < hi;
        reset();
        bool decided = !open, feasible = false;
        // (crossing + 2 windows bound the iteration; the loop runs until every lane of the wave has decided)
        for (int w = 0; w < kMaxKW * kMaxNRW + kMaxDW + 2; w++) {
            if (__ballot(!decided) == 0) break;
            sweep_window_dag<CNT::kTypeBits>(P, Tb, prog, state);
            uint32_t zero = 0, top, most;
            const bool rest = boundary_dag<DM>(P, Tb, state, lead, prevfree, mid, false, zero, top, most);
            if (!decided) {
                if (rest) { decided = true; feasible = true; }
                else if (top > (uint32_t)P.UB || w > crossing + 1) { decided = true; feasible = false; }
            }
        }
        if (open) { if (feasible) hi = mid; else lo = mid + 1u; }
    }
    return (int)hi;
}

// One candidate of a problem whose dependency graph is not a set of chains, or that is too wide for the other paths
// (general kernel only).  A device's order is kept as three bit planes of its symbols (bit p of plane k = bit k of the
// symbol at position p; up to eight block types per device) and the mask of the entries not yet placed.
__device__ __forceinline__ uint32_t even_bits(uint64_t x);
template <int DM, class CNT>
__device__ __forceinline__ int evaluate_dag(const KParams &P, const DagTables &Tb, uint64_t idx, uint16_t *prog, uint32_t *state,
                                            int &period, int (&peak)[DM])
{
    uint32_t p0[DM], p1[DM], p2[DM], alive[DM];
    CNT mu;
    period = 0;
#pragma unroll
    for (int d = 0; d < DM; d++) peak[d] = 0;
    {
        uint64_t rem[DM];
        int remlen[DM];
        int st = decode_candidate<DM, CNT>(P, idx, rem, remlen, mu, p2);
        if (st != kOk) return st;
#pragma unroll
        for (int d = 0; d < DM; d++) {
            p0[d] = even_bits(rem[d]); p1[d] = even_bits(rem[d] >> 1);
            alive[d] = remlen[d] >= 32 ? 0xFFFFFFFFu : (1u << remlen[d]) - 1u;
        }
    }
    const CNT lead = mu;
    auto type_at = [&](int d, uint32_t y) -> uint32_t { return y < 4u ? byte_of(P.type_of[d], y) : byte_of(P.type_of_hi[d], y - 4u); };
    int memcur[DM];
#pragma unroll
    for (int d = 0; d < DM; d++) {
        memcur[d] = 0;
        if (d < P.D)
            for (int y = 0; y < P.ntd[d]; y++)
                memcur[d] += P.m_of[d][y] * (int)mu.get(type_at(d, (uint32_t)y));
        peak[d] = INT_MIN;
    }
    const bool repair = P.space == kSampledRepair;
    int placed = 0;
    const int total = P.total;
    // a block may run when every producer has handled its micro-batch: in this window (counter ahead) or in the last
    // one (micro-batch below the producer's lead, which the counter is ahead of too)
    auto ready = [&](uint32_t g, uint64_t preds) -> bool {
        const uint32_t mg = mu.get(g);
        bool ok = true;
        for (uint64_t rest = preds; rest; rest &= rest - 1ull) ok = ok && mu.get((uint32_t)__builtin_ctzll(rest)) > mg;
        return ok;
    };
    // symbol at position pos of device d; entries of symbol y still to be placed
    auto symbol = [&](uint32_t a0, uint32_t a1, uint32_t a2, uint32_t pos) -> uint32_t {
        return ((a0 >> pos) & 1u) | (((a1 >> pos) & 1u) << 1) | (((a2 >> pos) & 1u) << 2);
    };
    auto left_of = [&](uint32_t a0, uint32_t a1, uint32_t a2, uint32_t al, uint32_t y) -> uint32_t {
        return al & (y & 1u ? a0 : ~a0) & (y & 2u ? a1 : ~a1) & (y & 4u ? a2 : ~a2);
    };
    // places the block of type g whose entry on device d_static sits at pos_d; on its other devices its earliest entry
    // (the head there when the block was placed as the head of all its lists)
    auto place = [&](uint32_t g, uint32_t mask, int m, uint32_t pos_d, int d_static) {
        prog[placed * kWave] = (uint16_t)(g | (mu.get(g) << CNT::kTypeBits));
        mu.inc(g);
        placed++;
#pragma unroll
        for (int dd = 0; dd < DM; dd++) {
            if (dd >= P.D || !((mask >> dd) & 1u)) continue;
            uint32_t pos = pos_d;
            if (dd != d_static) {
                uint32_t ysym = 0;
                for (int y = 0; y < P.ntd[dd]; y++) if (type_at(dd, (uint32_t)y) == g) ysym = (uint32_t)y;
                const uint32_t mine = left_of(p0[dd], p1[dd], p2[dd], alive[dd], ysym);
                pos = mine ? (uint32_t)__builtin_ctz(mine) : 0u;
            }
            alive[dd] &= ~(1u << pos);
            memcur[dd] += m;
            peak[dd] = max(peak[dd], memcur[dd]);
        }
    };
    bool deadlock = false;
    while (placed < total && !deadlock) {
        bool progress = false;
#pragma unroll
        for (int d = 0; d < DM; d++) {
            if (d >= P.D || alive[d] == 0) continue;
            const uint32_t pos = (uint32_t)__builtin_ctz(alive[d]);
            const uint32_t y = symbol(p0[d], p1[d], p2[d], pos);
            const uint32_t g = type_at(d, y), mask = Tb.mask[g];
            bool ok = ready(g, sel8(P.predmask_of[d], y));
            if (mask != (1u << d)) {
                // a multi-device block runs when it heads the list of all its devices; it is placed from its lowest device
                if ((mask & ((1u << d) - 1u)) != 0) ok = false;
#pragma unroll
                for (int dd = 0; dd < DM; dd++) {
                    if (dd >= P.D || dd == d || !((mask >> dd) & 1u)) continue;
                    const uint32_t hp = (uint32_t)__builtin_ctz(alive[dd] | 0x80000000u);
                    if (!(alive[dd] != 0 && type_at(dd, symbol(p0[dd], p1[dd], p2[dd], hp)) == g)) ok = false;
                }
            }
            if (ok) { place(g, mask, sel8(P.m_of[d], y), pos, d); progress = true; }
        }
        if (progress) continue;
        if (!repair) { deadlock = true; break; }
        bool done = false;
#pragma unroll
        for (int d = 0; d < DM; d++) {
            if (done || d >= P.D || alive[d] == 0) continue;
            uint32_t best_pos = 64u, best_y = 0;
#pragma unroll
            for (int y = 0; y < kMaxLTW; y++) {
                if (y >= P.ntd[d]) continue;
                const bool ok = ready(type_at(d, (uint32_t)y), P.predmask_of[d][y]);
                const uint32_t mine = left_of(p0[d], p1[d], p2[d], alive[d], (uint32_t)y);
                const uint32_t pos = ok && mine ? (uint32_t)__builtin_ctz(mine) : 64u;
                if (pos < best_pos) { best_pos = pos; best_y = (uint32_t)y; }
            }
            if (best_pos < 64u) {
                const uint32_t g = type_at(d, best_y);
                place(g, Tb.mask[g], sel8(P.m_of[d], best_y), best_pos, d);
                done = true;
            }
        }
        if (!done) deadlock = true;         // cannot happen: unplaced blocks form a DAG
    }
    if (deadlock) {
#pragma unroll
        for (int d = 0; d < DM; d++) peak[d] = 0;
        return kDeadlock;
    }
    int peak_max = INT_MIN;
#pragma unroll
    for (int d = 0; d < DM; d++) {
        if (d >= P.D || peak[d] == INT_MIN) peak[d] = 0;
        if (d < P.D) peak_max = max(peak_max, peak[d]);
    }
    if (peak_max > P.M) return kMem;
    period = least_period_dag<DM, CNT>(P, Tb, prog, state, lead);
    return kOk;
}

// ==================================================================== fast path
// Single-device blocks only.  Block types are addressed by their code c = device*4 + symbol, so
// that bit c of a 32-bit mask means "type c": R = types whose next occurrence may be placed now
// (producer ahead and occurrences left), HM = the type at the head of every device's list.
// One block is placed per step and lane:
//   heads first   : lowest set bit of R & HM            (any order of runnable heads gives the
//                                                         same per-device orders)
//   else repair   : lowest device with a runnable type = lowest set bit of R; inside the device
//                   the earliest remaining entry whose type is runnable
// A device's order is kept as two bit planes (bit p of lo/hi = low/high bit of the symbol at
// position p) and a mask of the entries not yet placed.  The per-device record is picked by a
// run-time device number and therefore lives in LDS [device][lane]; masks and the 4-bit
// micro-batch counters stay in VGPRs.

// the window's program: six 5-bit type codes a word, in executable order.  It is written and read with a
// wave-uniform word index, so it can live in VGPRs (indirect register addressing) and costs no LDS.
typedef uint32_t u32x32 __attribute__((ext_vector_type(32)));
typedef uint32_t u32x16 __attribute__((ext_vector_type(16)));
struct FastProgram {
    u32x32 a;
    u32x16 b;
    __device__ __forceinline__ uint32_t get(int i) const { return i < 32 ? a[i] : b[i - 32]; }
    __device__ __forceinline__ void set(int i, uint32_t v) { if (i < 32) a[i] = v; else b[i - 32] = v; }
};

constexpr int kFastTableWords = 16 * kMaxK;      // uniform tables at the start of the fast kernel's LDS
constexpr int kSweepTabWord = 12 * kMaxK;        // ... of which the sweeps' three tables by code; a multiple of 64 words, so
                                                 // that one two-address LDS read fetches a code's first and third word
constexpr int kTpListWord = 6 * kMaxK + kMaxD;
// the TP variants' own tables behind them, and their list of candidates (up to a multiple of 64 words: rows of 256 bytes)
constexpr int kTpTableWords = (kTpListWord + 2 * kWave + kWave - 1) / kWave * kWave;
// Everything a lane reads by a run-time index lies word by word: word w of entry i at w * 64 + i words, so that
// lanes with different entries hit different banks, a lane's words of one entry come with two-address reads
// (stride 64 words), and an LDS atomic on one word of the records meets no bank twice.

struct FastLds {
    uint32_t *sw_tab;     // [32]  by code, for the sweeps of problems without blocks on several devices:
                          //       t << 16 | LDS address of the time of the code's device (lane 0)
    uint32_t *ch_tab;     // [32]  by code, right behind sw_tab: LDS address of the first token of the code's chain (lane 0)
    uint32_t *in_tab;     // [32]  by code, behind ch_tab: 1 << s | s - 8, s = 16 + 4 * symbol: counter increment; shift that leaves the field times 256
    uint4 *tt_tab;        // [32]  by code, for the sweeps of the TP variants: x: t, y: byte offset of the first token slot of the code's
                          //       chain, z: byte offset of its device's words, w: bit offset of its micro-batch counter, bit 31: on several devices
    uint32_t *type_tab;   // [4][64], code in the low half of every 64: what placing one block of the type does:
                          //   word 0: added to the last word of its device record: memory delta << 16, one waiting
                          //      micro-batch of the type less, one more for its consumer if that sits on the same device
                          //   word 1: the consumer's codes (0: none)
                          //   word 2: LDS address of the last word (lane 0) of the record of the consumer's lowest device, if that is another one,
                          //      else of the type's own device (word 3 is 0 then); plus 4 * symbol of the type (rows are 256 bytes)
                          //   word 3: the increment of that word (one waiting micro-batch of the consumer)
                          // the upper half of the first holds chain_tab
    uint32_t *chain_tab;  // [32]  KParams::chain_tab
    uint32_t *grp_tab;    // [32]  TP variants: KParams::grp_code
    uint32_t *mem_tab;    // [32]  TP variants: by code, memory delta << 16
    uint32_t *tpg_tab;    // [8]   TP variants: KParams::tp_group (read in every build step with a uniform index; an array in
                          //       registers indexed at run time went to scratch memory)
    uint32_t rec;         // build: LDS address of the records [DM][4][64]: word 0: low plane, 1: high plane,
                          //        2: not-yet-placed mask, 3: micro-batches waiting at the input of the 4 types
                          //        (4 bits each) | memory now (signed) << 16
    // sweeps: three arrays [slot][64] in a row at distances known at compile time
    uint32_t *dfree;      // [DM] time at which the device is free
    uint32_t *dcnt;       // [DM] next micro-batch of the device's 4 types (4 bits each, in the upper half of the word)
    uint32_t *tok;        // [token slots] end time of the micro-batch's latest block
};

// problem scalars, read once per workgroup
template <int DM>
struct FastConst {
    int D, K, NR, M, total, nslots, npaths, nsweeps, space, has_fixed, nwords, ndeps;
    uint32_t step_q16;
    uint64_t seed;
    int ntd[DM];
    uint32_t mpack[DM];
    // blocks on several devices (TP variants of the kernel only)
    int ntp, tp_all;
    uint32_t several;                // codes of types on several devices
};

// One block of the window: s = max(device free, previous block of the micro-batch); both become s + t.  The
// micro-batch it handles is the device's counter of its type in `cnt`, the counter word as it was before the
// caller's atomic incremented it (the caller may have the next node's atomic in flight already).
__device__ __forceinline__ void sweep_node(const FastLds &L, const uint4 tt, uint32_t cnt, uint32_t lane4)
{
    // device times, counters and tokens lie at fixed distances in one array, so the three addresses of a block
    // share their registers: tt.z = the device's offset, tt.y = the chain's first token slot
    const uint32_t mu = __builtin_amdgcn_ubfe(cnt, tt.w, 4);
    uint32_t *fr = (uint32_t *)((char *)L.dfree + (tt.z + lane4));
    uint32_t *tk = (uint32_t *)((char *)L.dfree + (tt.y + lane4 + (mu << 8)));
    const uint32_t en = max(*fr, *tk) + tt.x;
    *fr = en;
    *tk = en;
}

// The same for problems with blocks on several devices: the block waits for all devices of its code group `G` (one
// nibble per device) and frees them together.  Counter and token are those of the type's code on its lowest device,
// which is the code the program holds.
template <int DM>
__device__ __forceinline__ void sweep_node_group(const FastLds &L, const uint4 tt, uint32_t cnt, uint32_t lane, uint32_t G, int D)
{
    const uint32_t mu = __builtin_amdgcn_ubfe(cnt, tt.w & 31u, 4);
    uint32_t *tk = (uint32_t *)((char *)L.dfree + (tt.y + lane * 4u + (mu << 8)));
    uint32_t s = *tk;
#pragma unroll
    for (int dd = 0; dd < DM; dd++)
        if (dd < D && ((G >> (4 * dd)) & 15u)) s = max(s, L.dfree[dd * kWave + lane]);
    const uint32_t en = s + tt.x;
#pragma unroll
    for (int dd = 0; dd < DM; dd++)
        if (dd < D && ((G >> (4 * dd)) & 15u)) L.dfree[dd * kWave + lane] = en;
    *tk = en;
}

// a lane's device record: four words at a stride of 64 words (two two-address accesses)
constexpr uint32_t kRecWordStep = kWave * 4u, kRecDevStep = 4u * kRecWordStep;
__device__ __forceinline__ uint4 rec_load(uint32_t a)
{
    return make_uint4(lds_load(a), lds_load(a + kRecWordStep), lds_load(a + 2u * kRecWordStep), lds_load(a + 3u * kRecWordStep));
}
__device__ __forceinline__ void rec_store(uint32_t a, const uint4 v)
{
    lds_store(a, v.x); lds_store(a + kRecWordStep, v.y); lds_store(a + 2u * kRecWordStep, v.z); lds_store(a + 3u * kRecWordStep, v.w);
}

// The blocks of one sweep for problems whose blocks sit on one device each, as a software pipeline four blocks deep.
// Per block: its table word is read (T); one returning LDS atomic reads and increments the counter word of its
// device (A), which names the micro-batch and with it the token; device time and token are read (R); s = max of the
// two, both become s + t (W).  As a dependent chain T -> A -> R -> W the wave would wait for the LDS three times a
// block, so block k + 3 does T, block k + 2 A and block k + 1 R before block k does W.  R(k + 1) then misses what
// W(k) writes: when block k + 1 runs on the same device or handles the same micro-batch as block k, the value read is
// replaced by block k's end time (two compares, two selects).  LDS keeps a wave's accesses in order, so W(k - 1) and
// everything older is seen.
// Table word of a code: t << 16 | LDS address of its device's time (lane 0); with several chains (MC) a second
// table holds the LDS address of the chain's first token (lane 0).  A device's counter word holds the next micro-batch
// of its four types in its upper half, four bits each; the third table word of a code, 1 << s | s - 8 with s =
// 16 + 4 * symbol, is both the increment of the atomic (the low half of the counter word only collects the s - 8, below 2^16
// over a window) and, by its low five bits, the shift that leaves the field times 256.
// Past the last block the stages T, A and R run on code 0 (a counter that the window boundary resets anyway, reads
// inside the arrays); stage W does not.
template <int DM, bool MC>
__device__ __forceinline__ void sweep_blocks(const FastConst<DM> &C, const FastLds &L, const FastProgram &prog, uint32_t lane4)
{
    const int total = C.total, nfull = total / 6, tail = total - 6 * nfull;
    constexpr uint32_t tab = kSweepTabWord * 4u;                // the kernel's LDS starts at address 0 (checked at its start)
    const uint32_t lane_tok = lds_address(L.dfree) + 2u * DM * kWave * 4u + lane4;
    struct Tst { uint32_t tt, w2, ch; };                        // T done
    struct Ast { uint32_t tt, fa, w2, cnt, ch; };               // A done
    struct Rst { uint32_t tt, fa, ta, fr, tk; };                // R done
    auto stage_t = [&](uint32_t w, int pos) -> Tst {
        Tst o;
        const uint32_t c4 = (pos == 0 ? w << 2 : w >> (5 * pos - 2)) & 0x7Cu;
        o.tt = lds_load(c4 + tab);
        o.w2 = lds_load(c4 + tab + 2u * kMaxK * 4u);
        o.ch = MC ? lds_load(c4 + tab + kMaxK * 4u) : 0u;
        return o;
    };
    auto stage_a = [&](const Tst &x) -> Ast {
        Ast o;
        o.tt = x.tt; o.ch = x.ch; o.w2 = x.w2;
        o.fa = (x.tt & 0xFFFFu) + lane4;
        o.cnt = lds_fetch_add(o.fa + DM * kWave * 4u, x.w2);
        return o;
    };
    auto stage_r = [&](const Ast &x) -> Rst {
        Rst o;
        o.tt = x.tt; o.fa = x.fa;
        const uint32_t mu = (x.cnt >> (x.w2 & 31u)) & 0xF00u;           // times 256
        o.ta = MC ? mu + lane4 + x.ch : mu + lane_tok;
        o.fr = lds_load(x.fa);
        o.tk = lds_load(o.ta);
        return o;
    };
    auto stage_w = [&](const Rst &x) {
        const uint32_t en = max(x.fr, x.tk) + (x.tt >> 16);
        lds_store(x.fa, en);
        lds_store(x.ta, en);
    };
    // per program word: the six table words first (they depend on the word only), then the blocks, the counter
    // atomic one block ahead of the times
    auto word = [&](uint32_t w, int nblocks) {
        Tst t[6];
#pragma unroll
        for (int j = 0; j < 6; j++) if (j < nblocks) t[j] = stage_t(w, j);
        Ast a = stage_a(t[0]);
#pragma unroll
        for (int j = 0; j < 6; j++)
            if (j < nblocks) {
                Ast an = a;
                if (j + 1 < nblocks) an = stage_a(t[j + 1]);
                stage_w(stage_r(a));
                a = an;
            }
    };
    for (int i = 0; i < nfull; i++) word(prog.get(i), 6);
    if (tail > 0) {
        const uint32_t w = prog.get(nfull);
        if (tail == 1) word(w, 1); else if (tail == 2) word(w, 2); else if (tail == 3) word(w, 3); else if (tail == 4) word(w, 4); else word(w, 5);
    }
}

// One sweep of the window over the program, then the window boundary.
template <int DM, bool TP>
__device__ __forceinline__ void sweep_fast(const FastConst<DM> &C, const FastLds &L, const FastProgram &prog, int lane,
                                           const Mu &lead_code, bool active)
{
    // a lane without a complete program (rejected candidate, lane past the end of the range) must not run one:
    // its counters would leave the token ring
    if (!active) return;
    const uint32_t lane4 = (uint32_t)lane * 4u;
    if (TP && C.tp_all) {
        // Every block on several devices sits on all of them: it waits for the latest end so far (one register) and
        // leaves a floor under all device times (another), instead of a visit to every device.  (36 blocks on 8 devices, all
        // of 2^24 candidates feasible: 25.8 -> 8.4 ms for the launch, with the tables of the build out of scratch memory.)
        uint32_t latest = 0, floor_all = 0;
#pragma unroll
        for (int d = 0; d < DM; d++) if (d < C.D) latest = max(latest, L.dfree[d * kWave + lane]);
        const int nwords = (C.total + 5) / 6;
        for (int wi = 0; wi < nwords; wi++) {
            uint32_t w = prog.get(wi);
            const int nj = min(6, C.total - 6 * wi);
#pragma unroll 1
            for (int j = 0; j < nj; j++, w >>= 5) {
                const uint4 tt = L.tt_tab[w & 31u];
                uint32_t *fr = (uint32_t *)((char *)L.dfree + (tt.z + lane4)), *cp = fr + DM * kWave;
                const uint32_t cnt = *cp;
                *cp = cnt + (1u << (tt.w & 31u));
                const uint32_t mu = __builtin_amdgcn_ubfe(cnt, tt.w & 31u, 4);
                uint32_t *tk = (uint32_t *)((char *)L.dfree + (tt.y + lane4 + (mu << 8)));
                const bool all = (int)tt.w < 0;
                const uint32_t en = max(*tk, all ? latest : max(*fr, floor_all)) + tt.x;
                *fr = en;
                *tk = en;
                latest = max(latest, en);
                floor_all = all ? en : floor_all;
            }
        }
#pragma unroll
        for (int d = 0; d < DM; d++) if (d < C.D) L.dfree[d * kWave + lane] = max(L.dfree[d * kWave + lane], floor_all);
    } else if (TP) {
        for (int k = 0; k < C.total; k++) {
            const uint32_t code = (prog.get(k / 6) >> (5 * (k % 6))) & 31u;
            const uint4 tt = L.tt_tab[code];
            uint32_t *cp = (uint32_t *)((char *)L.dfree + (tt.z + lane4)) + DM * kWave;
            const uint32_t cnt = *cp;
            *cp = cnt + (1u << (tt.w & 31u));
            sweep_node_group<DM>(L, tt, cnt, (uint32_t)lane, L.grp_tab[code], C.D);
        }
    } else {
        if (C.npaths > 1) sweep_blocks<DM, true>(C, L, prog, lane4);
        else sweep_blocks<DM, false>(C, L, prog, lane4);
    }
    // window boundary: micro-batches mu >= N_R are mu - N_R of the next window; counters restart at the leads
    for (int p = 0; p < C.npaths; p++)
        for (int mu = 0; mu < C.NR; mu++) {
            int base = p * 2 * C.NR + mu;
            L.tok[base * kWave + lane] = L.tok[(base + C.NR) * kWave + lane];
            L.tok[(base + C.NR) * kWave + lane] = 0;
        }
#pragma unroll
    for (int d = 0; d < DM; d++)
        if (d < C.D) L.dcnt[d * kWave + lane] = (uint32_t)((d < 4 ? lead_code.lo : lead_code.hi) >> (16 * (d & 3))) << 16;
}

template <int DM>
__device__ __forceinline__ void reset_sweep_state(const FastConst<DM> &C, const FastLds &L, int lane, const Mu &lead_code)
{
    for (int d = 0; d < C.D; d++) L.dfree[d * kWave + lane] = 0;
    for (int s = 0; s < C.nslots - C.D; s++) L.tok[s * kWave + lane] = 0;
#pragma unroll
    for (int d = 0; d < DM; d++)
        if (d < C.D) L.dcnt[d * kWave + lane] = (uint32_t)((d < 4 ? lead_code.lo : lead_code.hi) >> (16 * (d & 3))) << 16;
}

// Period of the repeated window.  The sweep is a max-plus linear map F on the boundary vector x
// (device free times, in-flight micro-batch end times).  If after some sweep every live component
// has grown by the same delta, x is an eigenvector of F and delta is its eigenvalue = the maximum
// cycle ratio, exactly.  Almost every candidate gets there within two or three sweeps; one that has
// not after the sweeps allowed (`tries`) is handed on by the caller: to a queue of candidates that get more
// sweeps, from there to the general kernel (Karp's formula).
// `settle`, in the longer search: the period is also found when the largest growth D was that of the boundary before and every value
// that grew by D then grew by D now.  No cycle ratio exceeds the largest growth; and a value that grew by D got its time from one that
// grew by D the time before (that one's growth bounds its own from above), which is again one of these, so following them
// closes a cycle of ratio D.  (Pipelines whose devices before the slowest one keep a smaller growth for ever: 8.7 M candidates of 70 blocks on
// five devices left so many to the general kernel that its pass took 563 of 1,690 us; a call 1,590 -> 1,090 us.  2^18 of 80 blocks on
// eight: 719 -> 159.)
template <int DM, int VM, bool TP>
__device__ __forceinline__ int period_fast(const KParams &P, const FastConst<DM> &C, const FastLds &L, const FastProgram &prog, int lane,
                                           const Mu &lead_code, bool want, int tries, bool settle,
                                           uint32_t &nsweeps_used)
{
    const int V = C.nsweeps - 1;
    const uint32_t lane4 = (uint32_t)lane * 4u;
    // byte offset (from the device times) of boundary value v: a device's free time or a carried token
    auto value_offset = [&](uint32_t e) -> uint32_t {
        const uint32_t slot = e & 63u;
        return ((e >> 6 & 1u) ? slot : 2u * DM + slot - (uint32_t)C.D) * (kWave * 4u) + lane4;
    };
    uint32_t live = 0;                                    // per lane: which boundary values mean anything
#pragma unroll
    for (int v = 0; v < VM; v++) {
        if (v < V) {
            // (the value's entry through scalar loads: its code is a constant of the wave)
            const uint32_t e = P.vtab[v], c = (e >> 7) & 31u;
            const uint32_t half = c & 16u ? (c & 8u ? (uint32_t)(lead_code.hi >> 32) : (uint32_t)lead_code.hi) : c & 8u ? (uint32_t)(lead_code.lo >> 32) : (uint32_t)lead_code.lo;
            const bool on = (e >> 6 & 1u) ? (e >> 17 & 1u) != 0 : (half >> (4u * (c & 7u)) & 15u) > ((e >> 13) & 15u);
            live |= (on ? 1u : 0u) << v;
        }
    }
    reset_sweep_state<DM>(C, L, lane, lead_code);
    uint32_t prev[VM];
#pragma unroll
    for (int v = 0; v < VM; v++) prev[v] = 0;
    int T = 0;
    bool done = !want;
    uint32_t top_before = 0, was = 0;
    for (int j = 0; j < tries; j++) {
        if (__ballot(!done) == 0) break;
        sweep_fast<DM, TP>(C, L, prog, lane, lead_code, !done);
        nsweeps_used += done ? 0u : 1u;
        if (settle) {
            uint32_t top = 0, now = 0;                    // the largest growth, and the values that have it
#pragma unroll
            for (int v = 0; v < VM; v++) {
                if (v < V) {
                    const uint32_t x = *(const uint32_t *)((const char *)L.dfree + value_offset(P.vtab[v]));
                    const uint32_t dv = live >> v & 1u ? x - prev[v] : 0u;
                    prev[v] = x;
                    now = dv > top ? 0u : now;
                    top = max(top, dv);
                    now |= (dv == top ? 1u : 0u) << v;
                }
            }
            now &= live;
            const bool held = j > 0 && top == top_before && (was & ~now) == 0;
            if (!done && (held || now == live) && live) { T = (int)top; done = true; }
            top_before = top; was = now;
            continue;
        }
        bool same = true, have = false;
        uint32_t delta = 0;
#pragma unroll
        for (int v = 0; v < VM; v++) {
            if (v < V) {
                const uint32_t x = *(const uint32_t *)((const char *)L.dfree + value_offset(P.vtab[v]));
                const uint32_t dv = x - prev[v];
                prev[v] = x;
                if (live >> v & 1u) {
                    if (!have) { delta = dv; have = true; }
                    else if (dv != delta) same = false;
                }
            }
        }
        if (!done && same && have) { T = (int)delta; done = true; }
    }
    return done ? T : -1;        // -1: no eigenvector within the sweeps allowed (the caller hands the candidate on)
}

// the quotient by n of a number below 2^32, of which the remainder stays: `inv` = floor(2^32 / n), 0 for n = 1
__device__ __forceinline__ uint32_t take_digit(uint32_t &x, uint32_t n, uint32_t inv)
{
    if (inv == 0) { const uint32_t q = x; x = 0; return q; }
    uint32_t q = __umulhi(x, inv);                            // the true one or one less
    x -= q * n;
    if (x >= n) { x -= n; q++; }
    return q;
}

// even bits of a word, compacted (bit 2p -> bit p)
__device__ __forceinline__ uint32_t even_bits(uint32_t x)
{
    x &= 0x55555555u;
    x = (x | (x >> 1)) & 0x33333333u;
    x = (x | (x >> 2)) & 0x0F0F0F0Fu;
    x = (x | (x >> 4)) & 0x00FF00FFu;
    return (x | (x >> 8)) & 0x0000FFFFu;
}
__device__ __forceinline__ uint32_t even_bits(uint64_t x)
{
    x &= 0x5555555555555555ull;
    x = (x | (x >> 1)) & 0x3333333333333333ull;
    x = (x | (x >> 2)) & 0x0F0F0F0F0F0F0F0Full;
    x = (x | (x >> 4)) & 0x00FF00FF00FF00FFull;
    x = (x | (x >> 8)) & 0x0000FFFF0000FFFFull;
    x = (x | (x >> 16)) & 0x00000000FFFFFFFFull;
    return (uint32_t)x;
}

// MODE: 0 exhaustive spaces, 1 sampled without repair, 2 sampled with repair.
// TP: some block type occupies several devices.  Such a type has one code on every device it occupies, and R, X
// hold all of them.  It is a runnable head only when it heads all its devices; placing it takes its earliest entry
// out of every one of them.
// Builds the candidate's window: validity, memory, the program of the window in executable order and the leads by
// code.  Returns kOk or the reason of the rejection; the period is the sweeps' business (period_fast).
// what the build carries from block to block besides the per-device records in LDS
// Sampled leads: every dependency between different device sets steps the lead with probability step_q16 / 65536; a lead is
// the number of steps from its type to the end of the chain, capped at N_R - 1.  The steps, a bit each:
template <int DM>
__device__ __forceinline__ uint32_t lead_steps(const KParams &P, const FastConst<DM> &C, uint32_t ka, uint32_t kb)
{
    uint32_t S = 0;
    for (int e = 0; e < C.ndeps; e += 2) {
        const uint32_t wv = stream_word(ka, kb, (kDrawLeadBase + (uint32_t)e) >> 1);
        // (the dependency's bit through scalar loads: the index is the same in every lane)
        const uint32_t b0 = P.dep_bit[e], b1 = e + 1 < C.ndeps ? P.dep_bit[e + 1] : 0u;
        S |= (wv & 0xFFFFu) < C.step_q16 ? b0 : 0u;
        S |= (wv >> 16) < C.step_q16 ? b1 : 0u;
    }
    return S;
}

// blocks that ran before the window: a device's leads, four bits each, times its memory deltas
__device__ __forceinline__ int entry_memory(uint32_t leads, uint32_t mpack)
{
    uint32_t leads4 = (leads & 0xFFu) | ((leads & 0xFF00u) << 8);
    leads4 = (leads4 | (leads4 << 4)) & 0x0F0F0F0Fu;
    return __builtin_amdgcn_sdot4((int)leads4, (int)mpack, 0, false);
}

// Sampled spaces with drawn leads: whether the memory at the window entry alone exceeds the cap on some device.  A device is back
// there after its last block (its deltas add up to nothing over a window), so the candidate's peak does too, whatever its orders.
// Its own phase in front of the decode for problems with blocks on several devices, whose memory is held on all of them at once: 86 % of 2^26
// candidates of 40 blocks with two on all of four devices leave here, 5.69 -> 1.68 ms.  In the others next to no lead vector
// exceeds a cap that any candidate meets.
template <int DM>
__device__ __forceinline__ bool entry_over(const KParams &P, const FastConst<DM> &C, uint64_t idx)
{
    uint32_t kb;
    const uint32_t ka = stream_keys(C.seed, idx, kb), S = lead_steps<DM>(P, C, ka, kb);
    int most = INT_MIN;
#pragma unroll
    for (int d = 0; d < DM; d++) {
        if (d >= C.D || C.ntd[d] == 0) continue;
        uint32_t leads = 0;
#pragma unroll
        for (int y = 0; y < kMaxLT; y++) leads |= min((uint32_t)C.NR - 1u, (uint32_t)__builtin_popcount(S & P.cum_code[4 * d + y])) << (4 * y);
        most = max(most, entry_memory(leads, C.mpack[d]));
    }
    return most > C.M;
}

struct BuildState {
    uint32_t R, HM, X;               // by code: runnable types, heads of the devices, exhausted types
    int worst;                       // largest memory prefix over all devices so far (Eq. 1 [2])
    int status;
};

template <int DM, int MODE, bool TP>
__device__ __forceinline__ void build_begin(const KParams &P, const FastConst<DM> &C, uint64_t idx, uint64_t last_idx, const FastLds &L,
                                            int lane, Mu &lead_code, BuildState &S)
{
    uint32_t plo[DM], phi[DM];       // order planes per device
    int nlen[DM];
    const uint32_t NR = (uint32_t)C.NR;
    int status = kOk;
    constexpr bool sampled = MODE != 0;    // kSampledStrict / kSampledRepair; else the exhaustive spaces
    Mu leads_type;                   // by type id (exhaustive spaces, fixed leads)
    leads_type.lo = 0; leads_type.hi = 0;
    const uint32_t *row = nullptr;
    uint32_t ka = 0, kb = 0;
    if (sampled) {
        const uint64_t z = mix64(C.seed + 0x9E3779B97F4A7C15ULL * (idx + 1));
        ka = (uint32_t)z; kb = (uint32_t)(z >> 32);
#pragma unroll
        for (int d = 0; d < DM; d++) {
            plo[d] = phi[d] = 0; nlen[d] = 0;
            if (d >= C.D) continue;
            const uint32_t n = (uint32_t)C.ntd[d] * NR;
            // cumulative counts of the remaining blocks by type, t1 <= t2 <= t3 <= 32: a digit below t1 picks
            // symbol 0, below t2 symbol 1, ...  The three are kept as bytes of one word, as 0x80 - t, so that
            // one add of the replicated digit leaves "digit >= t" in bit 7 of every byte (no carry between
            // bytes: 0x60 <= 0x80 - t + digit < 0xA0).
            const uint32_t c1 = C.ntd[d] > 0 ? NR : 0u, c2 = c1 + (C.ntd[d] > 1 ? NR : 0u), c3 = c2 + (C.ntd[d] > 2 ? NR : 0u);
            uint32_t tq = 0x808080u - (c1 | (c2 << 8) | (c3 << 16));
            // Outcomes of the three comparisons, one in bit 7 of each byte: the symbol is their number.
            auto pick = [&](uint32_t draw, uint32_t left) -> uint32_t {
                const uint32_t digit = (uint32_t)(((uint64_t)draw * (uint64_t)((left << 16) & 0xFFFFFFu)) >> 32);    // (draw * left) >> 16 as a
                                                                                                       // 24-bit high multiply (left <= 32)
                const uint32_t ge = mad24(digit, 0x010101u, tq) & 0x808080u;
                tq += (ge >> 7) ^ 0x010101u;                     // a threshold above the digit loses one block
                return ge;
            };
            // With repair they are collected as they are, eight positions to a word: byte k holds "at or above threshold k" of the
            // eight, so the symbols' high bits are the second byte, their low bits the three bytes' exclusive or.  (A count a position,
            // and 110 cycles a device to split pairs of bits into planes, less.)  Without repair the symbols are counted and
            // collected by pairs of bits, 16 to a word: together with the build step's other form (build_words) 1,000,003 scores of one or two
            // micro-batches of 10 to 16 types on 5 to 8 devices take 0.96 to 0.98 of the time.
            constexpr uint32_t kPer = MODE == 2 ? 8u : 16u;
            uint32_t seen[32u / kPer] = {};
#pragma unroll
            for (uint32_t h = 0; h < 32u / kPer; h++) {
                const uint32_t from = kPer * h, to = min(n, from + kPer);
                auto collect = [&](uint32_t ge, uint32_t at) { seen[h] |= MODE == 2 ? (ge >> 7) << at : (uint32_t)__builtin_popcount(ge) << (2u * at); };
                for (uint32_t pos = from; pos < to; pos += 2) {
                    const uint32_t word = stream_word(ka, kb, (kDrawOrdBase + 32u * (uint32_t)d + pos) >> 1);
                    collect(pick(word & 0xFFFFu, n - pos), pos - from);
                    if (pos + 1 < n) collect(pick(word >> 16, n - pos - 1u), pos + 1u - from);
                }
            }
            uint32_t lo, hi;
            if constexpr (MODE == 2) {
                // (bytes 0 of the four words to one, bytes 1 likewise)
                uint32_t low[4];
#pragma unroll
                for (int h = 0; h < 4; h++) low[h] = seen[h] ^ (seen[h] >> 8) ^ (seen[h] >> 16);
                auto bytes = [](uint32_t a, uint32_t b, uint32_t c, uint32_t e, uint32_t pair) -> uint32_t {
                    return __builtin_amdgcn_perm(__builtin_amdgcn_perm(e, c, pair), __builtin_amdgcn_perm(b, a, pair), 0x05040100u);
                };
                lo = bytes(low[0], low[1], low[2], low[3], 0x0C0C0400u);
                hi = bytes(seen[0], seen[1], seen[2], seen[3], 0x0C0C0501u);
            } else {
                lo = even_bits(seen[0]) | (even_bits(seen[1]) << 16);
                hi = even_bits(seen[0] >> 1) | (even_bits(seen[1] >> 1) << 16);
            }
            plo[d] = lo; phi[d] = hi; nlen[d] = (int)n;
        }
        if (C.has_fixed)
            for (int g = 0; g < C.K; g++) leads_type.set((uint32_t)g, P.fixed[g]);
    } else if (P.ranked) {
        // Ranks by mixed-radix digits of the index, orders and leads from tables by rank.  (Unranking symbol by symbol, up to
        // four 64-bit counts from memory per position, and 64-bit divisions were most of the time of a space whose
        // candidates mostly deadlock in their first blocks: 2^26 candidates of 32 blocks on 4 devices 6.8 -> 2.5 ms.)
        uint64_t rest = idx;
#pragma unroll
        for (int d = 0; d < DM; d++) {
            plo[d] = phi[d] = 0; nlen[d] = 0;
            if (d >= C.D) continue;
            nlen[d] = C.ntd[d] * (int)NR;
            const uint32_t n = (uint32_t)P.cdev[d], inv = P.recip[d];
            uint32_t rank = 0;
            if (inv != 0) {                                       // (one arrangement: nothing to take off the index)
                if ((last_idx >> 32) == 0) {
                    rank = (uint32_t)rest;
                    rest = take_digit(rank, n, inv);
                } else { rank = (uint32_t)(rest % n); rest /= n; }
            }
            const uint64_t o = P.orders[P.order_at[C.ntd[d]] + rank];
            plo[d] = (uint32_t)o; phi[d] = (uint32_t)(o >> 32);
        }
        row = P.leadrows + rest * (uint64_t)kLeadRow;
    } else {
        uint64_t ord[DM];
        status = decode_candidate<DM>(P, idx, ord, nlen, leads_type);
#pragma unroll
        for (int d = 0; d < DM; d++) { plo[d] = even_bits(ord[d]); phi[d] = even_bits(ord[d] >> 1); }
    }

    // leads by code, walking every chain from its last block to its first; R gets a type as soon
    // as its producer's lead is ahead (the previous window already handled that micro-batch)
    Mu mu, Q;                        // leads by code; micro-batches waiting at the input of every type
    mu.lo = 0; mu.hi = 0;
    Q.lo = Q.hi = 0xFFFFFFFFFFFFFFFFull;          // 15: a chain's first block never waits
    uint32_t R = 0, HM = 0, X = 0;
    const bool draw_leads = sampled && !C.has_fixed;
    if (draw_leads) {
        const uint32_t S = lead_steps<DM>(P, C, ka, kb);
#pragma unroll
        for (int d = 0; d < DM; d++) {
            if (d >= C.D) continue;
            // (The tables through scalar loads: what a code has of its own is the operand of one instruction.  By words from LDS, with a
            // compare and a select for a type without a producer, 16 instructions a code instead of nine.)
            const uint32_t pos = P.pred_pos[d];
            uint32_t mud = 0, qd = P.no_pred[d];             // 15: no producer, never waits
#pragma unroll
            for (int y = 0; y < kMaxLT; y++) {               // (a code without a type has no bits in the tables: lead 0, never read)
                const uint32_t lead = min(NR - 1u, (uint32_t)__builtin_popcount(S & P.cum_code[4 * d + y]));
                // its producer handled one micro-batch more in the previous window if their dependency steps and the cap is not reached
                const uint32_t wait = min((S >> (pos >> (8 * y) & 31u)) & 1u, NR - 1u - lead);
                mud |= lead << (4 * y);
                qd |= wait << (4 * y);
                R |= wait << (4 * d + y);
            }
            if (d < 4) { mu.lo |= (uint64_t)mud << (16 * d); Q.lo = (Q.lo & ~(0xFFFFull << (16 * d))) | ((uint64_t)qd << (16 * d)); }
            else { mu.hi |= (uint64_t)mud << (16 * (d - 4)); Q.hi = (Q.hi & ~(0xFFFFull << (16 * (d - 4)))) | ((uint64_t)qd << (16 * (d - 4))); }
        }
        R |= P.first_codes;
    } else if (!sampled && P.ranked) {
        const uint4 a = ((const uint4 *)row)[0], b = ((const uint4 *)row)[1];
        mu.lo = (uint64_t)a.x | ((uint64_t)a.y << 32); mu.hi = (uint64_t)a.z | ((uint64_t)a.w << 32);
        Q.lo = (uint64_t)b.x | ((uint64_t)b.y << 32); Q.hi = (uint64_t)b.z | ((uint64_t)b.w << 32);
        R = row[8];
    } else {
        for (int k = 0; k < C.K; k++) {
            const uint32_t ct = L.chain_tab[k];
            const uint32_t c = ct & 63u, sc = (ct >> 6) & 63u;
            const bool has_succ = sc != 63u;
            const uint32_t lead_succ = mu.get(sc & 31u);
            const uint32_t lead = leads_type.get(ct >> 21);
            mu.set(c, lead);
            if (has_succ) Q.set(sc & 31u, lead - lead_succ);          // handled by the previous window already
            if (has_succ && lead > lead_succ) R |= 1u << (sc & 31u);
            if ((ct >> 20) & 1u) R |= 1u << c;
        }
        if (TP)
            for (int c = 0; c < 4 * C.D; c++) {           // the other codes of a type copy its lowest device's
                const uint32_t h = P.home_code[c];
                if (h == 63u || h == (uint32_t)c) continue;
                mu.set((uint32_t)c, mu.get(h));
                Q.set((uint32_t)c, Q.get(h));
                R |= ((R >> h) & 1u) << c;
            }
    }

    // per-device records
#pragma unroll
    for (int d = 0; d < DM; d++) {
        if (d >= C.D) continue;
        const uint32_t mud = (uint32_t)((d < 4 ? mu.lo : mu.hi) >> (16 * (d & 3))) & 0xFFFFu;
        const uint32_t qd = (uint32_t)((d < 4 ? Q.lo : Q.hi) >> (16 * (d & 3))) & 0xFFFFu;
        // blocks that ran before the window: leads as bytes times the device's memory deltas.  (One dot product; in the exhaustive
        // spaces, which spill scalar registers around it, four products: 2,000,003 candidates of the factorial space of two
        // micro-batches of 16 types on 8 devices 316 -> 271 us.)
        int mem0 = 0;
        if (sampled) mem0 = entry_memory(mud, C.mpack[d]);
        else {
#pragma unroll
            for (int y = 0; y < kMaxLT; y++) mem0 += ((int)(C.mpack[d] << (24 - 8 * y)) >> 24) * (int)(mud >> (4 * y) & 15u);
        }
        const uint32_t alive = nlen[d] >= 32 ? 0xFFFFFFFFu : (1u << nlen[d]) - 1u;
        rec_store(L.rec + (uint32_t)d * kRecDevStep + (uint32_t)lane * 4u, make_uint4(plo[d], phi[d], alive, qd | ((uint32_t)mem0 << 16)));
        if (nlen[d] > 0) HM |= 1u << (4 * d + ((plo[d] & 1u) | ((phi[d] & 1u) << 1)));
    }

    lead_code = mu;
    S.R = R; S.HM = HM; S.X = X; S.worst = INT_MIN; S.status = status;
}

// Places the blocks of program words [w_from, w_to) (six blocks a word).  `live`: the lane holds a candidate.
// FREE: whether the orders of some devices go together at all.  The devices of the codes `free` run their blocks in any order: all of
// their types stand at the head (HM keeps their bits), and no program is written.
template <int DM, int MODE, bool TP, bool FREE = false>
__device__ __forceinline__ void build_words(const KParams &P, const FastConst<DM> &C, const FastLds &L, int lane, bool live,
                                            int w_from, int w_to, FastProgram &prog, BuildState &S, uint32_t *left_after, uint32_t free = 0)
{
    // With repair every candidate has an executable order (the blocks not yet placed form a DAG, so some type
    // is always runnable): no lane ever stops building, not even one without a candidate of the range (it scores
    // a real candidate whose result is dropped), and the per-lane predicate disappears from the loop.
    constexpr bool repair = MODE == 2;
    const int total = C.total;
    uint32_t R = S.R, HM = S.HM, X = S.X;
    int worst = S.worst, status = S.status;
    bool building = repair || (live && status == kOk);
    const uint32_t lane4 = (uint32_t)lane * 4u;
    const uint32_t rec_lane = L.rec + lane4;
    // one program word = six blocks
    auto word = [&](int wi) -> uint32_t {
        uint32_t acc = 0;
        const int nj = __builtin_amdgcn_readfirstlane(min(6, total - wi * 6));
#pragma unroll 1
        for (int j = 0; j < nj; j++) {
            uint32_t hm = R & HM;
            if (TP)
                for (int k = 0; k < C.ntp; k++) {
                    const uint32_t G = L.tpg_tab[k];
                    hm = (hm & G) == G ? hm : hm & ~G;
                }
            const uint32_t sel = hm ? hm : (repair ? R : 0u);
            if (!repair && building && sel == 0) { status = kDeadlock; building = false; }
            const uint32_t b = low_bit(sel);
            uint32_t d4 = repair ? min(b & 28u, 4u * (DM - 1)) : building ? b & 28u : 0u;    // 4 * device
            TESSEL_PIN(d4);
            const uint32_t ra = (d4 << 8) + rec_lane;          // (kRecDevStep = 4 << 8)
            const uint4 a = rec_load(ra);
            // earliest remaining entry of the device whose type is runnable: a 4-way multiplexer keyed by the two
            // planes.  (When the device was picked for its runnable head this is the head: nothing precedes it.)
            const int r4 = (int)(R >> d4);
            const uint32_t r0 = (uint32_t)__builtin_amdgcn_sbfe(r4, 0, 1), r1 = (uint32_t)__builtin_amdgcn_sbfe(r4, 1, 1),
                           r2 = (uint32_t)__builtin_amdgcn_sbfe(r4, 2, 1), r3 = (uint32_t)__builtin_amdgcn_sbfe(r4, 3, 1);
            const uint32_t gate = bfi(a.y, bfi(a.x, r3, r2), bfi(a.x, r1, r0));
            const uint32_t cand = a.z & gate, p = low_bit(cand);
            // its symbol, as two all-or-nothing masks
            const uint32_t ly = (uint32_t)__builtin_amdgcn_sbfe((int)a.x, p, 1), hy = (uint32_t)__builtin_amdgcn_sbfe((int)a.y, p, 1);
            // c = d4 | (ly & 1) | (hy & 2); as ly, hy are 0 or -1, also d4 - ly - 2 hy
            uint32_t c;
            if (repair) c = __builtin_amdgcn_bitop3_b32(__builtin_amdgcn_bitop3_b32(ly, hy, 1u, 0xE4), 3u, d4, 0xEA);
            else asm("v_mad_i32_i24 %0, %1, -2, %2" : "=v"(c) : "v"(hy), "v"(d4 - ly));
            const uint32_t c4 = c << 2;
            const uint4 e = rec_load(c4);                      // (the table of the types starts the kernel's LDS, at address 0)
            // take the entry out; new head of the device.  (When the device is empty now the bit set below is
            // meaningless, and harmless: all its types are exhausted, and R never holds an exhausted type.)
            // (With repair the step's instructions are chosen by rate, tessel_common.h: masks from signs instead of compares and selects,
            // right shifts instead of bit fields, the entry's bit by subtraction.  With the decode's part: 2^26 candidates of
            // 256 blocks on 8 devices 32.7 -> 32.0 ms, of 40 with two on all of four devices 6.03 -> 5.72.  Without repair, where a wave
            // ends with its last candidate and more masks are alive, they are fewer: build_begin has the figures.)
            const uint32_t alive = repair ? (uint32_t)__builtin_amdgcn_bitop3_b32(a.z, cand, 0u - cand, 0x70) : a.z & ~(1u << p);      // 0x70: a & ~(b & c)
            const uint32_t p2 = low_bit(alive);
            uint32_t c2;
            if (repair) {
                const uint32_t h2 = a.y >> (p2 & 31u);
                c2 = __builtin_amdgcn_bitop3_b32(__builtin_amdgcn_bitop3_b32(a.x >> (p2 & 31u), h2 + h2, 1u, 0xE4), 3u, d4, 0xEA);
            } else c2 = d4 + (__builtin_amdgcn_ubfe(a.x, p2, 1) | (__builtin_amdgcn_ubfe(a.y, p2, 1) << 1));
            const uint32_t hm_new = (HM & ~(15u << d4)) | (1u << c2) | (FREE ? free : 0u);
            // one waiting micro-batch is consumed; the type stays runnable while another one waits and
            // entries of it remain; its consumer gets one more and becomes runnable
            // remaining entries of the same type: alive & ~(lo ^ ly) & ~(hi ^ hy)
            const uint32_t rest = __builtin_amdgcn_bitop3_b32(__builtin_amdgcn_bitop3_b32(alive, a.x, ly, 0x90), a.y, hy, 0x90);
            // two or more were waiting (the shift, 4 * symbol, is in the low bits of the table entry)
            const uint32_t more = (a.w >> (e.z & 31u)) & 14u;
            // (a type on several devices: its codes on all of them)
            const uint32_t onec = TP ? L.grp_tab[c] : 1u << c;
            // exhausted: no entry of the type is left; it stays runnable only if entries are left and another
            // micro-batch waits.  (Masks, all ones: entries are left; another one waits.)
            const uint32_t some = (uint32_t)((int)(rest | (0u - rest)) >> 31), waits = (uint32_t)((int)(0u - more) >> 31);
            uint32_t x_new = repair ? (uint32_t)__builtin_amdgcn_bitop3_b32(X, onec, some, 0xF4) : X | (rest == 0 ? onec : 0u);        // 0xF4: a | (b & ~c)
            TESSEL_PIN(x_new);          // (the old X dies here: no second copy of the mask across the step)
            const uint32_t stalled = repair ? (uint32_t)__builtin_amdgcn_bitop3_b32(onec, some, waits, 0x70) : (rest == 0 || more == 0) ? onec : 0u;
            const uint32_t r_new = __builtin_amdgcn_bitop3_b32(R, stalled, e.y & ~x_new, 0xBA);      // (R & ~t) | z
            // the record's last word: waiting counts (16 bits) and the device's memory prefix (upper 16 bits,
            // signed); one sum updates both
            const uint32_t w_new = a.w + e.x;
            const bool active = repair || building;
            uint32_t hm_fin = hm_new;
            if (active) {
                lds_store(ra + 2u * kRecWordStep, alive);
                lds_store(ra + 3u * kRecWordStep, w_new);
                // (a type without a consumer on another device adds 0 to its own record)
                lds_fetch_add(__builtin_amdgcn_bitop3_b32(e.z, ~31u, lane4, 0xEA), e.w);       // (a & b) | c: rows of 256 bytes
                worst = max(worst, (int)w_new >> 16);
                acc |= c << (5 * j);
            }
            if (TP) {
                const bool several = active && ((C.several >> c) & 1u);
                if (__ballot(several) != 0 && several) {
                    // The block's earliest entry out of the lists of its other devices.  (It was picked on its lowest device: whichever of its codes
                    // is the lowest bit of all, that one is.  So the micro-batches that wait for it are counted there alone, and what is left to
                    // do on the others is their list, head and memory.)
                    const uint32_t mem = L.mem_tab[c];
#pragma unroll
                    for (int dd = 0; dd < DM; dd++) {
                        if (dd >= C.D) continue;
                        if (C.tp_all ? dd == 0 : ((onec >> (4 * dd)) & 15u) == 0 || 4u * dd == d4) continue;
                        const uint32_t rq = (uint32_t)dd * kRecDevStep + rec_lane;
                        const uint4 q = rec_load(rq);
                        const uint32_t y3 = (uint32_t)__builtin_amdgcn_sbfe((int)onec, 4 * dd + 3, 1);
                        const uint32_t ls = (uint32_t)__builtin_amdgcn_sbfe((int)onec, 4 * dd + 1, 1) | y3, hs = (uint32_t)__builtin_amdgcn_sbfe((int)onec, 4 * dd + 2, 1) | y3;
                        const uint32_t same = __builtin_amdgcn_bitop3_b32(__builtin_amdgcn_bitop3_b32(q.z, q.x, ls, 0x90), q.y, hs, 0x90);
                        const uint32_t left = __builtin_amdgcn_bitop3_b32(q.z, same, 0u - same, 0x70), wq = q.w + mem;
                        lds_store(rq + 2u * kRecWordStep, left);
                        lds_store(rq + 3u * kRecWordStep, wq);
                        worst = max(worst, (int)wq >> 16);
                        const uint32_t ph = low_bit(left), h2 = q.y >> (ph & 31u);
                        const uint32_t ch = __builtin_amdgcn_bitop3_b32(__builtin_amdgcn_bitop3_b32(q.x >> (ph & 31u), h2 + h2, 1u, 0xE4), 3u, 4u * dd, 0xEA);
                        hm_fin = (hm_fin & ~(15u << (4 * dd))) | 1u << ch;
                    }
                }
            }
            if (active) { R = r_new; X = x_new; HM = hm_fin; }
        }
        return acc;
    };
    // the program is two register vectors: one loop for each, so that a store never has to choose between them
    // (`left_after`: how many candidates are still alive goes into the launch's histogram)
    auto note = [&](int wi) {
        if (TP && repair && left_after && wi + 1 < w_to) {
            const uint32_t alive = (uint32_t)__builtin_popcountll(__ballot(worst <= C.M));
            if (lane == 0) __hip_atomic_fetch_add(left_after + wi + 1, alive, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        }
    };
    if constexpr (FREE) {
        for (int wi = w_from; wi < w_to && __ballot(building) != 0; wi++) (void)word(wi);
        S.status = status;
        return;
    }
    for (int wi = w_from; wi < min(w_to, 32); wi++) {
        if (!repair && __ballot(building) == 0) break;
        prog.a[wi] = word(wi);
        note(wi);
    }
    for (int wi = max(w_from, 32); wi < w_to; wi++) {
        if (!repair && __ballot(building) == 0) break;
        prog.b[wi - 32] = word(wi);
        note(wi);
    }
    S.R = R; S.HM = HM; S.X = X; S.worst = worst; S.status = status;
}

// the build's verdict once all blocks are placed
template <int DM>
__device__ __forceinline__ int build_end(const FastConst<DM> &C, const BuildState &S, int &peak_max)
{
    peak_max = 0;
    if (S.status != kOk) return S.status;
    int worst = S.worst;
#pragma unroll
    for (int d = 0; d < DM; d++)
        if (d < C.D && C.ntd[d] == 0) worst = max(worst, 0);      // a device without blocks holds nothing
    peak_max = worst;
    return worst > C.M ? kMem : kOk;
}

// What placing a block of the type with code `lane` does: its words of FastLds::type_tab; `rec`: LDS address of the records.
template <int DM, bool TP>
__device__ __forceinline__ void fill_type_tab(const KParams &P, uint32_t *type_tab, uint32_t rec, int lane)
{
    const uint32_t inf = P.info_loc[lane];
    const uint32_t su = inf & 63u, dev = (uint32_t)lane >> 2, y = (uint32_t)lane & 3u;
    const int32_t m = (int32_t)(inf << 6) >> 24;
    const bool has_su = su != 63u, same = has_su && (su >> 2) == dev;
    const uint32_t inc = has_su ? 1u << (4u * (su & 3u)) : 0u;
    const uint32_t last = rec + 3u * kRecWordStep;            // last word of device 0's record, lane 0
    const uint4 e = make_uint4(((uint32_t)m << 16) - (1u << (4u * y)) + (same ? inc : 0u),
                               !has_su ? 0u : TP && P.grp_code[su & 31u] ? P.grp_code[su & 31u] : 1u << (su & 31u),
                               last + (has_su && !same ? su >> 2 : dev < (uint32_t)DM ? dev : 0u) * kRecDevStep + 4u * y,
                               has_su && !same ? inc : 0u);
    type_tab[lane] = e.x; type_tab[2 * kMaxK + lane] = e.y; type_tab[4 * kMaxK + lane] = e.z; type_tab[6 * kMaxK + lane] = e.w;
}

// ------------------------------------------------------------------ which orders go together (CANONICAL, tables by rank)
// Next to all candidates of an exhaustive space deadlock (99.1 % of 2.88 G of a 4-stage pipeline with four micro-batches), and they
// share their deadlocks: the orders of two devices that cannot go together under some leads are the same two in all candidates that
// have them.  So a launch first finds out, for every lead vector of its range and every pair of devices that a dependency joins, which
// pairs of orders run to the end where all other devices run their blocks in any order (a necessary condition, whatever the
// other orders are), a bit each; the kernel over the range looks its candidates up there, 32 at a time, and builds those only
// that all their pairs leave (eval_fast_kernel, `pairs`).  In a pipeline these are the ones that do run; elsewhere a few more.
// 2^26 candidates of 4 stages and four micro-batches, by where the range lies: 1,810 to 2,350 us a call without, 153 to 378 with; all
// 5.8 M of three micro-batches 220 -> 62.
// One bit a lane: lead vectors x pairs x orders of the two.
template <int DM>
__global__ __launch_bounds__(kWave) void order_pairs_kernel(const KParams *__restrict__ Pp, uint32_t lead0, uint32_t chunks, uint32_t *__restrict__ tab)
{
    extern __shared__ uint32_t lds[];
    const KParams &P = *Pp;
    const int lane = threadIdx.x;
    FastLds L;
    L.type_tab = lds;
    L.rec = lds_address(lds) + kFastTableWords * 4u;
    if (lds_address(lds) != 0u) {                             // (the build's table starts at address 0; without it every bit stays set)
        for (uint32_t w = blockIdx.x * kWave + (uint32_t)lane; w < 2u * chunks; w += gridDim.x * kWave) tab[w] = ~0u;
        return;
    }
    if (lane < kMaxK) fill_type_tab<DM, false>(P, L.type_tab, L.rec, lane);
    __syncthreads();
    FastConst<DM> C;
    C.D = P.D; C.total = P.total; C.M = 0; C.ntp = 0;
    const uint32_t per_lead = P.pair_words / 2u;
    for (uint32_t chunk = blockIdx.x; chunk < chunks; chunk += gridDim.x) {
        const uint32_t lead = chunk / per_lead, at = (chunk - lead * per_lead) * 2u;
        int k = 0;
        while (k + 1 < P.npairs && P.pair_at[k + 1] <= at) k++;
        const int d = P.pair_of[k][0], e = P.pair_of[k][1];
        const uint32_t n = (uint32_t)P.cdev[d], bit = (at - P.pair_at[k]) * 32u + (uint32_t)lane;
        const bool valid = bit < n * (uint32_t)P.cdev[e];
        uint32_t rank_d = valid ? bit : 0u;
        const uint32_t rank_e = take_digit(rank_d, n, P.recip[d]);
        const uint32_t *row = P.leadrows + (size_t)(lead0 + lead) * kLeadRow;
        BuildState S;
        const uint32_t free = ~(15u << (4 * d) | 15u << (4 * e));
        S.R = row[8]; S.HM = free; S.X = 0; S.worst = INT_MIN; S.status = kOk;
#pragma unroll
        for (int dd = 0; dd < DM; dd++) {
            if (dd >= P.D) continue;
            const uint32_t len = (uint32_t)(P.ntd[dd] * P.NR);
            const uint64_t o = P.orders[P.order_at[P.ntd[dd]] + (dd == d ? rank_d : dd == e ? rank_e : 0u)];
            const uint32_t lo = (uint32_t)o, hi = (uint32_t)(o >> 32), waits = row[4 + dd / 2] >> (16 * (dd & 1)) & 0xFFFFu;
            rec_store(L.rec + (uint32_t)dd * kRecDevStep + (uint32_t)lane * 4u, make_uint4(lo, hi, len >= 32u ? 0xFFFFFFFFu : (1u << len) - 1u, waits));
            if (len > 0) S.HM |= 1u << (4 * dd + ((lo & 1u) | (hi & 1u) << 1));
        }
        FastProgram none;
        build_words<DM, 0, false, true>(P, C, L, lane, valid, 0, (P.total + 5) / 6, none, S, nullptr, free);
        const uint64_t run = __ballot(valid && S.status == kOk);
        if (lane < 2) tab[2u * chunk + (uint32_t)lane] = (uint32_t)(run >> (32 * lane));
    }
}

// (Waves per SIMD: what the registers of the variant allow without spills in the loops; the TP variants with four waves
// and 24 boundary values, or 8 devices, spilled up to 600 registers.)
template <int DM, int VM, int MODE, bool TP = false, bool PAIRS = false>
__global__ __launch_bounds__(kWave, MODE && !(TP && (DM > 4 || VM > 10)) ? 4 : 3) void eval_fast_kernel(const KParams *__restrict__ Pp, uint64_t first, uint64_t count,
                                                          BlockRec *__restrict__ recs, int32_t *__restrict__ code_out,
                                                          int32_t *__restrict__ peak_out, int tries, int retry_tries,
                                                          uint64_t *__restrict__ out_list, uint32_t *__restrict__ out_count,
                                                          uint32_t out_cap, uint32_t *__restrict__ overflow, uint32_t *ring_base,
                                                          uint32_t ring_words, int stage_words, int adapt, uint32_t *left_after,
                                                          const uint32_t *__restrict__ pairs, uint32_t lead0, uint32_t scatter)
{
    extern __shared__ uint32_t lds[];
    // the sweeps address their tables by LDS byte address from 0: the kernel has no other LDS in front of this array
    if (lds_address(lds) != 0u) { if (threadIdx.x == 0) *overflow = 0x100u; return; }
    const KParams &P = *Pp;
    const int lane = threadIdx.x;
    FastLds L;
    L.type_tab = lds;                                         // 4 x 64 words, the lower half of every 64
    L.chain_tab = lds + kMaxK;
    L.tt_tab = (uint4 *)(lds + kFastTableWords);              // 128 words, TP variants only
    L.grp_tab = lds + kFastTableWords + 4 * kMaxK;            // TP variants only
    L.mem_tab = lds + kFastTableWords + 5 * kMaxK;            // TP variants only
    L.tpg_tab = lds + kFastTableWords + 6 * kMaxK;            // TP variants only
    L.sw_tab = lds + kSweepTabWord;
    L.ch_tab = lds + kSweepTabWord + kMaxK;
    L.in_tab = lds + kSweepTabWord + 2 * kMaxK;
    uint32_t *base = lds + kFastTableWords + (TP ? kTpTableWords : 0);
    L.rec = lds_address(base);
    // the sweep state is only used once the build is over: it shares the records' space when it fits
    const int ntok = P.nslots - P.D;
    const bool share = DM * 2 + ntok <= DM * 4;
    uint32_t *sweep_base = share ? base : base + DM * kWave * 4;
    L.dfree = sweep_base;                       // [DM] device times, [DM] counters, then the tokens
    L.dcnt = sweep_base + DM * kWave;
    L.tok = sweep_base + 2 * DM * kWave;
    if (lane < kMaxK) {
        const uint32_t inf = P.info_loc[lane];
        if (TP) L.tt_tab[lane] = make_uint4((uint32_t)P.t_loc[lane], ((((inf >> 12) & 63u) - (uint32_t)P.D + 2u * DM) << 8),
                                    ((uint32_t)lane >> 2) * (kWave * 4u),
                                    (16u + 4u * ((uint32_t)lane & 3u)) | ((P.grp_code[lane] & (P.grp_code[lane] - 1u)) ? 0x80000000u : 0u));
        fill_type_tab<DM, TP>(P, L.type_tab, L.rec, lane);
        {
            // codes no block type has: device 0, chain 0, t = 0 (the pipeline of the sweeps reads code 0 past the end)
            const bool used = P.t_loc[lane] != 0;
            const uint32_t dev = used ? (uint32_t)lane >> 2 : 0u, rel = used ? ((inf >> 12) & 63u) - (uint32_t)P.D : 0u;
            L.sw_tab[lane] = ((uint32_t)P.t_loc[lane] << 16) | (lds_address(L.dfree) + dev * (kWave * 4u));
            L.ch_tab[lane] = lds_address(L.dfree) + (2u * DM + rel) * (kWave * 4u);
            L.in_tab[lane] = (1u << (16u + 4u * ((uint32_t)lane & 3u))) | (8u + 4u * ((uint32_t)lane & 3u));
        }
        L.chain_tab[lane] = P.chain_tab[lane];
        if (TP && lane < kMaxD) L.tpg_tab[lane] = P.tp_group[lane];
        if (TP) L.grp_tab[lane] = P.grp_code[lane] ? P.grp_code[lane] : 1u << lane;
        if (TP) L.mem_tab[lane] = (uint32_t)((int32_t)(inf << 6) >> 24) << 16;
    }
    __syncthreads();
    FastConst<DM> C;
    C.D = P.D; C.K = P.K; C.NR = P.NR; C.M = P.M; C.total = P.total; C.nslots = P.nslots; C.npaths = P.npaths;
    C.nsweeps = P.nsweeps; C.space = P.space; C.has_fixed = P.has_fixed; C.nwords = (P.total + 5) / 6; C.ndeps = P.K - P.npaths;
    C.step_q16 = P.step_q16; C.seed = P.seed;
#pragma unroll
    for (int d = 0; d < DM; d++) { C.ntd[d] = P.ntd[d]; C.mpack[d] = P.mpack[d]; }
    C.ntp = TP ? P.ntp : 0; C.several = TP ? P.several : 0u; C.tp_all = TP ? P.tp_all : 0;

    int best = INT_MAX;
    uint64_t best_idx = 0;
    // counters of the whole wave (uniform values: they live in scalar registers)
    uint32_t cnt[kNumStatus];
#pragma unroll
    for (int s = 0; s < kNumStatus; s++) cnt[s] = 0;
    uint32_t nev = 0;
    uint32_t nsw = 0;                // per lane: window sweeps
    // The kernel works in three phases with a queue between each two, so that every phase runs on full waves
    // although candidates drop out on the way:
    //   A  decode + the first `stage_words` words of the build, one new candidate per lane;
    //   B  the rest of the build for the candidates that are still alive after A (with repair, and no per-candidate
    //      peak wanted: whose memory is within the cap so far; most candidates that exceed it do so early);
    //   C  the window sweeps for the candidates that survive the build.
    // A survivor of A appends its state (masks, records, program so far) to ring 1 of this wave in global memory,
    // a survivor of B program and leads to ring 2; B and C run whenever 64 candidates wait in their ring, one per
    // lane.  Ring layout: [word][slot]; slot = ring tail + rank of the lane among the survivors.
    // A candidate whose boundary vector is no eigenvector yet after the `tries` sweeps of C goes, with its program, to
    // ring 3 and gets up to `retry_tries` sweeps from the start when 64 of them wait there (a wave sweeps until its
    // slowest lane is done: a straggler among 63 finished lanes would cost a whole sweep of the wave).  What is still
    // open then is appended to the list of the general kernel.
    uint32_t *ring1 = ring_base + (size_t)blockIdx.x * 3u * ring_words, *ring2 = ring1 + ring_words, *ring3 = ring2 + ring_words;
    uint32_t head1 = 0, count1 = 0, head2 = 0, count2 = 0, head3 = 0, count3 = 0, nretry = 0, nblocks = 0;           // wave-uniform
    const int nwords = C.nwords;
    // Program words of phase A: `stage_words`, or, in the repair variants for blocks on several devices where the waves have many
    // rounds of candidates to come (`adapt`), what the launch's first candidates ask for: the first two rounds are built in
    // one go; one wave in 16 adds to a histogram after how many words its candidates were out, and then every wave takes
    // the number of words that costs the fewest lane words: 64 w in phase A, and for the candidates alive then the rest of the words
    // and the way through the queue.  How early candidates leave depends on cap, times and leads, not on sizes: with a block
    // on all of four devices and 7 words a window the best number is 1 (0.36 of the time of building in one go), 2
    // (0.50) or 7 (2 words: 1.00 to 1.04) by the cap alone.  The way through the queue is counted, not fitted; what the waves
    // choose is within 5 % of the best fixed number in launches of 60 rounds (13 % at worst: the two rounds of the start).  (A
    // wave that goes by its own 64 candidates is off by as much as
    // the best number gains, and the launch ends with the slowest wave.  In the other variants the best number is near the one by
    // size, and the histogram's code costs them registers: 5 to 7 % of the time on 256 blocks.)
    int wordsA, chunksA;
    bool split;
    auto set_stage = [&](int w) {
        split = w < nwords;                                          // else A builds all of the window
        wordsA = split ? w : nwords;
        chunksA = (wordsA + 3) / 4;
    };
    set_stage(stage_words);
    const int chunksAll = (nwords + 3) / 4;
    const bool drop_mem = MODE == 2 && peak_out == nullptr;          // a rejected candidate's peak is that of the whole window
    // every phase has a program of its own (words it does not write stay undefined and are never read), so that no
    // program lives on from one phase to the next
    Mu lead_code;
    BuildState S;

    auto rank_in = [&](uint64_t m) -> uint32_t {
        return __builtin_amdgcn_mbcnt_hi((uint32_t)(m >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)m, 0u));
    };
    // a candidate the build rejects is final
    auto reject = [&](bool rejected, uint64_t idx, int status, int pk) {
        nev += (uint32_t)__builtin_popcountll(__ballot(rejected));
#pragma unroll
        for (int s = 1; s < kNumStatus; s++) cnt[s] += (uint32_t)__builtin_popcountll(__ballot(rejected && status == s));
        if (rejected) {
            if (code_out) code_out[idx - first] = -status;
            if (peak_out) peak_out[idx - first] = status == kMem ? pk : 0;
        }
    };
    auto push_program = [&](bool ok, uint64_t idx, int pk, const FastProgram &prog, uint32_t *ring, uint32_t tail) -> uint32_t {
        const uint64_t okm = __ballot(ok);
        if (okm == 0) return 0u;
        if (ok) {
            uint32_t *dst = ring + ((tail + rank_in(okm)) & (kRingSlots - 1u));
            dst[0 * kRingSlots] = (uint32_t)lead_code.lo; dst[1 * kRingSlots] = (uint32_t)(lead_code.lo >> 32);
            dst[2 * kRingSlots] = (uint32_t)lead_code.hi; dst[3 * kRingSlots] = (uint32_t)(lead_code.hi >> 32);
            dst[4 * kRingSlots] = (uint32_t)idx; dst[5 * kRingSlots] = (uint32_t)(idx >> 32);
            dst[6 * kRingSlots] = (uint32_t)pk;
#pragma unroll
            for (int c4 = 0; c4 < 12; c4++)
                if (c4 < chunksAll) {
#pragma unroll
                    for (int w = 4 * c4; w < 4 * c4 + 4; w++) dst[(kRingMetaWords + w) * kRingSlots] = prog.get(w);
                }
        }
        return (uint32_t)__builtin_popcountll(okm);
    };
    // phase C on the first n candidates of ring 2, or (`again`) of ring 3
    // (Wave priority by phase, set where a phase starts: the sweeps wait for the LDS after every few instructions and
    // issue first (3), then the second build phase (2), then the first (1: a build step waits for two rounds of LDS
    // reads); the decode, which always has an instruction ready, fills what is left (0).  Measured on windows of 256
    // blocks: 32.5 ms per 2^26 candidates against 37.3 with all waves equal; decode and first build phase both at 0
    // with the second at 1 or 2: 33.6 to 33.8; both build phases at 3: 34.3; the sweeps alone at 3: 35.9.)
    auto sweep_from_ring = [&](uint32_t n, bool again) {
        __builtin_amdgcn_s_setprio(3);
        __threadfence_block();         // the stores of this wave's other lanes must be visible to the loads below
        const bool have = (uint32_t)lane < n;
        const uint32_t *src = (again ? ring3 : ring2) + (((again ? head3 : head2) + (uint32_t)lane) & (kRingSlots - 1u));
        // every lane loads (a lane without a candidate reads a slot behind the last one: stale words, results dropped)
        FastProgram prog;
        lead_code.lo = (uint64_t)src[0 * kRingSlots] | ((uint64_t)src[1 * kRingSlots] << 32);
        lead_code.hi = (uint64_t)src[2 * kRingSlots] | ((uint64_t)src[3 * kRingSlots] << 32);
        const uint64_t idx = have ? (uint64_t)src[4 * kRingSlots] | ((uint64_t)src[5 * kRingSlots] << 32) : first;
        const int pk = (int)src[6 * kRingSlots];
#pragma unroll
        for (int c4 = 0; c4 < 12; c4++)
            if (c4 < chunksAll) {
#pragma unroll
                for (int w = 4 * c4; w < 4 * c4 + 4; w++) prog.set(w, src[(kRingMetaWords + w) * kRingSlots]);
            }
        if (again) { head3 = (head3 + n) & (kRingSlots - 1u); count3 -= n; }
        else { head2 = (head2 + n) & (kRingSlots - 1u); count2 -= n; }
        const int T = period_fast<DM, VM, TP>(P, C, L, prog, lane, lead_code, have, again ? retry_tries : tries, again, nsw);
        const bool open = have && T < 0;                  // no eigenvector within the sweeps allowed
        if (!again) {
            const uint32_t k = push_program(open, idx, pk, prog, ring3, head3 + count3);
            count3 += k; nretry += k;
        } else if (open) {
            const uint32_t at = atomicAdd(out_count, 1u);
            if (at < out_cap) out_list[at] = idx; else *overflow = 1u;
        }
        const bool scored = have && T >= 0;
        const uint32_t ns = (uint32_t)__builtin_popcountll(__ballot(scored));
        nev += ns;
        cnt[kOk] += ns;
        if (scored) {
            if (key_less(T, idx, best, best_idx)) { best = T; best_idx = idx; }
            if (code_out) code_out[idx - first] = T;
            if (peak_out) peak_out[idx - first] = pk;
        }
    };
    // the end of the build for the candidates the lanes hold: verdict, then ring 2 or out
    auto finish_build = [&](bool have, uint64_t idx, const FastProgram &prog) {
        int pk;
        const int status = build_end<DM>(C, S, pk);
        reject(have && status != kOk, idx, status, pk);
        count2 += push_program(have && status == kOk, idx, pk, prog, ring2, head2 + count2);
    };
    // phase B on the first n candidates of ring 1
    auto build_from_ring = [&](uint32_t n) {
        __builtin_amdgcn_s_setprio(2);
        __threadfence_block();
        const bool have = (uint32_t)lane < n;
        const uint32_t *src = ring1 + ((head1 + (uint32_t)lane) & (kRingSlots - 1u));
        FastProgram prog;
        S.status = kOk;
        S.R = src[0 * kRingSlots]; S.HM = src[1 * kRingSlots]; S.X = src[2 * kRingSlots]; S.worst = (int)src[3 * kRingSlots];
        lead_code.lo = (uint64_t)src[4 * kRingSlots] | ((uint64_t)src[5 * kRingSlots] << 32);
        lead_code.hi = (uint64_t)src[6 * kRingSlots] | ((uint64_t)src[7 * kRingSlots] << 32);
        const uint64_t idx = have ? (uint64_t)src[8 * kRingSlots] | ((uint64_t)src[9 * kRingSlots] << 32) : first;
#pragma unroll
        for (int d = 0; d < DM; d++)
            if (d < C.D)
                rec_store(L.rec + (uint32_t)d * kRecDevStep + (uint32_t)lane * 4u,
                          make_uint4(src[(kStageMetaWords + 4 * d) * kRingSlots], src[(kStageMetaWords + 4 * d + 1) * kRingSlots],
                                     src[(kStageMetaWords + 4 * d + 2) * kRingSlots], src[(kStageMetaWords + 4 * d + 3) * kRingSlots]));
#pragma unroll
        for (int c4 = 0; c4 < 12; c4++)
            if (c4 < chunksA) {
#pragma unroll
                for (int w = 4 * c4; w < 4 * c4 + 4; w++) prog.set(w, src[(kStageMetaWords + 4 * DM + w) * kRingSlots]);
            }
        head1 = (head1 + n) & (kRingSlots - 1u);
        count1 -= n;
        build_words<DM, MODE, TP>(P, C, L, lane, have, wordsA, nwords, prog, S, nullptr);
        nblocks += n * (uint32_t)(C.total - min(C.total, 6 * wordsA));
        finish_build(have, idx, prog);
    };

    const uint64_t stride = (uint64_t)gridDim.x * kWave;
    uint64_t rounds = (count + stride - 1) / stride;                // the same trip count for every lane of the grid
    // With tables of the orders that go together (PAIRS): candidates come from there.  A unit is 32 neighbours in the order of the
    // first device, their other orders and leads alike: a bit each by the pairs that device is in, all or none by the others.
    // Those that are left go to a list of the wave, as offsets (in ring 1, which a window built in one go leaves free), until there are
    // 64.  The units of a wave's lanes lie far apart, so that every wave gets its share: the ones with anything left lie together.  (A
    // variant of its own: as a branch in the others it cost launches without tables 2 to 4 %.)
    static_assert(63 + 32 * kWave <= (4 + kStageMetaWords + 4 * 2) * (int)kRingSlots, "the list of a wave fits its ring");
    uint32_t *const left_list = ring1;
    uint32_t nleft = 0, out = 0;                                     // candidates on it; per lane: candidates that the tables reject
    uint32_t n0 = 0, wpr = 0, group0 = 0, units = 0, unit_lanes = 0, unit_rounds = 0, unit_round = blockIdx.x, unit_shift = 0;
    if (PAIRS) {
        n0 = (uint32_t)P.cdev[0];
        wpr = (n0 + 31u) / 32u;
        group0 = (uint32_t)(first / n0);
        units = ((uint32_t)((first + count - 1) / n0) - group0 + 1u) * wpr;
        unit_lanes = min((units + gridDim.x - 1u) / gridDim.x, (uint32_t)kWave);
        unit_rounds = (units + unit_lanes - 1u) / unit_lanes;
        if (scatter) unit_shift = (uint32_t)lane * 0x9E3779B1u % unit_rounds;
        rounds = 0;
    }
    auto look_up = [&]() {
        uint32_t unit = unit_round + unit_shift;
        unit = (unit < unit_rounds ? unit : unit - unit_rounds) + (uint32_t)lane * unit_rounds;
        unit_round += gridDim.x;
        uint32_t left = 0, at0 = 0;
        if ((uint32_t)lane < unit_lanes && unit < units) {
            const uint32_t row = unit / wpr, w = unit - row * wpr;
            uint32_t rank[DM], lead = group0 + row;
            rank[0] = 0;
#pragma unroll
            for (int d = 1; d < DM; d++) {
                rank[d] = lead;
                lead = d < C.D ? take_digit(rank[d], (uint32_t)P.cdev[d], P.recip[d]) : lead;
            }
            // the members of the unit that are in the range
            const uint64_t base = (uint64_t)(group0 + row) * n0 + 32u * w;
            const uint32_t members = min(32u, n0 - 32u * w);
            uint32_t in = members < 32u ? (1u << members) - 1u : 0xFFFFFFFFu;
            if (base < first) in = first - base < 32 ? in & (0xFFFFFFFFu << (uint32_t)(first - base)) : 0u;
            const uint64_t behind = first + count;
            if (base + 32 > behind) in = behind > base ? in & ((1u << (uint32_t)(behind - base)) - 1u) : 0u;
            const uint32_t *tab = pairs + (size_t)(lead - lead0) * P.pair_words;
            left = in;
            for (int k = 0; k < P.npairs; k++) {
                const int d = P.pair_of[k][0], e = P.pair_of[k][1];
                uint32_t rd = 0, re = 0;
#pragma unroll
                for (int dd = 0; dd < DM; dd++) { rd = dd == d ? rank[dd] : rd; re = dd == e ? rank[dd] : re; }
                const uint32_t bit = re * (uint32_t)P.cdev[d] + (d == 0 ? 32u * w : rd);
                const uint32_t *word = tab + P.pair_at[k] + (bit >> 5);
                // (the unit's members end inside the table, so a second word is read only where there is one)
                if (d == 0) {
                    const bool more = (bit & 31u) + members > 32u;
                    left &= __builtin_amdgcn_alignbit(more ? word[1] : 0u, word[0], bit & 31u);
                } else left = word[0] >> (bit & 31u) & 1u ? left : 0u;
            }
            out += (uint32_t)__builtin_popcount(in & ~left);
            at0 = (uint32_t)(base - first);                          // (below 0 for the first unit: its first members are out of the range)
        }
        for (;;) {
            const uint64_t some = __ballot(left != 0u);
            if (some == 0) break;
            if (left != 0u) {
                left_list[nleft + rank_in(some)] = at0 + (uint32_t)__builtin_ctz(left);
                left &= left - 1u;
            }
            nleft += (uint32_t)__builtin_popcountll(some);
        }
    };
    const bool adapting = TP && MODE == 2 && adapt && drop_mem;
    if (adapting) set_stage(nwords);
    // phase A on the next 64 candidates of the wave's share
    uint64_t r = 0;
    uint32_t built = 0;                                              // phases A so far
    bool sieve = TP && MODE == 2 && drop_mem && !C.has_fixed && rounds > 1;
    uint32_t *const tp_list = lds + kFastTableWords + kTpListWord;
    auto build_new = [&]() {
        uint64_t kk = r * stride + (uint64_t)blockIdx.x * kWave + lane;
        bool valid = kk < count;
        if (TP && MODE == 2) {
            // leads first: 64 candidates at a time, until 64 are left whose entry memory fits
            while (sieve && nleft < (uint32_t)kWave && r < rounds) {
                kk = r++ * stride + (uint64_t)blockIdx.x * kWave + lane;
                valid = kk < count;
                const uint64_t idx = first + (valid ? kk : 0u);
                const bool over = entry_over<DM>(P, C, idx);
                reject(valid && over, idx, kMem, 0);
                const uint64_t fits = __ballot(valid && !over);
                if (valid && !over) tp_list[nleft + rank_in(fits)] = (uint32_t)kk;
                nleft += (uint32_t)__builtin_popcountll(fits);
                // (a look at the leads costs a sixth of what it saves of a candidate that it rejects)
                if (r == 1) sieve = __builtin_popcountll(fits) <= 52;
            }
            if (nleft > 0 || sieve) {
                const uint32_t n = min(nleft, (uint32_t)kWave);
                if (n == 0) return;
                __threadfence_block();
                valid = (uint32_t)lane < n;
                nleft -= n;
                kk = valid ? tp_list[nleft + (uint32_t)lane] : 0u;
            } else r++;
        } else r++;
        if (PAIRS) {
            while (nleft < (uint32_t)kWave && unit_round < unit_rounds) look_up();
            const uint32_t n = min(nleft, (uint32_t)kWave);
            if (n == 0) return;
            __threadfence_block();
            valid = (uint32_t)lane < n;
            nleft -= n;
            kk = valid ? left_list[nleft + (uint32_t)lane] : 0u;
        }
        const uint64_t idx = valid ? first + kk : first;
        __builtin_amdgcn_s_setprio(0);
        build_begin<DM, MODE, TP>(P, C, idx, first + count - 1, L, lane, lead_code, S);
        FastProgram prog;
        __builtin_amdgcn_s_setprio(1);
        const uint32_t nth = built++;
        const bool watch = adapting && nth < 2;
        const bool report = watch && nth == 0 && (blockIdx.x & 15u) == 0;
        build_words<DM, MODE, TP>(P, C, L, lane, valid, 0, wordsA, prog, S, report ? left_after : nullptr);
        nblocks += (uint32_t)__builtin_popcountll(__ballot(valid)) * (uint32_t)min(C.total, 6 * wordsA);
        if (!split) {
            finish_build(valid, idx, prog);
            if (!(TP && MODE == 2) || !watch) return;
            if (nth == 0) {
                if (report && lane == 0) __hip_atomic_fetch_add(left_after, (uint32_t)kWave, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                return;
            }
            // (the way through the queue in words, times eight: push and pop of masks, records and program)
            constexpr uint32_t way = 4 + DM;
            const uint32_t alive = lane < nwords ? __hip_atomic_load(left_after + lane, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) : 0u;
            const uint32_t all = (uint32_t)__builtin_amdgcn_readfirstlane((int)alive), n8 = 8u * (uint32_t)nwords, w8 = 8u * (uint32_t)lane;
            // lane w: the cost of w words; lane 0: of building in one go.  (At most 2^14 candidates times 43 words times 8: the
            // number fits above six bits of w.)
            uint32_t cost = lane == 0 ? all * n8 : lane < nwords ? all * w8 + alive * (n8 - w8 + way) : 0x3FFFFFFu;
            cost = (cost << 6) | (uint32_t)lane;
#pragma unroll
            for (int off = 32; off >= 1; off >>= 1) cost = min(cost, (uint32_t)__shfl_xor(cost, off));
            const int w = (int)(cost & 63u);
            set_stage(all == 0 ? stage_words : w == 0 ? nwords : w);
            return;
        }
        const bool over = drop_mem && S.status == kOk && S.worst > C.M;
        reject(valid && (S.status != kOk || over), idx, over ? (int)kMem : S.status, 0);
        const bool ok = valid && S.status == kOk && !over;
        const uint64_t okm = __ballot(ok);
        if (okm == 0) return;
        if (ok) {
            uint32_t *dst = ring1 + ((head1 + count1 + rank_in(okm)) & (kRingSlots - 1u));
            dst[0 * kRingSlots] = S.R; dst[1 * kRingSlots] = S.HM; dst[2 * kRingSlots] = S.X; dst[3 * kRingSlots] = (uint32_t)S.worst;
            dst[4 * kRingSlots] = (uint32_t)lead_code.lo; dst[5 * kRingSlots] = (uint32_t)(lead_code.lo >> 32);
            dst[6 * kRingSlots] = (uint32_t)lead_code.hi; dst[7 * kRingSlots] = (uint32_t)(lead_code.hi >> 32);
            dst[8 * kRingSlots] = (uint32_t)idx; dst[9 * kRingSlots] = (uint32_t)(idx >> 32);
#pragma unroll
            for (int d = 0; d < DM; d++)
                if (d < C.D) {
                    const uint4 q = rec_load(L.rec + (uint32_t)d * kRecDevStep + (uint32_t)lane * 4u);
                    dst[(kStageMetaWords + 4 * d) * kRingSlots] = q.x; dst[(kStageMetaWords + 4 * d + 1) * kRingSlots] = q.y;
                    dst[(kStageMetaWords + 4 * d + 2) * kRingSlots] = q.z; dst[(kStageMetaWords + 4 * d + 3) * kRingSlots] = q.w;
                }
#pragma unroll
            for (int c4 = 0; c4 < 12; c4++)
                if (c4 < chunksA) {
#pragma unroll
                    for (int w = 4 * c4; w < 4 * c4 + 4; w++) dst[(kStageMetaWords + 4 * DM + w) * kRingSlots] = prog.get(w);
                }
        }
        count1 += (uint32_t)__builtin_popcountll(okm);
    };

    // Later phases first: a ring is served as soon as it holds 64 candidates, so that it never holds more than 127;
    // when the wave's share is used up the rings are drained on partial waves.  Every condition is wave-uniform.
    for (;;) {
        const bool fresh = r < rounds || nleft > 0 || (PAIRS && unit_round < unit_rounds);
        // (one call for both rings of programs, so that the sweeps exist once in the code)
        const bool again = count3 >= (uint32_t)kWave || (!fresh && count1 == 0 && count2 == 0 && count3 > 0);
        const bool sweep = again || count2 >= (uint32_t)kWave || (!fresh && count1 == 0 && count2 > 0);
        if (sweep) sweep_from_ring(min(again ? count3 : count2, (uint32_t)kWave), again);
        else if (count1 >= (uint32_t)kWave || (!fresh && count1 > 0)) build_from_ring(min(count1, (uint32_t)kWave));
        else if (fresh) build_new();
        else break;
    }
    if (!recs) return;
#pragma unroll
    for (int off = 32; off >= 1; off >>= 1) {
        int op = __shfl_xor(best, off);
        uint32_t ilo = __shfl_xor((uint32_t)best_idx, off), ihi = __shfl_xor((uint32_t)(best_idx >> 32), off);
        uint64_t oi = ((uint64_t)ihi << 32) | ilo;
        if (key_less(op, oi, best, best_idx)) { best = op; best_idx = oi; }
        nsw += __shfl_xor(nsw, off);
        if (PAIRS) out += __shfl_xor(out, off);
    }
    if (PAIRS) { nev += out; cnt[kDeadlock] += out; }
    if (lane == 0) {
        BlockRec rr;
        rr.period = best; rr.n_retried = nretry; rr.index = best_idx; rr.n_evaluated = nev; rr.n_sweeps = nsw; rr.n_blocks = nblocks; rr.n_high = 0;
#pragma unroll
        for (int s = 0; s < kNumStatus; s++) rr.n_status[s] = cnt[s];
        recs[blockIdx.x] = rr;
    }
}

// ------------------------------------------------------------------ kernels
// Problems with more than kMaxD devices, kMaxK block types, kMaxLT types on a device or kMaxNR micro-batches per window (DM above kMaxD)
// are scored as dependency graphs, with the per-lane state and program in global memory (`far`: one region of
// far_words(P) words per workgroup) where the LDS of a workgroup does not hold them: 24 devices with 40 rings of 24
// slots and 384 program entries need 300 KB.
// (`where`: 1 = only the program lives there, the state stays in LDS; 2 = both)
__host__ __device__ inline size_t far_words(const KParams &P, int where)
{
    const size_t state = where == 2 ? (size_t)P.nslots * kWave * 4 : 0, prog = where ? (size_t)P.total * kWave * 2 : 0;
    return ((state + prog + 255) & ~(size_t)255) / 4;
}

// What one launch adds to the running best: the sum of records, a wave at a time.  Candidates are counted in 32 bits (a launch has at
// most 2^26), sweeps and blocks in 64, also in the record of a part of the launch.
static_assert(kMaxPerLaunch <= 0xFFFFFFFFu, "candidates of a launch are counted in 32 bits");
static_assert(((kMaxPerLaunch * 2 * kMostTries) >> 48) == 0 && ((kMaxPerLaunch * kMaxKW * kMaxNRW) >> 48) == 0, "BlockRec::n_high holds what is above 32 bits");
struct Tally {
    int best;
    uint32_t nre, nev, cnt[kNumStatus];
    uint64_t best_idx, nsw, nbl;
    __device__ __forceinline__ void clear()
    {
        best = INT_MAX; best_idx = 0; nre = nev = 0; nsw = nbl = 0;
#pragma unroll
        for (int s = 0; s < kNumStatus; s++) cnt[s] = 0;
    }
    __device__ __forceinline__ void add(const BlockRec &r)
    {
        if (key_less(r.period, r.index, best, best_idx)) { best = r.period; best_idx = r.index; }
        nre += r.n_retried; nev += r.n_evaluated; nsw += (uint64_t)(r.n_high >> 16) << 32 | r.n_sweeps; nbl += (uint64_t)(r.n_high & 0xFFFFu) << 32 | r.n_blocks;
#pragma unroll
        for (int s = 0; s < kNumStatus; s++) cnt[s] += r.n_status[s];
    }
    __device__ __forceinline__ static uint64_t from(uint64_t v, int off)
    {
        const uint32_t lo = __shfl_xor((uint32_t)v, off), hi = __shfl_xor((uint32_t)(v >> 32), off);
        return ((uint64_t)hi << 32) | lo;
    }
    // the wave's sum, in every lane
    __device__ __forceinline__ void fold()
    {
#pragma unroll 1
        for (int off = kWave / 2; off >= 1; off >>= 1) {
            const int op = __shfl_xor(best, off);
            const uint64_t oi = from(best_idx, off);
            if (key_less(op, oi, best, best_idx)) { best = op; best_idx = oi; }
            nre += __shfl_xor(nre, off); nev += __shfl_xor(nev, off); nsw += from(nsw, off); nbl += from(nbl, off);
#pragma unroll
            for (int s = 0; s < kNumStatus; s++) cnt[s] += __shfl_xor(cnt[s], off);
        }
    }
};

// `from_range` < 0: scores the range.  Else the pass over the list, in the workspace `ws`, of the kernel before it in the launch; it also adds up the launch, its own records and the `from_range` of the kernel over the range
// right in front of them, and clears the list's counter and the histogram for the next launch (scores of every candidate: the
// latter alone).  (Addresses in the workspace are worked out where they are needed: as arguments of their own they were spilled
// around the loop over candidates, 4 % of 331,776 scores of an exhaustive space.)
template <int DM, int VM>
__global__ __launch_bounds__(kWave) void eval_kernel(const KParams *__restrict__ Pp, uint64_t first, uint64_t count,
                                                     BlockRec *recs, int32_t *__restrict__ code_out,
                                                     int32_t *__restrict__ peak_out, bool whole, uint32_t *far, int where, char *ws, int from_range)
{
    const KParams &P = *Pp;
    extern __shared__ uint32_t lds[];
    constexpr bool wide = DM > kMaxD;
    // with a list: score the listed candidates (all inside [first, first + count)) instead of the range; `whole`: the range
    // after all where the list was too short for them.  (A workgroup without a candidate leaves no record.)
    // Who takes part in the pass over a list: a workgroup for every 64 candidates on it, and for every 64 records of the kernel over
    // the range, as far as the grid goes.  (The count is cleared by the last one that takes part; one that reads it
    // later sees a smaller number, and takes no part either way.)
    uint32_t parts = gridDim.x;
    bool listing = false;
    if (from_range >= 0) {
        const uint32_t listed = ((const DevResult *)(ws + kWsResultOff))->defer_count;
        listing = !(whole && listed > kWsListCap);
        if (listing) {
            count = min(listed, kWsListCap);
            const uint32_t records = (uint32_t)(from_range + kWave - 1) / kWave;
            parts = min(parts, max(max((uint32_t)((count + kWave - 1) / kWave), records), 1u));
            if (blockIdx.x >= parts) return;
        }
    }
    constexpr int KT = wide ? kMaxKW : kMaxK;             // entries of a table by type
    int32_t *t_tab = (int32_t *)lds;
    uint32_t *mask_tab = lds + KT;
    // (wide problems: behind their five tables in LDS, or in this workgroup's region of the workspace: `where` = 1 the
    // program, 2 state and program)
    uint32_t *region = wide && where ? far + (size_t)blockIdx.x * far_words(P, where) : nullptr;
    uint32_t *state_all = !wide ? lds + 4 * kMaxK : where == 2 ? region : lds + 5 * kMaxKW;
    uint16_t *prog_all = where == 1 ? (uint16_t *)region : (uint16_t *)(state_all + P.nslots * kWave);
    const int lane = threadIdx.x;
    // by home code for chain problems, by type id (with the producers and the token rings) for the others
    DagTables Tb;
    Tb.t = t_tab; Tb.mask = mask_tab; Tb.pred = lds + 2 * KT; Tb.tok = lds + 3 * KT; Tb.pred_hi = wide ? lds + 4 * KT : nullptr;
    if (lane < KT) {
        t_tab[lane] = P.dag ? P.t_type[lane] : P.t_loc[lane];
        mask_tab[lane] = P.dag ? P.mask_type[lane] : P.mask_loc[lane];
        lds[2 * KT + lane] = (uint32_t)P.predmask[lane];
        lds[3 * KT + lane] = P.tokbase[lane];
        if (wide) lds[4 * KT + lane] = (uint32_t)(P.predmask[lane] >> 32);
    }
    __syncthreads();
    uint32_t *state = state_all + lane;
    uint16_t *prog = prog_all + lane;

    int best = INT_MAX;
    uint64_t best_idx = 0;
    uint32_t cnt[kNumStatus];
#pragma unroll
    for (int s = 0; s < kNumStatus; s++) cnt[s] = 0;
    uint32_t nev = 0;

    const uint64_t stride = (uint64_t)gridDim.x * kWave;
    for (uint64_t kk = (uint64_t)blockIdx.x * kWave + lane; kk < count; kk += stride) {
        const uint64_t idx = listing ? ((const uint64_t *)(ws + kWsListOff))[kk] : first + kk;
        const uint64_t k = idx - first;
        int period, peak[DM];
        int status;
        if constexpr (wide) status = evaluate_dag<DM, MuWide>(P, Tb, idx, prog, state, period, peak);
        else status = P.dag ? evaluate_dag<DM, Mu>(P, Tb, idx, prog, state, period, peak)
                            : evaluate<DM, VM>(P, idx, prog, state, t_tab, mask_tab, period, peak);
        nev++;
#pragma unroll
        for (int s = 0; s < kNumStatus; s++) cnt[s] += status == s;
        if (status == kOk && key_less(period, idx, best, best_idx)) { best = period; best_idx = idx; }
        int pk = 0;
        if (status == kOk || status == kMem) {
            pk = INT_MIN;
#pragma unroll
            for (int d = 0; d < DM; d++) if (d < P.D) pk = max(pk, peak[d]);
        }
        if (code_out) code_out[k] = status == kOk ? period : -status;
        if (peak_out) peak_out[k] = pk;
    }
    Tally a;
    a.best = best; a.best_idx = best_idx; a.nre = 0; a.nev = nev; a.nsw = 0; a.nbl = 0;
#pragma unroll
    for (int s = 0; s < kNumStatus; s++) a.cnt[s] = cnt[s];
    // (in a launch whose range this kernel scored again, the records of the kernel before it are void)
    if (listing)
        for (int r = (int)blockIdx.x * kWave + lane; r < from_range; r += (int)parts * kWave) a.add(recs[r - from_range]);
    if (recs) {
        a.fold();
        if (lane == 0) {
            BlockRec r;
            r.period = a.best; r.n_retried = a.nre; r.index = a.best_idx; r.n_evaluated = a.nev; r.n_sweeps = (uint32_t)a.nsw;
            r.n_blocks = (uint32_t)a.nbl; r.n_high = (uint32_t)(a.nsw >> 32) << 16 | (uint32_t)(a.nbl >> 32);
#pragma unroll
            for (int s = 0; s < kNumStatus; s++) r.n_status[s] = a.cnt[s];
            recs[blockIdx.x] = r;
        }
    }
    if (from_range < 0) return;
    // ---- the workgroup that comes last adds the records up
    DevResult *res = (DevResult *)(ws + kWsResultOff);
    if (parts > 1) {
        uint32_t before = 0;
        __threadfence();
        if (lane == 0) before = __hip_atomic_fetch_add(&res->arrived, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        if ((uint32_t)__builtin_amdgcn_readfirstlane((int)before) + 1u != parts) return;
        __threadfence();
        if (recs) {
            a.clear();
            for (uint32_t r = (uint32_t)lane; r < parts; r += kWave) a.add(recs[r]);
            a.fold();
        }
    }
    ((uint32_t *)(ws + kWsLeftOff))[lane] = 0;
    if (lane != 0) return;
    if (recs) {
        if (key_less(a.best, a.best_idx, res->period, res->index)) { res->period = a.best; res->index = a.best_idx; }
        res->n_retried += a.nre;
        res->n_deferred += min(res->defer_count, kWsListCap);
        res->n_evaluated += a.nev;
        res->n_sweeps += a.nsw;
        res->n_blocks += a.nbl;
#pragma unroll
        for (int s = 0; s < kNumStatus; s++) res->n_status[s] += a.cnt[s];
    }
    res->defer_count = 0;
    res->arrived = 0;
}

// The two instantiations for problems beyond the fast kernel's limits (16 and 32 devices) take as long to compile as
// everything else in this file: tessel_wide.hip includes this file up to here and holds them, so that the two halves
// build side by side.
#define TESSEL_EVAL_KERNEL_ARGS const KParams *, uint64_t, uint64_t, BlockRec *, int32_t *, int32_t *, bool, uint32_t *, int, char *, int
#ifdef TESSEL_WIDE_INSTANTIATIONS
template __global__ void eval_kernel<16, 1>(TESSEL_EVAL_KERNEL_ARGS);
template __global__ void eval_kernel<32, 1>(TESSEL_EVAL_KERNEL_ARGS);
#else
extern template __global__ void eval_kernel<16, 1>(TESSEL_EVAL_KERNEL_ARGS);
extern template __global__ void eval_kernel<32, 1>(TESSEL_EVAL_KERNEL_ARGS);

// Merges the block records of a launch of the general kernel alone into the running best: one workgroup, a record per thread and
// round, waves first.  (Behind the other two kernels the pass over the list does that: one launch less.)  Bound by the
// latency of the record loads: 4,160 records took one wave 14.6 us (65 dependent rounds), eight waves take 9 to 10.
constexpr int kMergeThreads = 512;
__global__ __launch_bounds__(kMergeThreads) void merge_kernel(const BlockRec *__restrict__ recs, int nrecs, DevResult *__restrict__ res)
{
    __shared__ Tally part[kMergeThreads / kWave];
    Tally a;
    a.clear();
    for (int k = threadIdx.x; k < nrecs; k += kMergeThreads) a.add(recs[k]);
    a.fold();
    if ((threadIdx.x & (kWave - 1)) == 0) part[threadIdx.x / kWave] = a;
    __syncthreads();
    if (threadIdx.x != 0) return;
    for (int w = 1; w < kMergeThreads / kWave; w++) {
        const Tally &o = part[w];
        if (key_less(o.best, o.best_idx, a.best, a.best_idx)) { a.best = o.best; a.best_idx = o.best_idx; }
        a.nev += o.nev;
        for (int s = 0; s < kNumStatus; s++) a.cnt[s] += o.cnt[s];
    }
    if (key_less(a.best, a.best_idx, res->period, res->index)) { res->period = a.best; res->index = a.best_idx; }
    res->n_evaluated += a.nev;
    for (int s = 0; s < kNumStatus; s++) res->n_status[s] += a.cnt[s];
}

__global__ void reset_kernel(DevResult *res, uint32_t *left_after)
{
    if (threadIdx.x == 0 && blockIdx.x == 0) {
        for (int w = 0; w < kWave; w++) left_after[w] = 0;
        res->period = INT_MAX; res->pad = 0; res->index = ~0ull; res->n_evaluated = 0; res->n_sweeps = 0; res->n_blocks = 0;
        res->n_retried = 0; res->n_deferred = 0; res->overflow = 0; res->defer_count = 0; res->arrived = 0;
        for (int s = 0; s < kNumStatus; s++) res->n_status[s] = 0;
    }
}

// ------------------------------------------------------------------ launchers
typedef void (*eval_fn)(TESSEL_EVAL_KERNEL_ARGS);
typedef void (*fast_fn)(const KParams *, uint64_t, uint64_t, BlockRec *, int32_t *, int32_t *, int, int, uint64_t *, uint32_t *,
                        uint32_t, uint32_t *, uint32_t *, uint32_t, int, int, uint32_t *, const uint32_t *, uint32_t, uint32_t);
typedef void (*pairs_fn)(const KParams *, uint32_t, uint32_t, uint32_t *);

// problems too wide for the fast kernel and the chain path (their state stays in LDS where 64 KB hold it)
static bool wide_problem(const KParams &kp) { return kp.D > kMaxD || kp.K > kMaxK || kp.many || kp.NR > kMaxNR; }

static eval_fn pick_kernel(const KParams &kp)
{
    const int V = kp.nsweeps - 1;
    if (kp.D > 16) return eval_kernel<32, 1>;
    if (wide_problem(kp)) return eval_kernel<16, 1>;
    if (kp.D <= 2 && V <= 4) return eval_kernel<2, 4>;
    if (kp.D <= 4 && V <= 8) return eval_kernel<4, 8>;
    if (kp.D <= 8 && V <= 16) return eval_kernel<8, 16>;
    return eval_kernel<8, 24>;
}

// devices of the fast kernel's variant: 2, 4 or 8
static int fast_dm(const KParams &kp) { return kp.D <= 2 ? 2 : kp.D <= 4 ? 4 : 8; }

// Boundary values of the variant: the fewest that hold the problem's.  Most windows of five and more micro-batches on up to four devices have
// 9 to 16.  With room for 24, which the registers do not hold without spills in the sweeps, 2^20 candidates of a pipeline at eight
// micro-batches take 198 us on two devices and 485 on four, with room for 16 172 and 435.  Two devices have 17 values at most (three chains at
// five micro-batches, five at three).  By the variant for four devices 2^21 candidates take 796 us with repair, 516 without and 616 in a canonical
// range, with room for 24 on two 428, 273 and 411.  (2^21 of the X-shape on three devices: 658 and 1,015 us at
// three and four micro-batches, 367 and 639 now: there the general kernel had to find periods that the longer search settles.)
template <int MODE, bool PAIRS = false>
static fast_fn pick_fast_mode(const KParams &kp)
{
    const int V = kp.nsweeps - 1;
    switch (fast_dm(kp)) {
    case 2: return V <= 4 ? eval_fast_kernel<2, 4, MODE, false, PAIRS> : V <= 16 ? eval_fast_kernel<2, 16, MODE, false, PAIRS> : eval_fast_kernel<2, 24, MODE, false, PAIRS>;
    case 4: return V <= 8 ? eval_fast_kernel<4, 8, MODE, false, PAIRS> : V <= 16 ? eval_fast_kernel<4, 16, MODE, false, PAIRS> : eval_fast_kernel<4, 24, MODE, false, PAIRS>;
    default: return V <= 16 ? eval_fast_kernel<8, 16, MODE, false, PAIRS> : eval_fast_kernel<8, 24, MODE, false, PAIRS>;
    }
}

static fast_fn pick_fast(const KParams &kp)
{
    const int V = kp.nsweeps - 1;
    if (!kp.fast_ok) return nullptr;
    if (kp.fast_tp) {
        // blocks on several devices
        if (kp.space == kSampledRepair)
            return kp.D <= 2 ? (V <= 10 ? eval_fast_kernel<2, 10, 2, true> : eval_fast_kernel<2, 24, 2, true>)
                 : kp.D <= 4 ? (V <= 8 ? eval_fast_kernel<4, 8, 2, true> : eval_fast_kernel<4, 24, 2, true>)
                             : (V <= 16 ? eval_fast_kernel<8, 16, 2, true> : eval_fast_kernel<8, 24, 2, true>);
        if (kp.space == kSampledStrict)
            return kp.D <= 2 ? eval_fast_kernel<2, 24, 1, true> : kp.D <= 4 ? eval_fast_kernel<4, 24, 1, true> : eval_fast_kernel<8, 24, 1, true>;
        return kp.D <= 2 ? eval_fast_kernel<2, 24, 0, true> : kp.D <= 4 ? eval_fast_kernel<4, 24, 0, true> : eval_fast_kernel<8, 24, 0, true>;
    }
    return kp.space == kSampledRepair ? pick_fast_mode<2>(kp) : kp.space == kSampledStrict ? pick_fast_mode<1>(kp) : pick_fast_mode<0>(kp);
}

// Whether a launch looks its candidates up in tables of the orders that go together (order_pairs_kernel), and for how many lead vectors
// from which on.  Tables and a launch for them cost a call 8 to 12 us, and a bit as much as a candidate that gets far: calls of 2^18 candidates
// take 30 to 59 us without them and 30 to 65 with (pipelines of 3 to 8 devices, two to five micro-batches), of 2^20 56 to 81 and 29 to 71;
// 2^22 candidates 147 and 150 us where the tables have 1.7 M bits (924 orders on each of three devices), 2^24 497 and 156.
constexpr uint64_t kPairCandidates = 1u << 19;
static uint32_t pair_leads(const KParams &kp, uint64_t first, uint64_t count, uint32_t &lead0)
{
    lead0 = 0;
    if (kp.npairs == 0 || kp.cdev[0] < 2) return 0;
    uint64_t orders = 1;
    for (int d = 0; d < kp.D; d++)
        if (__builtin_mul_overflow(orders, kp.cdev[d], &orders)) return 0;
    const uint64_t l0 = first / orders, n = (first + count - 1) / orders - l0 + 1;
    if ((first + count - 1) / kp.cdev[0] >= 0xFFFFFFFFull || n * kp.pair_words > kp.pair_room) return 0;
    int always = 0;
    if (const char *env = getenv("TESSEL_PAIRS")) {                 // tuning knob
        if (atoi(env) == 0) return 0;
        always = 1;
    }
    if (!always && (count < kPairCandidates || n * kp.pair_bits * 4 > count)) return 0;
    lead0 = (uint32_t)l0;
    return (uint32_t)n;
}

// How eval_fast_kernel shares the units of such a launch out: a lane's lie one behind the other, those of a wave's lanes at equal distances.
// Where that distance comes back to nearly the same order of the second device with every lane, every second or third, the lanes start at
// places without an order instead (2,000,003 candidates of 252 orders a device, 378 of them between lanes: 194 -> 117 us and 246 -> 143 on three
// and four devices, 171 and 223 without tables).  Equal distances are better by up to 15 % otherwise, and with few orders there is no
// telling (0.89 to 1.12).
static uint32_t scatter_units(const KParams &kp, uint64_t first, uint64_t count, uint32_t blocks)
{
    const uint64_t n0 = kp.cdev[0], words = (n0 + 31) / 32, units = ((first + count - 1) / n0 - first / n0 + 1) * words;
    const uint64_t lanes = std::min<uint64_t>((units + blocks - 1) / blocks, kWave), apart = (units + lanes - 1) / lanes;
    const uint64_t turn = kp.cdev[1] * words;
    if (turn <= 512) return 0;
    for (uint64_t k = 1; k <= 3; k++) {
        const uint64_t off = apart * k % turn;
        if (std::min(off, turn - off) < turn / 16) return 1;
    }
    return 0;
}

// state and program of the general kernel's lanes: in LDS, except for wide problems that 64 KB do not hold
// (the LDS one workgroup may ask for: what the device reports, 64 KB where there is none to ask)
static size_t lds_per_workgroup()
{
    static size_t cap = 0;
    if (!cap) {
        int dev = 0, v = 0;
        if (hipGetDevice(&dev) == hipSuccess && hipDeviceGetAttribute(&v, hipDeviceAttributeMaxSharedMemoryPerBlock, dev) == hipSuccess &&
            v >= 64 * 1024)
            cap = (size_t)v < (size_t)160 * 1024 ? (size_t)v : (size_t)160 * 1024;
        else {
            (void)hipGetLastError();
            cap = 64 * 1024;
        }
    }
    return cap;
}
constexpr size_t kLdsAllBytes = 20 * 1024;       // state and program in LDS up to this much per workgroup (8 workgroups per CU)
constexpr size_t kLdsStateBytes = 40 * 1024;     // the state alone up to this much (4 per CU)
// Where the lanes' state and program of a wide problem live: 0 = in LDS, 1 = the program in the workspace, 2 = both.
// (TESSEL_FAR_MODE: tuning knob, honoured where the LDS allows it.)
static int far_mode(const KParams &kp)
{
    if (!wide_problem(kp)) return 0;
    const size_t tables = (size_t)5 * kMaxKW * 4, state = (size_t)kp.nslots * kWave * 4, prog = (size_t)kp.total * kWave * 2;
    int mode = tables + state + prog <= kLdsAllBytes ? 0 : tables + state <= kLdsStateBytes ? 1 : 2;
    if (const char *env = getenv("TESSEL_FAR_MODE")) {
        const int want = atoi(env);
        if (want == 2 || (want == 1 && tables + state <= lds_per_workgroup()) || (want == 0 && tables + state + prog <= lds_per_workgroup()))
            mode = want;
    }
    if (mode == 0 && tables + state + prog > lds_per_workgroup()) mode = 1;
    if (mode == 1 && tables + state > lds_per_workgroup()) mode = 2;
    return mode;
}
static size_t far_bytes(const KParams &kp) { return far_words(kp, far_mode(kp)) * 4; }

static size_t general_lds_bytes(const KParams &kp)
{
    if (wide_problem(kp)) {
        const int where = far_mode(kp);
        return (size_t)5 * kMaxKW * 4 + (where == 2 ? 0 : (size_t)kp.nslots * kWave * 4) + (where ? 0 : (((size_t)kp.total * kWave * 2 + 255) & ~(size_t)255));
    }
    return (size_t)4 * kMaxK * 4 + (size_t)kp.nslots * kWave * 4 + (size_t)kp.total * kWave * 2;
}

static size_t fast_lds_bytes(const KParams &kp)
{
    const int ntok = kp.nslots - kp.D;
    const bool share = fast_dm(kp) * 2 + ntok <= fast_dm(kp) * 4;
    return (size_t)(kFastTableWords + (kp.fast_tp ? kTpTableWords : 0)) * 4 + (size_t)fast_dm(kp) * kWave * 16 +
           (share ? 0 : (size_t)(fast_dm(kp) * 2 + ntok) * kWave * 4);
}

// Workgroups whose LDS a CU holds: it is given out in pieces of 1,280 bytes.  (The runtime's occupancy call counts finer.  With 13 workgroups of 12,288
// bytes for each CU, where 12 fit, the last 256 began when the others had ended: 2^21 candidates of 30 blocks, ten of them on two of three
// devices, 926 us, with 12 592.)
static int lds_blocks(size_t lds_bytes) { return (int)(160 * 1024 / 1280 / ((std::max<size_t>(lds_bytes, 1) + 1279) / 1280)); }

// resident workgroups per CU by LDS and, as the runtime computes them, by registers, 16 at most
static int blocks_per_cu(const void *fn, size_t lds_bytes)
{
    int per_cu = 0;
    if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, fn, kWave, lds_bytes) != hipSuccess || per_cu < 1) {
        (void)hipGetLastError();
        per_cu = 16;
    }
    per_cu = std::min({per_cu, lds_blocks(lds_bytes), 16});
    if (const char *env = getenv("TESSEL_BLOCKS_PER_CU")) {        // tuning knob: fewer resident workgroups per CU
        int want = atoi(env);
        if (want >= 1 && want < per_cu) per_cu = want;
    }
    return per_cu < 1 ? 1 : per_cu;
}

static int general_blocks_per_cu(const KParams &kp)
{
    const int per_cu = blocks_per_cu((const void *)pick_kernel(kp), general_lds_bytes(kp));
    return far_mode(kp) == 2 && per_cu > 4 ? 4 : per_cu;             // (keeps the state regions of a launch small)
}

static size_t ring_offset(int records, int num_cus);

// Behind the graph kernel the general one gets the grid that it has where it scores a problem alone: there are problems
// whose periods the graph kernel's sweeps hardly ever settle (cycles whose time is no multiple of the windows they cross; 32
// chains of two blocks round a ring of 32 devices: none in 2^18), and on 64 workgroups these took 571 ms where the general kernel
// alone takes 45.  Workgroups beyond the list end at once.
LaunchShape eval_launch_shape(const KParams &kp, int num_cus, int max_blocks)
{
    LaunchShape s;
    s.threads = kWave;
    s.list_blocks = kDeferBlocks;
    if (fast_fn ff = pick_fast(kp)) {
        s.lds_bytes = fast_lds_bytes(kp);
        s.blocks = num_cus * blocks_per_cu((const void *)ff, s.lds_bytes);
    } else if (kp.graph_ok) {
        s.lds_bytes = kp.graph_lds;
        s.blocks = num_cus * blocks_per_cu(graph_kernel(kp), s.lds_bytes);
        s.list_blocks = num_cus * general_blocks_per_cu(kp);
    } else {
        s.lds_bytes = general_lds_bytes(kp);
        s.blocks = num_cus * general_blocks_per_cu(kp);
    }
    if (max_blocks > 0) {                                            // the library's own buffer: room for fewer
        if (s.blocks > max_blocks) s.blocks = max_blocks;
        if (kp.graph_ok && far_bytes(kp) > 0) {
            const size_t fit = (kScratchBytes - ring_offset(s.blocks + s.list_blocks, num_cus)) / far_bytes(kp);
            if ((size_t)s.list_blocks > fit) s.list_blocks = (int)fit;
        }
    }
    return s;
}

// Program words the fast kernel builds before the candidates that are still alive queue for the rest (most candidates
// that exceed the memory cap do so within the first blocks of the window).  Windows of ten words and more: 3 of 11, 6 of 22, 9 of
// 32, 12 of 43, between the best numbers under tight and under wide caps (against two sevenths rounded up to four: 0.96 to
// 1.00 of the time; smaller windows lose 5 to 10 % by a queue where most candidates fit, and gain as much where few do).
// With repair, when every candidate's peak is wanted, none leaves early: all of the window, no queue, on more than 4 devices where the
// last round of candidates is full to five eighths or the only one (160 to 256 blocks on 5 to 8 devices: 0.98 of the time in up to one
// round, 1.75, 2, 3 and 4 rounds; but 1.06, 1.04, 1.02 in 1.1, 1.3, 1.5 and 1.03, 1.02 in 2.1, 3.1, where the waves of a nearly empty round
// share less of the chip with the queue's phases).  On up to 4 devices, whose queue moves half the words, 0.98 to 1.07 without an order to
// it: they keep it.  Blocks on several devices: always (0.94 to 0.99).
// Blocks on several devices, with repair, by the rounds of candidates that a wave of the grid has.  (Geometric means over 2 to 8
// devices, 2 to 4 micro-batches, five caps, blocks on all devices or two; windows of 3 to 12 words.)
//   windows below ten words: all of the window in one round, else two words, whose steps are the dearest: 0.98 of the time of all
//   of it in one round (0.74 to 1.10), 0.92 in 1.15 rounds, 0.79 in four, 0.69 in eleven; under caps that all candidates
//   meet 1.02 to 1.05
//   ten words and more: two sevenths rounded up to four words in up to two rounds, where a second phase for a few
//   candidates of a wave takes as long as for 64 (two words: 1.15, at worst 1.9 of the time; all of it 1.4), else two words (0.97 in 2.5
//   rounds, 0.78 in eleven)
//   24 rounds and more: with `adapt` the waves find the number themselves (against two words: 1.05 in 12 rounds, 1.01 in 16,
//   0.97 in 24, 0.90 in 60; the kernel says how)
// Blocks on several devices without repair: all of the window, since a wave stops when its last candidate is out anyway and
// the memory verdict has to wait (two words 1.00 to 1.05 of the time at 5,000 to 2,000,000 candidates).
static int stage_words(const KParams &kp, bool peaks, uint64_t count, int blocks, int &adapt)
{
    const int nwords = (kp.total + 5) / 6;
    adapt = 0;
    if (const char *env = getenv("TESSEL_STAGE_WORDS")) {           // tuning knob
        const int want = atoi(env);
        if (want >= 0 && want <= nwords) return want;
    }
    const uint64_t round = (uint64_t)blocks * kWave;
    if (peaks && kp.space == kSampledRepair && (kp.fast_tp || (kp.D > 4 && (count <= round || 8 * ((count - 1) % round + 1) >= 5 * round))))
        return nwords;
    if (kp.fast_tp) {
        if (kp.space != kSampledRepair) return nwords;
        adapt = count >= 24 * round;
        if (nwords < 10) return nwords > 2 && count > round ? 2 : nwords;
        return count > 2 * round ? 2 : (nwords * 2 / 7 + 3) / 4 * 4;
    }
    return nwords >= 10 ? 3 + (nwords - 10) * 9 / 33 : nwords;
}

// the rings of the fast kernel's waves lie behind the block records, two per wave; words of one ring
static uint32_t ring_words(const KParams &kp)
{
    const int nwords = (kp.total + 5) / 6;
    const int program = (nwords + 3) / 4 * 4 + kRingMetaWords;
    const int stage = (nwords + 3) / 4 * 4 + kStageMetaWords + 4 * fast_dm(kp);     // any stage_words
    return (uint32_t)(program > stage ? program : stage) * kRingSlots;
}

// behind the records of one launch (one per workgroup of the scoring kernels), or one (smaller) per workgroup of the
// completion search, whose grid is 16 workgroups per compute unit at most
static size_t ring_offset(int records, int num_cus)
{
    const size_t eval = (size_t)records * sizeof(BlockRec), comp = (size_t)num_cus * 16 * sizeof(CompRec);
    return (kWsBlockRecOff + (eval > comp ? eval : comp) + 256 + 255) & ~(size_t)255;
}
static size_t ring_offset(const LaunchShape &s, int num_cus) { return ring_offset(s.blocks + s.list_blocks, num_cus); }

// what a workgroup of the scoring kernel owns behind the records: queues of the fast kernel, slots of the graph kernel, or
// state and program of the general one
static size_t block_bytes(const KParams &kp)
{
    return pick_fast(kp) ? (size_t)3 * ring_words(kp) * 4 : kp.graph_ok ? (size_t)kp.graph_slot_words * kGraphSlots * 4 : far_bytes(kp);
}

size_t eval_workspace_bytes(const KParams &kp, int num_cus, int max_blocks)
{
    const LaunchShape s = eval_launch_shape(kp, num_cus, max_blocks);
    // (state and program of the general kernel's workgroups lie where the graph kernel's slots lay: it runs afterwards)
    const size_t own = (size_t)s.blocks * block_bytes(kp), list = kp.graph_ok ? (size_t)s.list_blocks * far_bytes(kp) : 0;
    return ring_offset(s, num_cus) + (own > list ? own : list);
}

static int launch_general(const KParams &kp, void *ws, uint64_t first, uint64_t count, int blocks, BlockRec *recs,
                          int32_t *code, int32_t *peak, bool whole, uint32_t *far, int from_range, hipStream_t st)
{
    const int where = far_mode(kp);
    if (where && !far) return (int)hipErrorInvalidValue;
    eval_fn fn = pick_kernel(kp);
    const size_t lds = general_lds_bytes(kp);
    if (lds > 64 * 1024) {
        hipError_t e = hipFuncSetAttribute((const void *)fn, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
        if (e != hipSuccess) return (int)e;
    }
    hipLaunchKernelGGL(fn, dim3(blocks), dim3(kWave), lds, st, (const KParams *)((char *)ws + kWsParamsOff), first, count, recs, code, peak, whole, far,
                       where, (char *)ws, from_range);
    return (int)hipGetLastError();
}

// How the waves of the graph kernel take turns on their SIMD (take_turn), by the rounds of candidates that a wave of the grid has.  Time with
// turns by that without, geometric means over 55 chains and graphs, least and most in brackets (2^22 candidates of the K-shape 538 -> 480 us a
// call; 100,003 windows of 288 blocks on 12 devices, one round of three waves a SIMD, 260 -> 235):
//   12 or 16 waves a CU, all alike
//       up to 0.3 of a round 1.01 (the clock), 0.4 0.98, 0.75 to one 0.96 (0.92, 1.01)
//       the last round filled to five eighths and more 0.92 to 0.97 (0.89, 1.02)
//       4.2 rounds and more 0.96 to 0.92 (0.87, 1.03)
//   fewer than that in the last round, of 1.06 to 3.5: the waves with candidates in it are the oldest and ended sooner at one priority, but where few
//   candidates survive the build a round more is a build more, and the sweeps are for the end
//       seven eighths of the candidates and more survive: all alike 1.00 to 1.08 (0.92, 1.15), so not so, but
//           from 2 on, to a quarter, these first, the others in turns on the three steps below: 0.98 (0.93, 1.02) in 2.1 rounds, 0.94 in 3.2
//           more of it, these first, both by twos: 0.98 (0.96, 1.02) in 1.3 to 2.6 rounds, 0.99 in 3.5
//       fewer: all alike 0.97 (0.91, 1.02)
//       up to 1.25 rounds, whoever survives: all alike 1.06 (0.97, 1.15), these first and the others below during the first build alone 1.02 (0.95, 1.05),
//           which is known by its end only, so none
//   other numbers of waves, unlike on the SIMDs, or fewer: 0.99 to 1.01 (0.91, 1.11) up to four rounds, no order to it; all alike in more, 5 to 14 waves a
//       CU, 9 to 26 rounds: 0.97 (0.91, 1.02; 613 us with and 674 without, 568 and 603, 939 and 974)
static GraphTurns graph_turns(uint64_t count, int blocks, int num_cus)
{
    const uint64_t round = (uint64_t)blocks * kWave, last = (count - 1) % round + 1;
    constexpr uint32_t alike = turns_of(3, 3, 0);
    constexpr uint32_t first = turns_of(0, 0, 3), below = turns_of(3, 2, 0);
    if (count > 4 * round && blocks > 4 * num_cus) return {0, alike, alike, alike, alike};
    if (blocks < 12 * num_cus || blocks % (4 * num_cus) != 0 || 3 * count < round) return {0, 0, 0, 0, 0};
    if (count <= round || 8 * last >= 5 * round) return {0, alike, alike, alike, alike};
    const uint32_t more = (uint32_t)((last + kWave - 1) / kWave);
    if (4 * last > round) return {more, turns_of(1, 1, 2), turns_of(1, 1, 0), alike, alike};
    if (count < 2 * round) return {0, 0, 0, 0, 0};
    return {more, first, below, alike, alike};
}

// Scores [first, first+count).  Where the problem allows it: the fast kernel (a short eigenvector search, a longer one
// for the candidates that did not converge) or the graph kernel, then the general kernel over what these could not finish (next
// to nothing in most problems).  Otherwise the general kernel alone.  `recs` may be null: per-candidate outputs only.
// Returns 0 or a HIP error.
static int launch_pass(const KParams &kp, uint64_t first, uint64_t count, void *ws, int num_cus, int max_blocks, BlockRec *recs,
                       int32_t *code, int32_t *peak, bool general, hipStream_t st)
{
    const KParams *kp_dev = (const KParams *)((char *)ws + kWsParamsOff);
    DevResult *res = (DevResult *)((char *)ws + kWsResultOff);
    uint64_t *list = (uint64_t *)((char *)ws + kWsListOff);
    uint32_t *left_after = (uint32_t *)((char *)ws + kWsLeftOff);
    const LaunchShape s = eval_launch_shape(kp, num_cus, max_blocks);
    const uint64_t need = (count + kWave - 1) / kWave;
    const int blocks = need < (uint64_t)s.blocks ? (int)need : s.blocks;
    const int list_blocks = need < (uint64_t)s.list_blocks ? (int)need : s.list_blocks;
    if (blocks < 1) return 0;
    uint32_t *behind = (uint32_t *)((char *)ws + ring_offset(s, num_cus));      // queues, slots, or the general kernel's state
    fast_fn ff = general ? nullptr : pick_fast(kp);
    const bool graph = !ff && kp.graph_ok && !general;
    if (!ff && !graph) {
        int rc = launch_general(kp, ws, first, count, blocks, recs, code, peak, false, behind, -1, st);
        if (rc || !recs) return rc;
        hipLaunchKernelGGL(merge_kernel, dim3(1), dim3(kMergeThreads), 0, st, recs, blocks, res);
        return (int)hipGetLastError();
    }
    int rc;
    if (graph) {
        // (every problem its tables hold: on 24 blocks of three devices 4.5 times the general kernel's rate, on 96 to 288
        // blocks 34 to 78 times; one to 4,096 scores of 6 to 12 blocks 33 to 54 us against 39 to 82)
        rc = launch_graph(kp, first, count, blocks, recs, code, peak, ws, behind, graph_turns(count, s.blocks, num_cus), st);
    } else {
        int adapt = 0;
        int stage = stage_words(kp, peak != nullptr, count, s.blocks, adapt);
        uint32_t lead0 = 0;
        const uint32_t leads = code ? 0u : pair_leads(kp, first, count, lead0);
        if (leads) {
            const uint32_t chunks = leads * (kp.pair_words / 2);
            const int dm = fast_dm(kp);
            const pairs_fn pf = dm == 2 ? order_pairs_kernel<2> : dm == 4 ? order_pairs_kernel<4> : order_pairs_kernel<8>;
            hipLaunchKernelGGL(pf, dim3(std::min<uint32_t>(chunks, (uint32_t)num_cus * 12u)), dim3(kWave),
                               (size_t)kFastTableWords * 4 + (size_t)fast_dm(kp) * kWave * 16, st, kp_dev, lead0, chunks, kp.pair_tab);
            rc = (int)hipGetLastError();
            if (rc) return rc;
            stage = (kp.total + 5) / 6;                             // (what is left mostly runs to the end)
        }
        if (leads) ff = pick_fast_mode<0, true>(kp);
        hipLaunchKernelGGL(ff, dim3(blocks), dim3(kWave), fast_lds_bytes(kp), st, kp_dev, first, count, recs, code, peak, kp.eigen_tries,
                           kp.retry_tries, list, &res->defer_count, kWsListCap, &res->overflow, behind, ring_words(kp), stage, adapt, left_after,
                           leads ? kp.pair_tab : nullptr, lead0, leads ? scatter_units(kp, first, count, (uint32_t)blocks) : 0u);
        rc = (int)hipGetLastError();
    }
    if (rc) return rc;
    return launch_general(kp, ws, first, count, list_blocks, recs ? recs + blocks : nullptr, code, peak, graph, graph ? behind : nullptr,
                          recs ? blocks : 0, st);
}

int launch_eval(const KParams &kp, uint64_t first, uint64_t count, void *ws, int num_cus, int max_blocks, void *stream, uint64_t max_piece)
{
    BlockRec *recs = (BlockRec *)((char *)ws + kWsBlockRecOff);
    // pieces of at most max_piece candidates, so that the lists of unfinished candidates stay small
    for (uint64_t done = 0; done < count;) {
        const uint64_t piece = count - done < max_piece ? count - done : max_piece;
        int rc = launch_pass(kp, first + done, piece, ws, num_cus, max_blocks, recs, nullptr, nullptr, false, (hipStream_t)stream);
        if (rc) return rc;
        done += piece;
    }
    return 0;
}

int launch_score(const KParams &kp, uint64_t first, uint64_t count, int32_t *code, int32_t *peak, void *ws, int num_cus,
                 int max_blocks, bool general, void *stream)
{
    // pieces in which no list can overflow: the per-candidate outputs of a dropped candidate would stay unwritten
    const uint64_t max_piece = kSafePerLaunch;
    for (uint64_t done = 0; done < count;) {
        const uint64_t piece = count - done < max_piece ? count - done : max_piece;
        int rc = launch_pass(kp, first + done, piece, ws, num_cus, max_blocks, nullptr, code + done, peak ? peak + done : nullptr, general,
                             (hipStream_t)stream);
        if (rc) return rc;
        done += piece;
    }
    return 0;
}

int launch_reset(void *ws, void *stream)
{
    hipLaunchKernelGGL(reset_kernel, dim3(1), dim3(1), 0, (hipStream_t)stream, (DevResult *)((char *)ws + kWsResultOff),
                       (uint32_t *)((char *)ws + kWsLeftOff));
    return (int)hipGetLastError();
}

size_t block_rec_bytes(int blocks) { return (size_t)blocks * sizeof(BlockRec); }

// ------------------------------------------------------------------ a workspace the library holds itself
// For callers that cannot allocate device memory: one buffer per GPU, part of the code object, shared by every call
// on that GPU (it keeps the last call's contents; the kernels clear what has to start at zero).  In host code the
// array's name stands for the symbol, not for device memory: its address on the current device comes from
// hipGetSymbolAddress, once per device.
static __device__ __align__(256) __attribute__((used)) unsigned char scratch[kScratchBytes];

int scratch_workspace(void **ptr, size_t *bytes)
{
    constexpr int kMaxGpus = 64;
    static void *address[kMaxGpus] = {};
    int dev = 0;
    hipError_t e = hipGetDevice(&dev);
    if (e != hipSuccess) return (int)e;
    if (dev < 0 || dev >= kMaxGpus) return (int)hipErrorInvalidDevice;
    if (!address[dev]) {
        void *p = nullptr;
        e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
        if (e != hipSuccess) return (int)e;
        if (!p) return (int)hipErrorInvalidSymbol;
        address[dev] = p;
    }
    *ptr = address[dev];
    *bytes = kScratchBytes;
    return 0;
}

// the largest grid of the scoring kernels whose records and queues fit `bytes`; 0: not even one workgroup
int eval_blocks_that_fit(const KParams &kp, int num_cus, size_t bytes)
{
    const size_t per_block = sizeof(BlockRec) + block_bytes(kp);
    const size_t fixed = ring_offset(eval_launch_shape(kp, num_cus, 0).list_blocks, num_cus) + 512;
    if (bytes < fixed + per_block) return 0;
    int blocks = (int)std::min<size_t>((bytes - fixed) / per_block, (size_t)num_cus * 16);
    while (blocks > 0 && eval_workspace_bytes(kp, num_cus, blocks) > bytes) blocks--;
    return blocks;
}


// ==================================================================== searched completion
// Warm-up and cool-down around R copies of the best window (Sec. IV-C).  The paper orders the two outer
// phases with a time-optimal solver; here many perturbed greedy list schedules are tried, one per lane,
// and the shortest complete schedule wins.  Completion candidate `ordinal`: per phase every block type
// offers its lowest unscheduled micro-batch (Property 1); an offered block is eligible when its producer's
// block of the same micro-batch is scheduled and its memory delta fits on all its devices; the eligible
// block with the smallest (earliest start + jitter, micro-batch, type id) is appended at its earliest
// start.  jitter(type, mu) = (draw * (J + 1)) >> 16 with draw number type*N + mu of the stream keyed by the
// ordinal; ordinal 0 has no jitter (the plain greedy schedule).
// ---- every type on one device, chains, at most eight of them (all pipeline placements without tensor parallelism) ----------------
// One lane a candidate; all lanes of a wave place the same number of blocks a phase, one a step.  Per lane, in LDS [row][lane]:
//   offer  per block type (rows by device and symbol): the block it offers, as the sort key it has by its producer alone, (end of
//          the producer's block + jitter) << 15 | micro-batch << 5 | type; bit 31: its producer has not handled that micro-batch;
//          all ones: nothing left to offer in this phase
//   device free time (16 bits) | memory << 16; the jitters of the blocks its types offer, a byte each; the smallest key of its types
//   token  end times of the micro-batches in flight, a ring a chain, 16 bits
// The key of an offer is max(offer, (free time + jitter) << 15 | the same low bits), with bit 31 where its memory does not fit.  A
// step changes the keys of the block's own device, worked out anew (four at most), and the offer of its consumer, if that waits
// for this very micro-batch: with the block's end and the jitter it has already.  So a pick is the smallest of eight words, not of the
// keys of all types, which were kept in LDS before and of which a step changed up to five.  It is known when the step ends: the
// smallest keys of the other devices and the offers of the block's own are read with the rest of the state, the block's own words all
// ones by then, and its new ones and the consumer's key join them in registers.
// Bound by vector issue at two waves a SIMD (LDS: 17.7 KB a wave for 8 devices and 32 types): 116 vector instructions and two rounds of LDS
// reads a step (table words; state).  With five rounds (smallest keys, table words, state, offers, all in a row) the same time, until the waves
// of a SIMD took turns, see below.  2^20 candidates of 64 micro-batches on 8 devices, as a call: 2.47 ms with a key a type, 1.38 with a key a device,
// 1.32 with turns, 1.23 with two rounds as well.
template <int DM, int SY>
struct ChainRows {
    static constexpr uint32_t kRowB = kWave * 4u;
    static constexpr uint32_t types = 0, more = 512, room = 640, init = 768, mpos = 896, rows = 1024;     // tables: by type (three), by code, by device
    static constexpr uint32_t least = rows, dev = least + DM * kRowB, jit = dev + DM * kRowB, offer = jit + DM * kRowB;
    static constexpr uint32_t ones = offer + DM * SY * kRowB, token = ones + kRowB;
};

template <int DM, int SY>
__global__ __launch_bounds__(kWave) void complete_chain_kernel(const CompParams *__restrict__ cpg, const CompMatrix *__restrict__ cmg,
                                                               uint64_t first, uint64_t count, CompRec *__restrict__ recs,
                                                               int32_t *__restrict__ makespan_out)
{
    typedef ChainRows<DM, SY> L;
    extern __shared__ uint32_t lds[];
    const int lane = threadIdx.x;
    // (all LDS addresses below are offsets from 0: nothing else of the kernel lies in front of this array)
    if (lds_address(lds) != 0u) {
        if (recs && lane == 0) { recs[blockIdx.x].makespan = INT_MAX; recs[blockIdx.x].ordinal = ~0ull; }
        return;
    }
    const uint32_t lane4 = (uint32_t)lane * 4u, lane2 = (uint32_t)lane * 2u;
    const int D = cpg->D, K = cpg->K, N = cpg->N, NR = cpg->NR, M = cpg->M, J = cpg->J, R = cpg->R, TR = cpg->tok_ring, nseq = cpg->nseq;
    const uint32_t ring_rows = (uint32_t)(cpg->npaths * TR), tmask = (uint32_t)(TR - 1) << 7, tring = (uint32_t)(TR - 1) << 5, oFree = ring_rows;
    const uint32_t seed_lo = cpg->seed_lo, seed_hi = cpg->seed_hi;
    const uint32_t replay = L::token + ((ring_rows * (uint32_t)(kWave * 2) + 255u) & ~255u);      // words of the windows' blocks (no matrix)
    const int nin = cmg->nin, nout = cmg->nout;
    // ---- tables, a type a lane (the parameter block is read from a copy behind the tables)
    uint32_t my_lead = 0, my_more = 0;
    {
        uint32_t *copy = lds + L::rows / 4;
        for (int w = lane; w < (int)(sizeof(CompParams) / 4); w += kWave) copy[w] = ((const uint32_t *)cpg)[w];
        for (int w = lane; w < (int)(L::rows / 4); w += kWave) lds[w] = 0;
        __syncthreads();
        const CompParams &cp = *(const CompParams *)copy;
        auto device_of = [&](int i) -> uint32_t { return (uint32_t)__builtin_ctz((uint32_t)cp.mask[i]); };
        auto symbol_of = [&](int i) -> uint32_t { uint32_t y = 0; for (int j = 0; j < i; j++) y += cp.mask[j] == cp.mask[i] ? 1u : 0u; return y; };
        auto offer_of = [&](int i) -> uint32_t { return L::offer + (device_of(i) * SY + symbol_of(i)) * L::kRowB; };
        if (lane < K) {
            const int i = lane, a = cp.pred[i];
            int c = -1;
            for (int j = 0; j < K; j++) if (cp.pred[j] == i) c = j;
            const uint32_t d = device_of(i), y = symbol_of(i);
            lds[L::types / 4 + 4 * i] = (d << 8) | ((uint32_t)cp.path[i] * (uint32_t)TR * (uint32_t)(kWave * 2) + L::token) << 16;
            lds[L::types / 4 + 4 * i + 1] = (uint32_t)cp.t[i] | (uint32_t)cp.m[i] << 16;
            lds[L::types / 4 + 4 * i + 2] = offer_of(i) | (c >= 0 ? offer_of(c) : L::ones) << 16;
            lds[L::types / 4 + 4 * i + 3] = (uint32_t)max(c, 0) | (c >= 0 ? device_of(c) << 8 | 8u * symbol_of(c) << 16 : 0u) | 8u * y << 24 | (a >= 0 ? 1u << 30 : 0u);
            // (goes to `more` when a phase starts, with the micro-batches the phase has of the type, times 32)
            my_more = (a >= 0 ? offer_of(a) : L::ones) | (c >= 0 ? (uint32_t)max((int)cp.m[c], 0) : 0u);
            my_lead = (uint32_t)cp.lead[i];
            atomicOr(&lds[L::mpos / 4 + d], (uint32_t)max((int)cp.m[i], 0) << (8u * y));
            // by code: type, lead, no producer, its micro-batch after the windows is there already, a type
            lds[L::init / 4 + d * SY + y] = (uint32_t)i | (uint32_t)cp.lead[i] << 8 | (a < 0 ? 1u << 16 : 0u) |
                                            (a < 0 || cp.lead[a < 0 ? 0 : a] > cp.lead[i] ? 1u << 17 : 0u) | 1u << 18;
        }
        if (nin == 0) {
            // one word per block of the window: device (3 bits), micro-batch within the first window (8), chain (3), has a producer, t (16)
            for (int s = lane; s < nseq; s += kWave) {
                const int i = cp.seq[s];
                lds_store(replay + 4u * (uint32_t)s, device_of(i) | ((uint32_t)cp.lead[i] + (uint32_t)cp.occ[s]) << 3 | (uint32_t)cp.path[i] << 11 |
                                                     (cp.pred[i] >= 0 ? 1u << 14 : 0u) | (uint32_t)cp.t[i] << 16);
            }
        }
        __syncthreads();
        if (lane < K) lds[L::room / 4 + lane] = lds[L::mpos / 4 + device_of(lane)];      // what the types of its device ask for
        __syncthreads();
    }
    auto uniform_word = [&](uint32_t a) -> uint32_t { return (uint32_t)__builtin_amdgcn_readfirstlane((int)lds_load(a)); };
    // What the start of a phase goes by, a word a lane: by code, by type, by device.  (A phase visits the codes that block types have.  All of a
    // device's codes with their words read from LDS one by one: 1 to 4 us of a call of 20 us for problems with fewer types than that.)
    const uint32_t by_code = lane < DM * SY ? lds_load(L::init + lane4) : 0u, by_type = lane < K ? lds_load(L::types + 4u * lane4) : 0u,
                   by_dev = lane < DM ? lds_load(L::mpos + lane4) : 0u;
    auto word_of = [](uint32_t words, uint32_t of) -> uint32_t { return (uint32_t)__builtin_amdgcn_readlane((int)words, (int)of); };
    const uint32_t codes = (uint32_t)__ballot(by_code != 0u);
    for (uint32_t k = 0; k < (uint32_t)(DM * SY); k++) lds_store(L::offer + k * L::kRowB + lane4, ~0u);
    lds_store(L::ones + lane4, ~0u);
    int best = INT_MAX;
    uint64_t best_ord = 0;
    const uint64_t stride = (uint64_t)gridDim.x * kWave;
    const uint64_t rounds = (count + stride - 1) / stride;          // the same trip count for every lane of the grid
    const uint32_t slot = __builtin_amdgcn_s_getreg((3 << 11) | 4);     // the wave's place on its SIMD (bits 0 to 3 of HW_ID)
    for (uint64_t r = 0; r < rounds; r++) {
        const uint64_t kk = r * stride + (uint64_t)blockIdx.x * kWave + lane;
        const bool live = kk < count;
        const uint64_t c = first + (live ? kk : 0);                 // (a lane past the end scores the first candidate and drops it)
        uint32_t kb;
        const uint32_t ka = stream_keys(((uint64_t)seed_hi << 32) | seed_lo, c, kb);
        const uint32_t jmul = c != 0 ? (uint32_t)(J + 1) : 0u;      // ordinal 0 has no jitter
        auto jitter = [&](uint32_t n) -> uint32_t { return __umul24(stream_draw16(ka, kb, n), jmul) >> 16; };
        for (uint32_t s = 0; s < ring_rows; s++) lds_store16(L::token + s * (kWave * 2u) + lane2, 0u);
        for (int d = 0; d < DM; d++) { lds_store(L::dev + (uint32_t)d * L::kRowB + lane4, 0u); lds_store(L::least + (uint32_t)d * L::kRowB + lane4, ~0u); }
        bool fail = false;
        // an offer's key: not before its device is free (jitter included); bit 31 where the memory left is below 0
        auto key_of = [](uint32_t o, uint32_t from, int room) -> uint32_t {
            return __builtin_amdgcn_bitop3_b32((uint32_t)room, 0x80000000u, max(o, from << 15 | (o & 0x7FFFu)), 0xEA);
        };
        // the smallest key of a device's offers: free time, jitters, memory left (not below 0)
        auto least_key = [&](const uint32_t *o, uint32_t fr, uint32_t jits, int room, uint32_t mp) -> uint32_t {
            uint32_t low = ~0u;
#pragma unroll
            for (int y = 0; y < SY; y++) low = min(low, key_of(o[y], fr + (jits >> (8 * y) & 255u), room - (int)(mp >> (8 * y) & 255u)));
            return low;
        };
        for (int phase = 0; phase < 2; phase++) {
            // ---- what every type offers at first: warm-up from micro-batch 0, cool-down from where the windows end
            int left = 0;                                           // blocks of this phase
            if (lane < K) lds_store(L::more + lane4, my_more | (phase ? (uint32_t)N : my_lead) << 21);
            for (uint32_t rest = codes; rest;) {
                const uint32_t d = (uint32_t)__builtin_ctz(rest) / SY, mine = rest >> (d * SY) & ((1u << SY) - 1u), dd = d * L::kRowB + lane4;
                uint32_t jits = 0;
                rest ^= mine << (d * SY);
                for (uint32_t y = 0; mine >> y; y++) {              // (a device's symbols start at 0)
                    const uint32_t I = word_of(by_code, d * SY + y);
                    const uint32_t id = I & 31u, lead = I >> 8 & 255u, mu = phase ? lead + (uint32_t)(NR * R) : 0u, hi = phase ? (uint32_t)N : lead;
                    uint32_t o = ~0u;
                    if (mu < hi) {
                        left += (int)(hi - mu);
                        const uint32_t j = jitter(id * (uint32_t)N + mu);
                        jits |= j << (8u * y);
                        const bool there = I >> (phase ? 17 : 16) & 1u;
                        const uint32_t from = I >> 16 & 1u ? 0u : lds_load16((word_of(by_type, id) >> 16) + (mu << 7 & tmask) + lane2);
                        o = (there ? (from + j) << 15 : 0x80000000u) | mu << 5 | id;
                    }
                    lds_store(L::offer + (d * SY + y) * L::kRowB + lane4, o);
                }
                lds_store(L::jit + dd, jits);
                const uint32_t fm = lds_load(L::dev + dd);
                uint32_t o[SY];
#pragma unroll
                for (int y = 0; y < SY; y++) o[y] = lds_load(L::offer + (d * SY + y) * L::kRowB + lane4);
                lds_store(L::least + dd, least_key(o, fm & 0xFFFFu, jits, max(M - ((int)fm >> 16), 0), word_of(by_dev, d)));
            }
            __syncthreads();
            // ---- a block a step
            auto least_of_all = [&]() -> uint32_t {
                uint32_t low = ~0u;
#pragma unroll
                for (int d = 0; d < DM; d++) low = min(low, lds_load(L::least + (uint32_t)d * L::kRowB + lane4));
                return low;
            };
            uint32_t pick = least_of_all();
            // (Sixteen steps at a time while some candidate of the wave still has a schedule: under a tight cap whole waves are stuck after a
            // few.  2^20 candidates of 250 blocks, all stuck: a call of 256 us without, 190 with it.  Looked at in every step it cost the others 8 %.)
            for (int from = 0; from < left && __ballot(live && (int)pick >= 0) != 0; from += 16) {
                // (the waves of a SIMD issue first in turns of 41 us.  All at the same priority, the older of two does: it was done after 1,010 us,
                // the younger after 1,350, alone on the SIMD for the rest.)
                if ((((uint32_t)__builtin_amdgcn_s_memrealtime() >> 12) + slot) & 1u) __builtin_amdgcn_s_setprio(1);
                else __builtin_amdgcn_s_setprio(0);
                for (int s = from; s < min(left, from + 16); s++) {
                    if ((int)pick < 0) continue;                        // blocks left, none eligible: the lane's state stays as it is
                    const uint32_t b = pick & 31u, low = pick & 0x7FE0u, low1 = low + 32u;
                    const uint32_t T0 = lds_load(L::types + 16u * b), T1 = lds_load(L::types + 16u * b + 4u), T2 = lds_load(L::types + 16u * b + 8u),
                                   T3 = lds_load(L::types + 16u * b + 12u), U = lds_load(L::more + 4u * b), mp = lds_load(L::room + 4u * b);
                    uint32_t jn = jitter(__umul24(b, (uint32_t)N) + (low1 >> 5));
                    TESSEL_PIN(jn);
                    // (second round: everything these words name)
                    const uint32_t dd = (T0 & 0xF00u) + lane4, cd = (T3 & 0xF00u) + lane4, ring = (T0 >> 16) + lane2, oc = (T2 >> 16) + lane4;
                    const uint32_t ob = (T2 & 0xFFFFu) + lane4, at = (T0 & 0xF00u) * SY + L::offer + lane4;
                    lds_store(L::least + dd, ~0u);
                    lds_store(ob, ~0u);
                    uint32_t fm = lds_load(L::dev + dd), jits = lds_load(L::jit + dd);
                    uint32_t off_c = lds_load(oc), fm_c = lds_load(L::dev + cd), jits_c = lds_load(L::jit + cd);
                    uint32_t off_p = lds_load((U & 0xFF00u) + lane4), tk = lds_load16(ring + ((low1 & tring) << 2));
                    uint32_t o[SY], others[DM];
#pragma unroll
                    for (int y = 0; y < SY; y++) o[y] = lds_load(at + (uint32_t)y * L::kRowB);
#pragma unroll
                    for (int d = 0; d < DM; d++) others[d] = lds_load(L::least + (uint32_t)d * L::kRowB + lane4);
                    TESSEL_PIN(fm); TESSEL_PIN(jits); TESSEL_PIN(off_c); TESSEL_PIN(fm_c); TESSEL_PIN(jits_c); TESSEL_PIN(off_p); TESSEL_PIN(tk);
                    const uint32_t yb = T3 >> 24 & 31u;
                    const uint32_t en = (pick >> 15) - (jits >> yb & 255u) + (T1 & 0xFFFFu);
                    const uint32_t fm_new = ((fm + (T1 & 0xFFFF0000u)) & 0xFFFF0000u) | en;
                    const uint32_t jits_new = (jits & ~(255u << yb)) | jn << yb;
                    // the type's next micro-batch: there if its producer's offer is beyond it (nothing left to offer: all ones)
                    const uint32_t from = T3 >> 30 & 1u ? tk : 0u, low_b = low1 | b;
                    const uint32_t there = (from + jn) << 15;
                    uint32_t off_b = ((off_p & 0x7FE0u) > low1 ? there : 0x80000000u) | low_b;
                    off_b = low1 >= U >> 16 ? ~0u : off_b;
                    lds_store(L::dev + dd, fm_new);
                    lds_store(L::jit + dd, jits_new);
                    lds_store16(ring + ((low & tring) << 2), en);
                    lds_store(ob, off_b);
                    const int room = max(M - ((int)fm_new >> 16), 0);
                    const uint32_t mine = min(least_key(o, en, jits_new, room, mp), key_of(off_b, en + jn, room - (int)(mp >> yb & 255u)));
                    lds_store(L::least + dd, mine);
                    // its consumer, if that waits for this block.  (No consumer: a row of all ones, which no block matches.)
                    {
                        const uint32_t jc = jits_c >> (T3 >> 16 & 31u) & 255u, low_c = off_c & 0x7FFFu;
                        const bool waits = off_c == (0x80000000u | low | (T3 & 31u));
                        const uint32_t now = (en + jc) << 15 | low_c;
                        lds_store(oc, waits ? now : off_c);
                        const uint32_t fm_now = cd == dd ? fm_new : fm_c;
                        uint32_t key = key_of(now, (fm_now & 0xFFFFu) + jc, max(M - ((int)fm_now >> 16), 0) - (int)(U & 127u));
                        TESSEL_PIN(key);
                        key = waits ? key : ~0u;
                        __hip_atomic_fetch_min((lds_word *)(uintptr_t)(L::least + cd), key, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
                        pick = min(mine, key);
#pragma unroll
                        for (int d = 0; d < DM; d++) pick = min(pick, others[d]);
                    }
                }
            }
            fail = fail | (pick != ~0u);                            // (what is left has a key, with bit 31; nothing left: all ones)
            __syncthreads();
            if (phase == 1 || __ballot(live && !fail) == 0) break;
            // ---- the R windows: the same blocks at the same micro-batches in every lane.  (Without the memory, which a whole
            // window leaves as it was: the deltas on a device sum to zero, and the window itself was scored against the cap.)
            auto slot_address = [&](uint32_t s) -> uint32_t {
                return s < oFree ? L::token + s * (kWave * 2u) + lane2 : L::dev + (s - oFree) * L::kRowB + lane4;
            };
            if (nin > 0) {
                // all R windows at once: every slot they write = max over the slots they read first of (value + longest path);
                // rows and slots are the same in every lane and come by scalar loads
                int x[kMatIn];
#pragma unroll
                for (int j = 0; j < kMatIn; j++) x[j] = j < nin ? (int)lds_load16(slot_address(cmg->in_slot[j])) : 0;
                for (int o = 0; o < nout; o++) {
                    int acc = 0;                         // (every output has a path from some input, and times are >= 0)
#pragma unroll
                    for (int j = 0; j < kMatIn; j++) acc = max(acc, x[j] + cmg->a[o][j]);
                    lds_store16(slot_address(cmg->out_slot[o]), (uint32_t)acc);
                }
            } else
                for (int w = 0; w < R; w++)
                    for (int s = 0; s < nseq; s++) {
                        const uint32_t rw = uniform_word(replay + 4u * (uint32_t)s);
                        const uint32_t mu = (rw >> 3 & 255u) + (uint32_t)(NR * w), fr = L::dev + (rw & 7u) * L::kRowB + lane4;
                        const uint32_t tok = L::token + (rw >> 11 & 7u) * (uint32_t)TR * (kWave * 2u) + (mu << 7 & tmask) + lane2;
                        uint32_t est = lds_load16(fr);
                        if (rw >> 14 & 1u) est = max(est, lds_load16(tok));
                        const uint32_t en = est + (rw >> 16);
                        lds_store16(fr, en);
                        lds_store16(tok, en);
                    }
            __syncthreads();
        }
        int makespan = 0;
        for (int d = 0; d < D; d++) makespan = max(makespan, (int)(lds_load(L::dev + (uint32_t)d * L::kRowB + lane4) & 0xFFFFu));
        if (fail) makespan = INT_MAX;
        if (live && makespan_out) makespan_out[kk] = makespan;
        if (live && (makespan < best || (makespan == best && c < best_ord))) { best = makespan; best_ord = c; }
    }
    if (!recs) return;
#pragma unroll
    for (int off = 32; off >= 1; off >>= 1) {
        int om = __shfl_xor(best, off);
        uint32_t ilo = __shfl_xor((uint32_t)best_ord, off), ihi = __shfl_xor((uint32_t)(best_ord >> 32), off);
        uint64_t oo = ((uint64_t)ihi << 32) | ilo;
        if (key_less(om, oo, best, best_ord)) { best = om; best_ord = oo; }
    }
    if (lane == 0) { CompRec rr; rr.makespan = best; rr.pad = 0; rr.ordinal = best_ord; recs[blockIdx.x] = rr; }
}

// ---- any other problem: blocks on several devices, graphs, more than eight chains ------------------------------------------
// Per lane, in LDS [row][lane]: per type the sort key that it has by its producers alone (as in the rows of chains; bit 31: some
// producer has not handled the micro-batch, all ones: nothing left to offer) and the same key without the producers' end, jitter << 15 |
// micro-batch << 5 | type; per device the free time << 15 and the memory left; the rings of end times, 16 bits, one a chain or, in graphs,
// one a consumed type.  So a type's key is the larger of its offer and one sum, and a step looks at the types of the phase four at a
// time, which no lane's choice delays; what the chosen block changes goes by its own tables (producers, consumers and devices as masks).
// (A scan with every type's producers, devices and memory read one after the other, a chain of reads a type, and all windows
// replayed block by block: 67,295 candidates of 38 micro-batches with two blocks on all of 8 devices 669 -> 177 us a call, 300,007 of 50 on
// the K-shape 341 -> 211, 1,000,003 of 64 on the diamond 2,877 -> 1,822.)
struct ScanRows {
    static constexpr uint32_t kRowB = kWave * 4u, kWords = 6, types = 0, rows = kWords * kMaxK * 4u;     // a word of the tables is at word * 4 kMaxK + 4 type
    __host__ __device__ static uint32_t devices(int K) { return rows + (uint32_t)K * 2u * kRowB; }
    __host__ __device__ static uint32_t token(int K, int D) { return devices(K) + (uint32_t)D * 2u * kRowB; }
    __host__ __device__ static uint32_t replay(int K, int D, int ring_rows) { return token(K, D) + (((uint32_t)ring_rows * (uint32_t)(kWave * 2) + 255u) & ~255u); }
};
static_assert(sizeof(CompParams) <= 4u * ScanRows::kRowB, "the parameter block's copy lies in the rows of two types");

__global__ __launch_bounds__(kWave) void complete_scan_kernel(const CompParams *__restrict__ cpg, const CompMatrix *__restrict__ cmg,
                                                              uint64_t first, uint64_t count, CompRec *__restrict__ recs,
                                                              int32_t *__restrict__ makespan_out)
{
    typedef ScanRows L;
    constexpr uint32_t kRowB = L::kRowB, kTab = 4u * kMaxK;
    extern __shared__ uint32_t lds[];
    const int lane = threadIdx.x;
    // (all LDS addresses below are offsets from 0: nothing else of the kernel lies in front of this array)
    if (lds_address(lds) != 0u) {
        if (recs && lane == 0) { recs[blockIdx.x].makespan = INT_MAX; recs[blockIdx.x].ordinal = ~0ull; }
        return;
    }
    const uint32_t lane4 = (uint32_t)lane * 4u, lane2 = (uint32_t)lane * 2u;
    const int D = cpg->D, K = cpg->K, N = cpg->N, NR = cpg->NR, M = cpg->M, J = cpg->J, R = cpg->R, TR = cpg->tok_ring, nseq = cpg->nseq;
    const uint32_t ring_rows = (uint32_t)(cpg->npaths * TR), tmask = (uint32_t)(TR - 1) << 7;
    const uint32_t seed_lo = cpg->seed_lo, seed_hi = cpg->seed_hi;
    const uint32_t devices = L::devices(K), token = L::token(K, D), replay = L::replay(K, D, (int)ring_rows);
    const int nin = cmg->nin, nout = cmg->nout;
    // ---- tables, a type a lane.  In LDS: 0 time, 1 producers, 2 consumers, 3 devices | memory delta << 16, 4 the ring it writes (0: none),
    // 5 micro-batches of the phase.  In registers, for what goes over all types: `info` devices | memory it asks for << 8 | lead << 16
    uint32_t info = 0, from_types = 0;
    {
        uint32_t *copy = lds + L::rows / 4;
        for (int w = lane; w < (int)(sizeof(CompParams) / 4); w += kWave) copy[w] = ((const uint32_t *)cpg)[w];
        __syncthreads();
        const CompParams &cp = *(const CompParams *)copy;
        uint32_t t = 0, m = 0, ring = 0, to_types = 0;
        if (lane < K) {
            const int i = lane;
            t = (uint32_t)cp.t[i]; m = (uint32_t)(int)cp.m[i];
            from_types = cp.dag ? cp.predmask[i] : cp.pred[i] >= 0 ? 1u << cp.pred[i] : 0u;
            for (int j = 0; j < K; j++)
                if (cp.dag ? cp.predmask[j] >> i & 1u : cp.pred[j] == i) to_types |= 1u << j;
            ring = cp.path[i] != 0xFF ? token + (uint32_t)cp.path[i] * (uint32_t)TR * (uint32_t)(kWave * 2) : 0u;
            info = (uint32_t)cp.mask[i] | (uint32_t)max((int)cp.m[i], 0) << 8 | (uint32_t)cp.lead[i] << 16;
        }
        if (nin == 0)
            for (int s = lane; s < nseq; s += kWave) {
                const int i = cp.seq[s];
                lds_store(replay + 4u * (uint32_t)s, (uint32_t)i | ((uint32_t)cp.lead[i] + (uint32_t)cp.occ[s]) << 8);
            }
        __syncthreads();
        if (lane < K) {
            lds_store(lane4, t); lds_store(lane4 + kTab, from_types); lds_store(lane4 + 2 * kTab, to_types);
            lds_store(lane4 + 3 * kTab, (info & 255u) | m << 16); lds_store(lane4 + 4 * kTab, ring);
        }
        __syncthreads();
    }
    const uint32_t times = lane < K ? lds_load(lane4) : 0u, rings = lane < K ? lds_load(lane4 + 4 * kTab) : 0u;
    auto word_of = [](uint32_t words, uint32_t of) -> uint32_t { return (uint32_t)__builtin_amdgcn_readlane((int)words, (int)of); };
    const uint32_t several = (uint32_t)__ballot(lane < K && (info & 255u & ((info & 255u) - 1u)) != 0u);       // types on several devices
    int best = INT_MAX;
    uint64_t best_ord = 0;
    const uint64_t stride = (uint64_t)gridDim.x * kWave;
    const uint64_t rounds = (count + stride - 1) / stride;          // the same trip count for every lane of the grid
    for (uint64_t r = 0; r < rounds; r++) {
        const uint64_t kk = r * stride + (uint64_t)blockIdx.x * kWave + lane;
        const bool live = kk < count;
        const uint64_t c = first + (live ? kk : 0);                 // (a lane past the end scores the first candidate and drops it)
        uint32_t kb;
        const uint32_t ka = stream_keys(((uint64_t)seed_hi << 32) | seed_lo, c, kb);
        const uint32_t jmul = c != 0 ? (uint32_t)(J + 1) : 0u;      // ordinal 0 has no jitter
        auto jitter = [&](uint32_t n) -> uint32_t { return __umul24(stream_draw16(ka, kb, n), jmul) >> 16; };
        for (uint32_t s = 0; s < ring_rows; s++) lds_store16(token + s * (kWave * 2u) + lane2, 0u);
        for (int d = 0; d < D; d++) {
            lds_store(devices + (uint32_t)d * 2u * kRowB + lane4, 0u);
            lds_store(devices + (uint32_t)d * 2u * kRowB + kRowB + lane4, (uint32_t)M);
        }
        bool fail = false;
        for (int phase = 0; phase < 2; phase++) {
            // ---- what every type offers at first: warm-up from micro-batch 0, cool-down from where the windows end
            int left = 0;                                           // blocks of this phase
            uint32_t active = 0;                                    // types that have some
            if (lane < K) lds_store(lane4 + 5 * kTab, phase ? (uint32_t)N : info >> 16 & 255u);
            for (int i = 0; i < K; i++) {
                const uint32_t lead = word_of(info, (uint32_t)i) >> 16 & 255u, before = phase ? (uint32_t)(NR * R) : 0u;
                const uint32_t mu = phase ? lead + before : 0u, hi = phase ? (uint32_t)N : lead;
                uint32_t offer = ~0u, low = mu << 5 | (uint32_t)i;
                if (mu < hi) {
                    left += (int)(hi - mu);
                    active |= 1u << i;
                    uint32_t from = 0;
                    bool there = true;
                    for (uint32_t rest = word_of(from_types, (uint32_t)i); rest; rest &= rest - 1u) {
                        const uint32_t a = (uint32_t)__builtin_ctz(rest);
                        there = there && (phase ? (word_of(info, a) >> 16 & 255u) + before : 0u) > mu;
                        from = max(from, lds_load16(word_of(rings, a) + (mu << 7 & tmask) + lane2));
                    }
                    const uint32_t j = jitter((uint32_t)(i * N) + mu);
                    offer = there ? (from + j) << 15 | low : 0x80000000u | low;
                    low |= j << 15;
                }
                lds_store(L::rows + (uint32_t)i * 2u * kRowB + lane4, offer);
                lds_store(L::rows + (uint32_t)i * 2u * kRowB + kRowB + lane4, low);
            }
            __syncthreads();
            // ---- a block a step, sixteen steps at a time while some candidate of the wave still has a schedule
            for (int from_step = 0; from_step < left && __ballot(live && !fail) != 0; from_step += 16)
            for (int s = from_step; s < min(left, from_step + 16); s++) {
                uint32_t pick = ~0u;
                for (uint32_t rest = active & ~several; rest;) {
                    uint32_t o[4], j[4], fr[4], asks[4];
                    int room[4];
#pragma unroll
                    for (int q = 0; q < 4; q++) {                   // (past the last one: the last one again)
                        const uint32_t i = (uint32_t)__builtin_ctz(rest), w = word_of(info, i);
                        const uint32_t more = rest & (rest - 1u);
                        rest = q < 3 ? (more ? more : rest) : more;
                        const uint32_t ra = L::rows + i * 2u * kRowB + lane4, rd = devices + (uint32_t)__builtin_ctz(w) * 2u * kRowB + lane4;
                        o[q] = lds_load(ra); j[q] = lds_load(ra + kRowB); fr[q] = lds_load(rd); room[q] = (int)lds_load(rd + kRowB);
                        asks[q] = w >> 8 & 255u;
                    }
#pragma unroll
                    for (int q = 0; q < 4; q++)
                        pick = min(pick, (uint32_t)__builtin_amdgcn_bitop3_b32((uint32_t)(max(room[q], 0) - (int)asks[q]), 0x80000000u,
                                                                              max(o[q], fr[q] + j[q]), 0xEA));        // (a & b) | c
                }
                for (uint32_t rest = active & several; rest; rest &= rest - 1u) {
                    const uint32_t i = (uint32_t)__builtin_ctz(rest), w = word_of(info, i), ra = L::rows + i * 2u * kRowB + lane4;
                    const uint32_t o = lds_load(ra), j = lds_load(ra + kRowB);
                    uint32_t fr = 0;
                    int room = INT_MAX;
                    for (uint32_t on = w & 255u; on; on &= on - 1u) {
                        const uint32_t rd = devices + (uint32_t)__builtin_ctz(on) * 2u * kRowB + lane4;
                        fr = max(fr, lds_load(rd)); room = min(room, (int)lds_load(rd + kRowB));
                    }
                    pick = min(pick, (uint32_t)__builtin_amdgcn_bitop3_b32((uint32_t)(max(room, 0) - (int)(w >> 8 & 255u)), 0x80000000u, max(o, fr + j), 0xEA));
                }
                const bool placed = (int)pick >= 0;
                fail = fail | !placed;                              // blocks left, none eligible: no schedule
                if (!placed) continue;                              // (such a lane's state stays as it is to the end of the phase)
                const uint32_t b = pick & 31u, low = pick & 0x7FE0u, low1 = low + 32u, b4 = b << 2, rb = L::rows + b * 2u * kRowB + lane4;
                const uint32_t t = lds_load(b4), pre = lds_load(b4 + kTab), post = lds_load(b4 + 2 * kTab), dm = lds_load(b4 + 3 * kTab),
                               ring = lds_load(b4 + 4 * kTab), hi = lds_load(b4 + 5 * kTab), mine = lds_load(rb + kRowB);
                const uint32_t jn = jitter(__umul24(b, (uint32_t)N) + (low1 >> 5));
                const uint32_t en = (pick >> 15) - (mine >> 15) + t;
                if (ring) lds_store16(ring + (low << 2 & tmask) + lane2, en);
                for (uint32_t on = dm & 255u; on; on &= on - 1u) {
                    const uint32_t rd = devices + (uint32_t)__builtin_ctz(on) * 2u * kRowB + lane4;
                    const uint32_t room = lds_load(rd + kRowB);
                    lds_store(rd, en << 15);
                    lds_store(rd + kRowB, room - (uint32_t)((int)dm >> 16));
                }
                // the type's next micro-batch
                const bool ends = low1 >> 5 >= hi;
                uint32_t from = 0;
                bool there = true;
                for (uint32_t rest = pre; rest; rest &= rest - 1u) {
                    const uint32_t a = (uint32_t)__builtin_ctz(rest);
                    there = there && (lds_load(L::rows + a * 2u * kRowB + kRowB + lane4) & 0x7FE0u) > low1;
                    from = max(from, lds_load16(lds_load(4u * a + 4 * kTab) + (low1 << 2 & tmask) + lane2));
                }
                lds_store(rb, ends ? ~0u : there ? (from + jn) << 15 | low1 | b : 0x80000000u | low1 | b);
                lds_store(rb + kRowB, (ends ? 0u : jn << 15) | low1 | b);
                // its consumers, if they wait for this block and it was the last of their producers'
                for (uint32_t rest = post; rest; rest &= rest - 1u) {
                    const uint32_t h = (uint32_t)__builtin_ctz(rest), rh = L::rows + h * 2u * kRowB + lane4;
                    const uint32_t oh = lds_load(rh), jh = lds_load(rh + kRowB) >> 15;
                    if (oh != (0x80000000u | low | h)) continue;
                    uint32_t last = en;
                    bool all = true;
                    for (uint32_t others = lds_load(4u * h + kTab) & ~(1u << b); others; others &= others - 1u) {
                        const uint32_t a = (uint32_t)__builtin_ctz(others);
                        all = all && (lds_load(L::rows + a * 2u * kRowB + kRowB + lane4) & 0x7FE0u) > low;
                        last = max(last, lds_load16(lds_load(4u * a + 4 * kTab) + (low << 2 & tmask) + lane2));
                    }
                    if (all) lds_store(rh, (last + jh) << 15 | low | h);
                }
            }
            __syncthreads();
            if (phase == 1 || __ballot(live && !fail) == 0) break;
            // ---- the R windows: the same blocks at the same micro-batches in every lane.  (Without the memory, which a whole
            // window leaves as it was.)
            auto load_slot = [&](uint32_t s) -> uint32_t {
                return s < ring_rows ? lds_load16(token + s * (kWave * 2u) + lane2) : lds_load(devices + (s - ring_rows) * 2u * kRowB + lane4) >> 15;
            };
            if (nin > 0) {
                int x[kMatIn];
#pragma unroll
                for (int j = 0; j < kMatIn; j++) x[j] = j < nin ? (int)load_slot(cmg->in_slot[j]) : 0;
                for (int o = 0; o < nout; o++) {
                    int acc = 0;
#pragma unroll
                    for (int j = 0; j < kMatIn; j++) acc = max(acc, x[j] + cmg->a[o][j]);
                    const uint32_t s = cmg->out_slot[o];
                    if (s < ring_rows) lds_store16(token + s * (kWave * 2u) + lane2, (uint32_t)acc);
                    else lds_store(devices + (s - ring_rows) * 2u * kRowB + lane4, (uint32_t)acc << 15);
                }
            } else
                for (int w = 0; w < R; w++)
                    for (int s = 0; s < nseq; s++) {
                        const uint32_t rw = (uint32_t)__builtin_amdgcn_readfirstlane((int)lds_load(replay + 4u * (uint32_t)s)), i = rw & 255u;
                        const uint32_t at = ((rw >> 8) + (uint32_t)(NR * w)) << 7 & tmask, on_all = word_of(info, i) & 255u, ring = word_of(rings, i);
                        uint32_t est = 0;
                        for (uint32_t rest = word_of(from_types, i); rest; rest &= rest - 1u)
                            est = max(est, lds_load16(word_of(rings, (uint32_t)__builtin_ctz(rest)) + at + lane2));
                        for (uint32_t on = on_all; on; on &= on - 1u) est = max(est, lds_load(devices + (uint32_t)__builtin_ctz(on) * 2u * kRowB + lane4) >> 15);
                        const uint32_t en = est + word_of(times, i);
                        for (uint32_t on = on_all; on; on &= on - 1u) lds_store(devices + (uint32_t)__builtin_ctz(on) * 2u * kRowB + lane4, en << 15);
                        if (ring) lds_store16(ring + at + lane2, en);
                    }
            __syncthreads();
        }
        int makespan = 0;
        for (int d = 0; d < D; d++) makespan = max(makespan, (int)(lds_load(devices + (uint32_t)d * 2u * kRowB + lane4) >> 15));
        if (fail) makespan = INT_MAX;
        if (live && makespan_out) makespan_out[kk] = makespan;
        if (live && (makespan < best || (makespan == best && c < best_ord))) { best = makespan; best_ord = c; }
    }
    if (!recs) return;
#pragma unroll
    for (int off = 32; off >= 1; off >>= 1) {
        int om = __shfl_xor(best, off);
        uint32_t ilo = __shfl_xor((uint32_t)best_ord, off), ihi = __shfl_xor((uint32_t)(best_ord >> 32), off);
        uint64_t oo = ((uint64_t)ihi << 32) | ilo;
        if (key_less(om, oo, best, best_ord)) { best = om; best_ord = oo; }
    }
    if (lane == 0) { CompRec rr; rr.makespan = best; rr.pad = 0; rr.ordinal = best_ord; recs[blockIdx.x] = rr; }
}

// Bound by the latency of its reads: 2,048 records one after the other, 32 a lane, took 10 us; here sixteen of a lane are on their way at a
// time (the last record again where there are no more): 4.6 us, 1 to 8 % of a search.  The last workgroup of the scoring kernel cannot do it for less: a fence in
// every workgroup cost 10 to 30 us.
__global__ __launch_bounds__(kWave) void complete_merge_kernel(const CompRec *__restrict__ recs, int nrecs, DevCompletion *__restrict__ res)
{
    constexpr int kAhead = 16;
    const int lane = threadIdx.x;
    int best = INT_MAX;
    uint64_t best_ord = ~0ull;
    for (int r = 0; r < nrecs; r += kWave * kAhead) {
        CompRec got[kAhead];
#pragma unroll
        for (int k = 0; k < kAhead; k++) got[k] = recs[min(r + k * kWave + lane, nrecs - 1)];
#pragma unroll
        for (int k = 0; k < kAhead; k++)
            if (key_less(got[k].makespan, got[k].ordinal, best, best_ord)) { best = got[k].makespan; best_ord = got[k].ordinal; }
    }
#pragma unroll
    for (int off = 32; off >= 1; off >>= 1) {
        int om = __shfl_xor(best, off);
        uint32_t ilo = __shfl_xor((uint32_t)best_ord, off), ihi = __shfl_xor((uint32_t)(best_ord >> 32), off);
        uint64_t oo = ((uint64_t)ihi << 32) | ilo;
        if (key_less(om, oo, best, best_ord)) { best = om; best_ord = oo; }
    }
    if (lane == 0 && best != INT_MAX && key_less(best, best_ord, res->makespan, res->ordinal)) { res->makespan = best; res->ordinal = best_ord; }
}

__global__ void completion_reset_kernel(DevCompletion *res)
{
    if (threadIdx.x == 0 && blockIdx.x == 0) { res->makespan = INT_MAX; res->pad = 0; res->ordinal = ~0ull; }
}

typedef void (*comp_fn)(const CompParams *, const CompMatrix *, uint64_t, uint64_t, CompRec *, int32_t *);

// The kernel and the LDS of a workgroup.  Chains whose types sit on one device each: rows for 4 or 8 devices with 2 or 4 types each, then
// the ring of every chain, then (no matrix) one word per block of the window.  Others: the rows of ScanRows.
constexpr size_t kCompLds = 64 * 1024;      // the size that problems are taken by
static comp_fn pick_completion(const CompParams &cp, const CompMatrix &cm, size_t &lds)
{
    bool chain = cp.npaths <= 8 && !cp.dag;
    int on[kMaxD] = {0}, most = 0;
    for (int i = 0; i < cp.K; i++) {
        chain = chain && cp.mask[i] != 0 && (cp.mask[i] & (cp.mask[i] - 1)) == 0;
        if (chain) most = std::max(most, ++on[__builtin_ctz((unsigned)cp.mask[i])]);
    }
    const size_t replay = cm.nin > 0 ? 0 : (size_t)cp.nseq * 4;
    const size_t behind = (((size_t)cp.npaths * cp.tok_ring * kWave * 2 + 255) & ~(size_t)255) + ((replay + 15) & ~(size_t)15);
    const size_t rows = cp.D <= 4 ? (most <= 2 ? ChainRows<4, 2>::token : ChainRows<4, 4>::token) : (most <= 2 ? ChainRows<8, 2>::token : ChainRows<8, 4>::token);
    lds = rows + behind;
    if (!chain) {
        lds = ScanRows::replay(cp.K, cp.D, cp.npaths * cp.tok_ring) + ((replay + 15) & ~(size_t)15);
        lds = std::max(lds, (size_t)ScanRows::rows + sizeof(CompParams));
        return complete_scan_kernel;
    }
    if (cp.D <= 4) return most <= 2 ? complete_chain_kernel<4, 2> : complete_chain_kernel<4, 4>;
    return most <= 2 ? complete_chain_kernel<8, 2> : complete_chain_kernel<8, 4>;
}

// Problems are taken up to 64 KB of parameters, 16-bit state, a key a type and the windows' words.  (The last two are those of
// an earlier kernel, and what it refused is still refused; the kernel for chains needs less, the other up to 5 KB more.  Only graphs and blocks on several devices come near, with a ring of 16
// rows for every consumed type; rings of chains have at most 16 rows too, the next power of two from twice the micro-batches of a window on,
// and there are at most eight.)
static_assert(ChainRows<8, 4>::token + 8 * 16 * kWave * 2 + kMaxSeq * 4 <= kCompLds && 2 * kMaxNR <= 16, "LDS of the completion kernel for chains");
bool completion_fits(const CompParams &cp, const CompMatrix &cm)
{
    bool chain = cp.npaths <= 8 && !cp.dag;
    for (int i = 0; i < cp.K; i++) chain = chain && (cp.mask[i] & (cp.mask[i] - 1)) == 0;
    const size_t replay = chain && cm.nin > 0 ? (size_t)(kMatIn + kMatOut + cm.nout * kMatIn) * 4 : (size_t)cp.nseq * 4;
    return (size_t)1408 + (size_t)((cp.npaths * cp.tok_ring + 2 * cp.D + cp.K + 1 + 1) / 2 * 2) * kWave * 2 +
           (size_t)(cp.K + 1) * kWave * 4 + ((replay + 15) & ~(size_t)15) <= kCompLds;
}

int launch_completions(const CompParams &cp, const CompMatrix &cm, uint64_t first, uint64_t count, int32_t *makespan_out, void *ws,
                       int num_cus, void *stream)
{
    hipStream_t st = (hipStream_t)stream;
    size_t lds;
    comp_fn fn = pick_completion(cp, cm, lds);
    if (lds > lds_per_workgroup()) return -1;
    if (lds > 48 * 1024) {
        hipError_t e = hipFuncSetAttribute((const void *)fn, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
        if (e != hipSuccess) return (int)e;
    }
    int per_cu = std::max(1, std::min(lds_blocks(lds), 16));
    // a multiple of 4, the same number on every SIMD: 9 a CU (3, 2, 2, 2) took 1.25 times as long a round of candidates as 8
    if (fn != complete_scan_kernel && per_cu > 4) per_cu &= ~3;
    uint64_t need = (count + kWave - 1) / kWave;
    const int blocks = need < (uint64_t)(num_cus * per_cu) ? (int)need : num_cus * per_cu;
    if (blocks < 1) return 0;
    CompRec *recs = makespan_out ? nullptr : (CompRec *)((char *)ws + kWsBlockRecOff);
    hipLaunchKernelGGL(fn, dim3(blocks), dim3(kWave), lds, st, (const CompParams *)((char *)ws + kWsCompParamsOff),
                       (const CompMatrix *)((char *)ws + kWsCompMatrixOff), first,
                       count, recs, makespan_out);
    int rc = (int)hipGetLastError();
    if (rc || !recs) return rc;
    hipLaunchKernelGGL(complete_merge_kernel, dim3(1), dim3(kWave), 0, st, (const CompRec *)recs, blocks,
                       (DevCompletion *)((char *)ws + kWsCompletionOff));
    return (int)hipGetLastError();
}

int launch_completion_reset(void *ws, void *stream)
{
    hipLaunchKernelGGL(completion_reset_kernel, dim3(1), dim3(1), 0, (hipStream_t)stream, (DevCompletion *)((char *)ws + kWsCompletionOff));
    return (int)hipGetLastError();
}

// ------------------------------------------------------------------ a rate of the VALU
// Sixteen independent accumulators per lane, one add and one unsigned max each per round: 32
// integer VALU instructions per round with no dependency closer than 16 instructions.  One operand of each is a scalar
// register: both are of the slower class (tessel_common.h), and what this kernel sustains, 38 T lane-operations/s, is that class's rate.
constexpr int kProbeAcc = 16;

__global__ __launch_bounds__(256) void alu_probe_kernel(uint32_t *out, int rounds, uint32_t inc, uint32_t floor_)
{
    uint32_t a[kProbeAcc];
#pragma unroll
    for (int j = 0; j < kProbeAcc; j++) a[j] = threadIdx.x * 2654435761u + j;
    for (int r = 0; r < rounds; r++) {
#pragma unroll
        for (int j = 0; j < kProbeAcc; j++) a[j] = max(a[j] + inc, floor_);
    }
    uint32_t x = 0;
#pragma unroll
    for (int j = 0; j < kProbeAcc; j++) x ^= a[j];
    out[(size_t)blockIdx.x * blockDim.x + threadIdx.x] = x;
}

int launch_alu_probe(uint32_t *out, int blocks, int rounds, void *stream)
{
    hipLaunchKernelGGL(alu_probe_kernel, dim3(blocks), dim3(256), 0, (hipStream_t)stream, out, rounds, 0x9E3779B9u, 12345u);
    return (int)hipGetLastError();
}

#endif  // TESSEL_WIDE_INSTANTIATIONS

}  // namespace tessel
