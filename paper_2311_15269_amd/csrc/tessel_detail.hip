// The decoded best candidate: leads, per-device orders after repair and per-device peaks of the candidate the running
// best names, by one wave, without memory reads in the loop over blocks.  Lane d keeps device d (order as three bit
// planes, entries not yet placed, memory); lane g keeps type g (how many micro-batches each of its producers is ahead,
// a byte each).  The types that may run are one ballot; all heads that may run are placed in one round (any order of
// them gives the same per-device orders); when there is none, the repair rule places one block.
//
// Bound by the chain of dependent instructions of a round.  One lane that walked the whole candidate and swept its
// window again took 0.93 ms for 256 blocks on 8 devices and 2.9 ms on 16, longer than scoring 10^5 candidates; this
// wave with counters in registers 0.149 and 0.119 ms.  Most problems have a lane for every block type of every device
// (detail_lanes_kernel below, 0.038 and 0.032 ms); this one takes the others.
// The period in the record is checked against the decoded orders by the host (check_period in tessel_api.cpp).
#include <hip/hip_runtime.h>
#include <stdint.h>
#include <limits.h>
#include <stddef.h>
#include <tuple>

#include "tessel_common.h"

namespace tessel {

// ------------------------------------------------------------------ mail
// Words to pinned host memory: written through to it one by one (system scope), the last one when all others have arrived.  What goes to the
// workspace is written through too: the caller may hand that memory on once it has the mail, before the kernel has ended and its
// L2 is written back.
template <typename T>
__device__ __forceinline__ void mail_word(T *to, T v) { __hip_atomic_store(to, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM); }
__device__ __forceinline__ void mail_words(uint32_t *to, const void *from, int words)
{
    for (int w = threadIdx.x; w < words; w += kWave) mail_word(to + w, ((const uint32_t *)from)[w]);
}
__device__ __forceinline__ void mail_end(DevMail *mail, uint32_t told, bool whole)
{
    if (threadIdx.x == 0) mail_word(&mail->whole, whole ? 1u : 0u);
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");             // (one wave: all lanes' words have arrived)
    if (threadIdx.x == 0) mail_word(&mail->told, told);
}
// the record, and the candidate as the workspace has it unless the host has it already
__device__ __forceinline__ void mail_stored(DevMail *mail, uint32_t told, const DevResult *res, const DevDetail *out, bool whole)
{
    if (!mail) return;
    mail_words(mail->words, res, sizeof(DevResult) / 4);
    if (whole) mail_words(mail->words + kMailDetail, out, sizeof(DevDetail) / 4);
    mail_end(mail, told, whole);
}

__global__ __launch_bounds__(kWave) void tell_kernel(const uint32_t *__restrict__ from, int words, DevMail *mail, uint32_t told)
{
    mail_words(mail->words, from, words);
    mail_end(mail, told, false);
}

// One wave; the launch's own status.  (hipGetLastError() would also report a call that failed before on this thread, and the caller would
// take back the mail of a kernel that is on its way.)
template <typename... Params, typename... Args>
static int launch_wave(void (*kernel)(Params...), void *stream, Args... args)
{
    std::tuple<Params...> params(args...);
    void *at[sizeof...(Params)];
    std::apply([&](Params &...one) { int k = 0; ((at[k++] = (void *)&one), ...); }, params);
    const hipError_t e = hipLaunchKernel((const void *)kernel, dim3(1), dim3(kWave), at, 0, (hipStream_t)stream);
    if (e != hipSuccess) (void)hipGetLastError();
    return (int)e;
}

int launch_tell(void *ws, size_t offset, size_t bytes, DevMail *mail, uint32_t told, void *stream)
{
    return launch_wave(tell_kernel, stream, (const uint32_t *)((char *)ws + offset), (int)(bytes / 4), mail, told);
}

__global__ __launch_bounds__(kWave) void detail_kernel(const KParams *__restrict__ Pp, const DevResult *__restrict__ res,
                                                       DevDetail *out, DevMail *mail, uint32_t told, int known_period,
                                                       uint64_t known_index)
{
    __shared__ uint32_t lead[kMaxKW], mask[kMaxKW];
    __shared__ uint64_t producers[kMaxKW];
    const KParams &P = *Pp;
    const uint64_t idx = res->index;
    const bool feasible = res->period != INT_MAX, known = res->period == known_period && idx == known_index;
    if (!feasible || (out->status >= 0 && out->index == idx)) {  // nothing feasible yet; the running best has not changed since it was decoded
        mail_stored(mail, told, res, out, feasible && !known);
        return;
    }
    const int lane = threadIdx.x, D = P.D, K = P.K, space = P.space;
    const uint32_t NR = (uint32_t)P.NR;
    const bool here = lane < D, sampled = space == kSampledStrict || space == kSampledRepair;
    const int dev = here ? lane : 0;
    const uint32_t ntd = here ? (uint32_t)P.ntd[dev] : 0u, n = ntd * NR;
    const uint32_t types_lo = P.type_of[dev], types_hi = P.type_of_hi[dev];
    auto type_at = [&](uint32_t y) -> uint32_t { return byte_of(y < 4u ? types_lo : types_hi, y & 3u); };
    lead[lane] = 0; mask[lane] = 0;
    producers[lane] = lane >= K ? 0ull : P.dag ? P.predmask[lane] : P.pred[lane & (kMaxK - 1)] >= 0 ? 1ull << P.pred[lane & (kMaxK - 1)] : 0ull;
    __syncthreads();
    for (uint32_t y = 0; y < ntd; y++) atomicOr(&mask[type_at(y)], 1u << lane);
    // ---- order of the lane's device
    uint32_t p0 = 0, p1 = 0, p2 = 0;
    auto put = [&](uint32_t y, uint32_t pos) {
        p0 |= (y & 1u) << pos; p1 |= ((y >> 1) & 1u) << pos; p2 |= (y >> 2) << pos;
    };
    uint32_t ka = 0, kb = 0;
    uint32_t firstlab = 0xFFFFFFFFu;
    if (sampled) {
        ka = stream_keys(P.seed, idx, kb);
        uint32_t word = 0;
        uint64_t left = 0;                                       // blocks left of every type, eight bits each
        for (uint32_t y = 0; y < ntd; y++) left |= (uint64_t)NR << (8u * y);
        for (uint32_t pos = 0; pos < n; pos++) {
            const uint32_t j = kDrawOrdBase + 32u * (uint32_t)dev + pos;
            if ((pos & 1u) == 0) word = stream_word(ka, kb, j >> 1);
            const uint32_t u = (word >> (16u * (pos & 1u))) & 0xFFFFu, digit = (u * (n - pos)) >> 16;
            uint32_t acc = 0, y = 0;                             // symbol = number of cumulative counts at or below the digit
#pragma unroll
            for (int k = 0; k < kMaxLTW - 1; k++) { acc += (uint32_t)(left >> (8 * k)) & 255u; y += digit >= acc ? 1u : 0u; }
            left -= 1ull << (8u * y);
            put(y, pos);
        }
    } else {
        uint64_t rest = idx, mine = 0;
        for (int d = 0; d < D; d++) {
            const uint64_t r = rest % P.cdev[d];
            rest /= P.cdev[d];
            if (d == lane) mine = r;
        }
        if (space == kCanonical) {
            const uint32_t B = NR + 1;
            uint32_t c[kMaxLT];
#pragma unroll
            for (int y = 0; y < kMaxLT; y++) c[y] = (uint32_t)y < ntd ? NR : 0u;
            for (uint32_t pos = 0; pos < n; pos++) {
                bool chosen = false;
#pragma unroll
                for (int y = 0; y < kMaxLT; y++) {
                    if (!chosen && c[y] > 0) {
                        c[y]--;
                        const uint64_t w = P.wtab[((c[0] * B + c[1]) * B + c[2]) * B + c[3]];
                        if (mine < w) { put((uint32_t)y, pos); chosen = true; } else { mine -= w; c[y]++; }
                    }
                }
            }
            if (lane < K) lead[lane] = (uint32_t)P.leadtab[rest * (uint64_t)K + (uint64_t)lane];
        } else {
            uint32_t r = (uint32_t)mine;
            uint64_t list = P.init_list[dev];
            for (uint32_t pos = 0; pos < n; pos++) {
                const uint32_t f = P.fact[n - 1 - pos], digit = r / f;
                r -= digit * f;
                const uint32_t code = (uint32_t)(list >> (5u * digit)) & 31u;
                const uint64_t low = list & ((1ull << (5u * digit)) - 1ull);
                list = low | (((list >> (5u * digit)) >> 5) << (5u * digit));
                const uint32_t y = code >> 3, lab = code & 7u;
                put(y, pos);
                if (byte_of(firstlab, y) == 0xFFu) firstlab = (firstlab & ~(0xFFu << (8u * y))) | (lab << (8u * y));
            }
            for (uint32_t y = 0; y < ntd; y++) lead[type_at(y)] = byte_of(firstlab, y);      // (one lead per type: the candidate is feasible)
        }
    }
    __syncthreads();
    // ---- leads of the sampled spaces: the least solution of lead = min(N_R - 1, max over dependencies of (consumer's
    // lead + step)), a dependency or two per lane, round by round from 0
    if (sampled && P.has_fixed) { if (lane < K) lead[lane] = P.fixed[lane]; }
    else if (sampled) {
        uint32_t src[2], dst[2], step[2];
        bool edge[2];
#pragma unroll
        for (int k = 0; k < 2; k++) {
            const int e = lane + k * kWave;
            uint32_t draw = 0;
            bool cross = false;
            src[k] = dst[k] = 0; edge[k] = false;
            if (P.dag) {
                if (e < P.ndeps) { edge[k] = true; src[k] = P.dsrc[e]; dst[k] = P.ddst[e]; cross = P.dcross[e] != 0; draw = (uint32_t)e; }
            } else if (e < K && P.succ[e] >= 0) {
                edge[k] = true; src[k] = (uint32_t)e; dst[k] = (uint32_t)P.succ[e]; cross = P.cross_out[e] != 0; draw = P.edge_out[e];
            }
            if (k == 1 && P.ndeps <= kWave) { edge[k] = false; step[k] = 0; continue; }
            step[k] = edge[k] && cross && stream_draw16(ka, kb, kDrawLeadBase + draw) < P.step_q16 ? 1u : 0u;
        }
        for (int round = 0; round < K; round++) {
            bool grew = false;
#pragma unroll
            for (int k = 0; k < 2; k++)
                if (edge[k]) {
                    const uint32_t v = min(NR - 1u, lead[dst[k]] + step[k]);
                    if (v > lead[src[k]]) { atomicMax(&lead[src[k]], v); grew = true; }
                }
            __syncthreads();
            if (__ballot(grew) == 0) break;
        }
    }
    __syncthreads();
    // ---- lane d: memory at the window entry, memory delta of its symbols
    int delta[kMaxLTW], mem = 0, peak = INT_MIN;
#pragma unroll
    for (uint32_t y = 0; y < (uint32_t)kMaxLTW; y++) {
        delta[y] = y < ntd ? P.m_of[dev][y] : 0;
        mem += y < ntd ? delta[y] * (int)lead[type_at(y)] : 0;
    }
    // ---- lane g: its producers (eight bits each) and how far each is ahead of it
    const int my_lead = (int)lead[lane], my_mask = (int)mask[lane];
    uint64_t who = 0, ahead = 0;
    uint32_t nprod = (uint32_t)__builtin_popcountll(producers[lane]);
    {
        int k = 0;
        for (uint64_t rest = producers[lane]; rest && k < 8; rest &= rest - 1ull, k++) {
            const uint32_t a = (uint32_t)__builtin_ctzll(rest);
            who |= (uint64_t)a << (8 * k);
            ahead |= (uint64_t)(lead[a] - (uint32_t)my_lead) << (8 * k);       // (Property 2: not negative)
        }
    }
    const bool many_in = __ballot(nprod > 8u) != 0;              // some type has more producers than that: all counts are compared
    const uint64_t my_producers = producers[lane];
    int mu = my_lead;
    uint32_t most_in = 0, most_types = 0;
    for (uint32_t k = 1; k <= 8u; k++) {
        if (__ballot(nprod >= k) != 0) most_in = k;
        if (__ballot(ntd >= k) != 0) most_types = k;
    }
    const uint64_t several = __ballot(lane < K && ((uint32_t)my_mask & ((uint32_t)my_mask - 1u)) != 0);      // types on several devices
    // ---- build
    uint32_t alive = n >= 32u ? 0xFFFFFFFFu : (1u << n) - 1u;
    int placed = 0, len = 0, status = kOk;
    const int total = P.total;
    auto take = [&](uint32_t pos, uint32_t y) {
        alive &= ~(1u << pos);
        const int a = y & 1u ? delta[1] : delta[0], b = y & 1u ? delta[3] : delta[2], c = y & 1u ? delta[5] : delta[4], d = y & 1u ? delta[7] : delta[6];
        const int lo = y & 2u ? b : a, hi = y & 2u ? d : c;
        mem += y & 4u ? hi : lo;
        peak = max(peak, mem);
        mail_word(&out->orders[dev][len++], (uint8_t)type_at(y));
    };
    while (placed < total) {
        // the types whose producers are all ahead
        bool ready = true;
        if (many_in) {
            for (int a = 0; a < K; a++) {
                const int other = __builtin_amdgcn_readlane(mu, a);
                ready = ready && !((my_producers >> a & 1ull) && other <= mu);
            }
        } else
            for (uint32_t k = 0; k < most_in; k++) ready = ready && !(k < nprod && (uint8_t)(ahead >> (8 * k)) == 0);
        const uint64_t R = __ballot(ready);
        const uint32_t r_lo = (uint32_t)R, r_hi = (uint32_t)(R >> 32);
        // lane d: its entries whose type may run
        uint32_t gate = 0;
        for (uint32_t y = 0; y < most_types; y++) {
            const uint32_t g = type_at(y), may = (g & 32u ? r_hi : r_lo) >> (g & 31u) & 1u;
            const uint32_t mine = (y & 1u ? p0 : ~p0) & (y & 2u ? p1 : ~p1) & (y & 4u ? p2 : ~p2);
            gate |= y < ntd && may ? mine : 0u;
        }
        gate &= alive;
        const uint32_t head_bit = alive & (0u - alive), pos = gate ? (uint32_t)__builtin_ctz(gate) : 0u;
        const uint32_t y = ((p0 >> pos) & 1u) | ((p1 >> pos) & 1u) << 1 | ((p2 >> pos) & 1u) << 2, g = type_at(y);
        bool ok = (gate & head_bit) != 0;                        // its head may run (and is the entry at pos)
        // a block on several devices runs when it heads the list of all its devices
        for (uint64_t rest = several & R; rest; rest &= rest - 1ull) {
            const int gt = __builtin_ctzll(rest);
            const uint32_t on = (uint32_t)__builtin_amdgcn_readlane(my_mask, gt);
            const bool heads = ok && g == (uint32_t)gt;
            if (((uint32_t)__ballot(heads) & on) != on && heads) ok = false;
        }
        uint64_t now = __ballot(ok), types = 0;
        if (now != 0) {
            if (ok) take(pos, y);
            for (; now; now &= now - 1ull) types |= 1ull << __builtin_amdgcn_readlane((int)g, __builtin_ctzll(now));
        } else {
            // nothing at the head of any list can run: the lowest device with a block that can places its earliest
            const uint64_t can = space == kSampledRepair ? __ballot(gate != 0) : 0ull;
            if (can == 0) { status = kDeadlock; break; }
            const int from = __builtin_ctzll(can);
            const uint32_t gs = (uint32_t)__builtin_amdgcn_readlane((int)g, from);
            const uint32_t on = (uint32_t)__builtin_amdgcn_readlane(my_mask, (int)gs);
            types = 1ull << gs;
            if (lane == from) take(pos, y);
            else if (here && (on >> lane & 1u)) {
                // its earliest entry on its other devices
                for (uint32_t ys = 0; ys < ntd; ys++) {
                    const uint32_t mine = alive & (ys & 1u ? p0 : ~p0) & (ys & 2u ? p1 : ~p1) & (ys & 4u ? p2 : ~p2);
                    if (type_at(ys) == gs && mine) { take((uint32_t)__builtin_ctz(mine), ys); break; }
                }
            }
        }
        placed += __builtin_popcountll(types);
        const uint32_t self = (uint32_t)(types >> lane) & 1u;
        mu += (int)self;
        for (uint32_t k = 0; k < most_in; k++) {
            const uint32_t a = (uint32_t)(who >> (8 * k)) & 63u, step = (uint32_t)(types >> a) & 1u;
            if (k < nprod) ahead += (uint64_t)((int64_t)step - (int64_t)self) << (8 * k);
        }
    }
    if (peak == INT_MIN) peak = 0;                               // a device without blocks
    if (status == kOk && __ballot(here && peak > P.M) != 0) status = kMem;
    if (lane < kMaxDW) { mail_word(&out->peak[lane], here ? peak : 0); mail_word(&out->order_len[lane], len); }
    if (lane < K) mail_word(&out->leads[lane], (int)lead[lane]);
    if (lane == 0) { mail_word(&out->status, status); mail_word(&out->index, idx); }
    __threadfence();                                             // (read back below by other lanes)
    mail_stored(mail, told, res, out, true);
}

// ------------------------------------------------------------------ a lane per (device, block type)
// Where 2^LG lanes a device (one for every type on it) fit one wave and no type has more than kLaneIn producers.  A lane
// keeps the positions its type still has in its device's order and one word of fields with a guard bit each, occurrences left
// and per producer the micro-batches waiting: one addition and one compare tell whether the type may run.  The earliest
// entries of a device, and the earliest that may run, are minima over its lanes (cross-lane moves inside a group of eight),
// and a round is two or three ballots with no table to look anything up in.
//
// Bound by the same chain of dependent instructions, which is shorter by that: a round takes 290 cycles.  256 blocks on 8
// devices 149 -> 38 us, on 16 devices 119 -> 32; 288 on 12 devices 149 -> 39; 96 on 4 devices, six types each, 77 -> 20; 8 on two
// devices 6.5 -> 4.5.  Code that runs once stays in loops: fetching it costs more than the cycles a longer body would save.
constexpr int kLaneIn = 4;
constexpr uint32_t kLaneOnes = 0x01041041u, kLaneAdd = 31u * kLaneOnes, kLaneGuard = 32u * kLaneOnes;      // five fields of five bits and a guard

template <int LG>
__device__ __forceinline__ uint32_t least_of_device(uint32_t x)
{
    if (LG >= 1) x = min(x, (uint32_t)__builtin_amdgcn_mov_dpp((int)x, 0xB1, 0xF, 0xF, true));        // the other lane of a pair
    if (LG >= 2) x = min(x, (uint32_t)__builtin_amdgcn_mov_dpp((int)x, 0x4E, 0xF, 0xF, true));        // the other pair of four
    if (LG >= 3) x = min(x, (uint32_t)__builtin_amdgcn_mov_dpp((int)x, 0x141, 0xF, 0xF, true));       // eight lanes mirrored: the other four
    return x;
}

// (WIDE: more than 32 lanes)
template <int LG, bool TP, bool WIDE>
__global__ __launch_bounds__(kWave) void detail_lanes_kernel(const KParams *__restrict__ Pp, const DevResult *__restrict__ res,
                                                             DevDetail *out, DevMail *mail, uint32_t told, int known_period,
                                                             uint64_t known_index)
{
    constexpr uint32_t G = 1u << LG;
    constexpr int NP = LG > 0 ? LG : 1;
    __shared__ uint32_t lead[kMaxKW], home[kMaxKW], ahead[kMaxKW], after[kMaxKW];
    __shared__ uint32_t mates[2 * kMaxKW];                       // by type: its lanes, below 32 and from 32 on
    __shared__ uint64_t producers[kMaxKW];
    __shared__ __attribute__((aligned(4))) uint8_t order[kMaxDW * kMaxPos];        // symbols in device order
    __shared__ uint32_t det[sizeof(DevDetail) / 4];              // DevDetail by words
    static_assert(sizeof(DevDetail) / 4 == 4 + 2 * kMaxDW + kMaxKW + kMaxDW * kMaxPos / 4 && offsetof(DevDetail, peak) == 16 &&
                  offsetof(DevDetail, leads) == 4 * (4 + kMaxDW) && offsetof(DevDetail, order_len) == 4 * (4 + kMaxDW + kMaxKW), "words of DevDetail");
    const KParams &P = *Pp;
    const int lane = threadIdx.x, period = res->period, decoded = out->status;
    const uint64_t idx = res->index, decoded_idx = out->index;
    const int D = P.D, K = P.K, space = P.space;
    const uint32_t NR = (uint32_t)P.NR;
    const bool here = lane < D << LG, sampled = space == kSampledStrict || space == kSampledRepair;
    const uint32_t dev = here ? (uint32_t)lane >> LG : 0u, y = (uint32_t)lane & (G - 1u);
    const uint32_t ntd = (uint32_t)P.ntd[dev], n = ntd * NR;
    const uint32_t types_lo = P.type_of[dev], types_hi = P.type_of_hi[dev];
    // (what is read later by numbers known here: the loads are all on their way at once)
    int delta[kMaxLTW];                                          // lane d: memory deltas of device d's symbols
    const uint32_t own = (uint32_t)lane < kMaxDW ? (uint32_t)lane : 0u;
    const uint32_t own_lo = P.type_of[own], own_hi = P.type_of_hi[own];
    const int own_ntd = P.ntd[own];
#pragma unroll
    for (int s = 0; s < kMaxLTW; s++) delta[s] = P.m_of[own][s];
    const int chain_pred = P.pred[lane & (kMaxK - 1)];
    const uint64_t graph_pred = P.predmask[lane];
    const int chain_succ = P.succ[lane & (kMaxK - 1)], chain_cross = P.cross_out[lane & (kMaxK - 1)], chain_edge = P.edge_out[lane & (kMaxK - 1)];
    uint32_t src[2], dst[2], crosses[2];
#pragma unroll
    for (int k = 0; k < 2; k++) { src[k] = P.dsrc[lane + k * kWave]; dst[k] = P.ddst[lane + k * kWave]; crosses[k] = P.dcross[lane + k * kWave]; }
    static_assert(kMaxDeps == 2 * kWave, "two dependencies a lane");
    if (period == INT_MAX || (decoded >= 0 && decoded_idx == idx)) {      // nothing feasible yet; the running best has not changed since it was decoded
        mail_stored(mail, told, res, out, period != INT_MAX && !(period == known_period && idx == known_index));
        return;
    }
    auto type_at = [&](uint32_t s) -> uint32_t { return byte_of(s < 4u ? types_lo : types_hi, s & 3u); };
    const bool block = here && y < ntd;                          // the lane has a block type
    const uint32_t type = block ? type_at(y) : 0u;
    lead[lane] = 0; home[lane] = 63u; ahead[lane] = 0; after[lane] = (uint32_t)lane; mates[lane] = mates[kMaxKW + lane] = 0;
    producers[lane] = lane >= K ? 0ull : P.dag ? graph_pred : chain_pred >= 0 ? 1ull << chain_pred : 0ull;
    __syncthreads();
    if (block) {
        atomicMin(&home[type], (uint32_t)lane);
        if (TP) atomicOr(&mates[lane < 32 ? type : kMaxKW + type], 1u << (lane & 31));
    }
    // ---- order of the lane's device
    uint32_t ka = 0, kb = 0, firstlab = 0xFFFFFFFFu;
    Planes<NP> o;
    o.clear();
    if (sampled) {
        ka = stream_keys(P.seed, idx, kb);
        sampled_order<NP>(ka, kb, (int)dev, ntd, NR, o);
    } else {
        uint64_t rest = idx, mine = 0;
        for (int d = 0; d < D; d++) {
            uint64_t r;
            if ((rest | P.cdev[d]) >> 32) { r = rest % P.cdev[d]; rest /= P.cdev[d]; }
            else { r = (uint32_t)rest % (uint32_t)P.cdev[d]; rest = (uint32_t)rest / (uint32_t)P.cdev[d]; }
            if ((uint32_t)d == dev) mine = r;
        }
        if (space == kCanonical) {
            if (P.ranked) {
                const uint64_t planes = P.orders[P.order_at[ntd] + mine];
                o.p0 = (uint32_t)planes; o.p1 = (uint32_t)(planes >> 32);
            } else {
                const uint32_t B = NR + 1;
                uint32_t c[kMaxLT];
#pragma unroll
                for (int s = 0; s < kMaxLT; s++) c[s] = (uint32_t)s < ntd ? NR : 0u;
                for (uint32_t pos = 0; pos < n; pos++) {
                    bool chosen = false;
#pragma unroll
                    for (int s = 0; s < kMaxLT; s++) {
                        if (!chosen && c[s] > 0) {
                            c[s]--;
                            const uint64_t w = P.wtab[((c[0] * B + c[1]) * B + c[2]) * B + c[3]];
                            if (mine < w) { o.put((uint32_t)s, pos); chosen = true; } else { mine -= w; c[s]++; }
                        }
                    }
                }
            }
            if (lane < K) lead[lane] = (uint32_t)P.leadtab[rest * (uint64_t)K + (uint64_t)lane];
        } else {
            uint32_t r = (uint32_t)mine;
            uint64_t list = P.init_list[dev];
            for (uint32_t pos = 0; pos < n; pos++) {
                const uint32_t f = P.fact[n - 1 - pos], digit = r / f;
                r -= digit * f;
                const uint32_t code = (uint32_t)(list >> (5u * digit)) & 31u;
                const uint64_t low = list & ((1ull << (5u * digit)) - 1ull);
                list = low | (((list >> (5u * digit)) >> 5) << (5u * digit));
                const uint32_t s = code >> 3, lab = code & 7u;
                o.put(s, pos);
                if (byte_of(firstlab, s) == 0xFFu) firstlab = (firstlab & ~(0xFFu << (8u * s))) | (lab << (8u * s));
            }
            if (block) lead[type] = byte_of(firstlab, y);        // (one lead per type: the candidate is feasible)
        }
    }
    __syncthreads();
    // ---- leads of the sampled spaces: the least solution of lead = min(N_R - 1, max over dependencies of (consumer's
    // lead + step))
    if (sampled && P.has_fixed) { if (lane < K) lead[lane] = P.fixed[lane]; }
    else if (sampled) {
        uint32_t step[2];
        bool edge[2];
#pragma unroll
        for (int k = 0; k < 2; k++) {
            const int e = lane + k * kWave;
            uint32_t draw = (uint32_t)e;
            bool cross = crosses[k] != 0;
            edge[k] = P.dag && e < P.ndeps;
            if (!P.dag) {
                edge[k] = e < K && chain_succ >= 0;
                src[k] = (uint32_t)e; dst[k] = (uint32_t)chain_succ & (kMaxKW - 1); cross = chain_cross != 0; draw = (uint32_t)chain_edge;
            }
            if (k == 1 && P.ndeps <= kWave) { edge[k] = false; step[k] = 0; continue; }
            step[k] = edge[k] && cross && stream_draw16(ka, kb, kDrawLeadBase + draw) < P.step_q16 ? 1u : 0u;
        }
        if (!P.dag || P.graph_chain) {
            // chains: the steps to the end of the chain, by doubling
#pragma unroll
            for (int k = 0; k < 2; k++)
                if (edge[k]) { after[src[k]] = dst[k]; atomicMax(&ahead[src[k]], step[k]); }
            __syncthreads();
            int sum = (int)ahead[lane], next = (int)after[lane];
            for (int far = 1; far < K; far *= 2) {
                const int s = __shfl(sum, next), m = __shfl(next, next);
                sum += next != lane ? s : 0;
                next = m;
            }
            lead[lane] = min(NR - 1u, (uint32_t)sum);
        } else
            for (int round = 0; round < K; round++) {            // graphs: round by round from 0
                bool grew = false;
#pragma unroll
                for (int k = 0; k < 2; k++)
                    if (edge[k]) {
                        const uint32_t v = min(NR - 1u, lead[dst[k]] + step[k]);
                        if (v > lead[src[k]]) { atomicMax(&lead[src[k]], v); grew = true; }
                    }
                __syncthreads();
                if (__ballot(grew) == 0) break;
            }
    }
    __syncthreads();
    // ---- the lane's type: its entries, its word, where its producers sit
    const uint32_t alive = n >= 32u ? 0xFFFFFFFFu : (1u << n) - 1u;
    uint32_t left = alive & (y & 1u ? o.p0 : ~o.p0);
    if (NP > 1) left &= y & 2u ? o.p1 : ~o.p1;
    if (NP > 2) left &= y & 4u ? o.p2 : ~o.p2;
    if (!block) left = 0;
    uint32_t word = block ? kLaneOnes - 1u + NR : 0u, minus = 1u, from[kLaneIn], plus[kLaneIn], nprod = 0;
    {
        uint64_t rest = block ? producers[type] : 0ull;
#pragma unroll
        for (int k = 0; k < kLaneIn; k++) {
            from[k] = plus[k] = 0;
            if (rest == 0) continue;
            const uint32_t a = (uint32_t)__builtin_ctzll(rest), one = 1u << (6 * (k + 1));
            rest &= rest - 1ull;
            word += (lead[a] - lead[type] - 1u) * one;           // (Property 2: not negative; the field starts at 1)
            minus |= one;
            from[k] = home[a]; plus[k] = one;
            nprod++;
        }
    }
    uint32_t most_in = 0;
    for (uint32_t k = 1; k <= (uint32_t)kLaneIn; k++) if (__ballot(nprod >= k) != 0) most_in = k;
    // the lanes of the lane's type, where types sit on several devices
    const uint32_t all_lo = TP ? mates[type] : 0u, all_hi = TP ? mates[kMaxKW + type] : 0u;
    // ---- build
    const uint64_t repair = space == kSampledRepair ? ~0ull : 0ull;
    const uint32_t group = ((1u << G) - 1u) << ((uint32_t)lane & 31u & ~(G - 1u));       // the device's lanes, of 32
    uint32_t at = dev * (uint32_t)kMaxPos;                       // the device's next place in `order`
    for (;;) {
        const uint32_t pos = low_bit(left);                      // (none left: the largest number)
        const bool may = ((word + kLaneAdd) & kLaneGuard) == kLaneGuard;
        const uint32_t head = least_of_device<LG>(pos), first = least_of_device<LG>(may ? pos : 0xFFFFFFFFu);
        const uint64_t ready = __builtin_amdgcn_ballot_w64(may);
        uint64_t heads = ready & __builtin_amdgcn_ballot_w64(pos == head);
        // a block on several devices runs when it heads the list of all its devices
        if (TP) heads &= __builtin_amdgcn_ballot_w64(((uint32_t)heads & all_lo) == all_lo && (!WIDE || ((uint32_t)(heads >> 32) & all_hi) == all_hi));
        // nothing at the head of any list can run: the lowest device with a block that can places its earliest
        const uint64_t can = ready & __builtin_amdgcn_ballot_w64(pos == first) & repair;
        uint64_t one = can & (0ull - can);
        if (TP && heads == 0 && can != 0) {
            const int by = __builtin_ctzll(can);
            one = (uint64_t)(uint32_t)__builtin_amdgcn_readlane((int)all_lo, by) | (uint64_t)(uint32_t)__builtin_amdgcn_readlane((int)all_hi, by) << 32;
        }
        const uint64_t now = heads ? heads : one;
        if (now == 0) break;
        const uint32_t lo = (uint32_t)now, hi = (uint32_t)(now >> 32), half = WIDE && lane >= 32 ? hi : lo;
        if (__builtin_amdgcn_inverse_ballot_w64(now)) {
            order[at] = (uint8_t)y;
            left &= left - 1u;
            word -= minus;
        }
        at += half & group ? 1u : 0u;
#pragma unroll
        for (int k = 0; k < kLaneIn; k++) {
            if (k > 0 && (uint32_t)k >= most_in) break;
            word += plus[k] & (uint32_t)__builtin_amdgcn_sbfe((int)(WIDE && (from[k] & 32u) ? hi : lo), from[k], 1);
        }
    }
    const uint64_t open = __ballot(left != 0);
    __syncthreads();
    // ---- lane d: the device's order and memory
    int status = open ? kDeadlock : kOk;
    {
        const bool dev_lane = lane < D;
        const int end = (int)__shfl(at, (lane << LG) & (kWave - 1)), len = dev_lane ? end - lane * kMaxPos : 0;
        int mem = 0, peak = INT_MIN;
#pragma unroll
        for (int s = 0; s < kMaxLTW; s++)
            if (s < own_ntd) mem += delta[s] * (int)lead[byte_of(s < 4 ? own_lo : own_hi, (uint32_t)s & 3u)];
        // (a loop: the kernel runs its code once, and fetching it costs more than the few cycles a longer body would save)
#pragma unroll 1
        for (int k = 0; k < len; k++) {
            const uint32_t s = order[own * kMaxPos + (uint32_t)k];
            const int a = s & 1u ? delta[1] : delta[0], b = s & 1u ? delta[3] : delta[2], c = s & 1u ? delta[5] : delta[4], e = s & 1u ? delta[7] : delta[6];
            const int low = s & 2u ? b : a, high = s & 2u ? e : c;
            mem += s & 4u ? high : low;
            peak = max(peak, mem);
        }
        if (peak == INT_MIN) peak = 0;                           // a device without blocks
        if (status == kOk && __ballot(dev_lane && peak > P.M) != 0) status = kMem;
        if (lane < kMaxDW) { det[4 + lane] = (uint32_t)(dev_lane ? peak : 0); det[4 + kMaxDW + kMaxKW + lane] = (uint32_t)len; }
    }
    if (lane == 0) { det[0] = (uint32_t)status; det[1] = 0; det[2] = (uint32_t)idx; det[3] = (uint32_t)(idx >> 32); }
    det[4 + kMaxDW + lane] = lane < K ? lead[lane] : 0u;
    // (places behind a device's last block hold nothing, and are not read)
    for (int k = lane; k < D * kMaxPos / 4; k += kWave) {
        const int d = k / (kMaxPos / 4);
        const uint32_t lo = P.type_of[d], hi = P.type_of_hi[d], four = ((const uint32_t *)order)[k];
        uint32_t types = 0;
        for (int q = 0; q < 4; q++) {
            const uint32_t s = four >> (8 * q) & 7u;
            types |= byte_of(s < 4u ? lo : hi, s & 3u) << (8 * q);
        }
        det[4 + 2 * kMaxDW + kMaxKW + k] = types;
    }
    __syncthreads();
    // to the workspace, and to the host
    const int words = 4 + 2 * kMaxDW + kMaxKW + D * kMaxPos / 4;
    for (int w = lane; w < words; w += kWave) mail_word((uint32_t *)out + w, det[w]);
    if (mail) {
        mail_words(mail->words, res, sizeof(DevResult) / 4);
        for (int w = lane; w < words; w += kWave) mail_word(mail->words + kMailDetail + w, det[w]);
        mail_end(mail, told, true);
    }
}

typedef void (*detail_fn)(const KParams *, const DevResult *, DevDetail *, DevMail *, uint32_t, int, uint64_t);

// lanes a device takes (log2), or -1: see detail_lanes_kernel
int detail_lanes(int devices, int most_types, int most_producers)
{
    int lg = 0;
    while ((1 << lg) < most_types) lg++;
    return (devices << lg) <= kWave && most_producers <= kLaneIn ? lg : -1;
}

template <int LG>
static detail_fn pick_lanes(const KParams &kp)
{
    const bool wide = (kp.D << LG) > 32;
    return kp.tp ? (wide ? detail_lanes_kernel<LG, true, true> : detail_lanes_kernel<LG, true, false>)
                 : (wide ? detail_lanes_kernel<LG, false, true> : detail_lanes_kernel<LG, false, false>);
}

static detail_fn pick_detail(const KParams &kp)
{
    switch (kp.detail_lanes) {
    case 0: return pick_lanes<0>(kp);
    case 1: return pick_lanes<1>(kp);
    case 2: return pick_lanes<2>(kp);
    case 3: return pick_lanes<3>(kp);
    default: return detail_kernel;
    }
}

int launch_detail(const KParams &kp, void *ws, DevMail *mail, uint32_t told, int32_t known_period, uint64_t known_index, void *stream)
{
    return launch_wave(pick_detail(kp), stream, (const KParams *)((char *)ws + kWsParamsOff), (const DevResult *)((char *)ws + kWsResultOff),
                       (DevDetail *)((char *)ws + kWsDetailOff), mail, told, known_period, known_index);
}

}  // namespace tessel
