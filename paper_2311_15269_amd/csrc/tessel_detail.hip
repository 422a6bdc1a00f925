// The decoded best candidate: leads, per-device orders after repair and per-device peaks of the candidate the running
// best names, by one wave, without memory reads in the loop over blocks.  Lane d keeps device d (order as three bit
// planes, entries not yet placed, memory); lane g keeps type g (how many micro-batches each of its producers is ahead,
// a byte each).  The types that may run are one ballot; all heads that may run are placed in one round (any order of
// them gives the same per-device orders); when there is none, the repair rule places one block.
//
// Bound by the chain of dependent instructions of a round.  One lane that walked the whole candidate and swept its
// window again took 0.93 ms for 256 blocks on 8 devices and 2.9 ms on 16, longer than scoring 10^5 candidates; this
// wave with counters in LDS 0.26 and 0.155 ms, with counters in registers 0.149 and 0.119 ms.
// The period in the record is checked against the decoded orders by the host (check_period in tessel_api.cpp).
#include <hip/hip_runtime.h>
#include <stdint.h>
#include <limits.h>

#include "tessel_common.h"

namespace tessel {

__global__ __launch_bounds__(kWave) void detail_kernel(const KParams *__restrict__ Pp, const DevResult *__restrict__ res,
                                                       DevDetail *__restrict__ out)
{
    __shared__ uint32_t lead[kMaxKW], mask[kMaxKW];
    __shared__ uint64_t producers[kMaxKW];
    const KParams &P = *Pp;
    if (res->period == INT_MAX) return;                          // nothing feasible yet
    const uint64_t idx = res->index;
    if (out->status >= 0 && out->index == idx) return;           // the running best has not changed since it was decoded
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
        out->orders[dev][len++] = (int)type_at(y);
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
    if (lane < kMaxDW) { out->peak[lane] = here ? peak : 0; out->order_len[lane] = len; }
    if (lane < K) out->leads[lane] = (int)lead[lane];
    if (lane == 0) { out->status = status; out->index = idx; }
}

int launch_detail(void *ws, void *stream)
{
    hipLaunchKernelGGL(detail_kernel, dim3(1), dim3(kWave), 0, (hipStream_t)stream, (const KParams *)((char *)ws + kWsParamsOff),
                       (const DevResult *)((char *)ws + kWsResultOff), (DevDetail *)((char *)ws + kWsDetailOff));
    return (int)hipGetLastError();
}

}  // namespace tessel
